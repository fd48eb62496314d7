// Salient-weight protection (Sec. 3.5; App. "Salient Weight Protection"): per unit, the
// n_p = floor(rate * n) weights with the largest saliency |w| * s_c are kept out of the
// low-bit quantizer and stored in INT8; Eq. 5 then charges them 8 bits each.
//
// windq_salient_select  finds the protected set EXACTLY: the saliency threshold T of a
//   unit is the n_p-th largest key (the bit pattern of the fp32 saliency).  A sample of the
//   unit (all of a small one) brackets T between two keys lo <= T < hi; ONE pass over W then writes every
//   mask bit that the bracket decides (key >= hi: protected, key < lo: not), counts the
//   first kind and lists the keys in between, about 1 % of the unit, with their positions.
//   The counts prove the bracket: T lies in it if and only if n_p lies between the number
//   above it and that plus the number in it.  The rest is settled per unit from the list alone:
//   T by radix selection over the bracket, the ties (weights equal to T are taken in
//   the order of their flat index inside the unit) by the same over their positions.
//   Units whose sample misled, or whose bracket outgrows the list (a thirty-second of the
//   unit: constant weights, say), are selected by digit passes over W instead (11 + 11 + 9
//   bits of the key), count their ties per tile where they are split between kept and
//   protected, and rank them in a last pass.  The result is a bit mask in the layout of W:
//   one byte per 8 columns.
// windq_salient_encode  stores the protected weights: per unit one symmetric scale
//   sigma = fp32(max|w_p| / 127), codes clamp(rne(w * fp32(1/sigma)), -127, 127) in
//   flat-index order, and the activation-weighted error of that INT8 part.
// Everything is integer or fixed-order fp64: bit-reproducible.  Select streams W once, and of
// each unit a sample of at most 32768 weights (the units that fall back: four times more, and a fifth for the
// tiles of those whose ties are split); encode reads of W only the pieces that hold protected weights, once (again for
// tiles that hold more of them than their scratch area).  Every kernel
// takes a batch of matrices, so a decoder block costs eight launches for select and four for encode.
// 7B-shaped block at 3 %: select and encode 301 us (586 with two passes over W, a histogram atomic per weight in the
// first, and two gathers).  By a kernel trace, whose times are a few per cent longer: sample 21, the pass over W 103
// (3.9 TB/s; a plain copy moves 5.1), lists 22, five passes that find nothing flagged 22; collect 108, the units' scales
// 5, codes 29, errors 4.
// None of this is on the per-step hot path (the mask of a matrix is computed once per
// protection rate).
#include <float.h>

#include "windq_common.hpp"
#include "windq_select.hpp"
#include "windq_ws.hpp"

namespace windq {

constexpr int SAL_THREADS = 256;

struct SalArgs {
    const void* W;
    const float* s;
    uint8_t* mask;          // [rows][mask_ld] bytes
    int64_t mask_ld;
    Geometry g;
    uint32_t* hist;         // [3][U][FEAT_BINS]  digit histograms of flagged units
    uint32_t* lo;           // [U]  the bracket: lo <= T < hi
    uint32_t* hi;           // [U]
    uint32_t* mid;          // [U]  where the sample puts T: what the pass over W takes for it inside the bracket
    uint64_t* count;        // [U]  upper half: keys >= hi; lower half: keys in the bracket
    uint32_t* cnt;          // [n_tiles]  select: keys equal to T; encode: protected weights, then those of earlier tiles
    uint32_t* flag;         // [U]  1: selected by digit passes over W; 0: from the unit's candidate list
    uint32_t* n_flagged;    // how many units are flagged, and ...
    uint32_t* flagged;      // [U]  ... which, in no particular order
    uint2* cand;            // [U][cap]  (key, flat position in the unit) of the keys in the bracket
    uint32_t cap;
    uint32_t use_list;      // 0: every unit takes the digit passes (mask not addressable in whole dwords)
    uint32_t n_p;           // protected weights per unit
    uint32_t rank0;         // ascending rank of T: n - n_p + 1
    // encode
    int8_t* prot_codes;     // [U][n_p]
    float* prot_scale;      // [U]
    float* err_prot;        // [U]
    float* tile_max;        // [n_tiles]
    double* err_part;       // [n_tiles]
};

// A launch covers up to WINDQ_MAX_BATCH matrices (one chunk width, one element type): tiles,
// and units are numbered one matrix after the other.
struct SalBatch {
    int32_t n;
    uint32_t* any_flagged;      // flagged units of all matrices
    int64_t tile_start[WINDQ_MAX_BATCH + 1];
    int64_t unit_start[WINDQ_MAX_BATCH + 1];
    int64_t band_start[WINDQ_MAX_BATCH + 1];     // workgroups of the candidate pass
    int32_t cand_tiles;         // tiles that one of them takes
    SalArgs m[WINDQ_MAX_BATCH];
};

__host__ __device__ constexpr int sal_shift(int level) { return level == 0 ? 20 : (level == 1 ? 9 : 0); }
__host__ __device__ constexpr int sal_bits(int level) { return level == 2 ? 9 : 11; }

// Saliency key: the bit pattern of fp32(|w| * |s_c|), one correctly rounded multiply.
// Non-negative floats order like their bit patterns.
__device__ __forceinline__ uint32_t sal_key(float w, float sc) { return __float_as_uint(fabsf(w) * fabsf(sc)); }

template <int DT>
__device__ __forceinline__ void load8g(const void* __restrict__ data, int64_t off, float (&w)[8]) {
    if (DT == WINDQ_BF16) {
        const uint4 raw = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(data) + off);
        w[0] = bf16_bits_to_f32(raw.x & 0xffffu); w[1] = __uint_as_float(raw.x & 0xffff0000u);
        w[2] = bf16_bits_to_f32(raw.y & 0xffffu); w[3] = __uint_as_float(raw.y & 0xffff0000u);
        w[4] = bf16_bits_to_f32(raw.z & 0xffffu); w[5] = __uint_as_float(raw.z & 0xffff0000u);
        w[6] = bf16_bits_to_f32(raw.w & 0xffffu); w[7] = __uint_as_float(raw.w & 0xffff0000u);
    } else {
        const float4* src = reinterpret_cast<const float4*>(static_cast<const float*>(data) + off);
        const float4 a = src[0], b = src[1];
        w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
        w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
    }
}

// The same eight weights in two steps: the raw bytes (4 or 8 registers), then the values.
template <int DT>
struct Raw8 {
    uint4 a, b;
};
template <>
struct Raw8<WINDQ_BF16> {
    uint4 a;
};
template <int DT>
__device__ __forceinline__ Raw8<DT> load8raw(const void* __restrict__ data, int64_t off) {
    Raw8<DT> r;
    if constexpr (DT == WINDQ_BF16) {
        r.a = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(data) + off);
    } else {
        const uint4* src = reinterpret_cast<const uint4*>(static_cast<const float*>(data) + off);
        r.a = src[0];
        r.b = src[1];
    }
    return r;
}
template <int DT>
__device__ __forceinline__ void unpack8raw(const Raw8<DT>& r, float (&w)[8]) {
    if constexpr (DT == WINDQ_BF16) {
        w[0] = bf16_bits_to_f32(r.a.x & 0xffffu); w[1] = __uint_as_float(r.a.x & 0xffff0000u);
        w[2] = bf16_bits_to_f32(r.a.y & 0xffffu); w[3] = __uint_as_float(r.a.y & 0xffff0000u);
        w[4] = bf16_bits_to_f32(r.a.z & 0xffffu); w[5] = __uint_as_float(r.a.z & 0xffff0000u);
        w[6] = bf16_bits_to_f32(r.a.w & 0xffffu); w[7] = __uint_as_float(r.a.w & 0xffff0000u);
    } else {
        w[0] = __uint_as_float(r.a.x); w[1] = __uint_as_float(r.a.y); w[2] = __uint_as_float(r.a.z); w[3] = __uint_as_float(r.a.w);
        w[4] = __uint_as_float(r.b.x); w[5] = __uint_as_float(r.b.y); w[6] = __uint_as_float(r.b.z); w[7] = __uint_as_float(r.b.w);
    }
}

// Register 0..3 by a run-time index.  By value: picked through a reference, weights lay in scratch (144 bytes a lane).
__device__ __forceinline__ uint32_t pick4(uint32_t x, uint32_t y, uint32_t z, uint32_t w, int d) {
    const uint32_t lower = (d & 1) != 0 ? y : x, upper = (d & 1) != 0 ? w : z;
    return (d & 2) != 0 ? upper : lower;
}
// Weight j (0..7, a run-time index) of the eight.  CHAIN (bf16): compares one after the other; the tree has fewer steps, but
// encode takes 163 us with it and 147 so (7B-shaped block, 3 %).
template <int DT, bool CHAIN>
__device__ __forceinline__ float raw_elem(const Raw8<DT>& r, int j) {
    if constexpr (DT == WINDQ_BF16) {
        const int d = j >> 1;
        const uint32_t dw = CHAIN ? (d == 0 ? r.a.x : (d == 1 ? r.a.y : (d == 2 ? r.a.z : r.a.w))) : pick4(r.a.x, r.a.y, r.a.z, r.a.w, d);
        return __uint_as_float((j & 1) != 0 ? dw & 0xffff0000u : dw << 16);
    } else {
        const uint32_t lower = pick4(r.a.x, r.a.y, r.a.z, r.a.w, j), upper = pick4(r.b.x, r.b.y, r.b.z, r.b.w, j);
        return __uint_as_float(j < 4 ? lower : upper);
    }
}

// Clears the mask of a matrix (rows x mask_ld bytes, dense).
__global__ __launch_bounds__(256) void sal_clear_mask_kernel(uint8_t* __restrict__ mask, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) mask[i] = 0;
}

// Block-wide sum of a per-thread u32 (all SAL_THREADS threads call it).
__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t* sh) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t t = 0;
    for (int w = 0; w < SAL_THREADS / 64; ++w) t += sh[w];
    return t;
}

// ------------------------------------------------------- selection by digit passes over W
// What the histograms of the digits so far say about a flagged unit: the threshold's digits, and the
// 1-based ascending rank still to find among the keys that carry them.  After the last digit the prefix is the
// threshold T, every key of the bin equals T, and the rank left over, r, says that the wanted key is
// the r-th of those e ties in ascending order: r - 1 of them count among the kept weights and
// e - r + 1 among the protected ones.
struct SalFound {
    uint32_t prefix, rank, in_bin;
};
// The step from digit `step` - 1 to `step` (1 to 3; 0: nothing is known yet), by every workgroup that comes to a unit in the pass
// after that digit's histogram; the one with the unit's first tile keeps it for the next pass (`keep`), in the words of the
// bracket or, so that nothing is written that another workgroup of the pass still reads, of the unit's counts.
__device__ __forceinline__ SalFound sal_step(const SalArgs& A, int64_t u, int step, bool keep, uint32_t* sh_part, uint32_t* sh_out) {
    SalFound f = {0u, A.rank0, 0u};
    if (step == 0) return f;
    if (step == 2) f = {A.lo[u], A.hi[u], 0u};
    if (step == 3) f = {(uint32_t)A.count[u], (uint32_t)(A.count[u] >> 32), 0u};
    const uint32_t* h = A.hist + ((size_t)(step - 1) * (size_t)A.g.U + (size_t)u) * FEAT_BINS;
    uint32_t bin;
    uint64_t below;
    __syncthreads();
    select_bin<SAL_THREADS>(h, 1 << sal_bits(step - 1), f.rank, sh_part, sh_out, &bin, &below);
    f.rank -= (uint32_t)below;
    f.prefix = (f.prefix << sal_bits(step - 1)) | bin;
    f.in_bin = h[bin];
    if (keep && threadIdx.x == 0) {
        if (step == 2) {
            A.count[u] = ((uint64_t)f.rank << 32) | f.prefix;
        } else {
            A.lo[u] = f.prefix;
            A.hi[u] = f.rank;
            A.mid[u] = f.in_bin;
        }
    }
    return f;
}

// The histogram of the next digit is emptied while the one before it is filled (by the workgroup with the unit's first tile).
template <int NT>
__device__ __forceinline__ void sal_clear_hist(const SalArgs& A, int64_t u, int level) {
    uint4* __restrict__ h = reinterpret_cast<uint4*>(A.hist + ((size_t)level * (size_t)A.g.U + (size_t)u) * FEAT_BINS);
    for (int32_t i = threadIdx.x; i < FEAT_BINS / 4; i += NT) h[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Histogram of digit `level` of the keys of one tile that carry the unit's prefix.
template <int DT>
__device__ __forceinline__ void sal_hist_tile(const SalArgs& A, const TileCoord& tc, const int level, const uint32_t prefix,
                                              uint32_t* lhist, float* scol) {
    const int32_t G = A.g.chunk_w;
    const int32_t nbins = 1 << sal_bits(level);
    for (int32_t b = threadIdx.x; b < nbins; b += SAL_THREADS) lhist[b] = 0;
    for (int32_t c = threadIdx.x; c < G; c += SAL_THREADS) scol[c] = A.s[tc.col0 + c];
    __syncthreads();
    const int32_t shift = sal_shift(level), bits = sal_bits(level);
    const uint32_t dmask = (1u << bits) - 1u;
    const int32_t pieces = G >> 3;
    const int32_t total = tc.nrows * pieces;
    PieceWalk at((int32_t)threadIdx.x, SAL_THREADS, pieces);
    for (int32_t i = threadIdx.x; i < total; i += SAL_THREADS, at.next()) {
        const int32_t r = at.r, pc = at.pc;
        float w[8];
        load8g<DT>(A.W, (tc.row0 + r) * A.g.ld + tc.col0 + pc * 8, w);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t key = sal_key(w[j], scol[pc * 8 + j]);
            if (level == 0 || (key >> (shift + bits)) == prefix) atomicAdd(&lhist[(key >> shift) & dmask], 1u);
        }
    }
    __syncthreads();
    uint32_t* __restrict__ gh = A.hist + ((size_t)level * (size_t)A.g.U + (size_t)tc.u) * FEAT_BINS;
    for (int32_t b = threadIdx.x; b < nbins; b += SAL_THREADS) {
        const uint32_t v = lhist[b];
        if (v != 0) atomicAdd(&gh[b], v);
    }
}

// Per tile of a unit whose ties are split (some protected, some not: only then does their order
// matter): how many keys equal the threshold.
template <int DT>
__device__ __forceinline__ void sal_count_tile(const SalArgs& A, const TileCoord& tc, const SalFound& f, float* scol, uint32_t* sh) {
    if (f.rank <= 1u) return;
    const int32_t G = A.g.chunk_w;
    for (int32_t c = threadIdx.x; c < G; c += SAL_THREADS) scol[c] = A.s[tc.col0 + c];
    const uint32_t T = f.prefix;
    __syncthreads();
    const int32_t pieces = G >> 3;
    const int32_t total = tc.nrows * pieces;
    uint32_t eq = 0;
    PieceWalk at((int32_t)threadIdx.x, SAL_THREADS, pieces);
    for (int32_t i = threadIdx.x; i < total; i += SAL_THREADS, at.next()) {
        const int32_t r = at.r, pc = at.pc;
        float w[8];
        load8g<DT>(A.W, (tc.row0 + r) * A.g.ld + tc.col0 + pc * 8, w);
#pragma unroll
        for (int j = 0; j < 8; ++j) eq += sal_key(w[j], scol[pc * 8 + j]) == T ? 1u : 0u;
    }
    eq = block_sum_u32(eq, sh);
    if (threadIdx.x == 0) A.cnt[(size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)tc.t] = eq;
}

// Exclusive prefix sum over a workgroup, in thread order (all SAL_THREADS threads call it);
// *total receives the sum.  T: u32 or u64 (two or four counts side by side).
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* sh, T* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T t = __shfl_up(inc, d, 64);
        if (lane >= d) inc += t;
    }
    __syncthreads();
    if (lane == 63) sh[wave] = inc;
    __syncthreads();
    T excl = inc - v, tot = 0;
    for (int w = 0; w < SAL_THREADS / 64; ++w) {
        if (w < wave) excl += sh[w];
        tot += sh[w];
    }
    *total = tot;
    return excl;
}

// Per tile: the protection bits.  A thread takes eight consecutive columns of a row, i.e. one
// byte of the mask, straight from HBM; threads walk the tile in flat-index order.  Where the
// unit's ties are split, a tie is protected when its rank among the unit's ties, in flat-index
// order, is below `need`: ties in earlier tiles, plus a scan over the workgroup's threads, plus
// the thread's own eight in order.  Elsewhere every tie is protected and nothing is ranked.
template <int DT>
__device__ __forceinline__ void sal_mask_tile(const SalArgs& A, const TileCoord& tc, const SalFound& f, float* scol, uint32_t* sh) {
    const int32_t G = A.g.chunk_w;
    for (int32_t c = threadIdx.x; c < G; c += SAL_THREADS) scol[c] = A.s[tc.col0 + c];
    const uint32_t T = f.prefix;
    const uint32_t need = f.in_bin - f.rank + 1u;
    const bool split = f.rank > 1u;
    uint32_t carry = 0;
    if (split) {
        for (int64_t i = threadIdx.x; i < tc.t; i += SAL_THREADS) carry += A.cnt[(size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)i];
        carry = block_sum_u32(carry, sh);
    }
    __syncthreads();
    const int32_t pieces = G >> 3;
    const int32_t total = tc.nrows * pieces;
    PieceWalk at((int32_t)threadIdx.x, SAL_THREADS, pieces);
    for (int32_t i0 = 0; i0 < total; i0 += SAL_THREADS, at.next()) {
        const int32_t i = i0 + threadIdx.x;
        const bool valid = i < total;
        const int32_t r = at.r, pc = at.pc;
        uint32_t key[8];
        uint32_t eq = 0;
        if (valid) {
            float w[8];
            load8g<DT>(A.W, (tc.row0 + r) * A.g.ld + tc.col0 + pc * 8, w);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                key[j] = sal_key(w[j], scol[pc * 8 + j]);
                eq += key[j] == T ? 1u : 0u;
            }
        }
        uint32_t byte = 0;
        if (split) {                                   // uniform over the workgroup
            uint32_t tot;
            uint32_t tie_rank = carry + block_exclusive_scan(eq, sh, &tot);
            carry += tot;
            if (valid) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    bool prot = key[j] > T;
                    if (key[j] == T) {
                        prot = tie_rank < need;
                        ++tie_rank;
                    }
                    byte |= (prot ? 1u : 0u) << j;
                }
            }
        } else if (valid) {
#pragma unroll
            for (int j = 0; j < 8; ++j) byte |= (key[j] >= T ? 1u : 0u) << j;
        }
        if (valid) A.mask[(tc.row0 + r) * A.mask_ld + (tc.col0 >> 3) + pc] = (uint8_t)byte;
    }
}

// The digits, the tie counts and the masks of the units that do not select from a list: a
// fixed grid walks the tiles of the listed ("flagged") units of every matrix of the launch; with
// none flagged it returns at once.
constexpr int SAL_FLAGGED_GRID = 1024;
constexpr int SAL_WHAT_HIST = 0, SAL_WHAT_COUNT = 1, SAL_WHAT_MASK = 2;
template <int DT, int WHAT>
__global__ __launch_bounds__(SAL_THREADS) void sal_flagged_kernel(const SalBatch B, const int level) {
    if (*B.any_flagged == 0u) return;
    __shared__ uint32_t lhist[WHAT == SAL_WHAT_HIST ? FEAT_BINS : 1];
    __shared__ float scol[WINDQ_MAX_CHUNK];
    __shared__ uint32_t sh[SAL_THREADS / 64], sh_part[SAL_THREADS / 64], sh_out[2];
    for (int mi = 0; mi < B.n; ++mi) {
        const SalArgs& A = B.m[mi];
        // a run of tiles to each workgroup, so that it comes to few units
        const int64_t items = (int64_t)*A.n_flagged * A.g.tiles_per_unit, run = (items + gridDim.x - 1) / gridDim.x;
        const int64_t last = (blockIdx.x + 1) * run < items ? (blockIdx.x + 1) * run : items;
        SalFound found = {0u, 0u, 0u};
        int64_t unit = -1;
        for (int64_t it = blockIdx.x * run; it < last; ++it) {
            const int64_t f = it / A.g.tiles_per_unit;
            const TileCoord tc = tile_coord_of_unit(A.g, (int64_t)A.flagged[f], it - f * A.g.tiles_per_unit);
            if (tc.u != unit) {
                unit = tc.u;
                if (WHAT == SAL_WHAT_MASK) found = {A.lo[unit], A.hi[unit], A.mid[unit]};
                else found = sal_step(A, unit, WHAT == SAL_WHAT_HIST ? level : 3, tc.t == 0, sh_part, sh_out);
            }
            if (WHAT == SAL_WHAT_HIST && level < 2 && tc.t == 0) sal_clear_hist<SAL_THREADS>(A, unit, level + 1);
            __syncthreads();        // the previous tile's shared state is no longer read
            if (WHAT == SAL_WHAT_HIST) sal_hist_tile<DT>(A, tc, level, found.prefix, lhist, scol);
            else if (WHAT == SAL_WHAT_COUNT) sal_count_tile<DT>(A, tc, found, scol, sh);
            else sal_mask_tile<DT>(A, tc, found, scol, sh);
        }
    }
}

// ------------------------------------------------- selection from the unit's candidate list
// The bin (of nbins, a multiple of 64 up to FEAT_BINS) of a histogram in LDS that holds the 1-based ascending rank, and
// the count below it, by one wavefront: a lane adds a run of bins (starting each at its own bank), the lanes of the
// run that holds the rank then take a bin each.
__device__ __forceinline__ void wave_select_bin(const uint32_t* __restrict__ h, int nbins, uint32_t rank, uint32_t* bin, uint32_t* below) {
    const int lane = threadIdx.x & 63, run = nbins >> 6;
    uint32_t sum = 0u;
    for (int j = 0; j < run; ++j) sum += h[lane * run + ((j + lane) % run)];
    uint32_t inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t v = __shfl_up(inc, d, 64);
        if (lane >= d) inc += v;
    }
    const uint64_t reached = __ballot(inc >= rank);
    const int at = reached != 0ull ? __ffsll((unsigned long long)reached) - 1 : 63;
    uint32_t base = __shfl(inc - sum, at, 64);
    const uint32_t own = lane < run ? h[at * run + lane] : 0u;
    uint32_t in = own;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t v = __shfl_up(in, d, 64);
        if (lane >= d) in += v;
    }
    const uint64_t hit = __ballot(lane < run && base + in >= rank);
    const int b = hit != 0ull ? __ffsll((unsigned long long)hit) - 1 : run - 1;
    *bin = (uint32_t)(at * run + b);
    *below = base + __shfl(in - own, b, 64);
}

// bits = 2 bits + (key >= limit): a compare into the carry and an add with carry, where the compiler makes a
// compare, a select, a shift and an or of the same in C.
__device__ __forceinline__ void push_ge(uint32_t& bits, uint32_t key, uint32_t limit) {
    asm("v_cmp_le_u32_e32 vcc, %2, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(key), "s"(limit) : "vcc");
}

// The bracket, from a sample of the unit: all of it up to 32768 weights (then the bracket is the 128th of an octave that
// holds T, and no count can refute it); of a larger one 32768 in SAL_SEG_BYTES segments of as many rows as that gives, evenly
// spread, neighbouring sampled rows in neighbouring columns.  With p_s protected weights expected in the sample
// the bracket reaches from rank p_s + d to p_s - d,
//     d = 4 standard deviations of the sample's count + 2, and no more than the list can take,
// to a 128th of an octave: 1 % of a 524288-weight unit at a 3 % rate.  The deviation is that of the counts of segments in the same
// columns: where rows differ in norm their weights rise above T together, and the count deviates by more than
// independent weights would (by half for a log-normal spread of 0.8).  The margin decides nothing but how often a
// unit has to be selected the long way; whether the bracket holds is counted.
constexpr int SAL_BIG = 1024;               // threads of the per-unit kernels
constexpr int SAL_SAMPLE_LOG = 12, SAL_SAMPLE_PIECES = 1 << SAL_SAMPLE_LOG;     // most 8-weight pieces a unit's sample holds
constexpr int SAL_SEG_BYTES = 64;
constexpr float SAL_MARGIN = 4.0f;          // standard deviations
template <int DT>
__global__ __launch_bounds__(SAL_BIG) void sal_sample_kernel(const SalBatch B) {
    __shared__ uint32_t lh[FEAT_BINS];
    __shared__ uint32_t sh_bin[3], sh_below[3], sh_dev;
    __shared__ float scol[WINDQ_MAX_CHUNK];
    const int mi = batch_index(B.unit_start, B.n, blockIdx.x);
    const SalArgs& A = B.m[mi];
    const int64_t u = (int64_t)blockIdx.x - B.unit_start[mi];
    if (threadIdx.x == 0) {
        A.count[u] = 0ull;
        A.flag[u] = A.use_list != 0u ? 0u : 1u;
        if (u == 0) *A.n_flagged = 0u;
        if (u == 0 && mi == 0) *B.any_flagged = 0u;
    }
    if (A.use_list == 0u) return;
    const int32_t G = A.g.chunk_w;
    const int32_t pieces = G >> 3;
    const int64_t rb = u / A.g.n_chunks;
    const int64_t col0 = (u - rb * A.g.n_chunks) * G;
    const bool whole = A.g.R_u * pieces <= SAL_SAMPLE_PIECES;
    const int32_t total = whole ? (int32_t)A.g.R_u * pieces : SAL_SAMPLE_PIECES;
    for (int32_t b = threadIdx.x; b < FEAT_BINS; b += SAL_BIG) lh[b] = 0u;
    for (int32_t c = threadIdx.x; c < G; c += SAL_BIG) scol[c] = A.s[col0 + c];
    if (threadIdx.x == 0) sh_dev = 0u;
    constexpr int PER = SAL_SAMPLE_PIECES / SAL_BIG;
    uint32_t key[PER][8];
    Raw8<DT> raw[PER];
    int32_t pc[PER];
    // segments of 1 << seg_log pieces, n_pos to a row, 1 << n_seg_log of them in the sample
    constexpr int SEG_MAX = SAL_SEG_BYTES / (8 * Elem<DT>::bytes);
    const int seg_log = min(31 - __builtin_clz(SEG_MAX), (int)__builtin_ctz(pieces)), n_seg_log = SAL_SAMPLE_LOG - seg_log;
    if (whole) {
        PieceWalk at((int32_t)threadIdx.x, SAL_BIG, pieces);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            pc[k] = at.pc;
            if (k * SAL_BIG + (int32_t)threadIdx.x < total) raw[k] = load8raw<DT>(A.W, (rb * A.g.R_u + at.r) * A.g.ld + col0 + at.pc * 8);
            at.next();
        }
    } else {
        const uint32_t n_pos = (uint32_t)pieces >> seg_log, in_seg = threadIdx.x & ((1u << seg_log) - 1u);
        const bool pow2 = (n_pos & (n_pos - 1u)) == 0u;
        const uint32_t seg0 = threadIdx.x >> seg_log, seg_step = (uint32_t)SAL_BIG >> seg_log;       // four steps are the sample
        const bool spread = A.g.R_u >= (int64_t)1 << n_seg_log;
        int64_t x = (int64_t)seg0 * A.g.R_u + (A.g.R_u >> 1);
        const int64_t x_step = (int64_t)seg_step * A.g.R_u;
#pragma unroll
        for (int k = 0; k < PER; ++k, x += x_step) {
            uint32_t at = seg0 + k * seg_step;
            int64_t r = x >> n_seg_log;
            if (!spread) {                                 // fewer rows than segments: several of a row, in different columns
                const uint32_t turn = at / (uint32_t)A.g.R_u;
                r = (int64_t)(at - turn * (uint32_t)A.g.R_u);
                at = (uint32_t)r + turn;
            }
            pc[k] = (int32_t)(((pow2 ? at & (n_pos - 1u) : at % n_pos) << seg_log) + in_seg);
            raw[k] = load8raw<DT>(A.W, (rb * A.g.R_u + r) * A.g.ld + col0 + pc[k] * 8);
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (k * SAL_BIG + (int32_t)threadIdx.x < total) {
            float w[8];
            unpack8raw<DT>(raw[k], w);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                key[k][j] = sal_key(w[j], scol[pc[k] * 8 + j]);
                atomicAdd(&lh[key[k][j] >> 20], 1u);
            }
        }
    }
    __syncthreads();
    // ranks from the top, 1-based, of the bracket's ends (fp32 is exact for a unit sampled whole)
    const float n_s = (float)total * 8.0f;
    const float f = whole ? 1.0f : n_s / ((float)A.g.R_u * (float)G), p_s = (float)A.n_p * f;
    const uint32_t ns = (uint32_t)total * 8u;
    const int wave = threadIdx.x >> 6;
    float d = 0.0f;
    bool open = false;
    uint32_t bin = 0, below = 0, rank = 0;
    // (the first three wavefronts look for one of them each)
    const auto find = [&]() {
        open = wave == 0 ? p_s + d >= n_s : (wave == 1 && p_s - d < 1.0f);
        const float place = wave == 0 ? p_s + d : (wave == 1 ? p_s - d : (p_s < 1.0f ? 1.0f : p_s));
        rank = open ? (wave == 0 ? 1u : ns) : ns - (uint32_t)place + 1u;      // ascending
        wave_select_bin(lh, FEAT_BINS, rank, &bin, &below);
        if ((threadIdx.x & 63) == 0) {
            sh_bin[wave] = bin;
            sh_below[wave] = below;
        }
    };
    const float var = p_s * (1.0f - p_s / n_s), most = 0.43f * (float)A.cap * f - 2.0f;
    if (!whole) d = fminf(SAL_MARGIN * sqrtf(var * (1.0f - f)) + 2.0f, most);
    if (wave < 3) find();
    __syncthreads();
    if (!whole) {
        // how far the number of keys from the middle bin upwards deviates: by two of the four segments that a thread's pieces
        // belong to, which are of the same columns, or nearly (n_pos divides the distance between them where it is a power of two)
        constexpr int K = 2;
        const uint32_t from = __builtin_amdgcn_readfirstlane(sh_bin[2] << 20);
        uint32_t sum = 0u, sq = 0u;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            uint32_t bits = 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) push_ge(bits, key[k][j], from);
            uint32_t c = (uint32_t)__builtin_popcount(bits);
            for (int m = 1; m < 1 << seg_log; m <<= 1) c += __shfl_xor(c, m, 64);
            sum += c;
            sq += c * c;
        }
        uint32_t dev = (threadIdx.x & ((1u << seg_log) - 1u)) == 0u ? K * sq - sum * sum : 0u;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) dev += __shfl_xor(dev, m, 64);
        if ((threadIdx.x & 63) == 0) atomicAdd(&sh_dev, dev);
        __syncthreads();
        const float seen = (float)sh_dev * PER / (K * (K - 1));
        if (seen > 1.2f * var) {                           // the same for all threads
            d = fminf(SAL_MARGIN * sqrtf(seen * (1.0f - f)) + 2.0f, most);
            if (wave < 2) find();
            __syncthreads();
        }
    }
    // the next four bits of the keys from the lowest of the three bins to the highest
    const uint32_t first = sh_bin[0], below0 = sh_below[0];
    const uint32_t span = (sh_bin[1] - first + 1u) * 16u;
    const bool narrow = span <= FEAT_BINS;                                                // else: sixteen octaves wide
    for (int32_t b = threadIdx.x; b < FEAT_BINS; b += SAL_BIG) lh[b] = 0u;
    __syncthreads();
    if (narrow) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int32_t i = k * SAL_BIG + (int32_t)threadIdx.x;
            if (i < total) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t q = (key[k][j] >> 16) - (first << 4);
                    if (q < span) atomicAdd(&lh[q], 1u);
                }
            }
        }
    }
    __syncthreads();
    if (wave < 3) {
        uint32_t q = (bin - first) << 4, lower = 0u;
        if (narrow) wave_select_bin(lh, FEAT_BINS, rank - below0, &q, &lower);
        const uint32_t start = ((first << 4) + q) << 16;                                  // of the 128th of an octave that holds the rank
        if ((threadIdx.x & 63) == 0) {
            if (wave == 0) A.lo[u] = open ? 0u : start;
            else if (wave == 1) A.hi[u] = open ? 0x80000000u : start + (narrow ? 0x10000u : 0x100000u);      // above every key where open
            else A.mid[u] = start;
            sh_below[wave] = open ? (wave == 0 ? 0u : ns) : below0 + lower + (wave == 1 && narrow ? lh[q] : 0u);       // keys below the end
        }
    }
    __syncthreads();
    // a bracket that holds clearly more of the sample than the list does of the unit (many equal keys): not tried
    if (threadIdx.x == 0 && narrow && (float)(sh_below[1] - sh_below[0]) > 1.25f * (float)A.cap * f) A.flag[u] = 1u;
}

// The pass over W: the mask (inside the bracket as if T were `mid`), the counts, the list.  Bound by vector issue (18.5 lane-slots per
// weight, 3.9 TB/s where a large copy reaches 5.1): per weight one multiply and two pushes of a bit.  A workgroup takes 256 rows of a unit and no wavefront waits for another in its loop: candidates go
// into the workgroup's LDS in any order (the list has none), and are moved to the unit's list with ONE global atomic at
// the end.  (With a scan, a global atomic and two barriers per 64-row tile the pass took 157 us per 7B-shaped block.)  A workgroup
// takes at most 32768 weights, and so has room for twice the share of them that the unit's list holds: one that needs more flags
// its unit for the digit passes and stops.  (Past the buffer with an atomic per weight, 4096 x 4096 of equal weights took 1.7 ms.)
constexpr int SAL_CAND_ITERS = 4;       // pieces of 8 weights that a thread has in flight: more take registers from the other wavefronts
// Tiles per workgroup: fewer than four where that leaves less than two workgroups per CU (512 x 512 fp32 at chunk 64, whole
// columns: the selection takes 26.4 us, 29.1 in the 16 workgroups of four tiles)
constexpr int SAL_CAND_TILES = 4;
constexpr int64_t SAL_CAND_WGS = 512;
constexpr uint32_t SAL_CAND_BUF = 2048; // candidates the LDS holds
// FIXED: a thread's pieces all lie in the same columns (the pieces of a row divide the workgroup), its scales stay in registers
template <int DT, bool FIXED>
__global__ __launch_bounds__(SAL_THREADS) void sal_cand_kernel(const SalBatch B) {
    __shared__ __align__(16) float scol[WINDQ_MAX_CHUNK];
    __shared__ uint2 buf[SAL_CAND_BUF];
    __shared__ uint32_t sh[SAL_THREADS / 64];
    __shared__ uint32_t n_buf, base, skip, full;
    const int mi = batch_index(B.band_start, B.n, blockIdx.x);
    const SalArgs& A = B.m[mi];
    // chunks side by side, then row ranges, then row blocks
    const uint32_t idx = (uint32_t)((int64_t)blockIdx.x - B.band_start[mi]), nc = (uint32_t)A.g.n_chunks;
    const uint32_t ranges = ((uint32_t)A.g.tiles_per_unit + (uint32_t)B.cand_tiles - 1u) / (uint32_t)B.cand_tiles;
    const uint32_t band = idx / nc, j0 = idx - band * nc;
    const uint32_t rb = band / ranges, rr = band - rb * ranges;
    const int64_t u = (int64_t)rb * nc + j0;
    const int32_t most = B.cand_tiles * TILE_ROWS;
    const int64_t lrow0 = (int64_t)rr * most, row0 = (int64_t)rb * A.g.R_u + lrow0;
    const int64_t left = A.g.R_u - lrow0;
    const int32_t nrows = left < most ? (int32_t)left : most;
    const int32_t G = A.g.chunk_w;
    const int64_t col0 = (int64_t)j0 * G;
    const int32_t pieces = G >> 3;
    for (int32_t c = threadIdx.x; c < G; c += SAL_THREADS) scol[c] = A.s[col0 + c];
    if (threadIdx.x == 0) {
        n_buf = 0u;
        skip = A.flag[u];
        full = 0u;
    }
    const uint32_t lo = A.lo[u], hi = A.hi[u], mid = A.mid[u];
    uint2* __restrict__ list = A.cand + (size_t)u * (size_t)A.cap;
    const int32_t total = nrows * pieces;
    PieceWalk walk((int32_t)threadIdx.x, SAL_THREADS, pieces);
    __syncthreads();
    if (skip != 0u) return;
    volatile uint32_t* stop = &full;
    float sc[8];
    if (FIXED) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sc[j] = scol[walk.pc * 8 + j];
    }
    constexpr int NB = SAL_CAND_ITERS;
    uint32_t n_above = 0u;
    for (int32_t i0 = threadIdx.x; i0 < total && *stop == 0u; i0 += NB * SAL_THREADS) {
        Raw8<DT> raw[NB];                       // kept as loaded: the keys of a candidate piece are formed again
        int32_t rk[NB], pk[NB];                 // row and piece of each
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            rk[k] = walk.r;
            pk[k] = walk.pc;
            walk.next();
            if (i0 + k * SAL_THREADS < total) raw[k] = load8raw<DT>(A.W, (row0 + rk[k]) * A.g.ld + col0 + pk[k] * 8);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (i0 + k * SAL_THREADS >= total) break;
            float w[8];
            unpack8raw<DT>(raw[k], w);
            if (!FIXED) {
#pragma unroll
                for (int j = 0; j < 8; ++j) sc[j] = scol[pk[k] * 8 + j];
            }
            uint32_t above = 0u, in = 0u;
#pragma unroll
            for (int j = 7; j >= 0; --j) {
                const uint32_t key = sal_key(w[j], sc[j]);
                push_ge(above, key, hi);
                push_ge(in, key, lo);
            }
            n_above += (uint32_t)__builtin_popcount(above);
            in ^= above;
            if (in != 0u) {
                const uint32_t pos0 = (uint32_t)(lrow0 + rk[k]) * (uint32_t)G + (uint32_t)pk[k] * 8u;
                uint32_t at = atomicAdd(&n_buf, (uint32_t)__builtin_popcount(in));
                for (uint32_t m = in; m != 0u; m &= m - 1u, ++at) {        // usually one bit
                    const int j = __ffs(m) - 1;
                    const uint2 e = make_uint2(sal_key(raw_elem<DT, false>(raw[k], j), scol[pk[k] * 8 + j]), pos0 + (uint32_t)j);
                    above |= (e.x >= mid ? 1u : 0u) << j;
                    if (at < SAL_CAND_BUF) buf[at] = e;
                    else *stop = 1u;
                }
            }
            A.mask[(row0 + rk[k]) * A.mask_ld + (col0 >> 3) + pk[k]] = (uint8_t)above;
        }
    }
    n_above = block_sum_u32(n_above, sh);       // (and a barrier: the buffer is complete)
    const uint32_t n = n_buf;
    if (n > SAL_CAND_BUF) {                     // the same for all threads
        if (threadIdx.x == 0) A.flag[u] = 1u;
        return;
    }
    if (threadIdx.x == 0 && (n | n_above) != 0u)
        base = (uint32_t)atomicAdd(reinterpret_cast<unsigned long long*>(&A.count[u]), ((unsigned long long)n_above << 32) | n);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += SAL_THREADS)
        if (base + i < A.cap) list[base + i] = buf[i];
}

// The bin of 1-based ascending rank `rank` among the list's entries that satisfy pred, by `value`; returns the bin,
// the count below it and the bin's own count.  All SAL_BIG threads call it.
template <typename Value, typename Pred>
__device__ __forceinline__ void list_digit(const uint2* __restrict__ list, uint32_t n, int bits, uint32_t rank, Value value, Pred pred,
                                           uint32_t* lh, uint32_t* sh_part, uint32_t* sh_out, uint32_t* bin, uint32_t* below,
                                           uint32_t* in_bin) {
    const int32_t nbins = 1 << bits;
    __syncthreads();
    for (int32_t b = threadIdx.x; b < nbins; b += SAL_BIG) lh[b] = 0u;
    __syncthreads();
    for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 4 * SAL_BIG) {       // four loads in flight per thread
        uint2 e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i0 + k * SAL_BIG < n) e[k] = list[i0 + k * SAL_BIG];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i0 + k * SAL_BIG < n && pred(e[k])) atomicAdd(&lh[value(e[k]) & (uint32_t)(nbins - 1)], 1u);
    }
    __syncthreads();
    uint64_t bl;
    select_bin<SAL_BIG>(lh, nbins, rank, sh_part, sh_out, bin, &bl);
    *below = (uint32_t)bl;
    *in_bin = lh[*bin];
}

// Corrects the mask bit of a listed weight where the pass over W guessed it wrong.  (Setting the bit of every protected
// weight on the list, half of them, took 35 us per 7B-shaped block: scattered atomics run at about 34 a nanosecond.)
__device__ __forceinline__ void settle(const SalArgs& A, int64_t rb, int64_t col0, uint32_t mid, const uint2& e, bool prot) {
    if (prot == (e.x >= mid)) return;
    const uint32_t G = (uint32_t)A.g.chunk_w;
    const uint32_t r = e.y / G, c = e.y - r * G;
    const int64_t byte = (rb * A.g.R_u + (int64_t)r) * A.mask_ld + ((col0 + (int64_t)c) >> 3);
    atomicXor(reinterpret_cast<uint32_t*>(A.mask + (byte & ~(int64_t)3)), 1u << (8u * (uint32_t)(byte & 3) + (c & 7u)));
}

// Per unit: does the bracket hold the threshold, and the list the bracket?  If not, the unit is flagged.  If so: the
// threshold's bin among 2048 over the bracket's width, by one pass over the list; a second settles the mask bits of the
// weights outside that bin and gathers the bin's own, a handful, which are ranked one against another (key, then flat
// position).  A bin of more than SAL_BIN weights (ties) is resolved digit by digit instead: the threshold, then, where
// ties are split, the last position taken, by three digits of the position (ranking a thousand ties one against another
// took this kernel 60 to 90 us, digits 12 to 29).
constexpr uint32_t SAL_BIN = 128;
__global__ __launch_bounds__(SAL_BIG) void sal_list_kernel(const SalBatch B) {
    __shared__ uint32_t lh[FEAT_BINS];
    __shared__ uint2 own[SAL_BIN];
    __shared__ uint32_t n_own;
    __shared__ uint32_t sh_part[SAL_BIG / 64];
    __shared__ uint32_t sh_out[2];
    const int mi = batch_index(B.unit_start, B.n, blockIdx.x);
    const SalArgs& A = B.m[mi];
    const int64_t u = (int64_t)blockIdx.x - B.unit_start[mi];
    const uint64_t count = A.count[u];
    const uint32_t n = (uint32_t)count, above = (uint32_t)(count >> 32);
    if (A.flag[u] != 0u || n > A.cap || above > A.n_p || A.n_p - above > n) {
        sal_clear_hist<SAL_BIG>(A, u, 0);
        if (threadIdx.x == 0) {
            const uint32_t at = atomicAdd(A.n_flagged, 1u);
            A.flagged[at] = (uint32_t)u;
            if (at == 0u) atomicAdd(B.any_flagged, 1u);
        }
        return;
    }
    const uint32_t take = A.n_p - above;                  // of the listed weights
    const uint2* __restrict__ list = A.cand + (size_t)u * (size_t)A.cap;
    const uint32_t lo = A.lo[u], width = A.hi[u] - 1u - lo, mid = A.mid[u];
    const int64_t rb = u / A.g.n_chunks;
    const int64_t col0 = (u - rb * A.g.n_chunks) * A.g.chunk_w;
    if (take == 0u) {
        for (uint32_t i = threadIdx.x; i < n; i += SAL_BIG) settle(A, rb, col0, mid, list[i], false);
        return;
    }
    uint32_t left = n - take + 1u, prefix = 0u, ties = n, below, bin;
    if (threadIdx.x == 0) n_own = 0u;
    for (int rem = width == 0u ? 0 : 32 - __builtin_clz(width); rem > 0;) {
        const int bits = rem < FEAT_DIGIT_BITS ? rem : FEAT_DIGIT_BITS, shift = rem - bits;
        list_digit(list, n, bits, left, [=](const uint2& e) { return (e.x - lo) >> shift; },
                   [=](const uint2& e) { return rem == 32 || ((e.x - lo) >> rem) == prefix; }, lh, sh_part, sh_out, &bin, &below, &ties);
        prefix = (prefix << bits) | bin;
        left -= below;
        rem = shift;
        if (ties > SAL_BIN) continue;
        // `ties` weights share the digits found so far; the last ties - left + 1 of them are protected, and so is all above
        for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 4 * SAL_BIG) {
            uint2 e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i0 + k * SAL_BIG < n) e[k] = list[i0 + k * SAL_BIG];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (i0 + k * SAL_BIG >= n) continue;
                const uint32_t d = (e[k].x - lo) >> shift;
                if (d == prefix) own[atomicAdd(&n_own, 1u)] = e[k];
                else settle(A, rb, col0, mid, e[k], d > prefix);
            }
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < ties; i += SAL_BIG) {
            uint32_t ahead = 0u;
            for (uint32_t q = 0; q < ties; ++q) ahead += own[q].x > own[i].x || (own[q].x == own[i].x && own[q].y < own[i].y) ? 1u : 0u;
            settle(A, rb, col0, mid, own[i], ahead < ties - left + 1u);
        }
        return;
    }
    const uint32_t T = lo + prefix;
    const uint32_t need = ties - left + 1u;              // the rank left over counts the ties that stay unprotected, plus one
    uint32_t pos_max = 0xffffffffu;                        // ties up to this position are protected
    if (need < ties) {
        // the need-th smallest position among the ties (positions are distinct): digits of 11, 11, 10 bits
        uint32_t p1, p2, p3, bl, in_bin;
        list_digit(list, n, 11, need, [](const uint2& e) { return e.y >> 21; }, [=](const uint2& e) { return e.x == T; }, lh, sh_part,
                   sh_out, &p1, &bl, &in_bin);
        const uint32_t n1 = need - bl;
        list_digit(list, n, 11, n1, [](const uint2& e) { return e.y >> 10; }, [=](const uint2& e) { return e.x == T && (e.y >> 21) == p1; },
                   lh, sh_part, sh_out, &p2, &bl, &in_bin);
        const uint32_t n2 = n1 - bl;
        list_digit(list, n, 10, n2, [](const uint2& e) { return e.y; },
                   [=](const uint2& e) { return e.x == T && (e.y >> 10) == ((p1 << 11) | p2); }, lh, sh_part, sh_out, &p3, &bl, &in_bin);
        pos_max = (p1 << 21) | (p2 << 10) | p3;
    }
    for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 4 * SAL_BIG) {
        uint2 e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i0 + k * SAL_BIG < n) e[k] = list[i0 + k * SAL_BIG];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i0 + k * SAL_BIG < n) settle(A, rb, col0, mid, e[k], e[k].x > T || (e[k].x == T && e[k].y <= pos_max));
    }
}

// ---------------------------------------------------------------------------- encode
// INT8 codes need the unit's largest protected weight first.  The first kernel therefore collects a tile's
// protected weights (value and column, in flat-index order) in the tile's part of the candidate area, so that the
// second, which knows the scale, need not fetch them from W again: at 3 % they touch most of W's 64-byte
// sectors.  A tile with more of them than its part holds is collected from W a second time, as is every tile
// of a mask that was not made by select at a rate the area is for.
template <int DT>
struct SalPart {                // of one tile
    uint16_t* col;
    uint16_t* w16;              // bf16
    float* w32;                 // fp32
    uint32_t cap;
};
template <int DT>
__device__ __forceinline__ SalPart<DT> sal_part(const SalArgs& A, const TileCoord& tc) {
    const uint64_t bytes = ((uint64_t)A.cap * sizeof(uint2) / (uint64_t)A.g.tiles_per_unit) & ~(uint64_t)15;
    char* p = reinterpret_cast<char*>(A.cand + (size_t)tc.u * (size_t)A.cap) + (uint64_t)tc.t * bytes;
    SalPart<DT> s;
    s.cap = (uint32_t)(bytes / (2 + Elem<DT>::bytes)) & ~1u;
    s.w32 = reinterpret_cast<float*>(p);
    s.w16 = reinterpret_cast<uint16_t*>(p);
    s.col = reinterpret_cast<uint16_t*>(p + (uint64_t)s.cap * Elem<DT>::bytes);
    return s;
}

// The tile of a wavefront: a workgroup's four take four neighbouring tiles, each by itself.
__device__ __forceinline__ bool sal_wave_tile(const SalBatch& B, int* mi, int64_t* tile) {
    const int64_t t = (int64_t)blockIdx.x * (SAL_THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (t >= B.tile_start[B.n]) return false;
    *mi = batch_index(B.tile_start, B.n, t);
    *tile = t - B.tile_start[*mi];
    return true;
}

// Calls f(index, column, weight) for the protected weights of a wavefront's tile; index counts them in flat order.  A lane
// takes 8 columns at a time, four such pieces in flight, and reads of W only the pieces that hold one.  Returns their number.
constexpr int SAL_ENC_ITERS = 4;
template <int DT, typename F>
__device__ __forceinline__ uint32_t for_protected(const SalArgs& A, const TileCoord& tc, F f) {
    const int lane = threadIdx.x & 63;
    const int32_t pieces = A.g.chunk_w >> 3;
    const int32_t total = tc.nrows * pieces;
    const uint8_t* __restrict__ mask = A.mask + tc.row0 * A.mask_ld + (tc.col0 >> 3);
    PieceWalk walk(lane, 64, pieces);
    uint32_t before = 0;
    for (int32_t i0 = 0; i0 < total; i0 += SAL_ENC_ITERS * 64) {
        uint32_t m[SAL_ENC_ITERS];
        int32_t rk[SAL_ENC_ITERS], pk[SAL_ENC_ITERS];
        Raw8<DT> raw[SAL_ENC_ITERS];
#pragma unroll
        for (int k = 0; k < SAL_ENC_ITERS; ++k) {
            rk[k] = walk.r;
            pk[k] = walk.pc;
            walk.next();
            m[k] = i0 + k * 64 + lane < total ? mask[rk[k] * A.mask_ld + pk[k]] : 0u;
        }
#pragma unroll
        for (int k = 0; k < SAL_ENC_ITERS; ++k)
            if (m[k] != 0u) raw[k] = load8raw<DT>(A.W, (tc.row0 + rk[k]) * A.g.ld + tc.col0 + pk[k] * 8);
#pragma unroll
        for (int h = 0; h < SAL_ENC_ITERS; h += 4) {
            uint64_t mine = 0;                  // 16 bits per round of four: at most 512 weights each
#pragma unroll
            for (int k = 0; k < 4; ++k) mine |= (uint64_t)__builtin_popcount(m[h + k]) << (16 * k);
            uint64_t inc = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint64_t v = __shfl_up(inc, d, 64);
                if (lane >= d) inc += v;
            }
            const uint64_t tot = __shfl(inc, 63, 64);
            const uint64_t excl = inc - mine;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t at = before + (uint32_t)((excl >> (16 * k)) & 0xffffu);
                for (uint32_t b = m[h + k]; b != 0u; b &= b - 1u) {
                    const int j = __ffs(b) - 1;
                    f(at++, pk[h + k] * 8 + j, raw_elem<DT, true>(raw[h + k], j));
                }
                before += (uint32_t)((tot >> (16 * k)) & 0xffffu);
            }
        }
    }
    return before;
}

// Per tile: its protected weights collected, their number, the largest magnitude.
template <int DT>
__global__ __launch_bounds__(SAL_THREADS) void sal_collect_kernel(const SalBatch B) {
    int mi;
    int64_t tile;
    if (!sal_wave_tile(B, &mi, &tile)) return;
    const SalArgs& A = B.m[mi];
    const TileCoord tc = tile_coord(A.g, tile);
    const SalPart<DT> part = sal_part<DT>(A, tc);
    float mx = 0.0f;
    const uint32_t n = for_protected<DT>(A, tc, [&](uint32_t at, int32_t c, float w) {
        mx = fmaxf(mx, fabsf(w));
        if (at < part.cap) {
            part.col[at] = (uint16_t)c;
            if (DT == WINDQ_BF16) part.w16[at] = (uint16_t)(__float_as_uint(w) >> 16);
            else part.w32[at] = w;
        }
    });
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
    if ((threadIdx.x & 63) == 0) {
        const size_t at = (size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)tc.t;
        A.tile_max[at] = mx;
        A.cnt[at] = n;
    }
}

// Per unit: the INT8 scale, and the tiles' counts turned into those of all earlier tiles.
__global__ __launch_bounds__(SAL_THREADS) void sal_unit_kernel(const SalBatch B) {
    __shared__ uint32_t sh[SAL_THREADS / 64];
    __shared__ float shm[SAL_THREADS / 64];
    const int mi = batch_index(B.unit_start, B.n, blockIdx.x);
    const SalArgs& A = B.m[mi];
    const int64_t u = (int64_t)blockIdx.x - B.unit_start[mi];
    const int64_t T = A.g.tiles_per_unit;
    const size_t base = (size_t)u * (size_t)T;
    float mx = 0.0f;
    uint32_t carry = 0;
    for (int64_t t0 = 0; t0 < T; t0 += SAL_THREADS) {
        const int64_t t = t0 + threadIdx.x;
        if (t < T) mx = fmaxf(mx, A.tile_max[base + (size_t)t]);
        const uint32_t n = t < T ? A.cnt[base + (size_t)t] : 0u;
        uint32_t tot;
        const uint32_t excl = block_exclusive_scan(n, sh, &tot);
        if (t < T) A.cnt[base + (size_t)t] = carry + excl;
        carry += tot;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
    if ((threadIdx.x & 63) == 0) shm[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < SAL_THREADS / 64; ++w) mx = fmaxf(mx, shm[w]);
        float sg = mx / 127.0f;
        if (!(sg >= FLT_MIN)) sg = 0.0f;
        A.prot_scale[u] = sg;
        A.count[u] = carry;                    // the unit's protected weights
    }
}

// Per tile: INT8 codes of the protected weights at their place in the unit's stream, and the
// activation-weighted error of the tile's INT8 part.
template <int DT>
__global__ __launch_bounds__(SAL_THREADS) void sal_encode_kernel(const SalBatch B) {
    int mi;
    int64_t tile;
    if (!sal_wave_tile(B, &mi, &tile)) return;
    const SalArgs& A = B.m[mi];
    const TileCoord tc = tile_coord(A.g, tile);
    const size_t slot = (size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)tc.t;
    const uint32_t first = A.cnt[slot];
    const uint32_t end = tc.t + 1 < A.g.tiles_per_unit ? A.cnt[slot + 1] : (uint32_t)A.count[tc.u];
    const float sg = A.prot_scale[tc.u];
    const float inv = sg > 0.0f ? 1.0f / sg : 0.0f;
    const float* __restrict__ s = A.s + tc.col0;
    int8_t* __restrict__ dst = A.prot_codes + (size_t)tc.u * (size_t)A.n_p;
    const SalPart<DT> part = sal_part<DT>(A, tc);
    double err = 0.0;
    auto encode = [&](uint32_t at, int32_t c, float w) {
        const float t = w * inv;
        const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(t), -127.0f, 127.0f);
        if (first + at < A.n_p) dst[first + at] = (int8_t)(int32_t)q;     // a mask with more bits than n_p writes nothing past the unit
        const double d = (double)w - (double)q * (double)sg;
        const double a = (double)s[c] * (double)s[c];
        err = fma(a * d, d, err);
    };
    const uint32_t n = end - first;
    if (n <= part.cap) {
#pragma unroll 4
        for (uint32_t at = threadIdx.x & 63; at < n; at += 64)
            encode(at, part.col[at], DT == WINDQ_BF16 ? bf16_bits_to_f32(part.w16[at]) : part.w32[at]);
    } else {
        for_protected<DT>(A, tc, encode);
    }
    err = wave_sum(err);
    if ((threadIdx.x & 63) == 0) A.err_part[slot] = err;
}

__global__ __launch_bounds__(256) void sal_err_kernel(const SalBatch B) {
    __shared__ double red[4];
    const int mi = batch_index(B.unit_start, B.n, blockIdx.x);
    const SalArgs& A = B.m[mi];
    const int64_t u = (int64_t)blockIdx.x - B.unit_start[mi];
    const double e = unit_partial_sum<256>(A.err_part + (size_t)u * (size_t)A.g.tiles_per_unit, A.g.tiles_per_unit, red);
    if (threadIdx.x == 0) A.err_prot[u] = (float)e;
}

// ------------------------------------------------------------------- unit saliency
// Saliency score of a unit (App. "Comparison with Heuristic Sensitivity Allocator"): the mean
// of |w| * |s_c| over the unit.  Per tile an fp64 sum in a fixed order, per unit the tiles in order.
template <int DT>
__global__ __launch_bounds__(SAL_THREADS) void unit_saliency_tile_kernel(const void* __restrict__ W, const float* __restrict__ s,
                                                                         const Geometry g, double* __restrict__ part) {
    __shared__ float scol[WINDQ_MAX_CHUNK];
    __shared__ double red[SAL_THREADS / 64];
    const TileCoord tc = tile_coord(g, blockIdx.x);
    const int32_t G = g.chunk_w;
    for (int32_t c = threadIdx.x; c < G; c += SAL_THREADS) scol[c] = fabsf(s[tc.col0 + c]);
    __syncthreads();
    const int32_t pieces = G >> 3;
    const int32_t total = tc.nrows * pieces;
    double acc = 0.0;
    PieceWalk at((int32_t)threadIdx.x, SAL_THREADS, pieces);
    for (int32_t i = threadIdx.x; i < total; i += SAL_THREADS, at.next()) {
        const int32_t r = at.r, pc = at.pc;
        float w[8];
        load8g<DT>(W, (tc.row0 + r) * g.ld + tc.col0 + pc * 8, w);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc = fma((double)fabsf(w[j]), (double)scol[pc * 8 + j], acc);
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < SAL_THREADS / 64; ++w) t += red[w];
        part[(size_t)tc.u * (size_t)g.tiles_per_unit + (size_t)tc.t] = t;
    }
}

__global__ __launch_bounds__(256) void unit_saliency_finalize_kernel(const double* __restrict__ part, const Geometry g,
                                                                    float* __restrict__ sal) {
    __shared__ double red[4];
    const int64_t u = blockIdx.x;
    const double t = unit_partial_sum<256>(part + (size_t)u * (size_t)g.tiles_per_unit, g.tiles_per_unit, red);
    if (threadIdx.x == 0) sal[u] = (float)(t / ((double)g.R_u * (double)g.chunk_w));
}

static void carve(SalArgs& A, void* ws, const SalientLayout& L) {
    char* base = static_cast<char*>(ws);
    A.hist = reinterpret_cast<uint32_t*>(base + L.hist);
    A.lo = reinterpret_cast<uint32_t*>(base + L.lo);
    A.hi = reinterpret_cast<uint32_t*>(base + L.hi);
    A.mid = reinterpret_cast<uint32_t*>(base + L.mid);
    A.count = reinterpret_cast<uint64_t*>(base + L.count);
    A.cnt = reinterpret_cast<uint32_t*>(base + L.cnt);
    A.flag = reinterpret_cast<uint32_t*>(base + L.flag);
    A.n_flagged = reinterpret_cast<uint32_t*>(base + L.n_flagged);
    A.flagged = reinterpret_cast<uint32_t*>(base + L.flagged);
    A.cand = reinterpret_cast<uint2*>(base + L.cand);
    A.cap = L.cap;
    A.tile_max = reinterpret_cast<float*>(base + L.tile_max);
    A.err_part = reinterpret_cast<double*>(base + L.err_part);
}

template <int DT>
static int launch_select(const SalBatch& B, hipStream_t hs) {
    const dim3 units((unsigned)B.unit_start[B.n]), some(SAL_FLAGGED_GRID);
    // units that select from their candidate list ...
    hipLaunchKernelGGL(sal_sample_kernel<DT>, units, dim3(SAL_BIG), 0, hs, B);
    const dim3 bands((unsigned)B.band_start[B.n]);
    if (SAL_THREADS % (B.m[0].g.chunk_w >> 3) == 0) hipLaunchKernelGGL((sal_cand_kernel<DT, true>), bands, dim3(SAL_THREADS), 0, hs, B);
    else hipLaunchKernelGGL((sal_cand_kernel<DT, false>), bands, dim3(SAL_THREADS), 0, hs, B);
    hipLaunchKernelGGL(sal_list_kernel, units, dim3(SAL_BIG), 0, hs, B);
    // ... and the others
    for (int level = 0; level < 3; ++level)
        hipLaunchKernelGGL((sal_flagged_kernel<DT, SAL_WHAT_HIST>), some, dim3(SAL_THREADS), 0, hs, B, level);
    hipLaunchKernelGGL((sal_flagged_kernel<DT, SAL_WHAT_COUNT>), some, dim3(SAL_THREADS), 0, hs, B, 0);
    hipLaunchKernelGGL((sal_flagged_kernel<DT, SAL_WHAT_MASK>), some, dim3(SAL_THREADS), 0, hs, B, 0);
    return hipPeekAtLastError() == hipSuccess ? WINDQ_OK : WINDQ_EHIP;
}

template <int DT>
static int launch_encode(const SalBatch& B, hipStream_t hs) {
    const dim3 tiles((unsigned)((B.tile_start[B.n] + SAL_THREADS / 64 - 1) / (SAL_THREADS / 64))), units((unsigned)B.unit_start[B.n]);
    hipLaunchKernelGGL(sal_collect_kernel<DT>, tiles, dim3(SAL_THREADS), 0, hs, B);
    hipLaunchKernelGGL(sal_unit_kernel, units, dim3(SAL_THREADS), 0, hs, B);
    hipLaunchKernelGGL(sal_encode_kernel<DT>, tiles, dim3(SAL_THREADS), 0, hs, B);
    hipLaunchKernelGGL(sal_err_kernel, units, dim3(256), 0, hs, B);
    return hipPeekAtLastError() == hipSuccess ? WINDQ_OK : WINDQ_EHIP;
}

}  // namespace windq

using namespace windq;

extern "C" int64_t windq_n_protected(int64_t n_unit, uint32_t rate_ppm) {
    if (n_unit < 0 || rate_ppm > 1000000u) return -1;
    // n * rate fits 64 bits for every n the kernels accept (n < 2^32)
    return (int64_t)(((unsigned __int128)(uint64_t)n_unit * rate_ppm) / 1000000u);
}

static int salient_common(const windq_mat* W, const float* s, int32_t chunk_w, int64_t unit_rows, uint32_t rate_ppm,
                          const uint8_t* mask, void* ws, size_t ws_bytes, SalArgs* A) {
    if (W == nullptr) return WINDQ_EINVAL;
    const int st = make_geometry(W, chunk_w, unit_rows, &A->g);
    if (st != WINDQ_OK) return st;
    if (s == nullptr || mask == nullptr || rate_ppm > 1000000u) return WINDQ_EINVAL;
    if ((uint64_t)A->g.R_u * (uint64_t)chunk_w > (uint64_t)0xffffffffu) return WINDQ_ESHAPE;   // u32 counts
    const SalientLayout L = salient_layout(A->g);
    if (ws == nullptr || ws_bytes < L.total || !aligned(ws, 256)) return WINDQ_EWORKSPACE;
    A->W = W->data;
    A->s = s;
    A->mask = const_cast<uint8_t*>(mask);
    A->mask_ld = W->cols / 8;
    const uint64_t n = (uint64_t)A->g.R_u * (uint64_t)chunk_w;
    A->n_p = (uint32_t)windq_n_protected((int64_t)n, rate_ppm);
    A->rank0 = (uint32_t)(n - A->n_p + 1);
    // the list route sets mask bits with 32-bit atomics: the mask has to be addressable in whole dwords
    A->use_list = aligned(mask, 4) && ((uint64_t)W->rows * (uint64_t)A->mask_ld) % 4 == 0 ? 1u : 0u;
    A->prot_codes = nullptr;
    A->prot_scale = nullptr;
    A->err_prot = nullptr;
    carve(*A, ws, L);
    return WINDQ_OK;
}

// Numbers the tiles and units of the first B->n matrices.  unit_threads: the most a kernel of the call gives a unit.
static int salient_number(SalBatch* B, int unit_threads) {
    int64_t tiles = 0, units = 0, bands;
    for (int32_t i = 0; i <= WINDQ_MAX_BATCH; ++i) {
        B->tile_start[i] = tiles;
        B->unit_start[i] = units;
        if (i < B->n) {
            tiles += B->m[i].g.n_tiles;
            units += B->m[i].g.U;
        }
    }
    const int32_t wide = 32768 / (TILE_ROWS * B->m[0].g.chunk_w);
    B->cand_tiles = 2 * (wide < SAL_CAND_TILES ? wide : SAL_CAND_TILES);
    do {
        B->cand_tiles /= 2;
        bands = 0;
        for (int32_t i = 0; i <= WINDQ_MAX_BATCH; ++i) {
            B->band_start[i] = bands;
            if (i < B->n) bands += B->m[i].g.U * ((B->m[i].g.tiles_per_unit + B->cand_tiles - 1) / B->cand_tiles);
        }
    } while (B->cand_tiles > 1 && bands < SAL_CAND_WGS);
    for (int32_t i = B->n; i < WINDQ_MAX_BATCH; ++i) B->m[i] = B->m[0];
    B->any_flagged = B->m[0].n_flagged + 1;       // in the 256 bytes of the first matrix's own count
    return fits_launch(units, unit_threads) && fits_launch(bands, SAL_THREADS) && fits_launch(tiles, 64) ? WINDQ_OK : WINDQ_ESHAPE;
}

static int salient_select_launch(const windq_salient_item* items, int32_t n, int32_t chunk_w, int64_t unit_rows,
                                 uint32_t rate_ppm, void* stream) {
    if (items == nullptr || n < 1 || n > WINDQ_MAX_BATCH) return WINDQ_EINVAL;
    SalBatch B;
    B.n = 0;
    const uint8_t* empty[WINDQ_MAX_BATCH];      // masks of matrices whose units protect nothing
    int64_t empty_bytes[WINDQ_MAX_BATCH];
    int32_t n_empty = 0;
    for (int32_t i = 0; i < n; ++i) {
        SalArgs& A = B.m[B.n];
        const int st = salient_common(items[i].W, items[i].s, chunk_w, unit_rows, rate_ppm, items[i].mask, items[i].ws,
                                      items[i].ws_bytes, &A);
        if (st != WINDQ_OK) return st;
        if (items[i].W->dtype != items[0].W->dtype) return WINDQ_EINVAL;      // one kernel per launch
        if (A.n_p == 0) {
            if (!fits_launch((items[i].W->rows * A.mask_ld + 255) / 256, 256)) return WINDQ_ESHAPE;
            empty[n_empty] = items[i].mask;
            empty_bytes[n_empty++] = items[i].W->rows * A.mask_ld;
        } else {
            ++B.n;
        }
    }
    if (B.n > 0) {
        const int st = salient_number(&B, SAL_BIG);
        if (st != WINDQ_OK) return st;
    }
    hipStream_t hs = static_cast<hipStream_t>(stream);
    for (int32_t i = 0; i < n_empty; ++i)
        hipLaunchKernelGGL(sal_clear_mask_kernel, dim3((unsigned)((empty_bytes[i] + 255) / 256)), dim3(256), 0, hs,
                           const_cast<uint8_t*>(empty[i]), empty_bytes[i]);
    if (B.n == 0) return hipPeekAtLastError() == hipSuccess ? WINDQ_OK : WINDQ_EHIP;
    const int32_t dtype = items[0].W->dtype;
    return dtype == WINDQ_BF16 ? launch_select<WINDQ_BF16>(B, hs) : launch_select<WINDQ_F32>(B, hs);
}

static int salient_encode_launch(const windq_salient_item* items, int32_t n, int32_t chunk_w, int64_t unit_rows,
                                 uint32_t rate_ppm, void* stream) {
    if (items == nullptr || n < 1 || n > WINDQ_MAX_BATCH) return WINDQ_EINVAL;
    SalBatch B;
    B.n = n;
    for (int32_t i = 0; i < n; ++i) {
        SalArgs& A = B.m[i];
        const int st = salient_common(items[i].W, items[i].s, chunk_w, unit_rows, rate_ppm, items[i].mask, items[i].ws,
                                      items[i].ws_bytes, &A);
        if (st != WINDQ_OK) return st;
        if (items[i].W->dtype != items[0].W->dtype) return WINDQ_EINVAL;
        if (items[i].prot_scale == nullptr || items[i].err_prot == nullptr) return WINDQ_EINVAL;
        if (items[i].prot_codes == nullptr && A.n_p != 0) return WINDQ_EINVAL;
        A.prot_codes = items[i].prot_codes;
        A.prot_scale = items[i].prot_scale;
        A.err_prot = items[i].err_prot;
    }
    const int st = salient_number(&B, SAL_THREADS);
    if (st != WINDQ_OK) return st;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const int32_t dtype = items[0].W->dtype;
    return dtype == WINDQ_BF16 ? launch_encode<WINDQ_BF16>(B, hs) : launch_encode<WINDQ_F32>(B, hs);
}

extern "C" int windq_salient_select(const windq_mat* W, const float* s, int32_t chunk_w, int64_t unit_rows,
                                    uint32_t rate_ppm, uint8_t* mask, void* ws, size_t ws_bytes, void* stream) {
    const windq_salient_item it = {W, s, mask, nullptr, nullptr, nullptr, ws, ws_bytes};
    return salient_select_launch(&it, 1, chunk_w, unit_rows, rate_ppm, stream);
}

extern "C" int windq_salient_select_batch(const windq_salient_item* items, int32_t n, int32_t chunk_w, int64_t unit_rows,
                                          uint32_t rate_ppm, void* stream) {
    return salient_select_launch(items, n, chunk_w, unit_rows, rate_ppm, stream);
}

extern "C" int windq_salient_encode(const windq_mat* W, const float* s, int32_t chunk_w, int64_t unit_rows,
                                    const uint8_t* mask, uint32_t rate_ppm, int8_t* prot_codes, float* prot_scale,
                                    float* err_prot, void* ws, size_t ws_bytes, void* stream) {
    const windq_salient_item it = {W, s, const_cast<uint8_t*>(mask), prot_codes, prot_scale, err_prot, ws, ws_bytes};
    return salient_encode_launch(&it, 1, chunk_w, unit_rows, rate_ppm, stream);
}

extern "C" int windq_salient_encode_batch(const windq_salient_item* items, int32_t n, int32_t chunk_w, int64_t unit_rows,
                                          uint32_t rate_ppm, void* stream) {
    return salient_encode_launch(items, n, chunk_w, unit_rows, rate_ppm, stream);
}

extern "C" int windq_unit_saliency(const windq_mat* W, const float* s, int32_t chunk_w, int64_t unit_rows, float* sal,
                                   void* ws, size_t ws_bytes, void* stream) {
    Geometry g;
    const int st = make_geometry(W, chunk_w, unit_rows, &g);
    if (st != WINDQ_OK) return st;
    if (s == nullptr || sal == nullptr) return WINDQ_EINVAL;
    if (ws == nullptr || ws_bytes < unit_saliency_ws_bytes(g) || !aligned(ws, 256)) return WINDQ_EWORKSPACE;
    double* part = static_cast<double*>(ws);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    if (!fits_launch(g.n_tiles, SAL_THREADS)) return WINDQ_ESHAPE;
    const dim3 tiles((unsigned)g.n_tiles);
    if (W->dtype == WINDQ_BF16)
        hipLaunchKernelGGL(unit_saliency_tile_kernel<WINDQ_BF16>, tiles, dim3(SAL_THREADS), 0, hs, W->data, s, g, part);
    else
        hipLaunchKernelGGL(unit_saliency_tile_kernel<WINDQ_F32>, tiles, dim3(SAL_THREADS), 0, hs, W->data, s, g, part);
    hipLaunchKernelGGL(unit_saliency_finalize_kernel, dim3((unsigned)g.U), dim3(256), 0, hs, part, g, sal);
    return hipPeekAtLastError() == hipSuccess ? WINDQ_OK : WINDQ_EHIP;
}
