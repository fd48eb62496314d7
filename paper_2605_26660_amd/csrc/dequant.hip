// windq_dequant_plan: the way back from the packed artefact.  Unpacks the codes of a plan,
// reconstructs every weight from the stored per-group scale and offset, and recomputes the
// activation-weighted reconstruction error per unit from the artefact alone: the same number
// windq_fit_score_all_bits reported for the plan's bit-width and clip index (Sec. 3.5 scores a
// fit by its reconstruction error; this closes the loop codes -> error), and the first piece of
// a path that serves the quantized weights.
//   uniform:  w_hat = offset + code * scale     ternary: scale * (trit - 1)     binary: +-scale
// Errors use w_hat in fp64 from the stored fp32 numbers, as the fit does; the optional fp32
// output is one fused multiply-add.  Reads 2 bytes per weight plus the codes.
// Two kernels.  Chunk widths of 8 x 2^k columns: a lane owns eight columns of a row, i.e. one
// 16-byte piece of W, one mask byte, `bits` bytes of codes (ternary: the two or three bytes
// its eight trits sit in), and G/8 neighbouring lanes cover a row with contiguous loads
// straight from HBM; a workgroup walks the 64 rows of a tile, each lane keeping the fp64
// weights s_c^2 of its columns.  Other widths, and buffers off those alignments: the same
// pieces, numbered through the tile, a thread's columns found per piece.
#include "windq_common.hpp"
#include "windq_order.hpp"
#include "windq_ws.hpp"

namespace windq {

struct DequantArgs {
    const void* W;
    const float* s;
    const uint8_t* mask;       // or null
    int64_t mask_ld;
    const uint8_t* action;
    const int64_t* code_off;
    const uint8_t* codes;
    int64_t codes_bytes;
    const float* scale;
    const float* offset;
    Geometry g;
    float* what;               // [rows][what_ld] or null
    int64_t what_ld;
    double* part;              // [n_tiles] or [n_tiles][passes]
    float* err;                // [U] or null
    int64_t per_unit;          // partials per unit
    // matrix-vector product from the artefact (the GEMV kernels), else unused
    const float* x;            // [cols]
    float* y;                  // [rows]
    double* gpart;             // [n_chunks][rows]  a row's partial product over each chunk
};

// A launch covers up to WINDQ_MAX_BATCH matrices (one chunk width, one element type): their
// tiles and units are numbered one matrix after the other.
struct DequantBatch {
    int32_t n;
    int32_t by_cost;            // the product: workgroups in the order of what their units cost
    int64_t tile_start[WINDQ_MAX_BATCH + 1];
    int64_t unit_start[WINDQ_MAX_BATCH + 1];
    int64_t row_start[WINDQ_MAX_BATCH + 1];
    DequantArgs m[WINDQ_MAX_BATCH];
};

__device__ __forceinline__ int64_t dq_bytes_per_group(int a, int G) {
    switch (a) {
        case 1: return G;
        case 2: return G >> 1;
        case 3: return (G * 3) >> 3;
        case 4: return G >> 2;
        case 5: return (G + 4) / 5;
        case 6: return G >> 3;
        default: return 0;
    }
}

// Eight consecutive weights of a row, straight from global memory.
template <int DT>
__device__ __forceinline__ void load8_global(const void* __restrict__ p, float (&w)[8]) {
    if (DT == WINDQ_BF16) {
        const uint4 raw = *reinterpret_cast<const uint4*>(p);
        w[0] = bf16_bits_to_f32(raw.x & 0xffffu); w[1] = __uint_as_float(raw.x & 0xffff0000u);
        w[2] = bf16_bits_to_f32(raw.y & 0xffffu); w[3] = __uint_as_float(raw.y & 0xffff0000u);
        w[4] = bf16_bits_to_f32(raw.z & 0xffffu); w[5] = __uint_as_float(raw.z & 0xffff0000u);
        w[6] = bf16_bits_to_f32(raw.w & 0xffffu); w[7] = __uint_as_float(raw.w & 0xffff0000u);
    } else {
        const float4 a = reinterpret_cast<const float4*>(p)[0];
        const float4 b = reinterpret_cast<const float4*>(p)[1];
        w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
        w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
    }
}

// Entry threadIdx.x of the table that turns a byte into its five trits, as five 2-bit fields.
__device__ __forceinline__ void fill_trits(uint16_t* __restrict__ trits_of) {
    uint32_t b = threadIdx.x, t = 0;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        t |= (b % 3u) << (2 * i);
        b /= 3u;
    }
    trits_of[threadIdx.x] = (uint16_t)t;
}

// Lanes-per-row kernel: chunk_w = 8 << lpr_shift columns.  A workgroup takes one pass of a
// 64-row tile, the 256 >> lpr_shift rows its threads cover at once: no loop over rows, so all
// of a workgroup's loads are in flight together.
constexpr int DQ_THREADS = 256;
template <int DT>
__global__ __launch_bounds__(DQ_THREADS) void dequant_split_kernel(const DequantBatch B, const int lpr_shift) {
    __shared__ double red[DQ_THREADS / 64];
    const int32_t passes = dequant_passes(8 << lpr_shift);
    const int64_t tile_b = blockIdx.x / passes;                 // tile of the launch
    const int32_t pass = (int32_t)(blockIdx.x - tile_b * passes);
    const int mi = batch_index(B.tile_start, B.n, tile_b);
    const DequantArgs& A = B.m[mi];
    const TileCoord tc = tile_coord(A.g, tile_b - B.tile_start[mi]);
    const int32_t G = A.g.chunk_w;
    constexpr int EB = Elem<DT>::bytes;
    const int sub = threadIdx.x & ((1 << lpr_shift) - 1);      // which 8 columns of the row
    const int rsub = threadIdx.x >> lpr_shift;                 // which row of a pass
    const int rows_per_pass = DQ_THREADS >> lpr_shift;
    const int32_t c = sub * 8;

    int a = A.action[tc.u];
    if (a >= WINDQ_N_ACTIONS) a = 0;
    const int64_t bpg = dq_bytes_per_group(a, G);
    const int64_t base = A.code_off[tc.u];
    if (base < 0 || (base & 15) != 0 || base > A.codes_bytes - bpg * A.g.R_u) a = 0;   // a malformed entry reads nothing; base + bytes could pass 2^63
    const int bits = a == 1 ? 8 : (a == 2 ? 4 : (a == 3 ? 3 : (a == 4 ? 2 : 1)));

    double ac[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const double sv = (double)A.s[tc.col0 + c + j];
        ac[j] = sv * sv;
    }
    // ternary: a byte's five trits as five 2-bit fields, from a table the workgroup fills once
    __shared__ uint16_t trits_of[256];
    if (a == 5) {
        fill_trits(trits_of);
        __syncthreads();
    }

    double acc = 0.0;
    {
        const int32_t r = pass * rows_per_pass + rsub;
        if (r < tc.nrows && r < TILE_ROWS) {
            const int64_t row = tc.row0 + r;
            const int64_t gidx = tc.u * A.g.R_u + tc.lrow0 + r;
            float w[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            load8_global<DT>(static_cast<const char*>(A.W) + (row * A.g.ld + tc.col0 + c) * EB, w);
            const uint32_t m = A.mask != nullptr ? A.mask[row * A.mask_ld + (tc.col0 >> 3) + sub] : 0u;
            float* __restrict__ orow = A.what != nullptr ? A.what + row * A.what_ld + tc.col0 + c : nullptr;
            float wh[8];
            if (a == 0) {
#pragma unroll
                for (int j = 0; j < 8; ++j) wh[j] = w[j];                     // a skip unit keeps its weights
            } else {
                const float sc = A.scale[gidx];
                const float of = A.offset[gidx];
                const uint8_t* __restrict__ src = A.codes + base + (tc.lrow0 + r) * bpg;
                double whd[8];
                if (a == 5) {
                    // eight trits, five to a byte: they sit in two or three neighbouring bytes
                    const int32_t b0 = c / 5;
                    const int32_t last = (int32_t)bpg - 1;
                    const uint32_t y0 = src[b0];
                    const uint32_t y1 = src[b0 + 1 <= last ? b0 + 1 : last];
                    const uint32_t y2 = src[b0 + 2 <= last ? b0 + 2 : last];
                    const uint32_t v = ((uint32_t)trits_of[y0] | ((uint32_t)trits_of[y1] << 10) | ((uint32_t)trits_of[y2] << 20)) >>
                                       (2 * (c - 5 * b0));
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        wh[j] = sc * ((float)((v >> (2 * j)) & 3u) - 1.0f);
                        whd[j] = (double)wh[j];
                    }
                } else {
                    // eight codes = `bits` bytes, aligned to their own size (units start on 16 bytes)
                    const uint8_t* p = src + sub * bits;
                    uint64_t v;
                    if (bits == 8) {
                        const uint2 t = *reinterpret_cast<const uint2*>(p);
                        v = (uint64_t)t.x | ((uint64_t)t.y << 32);
                    } else if (bits == 4) {
                        v = *reinterpret_cast<const uint32_t*>(p);
                    } else if (bits == 3) {
                        const uint32_t t0 = p[0], t1 = p[1], t2 = p[2];
                        v = t0 | (t1 << 8) | (t2 << 16);
                    } else if (bits == 2) {
                        v = *reinterpret_cast<const uint16_t*>(p);
                    } else {
                        v = p[0];
                    }
                    if (a == 6) {
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            wh[j] = ((v >> j) & 1u) != 0u ? sc : -sc;
                            whd[j] = (double)wh[j];
                        }
                    } else {
                        const double scd = (double)sc, ofd = (double)of;
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const uint32_t code = (uint32_t)(v >> (j * bits)) & ((1u << bits) - 1u);
                            wh[j] = fmaf((float)code, sc, of);
                            whd[j] = ofd + (double)code * scd;
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool prot = ((m >> j) & 1u) != 0u;              // lives in the INT8 side stream
                    const double d = (double)w[j] - whd[j];
                    acc = fma(prot ? 0.0 : ac[j] * d, d, acc);
                    wh[j] = prot ? 0.0f : wh[j];
                }
            }
            if (orow != nullptr) {
                reinterpret_cast<float4*>(orow)[0] = make_float4(wh[0], wh[1], wh[2], wh[3]);
                reinterpret_cast<float4*>(orow)[1] = make_float4(wh[4], wh[5], wh[6], wh[7]);
            }
        }
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < DQ_THREADS / 64; ++i) t += red[i];
        A.part[((size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)tc.t) * (size_t)passes + (size_t)pass] = t;
    }
}

// Eight columns of row r of a tile: unpacked, reconstructed, written, and their error added to acc.
template <int DT, bool ALIGNED>
__device__ __forceinline__ void dequant_piece(const DequantArgs& A, const TileCoord& tc, int a, int64_t bpg, int64_t base, int32_t r, int32_t sub,
                                              const double (&ac)[8], const uint16_t* __restrict__ trits_of, double* acc) {
    constexpr int EB = Elem<DT>::bytes;
    const int bits = a == 1 ? 8 : (a == 2 ? 4 : (a == 3 ? 3 : (a == 4 ? 2 : 1)));
    const int32_t c = sub * 8;
    const int64_t row = tc.row0 + r;
    const int64_t gidx = tc.u * A.g.R_u + tc.lrow0 + r;
    float w[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    load8_global<DT>(static_cast<const char*>(A.W) + (row * A.g.ld + tc.col0 + c) * EB, w);
    const uint32_t m = A.mask != nullptr ? A.mask[row * A.mask_ld + (tc.col0 >> 3) + sub] : 0u;
    float* __restrict__ orow = A.what != nullptr ? A.what + row * A.what_ld + tc.col0 + c : nullptr;
    float wh[8];
    if (a == 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) wh[j] = w[j];                     // a skip unit keeps its weights
    } else {
        const float sc = A.scale[gidx];
        const float of = A.offset[gidx];
        const uint8_t* __restrict__ src = A.codes + base + (tc.lrow0 + r) * bpg;
        double whd[8];
        if (a == 5) {
            // eight trits, five to a byte: they sit in two or three neighbouring bytes
            const int32_t b0 = c / 5;
            const int32_t last = (int32_t)bpg - 1;
            const uint32_t y0 = src[b0];
            const uint32_t y1 = src[b0 + 1 <= last ? b0 + 1 : last];
            const uint32_t y2 = src[b0 + 2 <= last ? b0 + 2 : last];
            const uint32_t v = ((uint32_t)trits_of[y0] | ((uint32_t)trits_of[y1] << 10) | ((uint32_t)trits_of[y2] << 20)) >>
                               (2 * (c - 5 * b0));
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                wh[j] = sc * ((float)((v >> (2 * j)) & 3u) - 1.0f);
                whd[j] = (double)wh[j];
            }
        } else {
            // eight codes = `bits` bytes, aligned to their own size (units start on 16 bytes)
            const uint8_t* p = src + sub * bits;
            uint64_t v;
            if (!ALIGNED) {
                v = 0;
                for (int b = 0; b < bits; ++b) v |= (uint64_t)p[b] << (8 * b);
            } else if (bits == 8) {
                const uint2 t = *reinterpret_cast<const uint2*>(p);
                v = (uint64_t)t.x | ((uint64_t)t.y << 32);
            } else if (bits == 4) {
                v = *reinterpret_cast<const uint32_t*>(p);
            } else if (bits == 3) {
                const uint32_t t0 = p[0], t1 = p[1], t2 = p[2];
                v = t0 | (t1 << 8) | (t2 << 16);
            } else if (bits == 2) {
                v = *reinterpret_cast<const uint16_t*>(p);
            } else {
                v = p[0];
            }
            if (a == 6) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    wh[j] = ((v >> j) & 1u) != 0u ? sc : -sc;
                    whd[j] = (double)wh[j];
                }
            } else {
                const double scd = (double)sc, ofd = (double)of;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t code = (uint32_t)(v >> (j * bits)) & ((1u << bits) - 1u);
                    wh[j] = fmaf((float)code, sc, of);
                    whd[j] = ofd + (double)code * scd;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool prot = ((m >> j) & 1u) != 0u;              // lives in the INT8 side stream
            const double d = (double)w[j] - whd[j];
            *acc = fma(prot ? 0.0 : ac[j] * d, d, *acc);
            wh[j] = prot ? 0.0f : wh[j];
        }
    }
    if (orow != nullptr) {
        if (ALIGNED) {
            reinterpret_cast<float4*>(orow)[0] = make_float4(wh[0], wh[1], wh[2], wh[3]);
            reinterpret_cast<float4*>(orow)[1] = make_float4(wh[4], wh[5], wh[6], wh[7]);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) orow[j] = wh[j];
        }
    }
}

// Every other case: widths that are not 8 x 2^k columns, w_hat off 16 bytes, codes off 8 (the last two: ALIGNED false).
// A pass is 256 pieces (eight columns of a row each, rows one after the other), one per thread; widths that are no multiple
// of 32 have a last pass of more (dequant_passes rounds down), whose threads take several.  Bound by the chain of waits
// from the unit's action to its codes.  1000 x 1056 fp32 at chunk 96: 6.4 us; a lane per row over a tile in LDS took 41
// (a division per trit, single words stored 96 apart).  Two or four passes per workgroup, with their loads in
// flight together, take 8.1 and 8.8: fewer workgroups.  The kernel above stays for its widths: finding a piece's row and
// columns here costs 10 % there, and even its own body in this function 5 % (7B-shaped block: 308 us against 325 to 341).
template <int DT, bool ALIGNED>
__global__ __launch_bounds__(DQ_THREADS) void dequant_any_kernel(const DequantBatch B, const int32_t chunk_w) {
    __shared__ double red[DQ_THREADS / 64];
    __shared__ uint16_t trits_of[256];
    const int32_t passes = dequant_passes(chunk_w);
    const uint32_t tile_b = blockIdx.x / (uint32_t)passes;      // tile of the launch
    const int32_t pass = (int32_t)(blockIdx.x - tile_b * (uint32_t)passes);
    const int mi = batch_index(B.tile_start, B.n, tile_b);
    const DequantArgs& A = B.m[mi];
    const TileCoord tc = tile_coord(A.g, (int64_t)tile_b - B.tile_start[mi]);
    const int32_t G = chunk_w;
    const int32_t pieces = G >> 3;
    const int32_t total = tc.nrows * pieces;
    const uint32_t inv = ((1u << 20) + (uint32_t)pieces - 1u) / (uint32_t)pieces;     // i / pieces = i * inv >> 20 for i < 64 * pieces

    int a = A.action[tc.u];
    if (a >= WINDQ_N_ACTIONS) a = 0;
    const int64_t bpg = dq_bytes_per_group(a, G);
    const int64_t base = A.code_off[tc.u];
    if (base < 0 || (base & 15) != 0 || base > A.codes_bytes - bpg * A.g.R_u) a = 0;   // a malformed entry reads nothing; base + bytes could pass 2^63
    if (a == 5) {
        fill_trits(trits_of);
        __syncthreads();
    }
    double acc = 0.0;
    for (int32_t i = pass * DQ_THREADS + (int32_t)threadIdx.x; i < total; i += passes * DQ_THREADS) {
        const int32_t r = (int32_t)(((uint32_t)i * inv) >> 20);
        const int32_t sub = i - r * pieces;
        double ac[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const double sv = (double)A.s[tc.col0 + sub * 8 + j];
            ac[j] = sv * sv;
        }
        dequant_piece<DT, ALIGNED>(A, tc, a, bpg, base, r, sub, ac, trits_of, &acc);
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < DQ_THREADS / 64; ++i) t += red[i];
        A.part[((size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)tc.t) * (size_t)passes + (size_t)pass] = t;
    }
}

// err[u] = the sum of unit u's per_unit partials; one workgroup per unit.
__global__ __launch_bounds__(256) void dequant_finalize_kernel(const DequantBatch B) {
    __shared__ double red[4];
    const int mi = batch_index(B.unit_start, B.n, blockIdx.x);
    const DequantArgs& A = B.m[mi];
    if (A.err == nullptr) return;
    const int64_t u = (int64_t)blockIdx.x - B.unit_start[mi];
    const double t = unit_partial_sum<256>(A.part + (size_t)u * (size_t)A.per_unit, A.per_unit, red);
    if (threadIdx.x == 0) A.err[u] = (float)t;
}

// ------------------------------------------------------------- the product from the artefact
// y = W_hat x for one vector.  The codes are a few bits a weight, so what bounds a straightforward kernel
// is not HBM (63 MB for a 7B-shaped block at 2 bits: 12 us) but taking codes apart: extract, convert, two
// multiply-adds per weight.  Units at 1, 1.58 and 2 bits - nearly all of a plan - are looked up instead, several
// weights at a time: for the workgroup's chunk of x a table holds, for every value that a piece of the stream can take,
//     sum_j (code_j - centre) x_j      (centre: 1/2 of a bit's two signs, trit 1, code 1.5)
// The centre keeps the entries as small as the products they stand for; what it leaves out is
// (offset + centre * scale) * sum_c x_c, added once per row in fp64.  Pieces are small on purpose: a nibble
// (four 1-bit or two 2-bit weights; 16 entries), and of a byte of trits the lower three (27 entries) and the upper two (10).
// A wavefront's 64 look-ups into up to 32 consecutive words meet no bank conflict; tables of whole bytes (256
// entries, half the look-ups) do, and take 16 times as long to make: four 4096 x 11008 matrices took 26.0 / 34.5 /
// 36.3 us at 1 / 1.58 / 2 bits with them, 21.3 / 28.3 / 30.1 with the small ones (92 to 98 us with one lane per eight weights).
//   A lane owns a row (its bytes are contiguous, and so are its neighbours': a unit's rows lie one after the
// other).  Tables and sums are fp64: what the centre leaves to (offset + centre * scale) may cancel.
//   The other routes, one weight at a time, same results to rounding: 3, 4 and 8 bits (little to
// share), units under a protection mask, and what infinite or NaN weights would show in: chunks of x that hold a value no
// fp32 sum of a few columns may meet (infinite, NaN or above 2^96), rows whose scale or offset is such a value.  Skip
// units read W, G/8 lanes a row.
//   7B-shaped block at a 2-bit plan: 34 to 38 us by the card (109 with G/8 lanes a row), of which the sums over chunks take 5; with 3 % of the
// weights protected 65 (115).  The six wavefronts per SIMD that 84 registers allow are worth 5 to 10 % over the four
// that the skip route's loads would take.
constexpr int GEMV_THREADS = 256;
// Dear units first (windq_order.hpp) where a launch has four workgroups per CU or more: skipped units and those taken weight by
// weight (8, 4 and 3 bits), then tables of trits and of 2 bits, then of 1 bit.  7B-shaped block at 2 bits 41.9 -> 37.8 us,
// 28672 x 8192 and the others of its block 60 -> 42; the look at the actions costs plans of one width 0.5 to 1.4 us
// (7B-shaped block, 4 bits 41.5 -> 42.2, 2 bits 30.5 -> 31.6, binary 24.2 -> 25.5; asking for x or the action ahead of it, or one wavefront
// looking for all, takes 0.2 of that back and costs mixed plans more), and with 392 workgroups 0.4 of 13.9.
constexpr uint32_t GEMV_CLASSES = (1u << 8) | (1u << 10) | (2u << 12);
constexpr int GEMV_TRIT_WORDS = 48;                 // of a byte of trits: 27 entries at 0, 10 at 32
constexpr size_t GEMV_BOTH_LDS = GEMV_THREADS * sizeof(double) + 256 * sizeof(uint16_t);        // of lanes that share a row, beside the others
// LDS of the largest table, trits of whole dwords (2 bits: 8 entries a column, 1 bit: 4), after the chunk's x.
static size_t gemv_lds(int32_t chunk_w) {
    return (size_t)WINDQ_MAX_CHUNK * sizeof(float) + (size_t)(((chunk_w + 4) / 5 + 3) & ~3) * GEMV_TRIT_WORDS * sizeof(double);
}

// n (1..16) bytes of a row's codes, n the same for all lanes; the rest zero.  Rows start at any byte.
__device__ __forceinline__ void load_code_bytes(const uint8_t* __restrict__ p, int n, uint32_t (&d)[4]) {
    if (n == 16) {
        __builtin_memcpy(d, p, 16);
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        d[i] = 0u;
        if (4 * i + 4 <= n) {
            __builtin_memcpy(&d[i], p + 4 * i, 4);
        } else {
#pragma unroll
            for (int b = 0; b < 3; ++b)
                if (4 * i + b < n) d[i] |= (uint32_t)p[4 * i + b] << (8 * b);
        }
    }
}

// The tables of a chunk, nb bytes a row; pieces up to the end of the row's last dword are cleared.
//   1 bit   nibble n covers columns 4n ..    2 bits   nibble n covers columns 2n, 2n + 1
//   trits   byte k covers columns 5k .. ; columns past the chunk (the last byte) count as zero
__device__ __forceinline__ void gemv_tables(int a, const float* __restrict__ x, int32_t G, int32_t nb, double* __restrict__ tab) {
    const int32_t nb4 = (nb + 3) & ~3;
    if (a == 5) {
        for (int32_t i = threadIdx.x; i < nb4 * GEMV_TRIT_WORDS; i += GEMV_THREADS) {
            const uint32_t k = (uint32_t)i / GEMV_TRIT_WORDS, e = (uint32_t)i - k * GEMV_TRIT_WORDS;
            const uint32_t v = e < 32u ? e : e - 32u;
            const int32_t c = (int32_t)k * 5 + (e < 32u ? 0 : 3);
            double t = 0.0;
            if (c < G) t = ((double)(v % 3u) - 1.0) * (double)x[c];
            if (c + 1 < G) t = fma((double)((v / 3u) % 3u) - 1.0, (double)x[c + 1], t);
            if (e < 32u && c + 2 < G) t = fma((double)((v / 9u) % 3u) - 1.0, (double)x[c + 2], t);
            tab[i] = (int32_t)k < nb ? t : 0.0;
        }
        return;
    }
    for (int32_t i = threadIdx.x; i < nb4 * 32; i += GEMV_THREADS) {
        const int32_t n = i >> 4;
        const uint32_t v = (uint32_t)i & 15u;
        double t = 0.0;
        if (n < 2 * nb) {
            if (a == 6) {
                const float4 q = *reinterpret_cast<const float4*>(x + 4 * n);
                t = ((v & 1u) != 0u ? (double)q.x : -(double)q.x) + ((v & 2u) != 0u ? (double)q.y : -(double)q.y);
                t += ((v & 4u) != 0u ? (double)q.z : -(double)q.z) + ((v & 8u) != 0u ? (double)q.w : -(double)q.w);
            } else {
                t = fma((double)(v & 3u) - 1.5, (double)x[2 * n], ((double)(v >> 2) - 1.5) * (double)x[2 * n + 1]);
            }
        }
        tab[i] = t;
    }
}

// The sum of the entries that up to sixteen bytes select, whose first piece's table is at tab.
__device__ __forceinline__ double gemv_lookup_nibbles(const uint32_t (&d)[4], int n, const double* __restrict__ tab) {
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (4 * i < n) {                                            // the same for all lanes
            const char* __restrict__ t = reinterpret_cast<const char*>(tab + i * 128);
            double e[8];
            e[0] = *reinterpret_cast<const double*>(t + ((d[i] << 3) & 0x78u));
#pragma unroll
            for (int k = 1; k < 8; ++k) e[k] = *reinterpret_cast<const double*>(t + 128 * k + ((d[i] >> (4 * k - 3)) & 0x78u));
            acc += ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
        }
    }
    return acc;
}
__device__ __forceinline__ double gemv_lookup_trits(const uint32_t (&d)[4], int n, const double* __restrict__ tab) {
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (4 * i < n) {
            const char* __restrict__ t = reinterpret_cast<const char*>(tab + i * 4 * GEMV_TRIT_WORDS);
            double e[8];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t v = (d[i] >> (8 * k)) & 0xffu;
                const uint32_t q = (v * 607u) >> 14;                // v / 27 for v < 256
                const uint32_t r = v - q * 27u;
                e[2 * k] = *reinterpret_cast<const double*>(t + 8 * GEMV_TRIT_WORDS * k + 8 * r);
                e[2 * k + 1] = *reinterpret_cast<const double*>(t + 8 * GEMV_TRIT_WORDS * k + 256 + 8 * q);
            }
            acc += ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
        }
    }
    return acc;
}

// The reconstruction of eight columns from c (a multiple of 8) of a row: `bits` bytes of its codes at any
// alignment, or the two or three bytes that hold eight trits (trits_of: fill_trits' table).
__device__ __forceinline__ void decode8(int a, int bits, const uint8_t* __restrict__ src, int32_t c, int32_t bpg, float sc,
                                        float of, const uint16_t* __restrict__ trits_of, float (&wh)[8]) {
    if (a == 5) {
        const int32_t b0 = c / 5, last = bpg - 1;
        const uint32_t y0 = src[b0];
        const uint32_t y1 = src[b0 + 1 <= last ? b0 + 1 : last];
        const uint32_t y2 = src[b0 + 2 <= last ? b0 + 2 : last];
        const uint32_t v = ((uint32_t)trits_of[y0] | ((uint32_t)trits_of[y1] << 10) | ((uint32_t)trits_of[y2] << 20)) >> (2 * (c - 5 * b0));
#pragma unroll
        for (int j = 0; j < 8; ++j) wh[j] = sc * ((float)((v >> (2 * j)) & 3u) - 1.0f);
        return;
    }
    uint64_t v = 0;
    const uint8_t* p = src + (c >> 3) * bits;
    if (bits == 8) {
        __builtin_memcpy(&v, p, 8);
    } else if (bits == 4) {
        __builtin_memcpy(&v, p, 4);
    } else if (bits == 3) {
        v = (uint64_t)((uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16));
    } else if (bits == 2) {
        __builtin_memcpy(&v, p, 2);
    } else {
        v = p[0];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t code = (uint32_t)(v >> (j * bits)) & ((1u << bits) - 1u);
        wh[j] = a == 6 ? (code != 0u ? sc : -sc) : fmaf((float)code, sc, of);
    }
}

// The product of a row at 2 bits, 1.58 or 1 bit with the chunk of x, weight by weight, without tables.
__device__ __forceinline__ double gemv_row_plain(int a, const uint8_t* __restrict__ src, int32_t G, float sc, float of,
                                                 const float* __restrict__ xs) {
    double acc = 0.0;
#pragma unroll 1
    for (int32_t c = 0; c < G; c += 8) {
        float dot = 0.0f;
#pragma unroll 1
        for (int32_t i = c; i < c + 8; ++i) {
            float wh;
            if (a == 5) {
                uint32_t v = src[i / 5];
                for (int k = i % 5; k > 0; --k) v /= 3u;
                wh = sc * ((float)(v % 3u) - 1.0f);
            } else if (a == 4) {
                wh = fmaf((float)((src[i >> 2] >> (2 * (i & 3))) & 3), sc, of);
            } else {
                wh = ((src[i >> 3] >> (i & 7)) & 1) != 0 ? sc : -sc;
            }
            dot = fmaf(wh, xs[i], dot);
        }
        acc += (double)dot;
    }
    return acc;
}

// The products of N rows with the chunk of x one weight at a time: the values windq_dequant_plan reconstructs, eight
// columns in fp32 in column order, those runs in fp64.  32 columns (4 BITS bytes of codes) of every
// row per step, the next step's on their way meanwhile; the mask 128 columns at a time: a lane's row of it is a line of the
// cache of its own, gone before four narrower loads have met it (7B-shaped block, mixed plan: 74 us, 138 in dwords).
template <int BITS, bool MASKED, int N>
__device__ __forceinline__ void gemv_rows(const uint8_t* const (&src)[N], const uint8_t* const (&mrow)[N], int32_t G,
                                          const float (&sc)[N], const float (&of)[N], const float* __restrict__ xs, double (&acc)[N]) {
    const int32_t G32 = G & ~31;
    uint32_t d[N][BITS], m[N][4];
    auto fetch = [&](int32_t c, uint32_t (&dd)[N][BITS]) {
#pragma unroll
        for (int k = 0; k < N; ++k) __builtin_memcpy(dd[k], src[k] + (c >> 3) * BITS, 4 * BITS);
    };
    if (G32 > 0) fetch(0, d);
#pragma unroll 1
    for (int32_t c = 0; c < G32; c += 32) {
        if (MASKED) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                if ((c & 127) == 0) {
                    load_code_bytes(mrow[k] + (c >> 3), (G - c) >> 3 < 16 ? (G - c) >> 3 : 16, m[k]);
                } else {
                    m[k][0] = m[k][1]; m[k][1] = m[k][2]; m[k][2] = m[k][3];
                }
            }
        }
        uint32_t dn[N][BITS];
        fetch(c + 32 < G32 ? c + 32 : c, dn);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = xs[c + 8 * q + j];
#pragma unroll
            for (int k = 0; k < N; ++k) {
                float dot = 0.0f;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int bit = (8 * q + j) * BITS, w = bit >> 5, sft = bit & 31;
                    uint32_t code = d[k][w] >> sft;
                    if (sft + BITS > 32) code |= d[k][w + 1 < BITS ? w + 1 : w] << (32 - sft);
                    code &= (1u << BITS) - 1u;
                    float wh = BITS == 1 ? (code != 0u ? sc[k] : -sc[k]) : fmaf((float)code, sc[k], of[k]);
                    if (MASKED) wh = ((m[k][0] >> (8 * q + j)) & 1u) != 0u ? 0.0f : wh;
                    dot = fmaf(wh, x[j], dot);
                }
                acc[k] += (double)dot;
            }
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
#pragma unroll
            for (int i = 0; i < BITS; ++i) d[k][i] = dn[k][i];
        }
    }
    for (int32_t c = G32; c < G; c += 8) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            float wh[8], dot = 0.0f;
            decode8(BITS == 1 ? 6 : 1, BITS, src[k], c, 0, sc[k], of[k], nullptr, wh);
            const uint32_t mb = MASKED ? mrow[k][c >> 3] : 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) dot = fmaf(((mb >> j) & 1u) != 0u ? 0.0f : wh[j], xs[c + j], dot);
            acc[k] += (double)dot;
        }
    }
}

template <bool MASKED, int N>
__device__ __forceinline__ void gemv_rows_of(int a, const uint8_t* const (&src)[N], const uint8_t* const (&mrow)[N],
                                             int32_t G, int32_t bpg, const float (&sc)[N], const float (&of)[N],
                                             const float* __restrict__ xs, const uint16_t* __restrict__ trits_of, double (&acc)[N]) {
    switch (a) {
        case 1: return gemv_rows<8, MASKED>(src, mrow, G, sc, of, xs, acc);
        case 2: return gemv_rows<4, MASKED>(src, mrow, G, sc, of, xs, acc);
        case 3: return gemv_rows<3, MASKED>(src, mrow, G, sc, of, xs, acc);
        case 4: return gemv_rows<2, MASKED>(src, mrow, G, sc, of, xs, acc);
        case 6: return gemv_rows<1, MASKED>(src, mrow, G, sc, of, xs, acc);
        default: break;                                                // trits
    }
    uint32_t m[N][4];
#pragma unroll 1
    for (int32_t c = 0; c < G; c += 8) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if (MASKED && (c & 127) == 0) load_code_bytes(mrow[k] + (c >> 3), (G - c) >> 3 < 16 ? (G - c) >> 3 : 16, m[k]);
            float wh[8], dot = 0.0f;
            decode8(5, 0, src[k], c, bpg, sc[k], of[k], trits_of, wh);
#pragma unroll
            for (int i = 0; i < 8; ++i) dot = fmaf(MASKED && ((m[k][0] >> i) & 1u) != 0u ? 0.0f : wh[i], xs[c + i], dot);
            acc[k] += (double)dot;
            if (MASKED) {
                m[k][0] = (m[k][0] >> 8) | (m[k][1] << 24); m[k][1] = (m[k][1] >> 8) | (m[k][2] << 24);
                m[k][2] = (m[k][2] >> 8) | (m[k][3] << 24); m[k][3] >>= 8;
            }
        }
    }
}

// RPT rows per thread: a workgroup takes RPT * 256 rows of a unit.  Where that leaves the chip short of workgroups, several
// (1 << parts_shift) are launched for each: they share the rows of a skip unit, all but the first leave any other at once.
// MASKED: matrices with a protection mask, in launches of their own (compiled into one kernel the two spilled registers:
// 7B-shaped block under a mask 180 us against 138).
template <int DT, int RPT, bool MASKED>
__device__ __forceinline__ void gemv_rows_wg(const DequantBatch& B, const uint32_t wgs, const int parts_shift, char* __restrict__ smem,
                                             double* __restrict__ red) {
    float* xs = reinterpret_cast<float*>(smem);
    double* tab = reinterpret_cast<double*>(smem + WINDQ_MAX_CHUNK * sizeof(float));
    constexpr int nt = RPT * GEMV_THREADS;         // rows
    uint32_t wg = blockIdx.x, part = 0u;
    if (parts_shift != 0) {
        part = wg / wgs;
        wg -= part * wgs;
    }
    // masked: neighbouring chunks, whose mask bytes share lines of the cache, on one XCD (workgroups go round the eight): 65 us
    // against 74 for a 7B-shaped block
    if (MASKED && wg < (wgs & ~7u)) wg = (wg & 7u) * (wgs >> 3) + (wg >> 3);
    const int mi = batch_index(B.tile_start, B.n, wg);
    const DequantArgs& A = B.m[mi];
    // workgroups of one matrix: chunks side by side, then row ranges, then row blocks
    const uint32_t at = (uint32_t)((int64_t)wg - B.tile_start[mi]);
    const uint32_t nc = (uint32_t)A.g.n_chunks;
    const uint32_t nr = (uint32_t)((A.g.R_u + nt - 1) / nt);
    uint32_t rb, rr, j;
    if (!MASKED && B.by_cost != 0 && A.g.U <= ORDER_MAX_UNITS) {
        const OrderedItem o = item_by_cost<false>(A.action, (int32_t)A.g.U, (int32_t)nr, (int32_t)nr, (int32_t)at, GEMV_CLASSES);
        rr = (uint32_t)o.item;
        rb = (uint32_t)o.unit / nc;
        j = (uint32_t)o.unit - rb * nc;
    } else {
        const uint32_t band = at / nc;
        j = at - band * nc;
        rb = band / nr;
        rr = band - rb * nr;
    }
    const int64_t u = (int64_t)rb * nc + j;
    const int64_t lrow0 = (int64_t)rr * nt;                            // first row, local to the unit
    const int64_t row0 = (int64_t)rb * A.g.R_u + lrow0;
    const int64_t left = A.g.R_u - lrow0;
    const int32_t nrows = left < nt ? (int32_t)left : nt;
    const int32_t G = A.g.chunk_w;
    const int64_t col0 = (int64_t)j * G;
    const int tid = threadIdx.x;

    int a = A.action[u];                           // on their way while x is looked over
    const int64_t base = A.code_off[u];
    const int32_t lpr = G >> 3;
    const bool lanes_split = (lpr & (lpr - 1)) == 0;
    // G/8 lanes side by side share a row of a skip unit and, under a mask, of 8-bit codes (a lane's own row of them is a line
    // of the cache that is gone before the lane has used it up): the routes whose rows the parts share
    const auto shared_rows = [&](int act) { return act == 0 || (MASKED && act == 1 && lanes_split); };
    if (part != 0u) {
        int act = a < WINDQ_N_ACTIONS ? a : 0;
        const int64_t bytes = dq_bytes_per_group(act, G);
        if (base < 0 || (base & 15) != 0 || base > A.codes_bytes - bytes * A.g.R_u) act = 0;
        if (!shared_rows(act)) return;
    }
    const int32_t share = nt >> parts_shift, first = (int32_t)part * share;             // this part's rows
    const int32_t end = first + share < nrows ? first + share : nrows;
    bool odd = false;
    double xsum = 0.0;
    for (int32_t c = tid; c < G; c += GEMV_THREADS) {
        const float v = A.x[col0 + c];
        xs[c] = v;
        xsum += (double)v;
        odd = odd || !(fabsf(v) <= 0x1p96f);
    }
    xsum = wave_sum(xsum);
    if ((tid & 63) == 0) red[tid >> 6] = xsum;
    const bool direct = __syncthreads_or(odd ? 1 : 0) != 0 || MASKED;
    if (a >= WINDQ_N_ACTIONS) a = 0;
    const int64_t bpg = dq_bytes_per_group(a, G);
    if (base < 0 || (base & 15) != 0 || base > A.codes_bytes - bpg * A.g.R_u) a = 0;   // a malformed entry reads nothing; base + bytes could pass 2^63
    double* __restrict__ out = A.gpart + (int64_t)j * A.g.rows + row0;

    if (a == 0) {
        constexpr int EB = Elem<DT>::bytes;
        const char* __restrict__ w0 = static_cast<const char*>(A.W) + (row0 * A.g.ld + col0) * EB;
        if (lanes_split) {                                 // G/8 lanes side by side share a row
            const int sub = tid & (lpr - 1);
            const int step = GEMV_THREADS / lpr;
            float xv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) xv[i] = A.x[col0 + sub * 8 + i];
            constexpr int NR = DT == WINDQ_BF16 ? 8 : 4;
            for (int32_t r0 = first + tid / lpr; r0 < end; r0 += NR * step) {  // NR rows in flight; lpr lanes keep together
                uint4 raw[NR][EB / 2];
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    const int32_t r = r0 + k * step;
                    __builtin_memcpy(raw[k], w0 + ((int64_t)(r < end ? r : end - 1) * A.g.ld + sub * 8) * EB, 8 * EB);
                }
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    float w[8], dot = 0.0f;
                    load8_global<DT>(raw[k], w);
#pragma unroll
                    for (int i = 0; i < 8; ++i) dot = fmaf(w[i], xv[i], dot);
                    double d = (double)dot;
                    for (int mk = 1; mk < lpr; mk <<= 1) d += __shfl_xor(d, mk, 64);
                    if (sub == 0 && r0 + k * step < end) out[r0 + k * step] = d;
                }
            }
        } else {
            for (int32_t r = first + tid; r < end; r += GEMV_THREADS) {
                double acc = 0.0;
                for (int32_t c = 0; c < G; c += 8) {
                    float w[8], dot = 0.0f;
                    load8_global<DT>(w0 + ((int64_t)r * A.g.ld + c) * EB, w);
#pragma unroll
                    for (int i = 0; i < 8; ++i) dot = fmaf(w[i], xs[c + i], dot);
                    acc += (double)dot;
                }
                out[r] = acc;
            }
        }
        return;
    }

    const int64_t g0 = u * A.g.R_u + lrow0;
    const uint8_t* __restrict__ src0 = A.codes + base + lrow0 * bpg;
    if (shared_rows(a)) {
        const int32_t sub = tid & (lpr - 1), step = GEMV_THREADS / lpr;
        const uint8_t* __restrict__ mask0 = A.mask + row0 * A.mask_ld + (col0 >> 3) + sub;
        float xv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) xv[i] = xs[sub * 8 + i];
        constexpr int NR = 4;
        for (int32_t r0 = first + tid / lpr; r0 < end; r0 += NR * step) {
            uint32_t d[NR][2], m[NR];
            float sc[NR], of[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const int32_t r = r0 + k * step, row = r < end ? r : end - 1;
                __builtin_memcpy(d[k], src0 + (int64_t)row * G + sub * 8, 8);
                m[k] = mask0[row * A.mask_ld];
                sc[k] = A.scale[g0 + row];
                of[k] = A.offset[g0 + row];
            }
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                float dot = 0.0f;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float wh = fmaf((float)((d[k][i >> 2] >> (8 * (i & 3))) & 0xffu), sc[k], of[k]);
                    dot = fmaf(((m[k] >> i) & 1u) != 0u ? 0.0f : wh, xv[i], dot);
                }
                double t = (double)dot;
                for (int mk = 1; mk < lpr; mk <<= 1) t += __shfl_xor(t, mk, 64);
                if (sub == 0 && r0 + k * step < end) out[r0 + k * step] = t;
            }
        }
        return;
    }
    if (!MASKED && a >= 4 && !direct) {
        // the rows' loads are on their way while the tables are made, the next bytes while these are looked up; a thread
        // past the last row reads the last row's data again and writes nothing
        uint32_t d[RPT][4];
        float sc[RPT], of[RPT];
        double acc[RPT];
        const int32_t nb = (int32_t)bpg;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int32_t r = k * GEMV_THREADS + tid, row = r < nrows ? r : nrows - 1;
            load_code_bytes(src0 + (int64_t)row * bpg, nb < 16 ? nb : 16, d[k]);
        }
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int32_t r = k * GEMV_THREADS + tid, row = r < nrows ? r : nrows - 1;
            sc[k] = A.scale[g0 + row];
            of[k] = a == 4 ? A.offset[g0 + row] : 0.0f;
            acc[k] = 0.0;
        }
        gemv_tables(a, xs, G, nb, tab);
        __syncthreads();
        const double* __restrict__ t = tab;
        for (int32_t b0 = 0; b0 < nb; b0 += 16, t += a == 5 ? 16 * GEMV_TRIT_WORDS : 16 * 32) {
            const int n = nb - b0 < 16 ? nb - b0 : 16;
            const int32_t b1 = b0 + 16;
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                const uint32_t now[4] = {d[k][0], d[k][1], d[k][2], d[k][3]};
                const int32_t r = k * GEMV_THREADS + tid, row = r < nrows ? r : nrows - 1;
                if (b1 < nb) load_code_bytes(src0 + (int64_t)row * bpg + b1, nb - b1 < 16 ? nb - b1 : 16, d[k]);
                acc[k] += a == 5 ? gemv_lookup_trits(now, n, t) : gemv_lookup_nibbles(now, n, t);
            }
        }
        const double xt = ((red[0] + red[1]) + red[2]) + red[3];
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int32_t r = k * GEMV_THREADS + tid;
            if (r < nrows) {
                const double scd = (double)sc[k];
                double t = a == 4 ? fma(fma(1.5, scd, (double)of[k]), xt, scd * acc[k]) : scd * acc[k];
                if (!(fabsf(sc[k]) <= 0x1p96f && fabsf(of[k]) <= 0x1p96f)) t = gemv_row_plain(a, src0 + (int64_t)r * bpg, G, sc[k], of[k], xs);
                out[r] = t;
            }
        }
        return;
    }

    uint16_t* trits_of = reinterpret_cast<uint16_t*>(tab);
    if (a == 5) {
        fill_trits(trits_of);
        __syncthreads();
    }
    const uint8_t *src[RPT], *mrow[RPT];
    float sc[RPT], of[RPT];
    double acc[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int32_t r = k * GEMV_THREADS + tid, row = r < nrows ? r : nrows - 1;
        src[k] = src0 + (int64_t)row * bpg;
        mrow[k] = MASKED ? A.mask + (row0 + row) * A.mask_ld + (col0 >> 3) : nullptr;
        sc[k] = A.scale[g0 + row];
        of[k] = A.offset[g0 + row];
        acc[k] = 0.0;
    }
    gemv_rows_of<MASKED>(a, src, mrow, G, (int32_t)bpg, sc, of, xs, trits_of, acc);
#pragma unroll
    for (int k = 0; k < RPT; ++k)
        if (k * GEMV_THREADS + tid < nrows) out[k * GEMV_THREADS + tid] = acc[k];
}
template <int DT, int RPT, bool MASKED>
__global__ __launch_bounds__(GEMV_THREADS, MASKED ? 4 : 6) void gemv_kernel(const DequantBatch B, const int parts_shift) {
    extern __shared__ __align__(16) char gemv_smem[];
    __shared__ double red[GEMV_THREADS / 64];
    gemv_rows_wg<DT, RPT, MASKED>(B, (uint32_t)B.tile_start[B.n], parts_shift, gemv_smem, red);
}

// Short units, and small matrices: G/8 lanes side by side share a row, eight columns each; no tables to make and no lanes
// without a row.  A workgroup takes a tile of 64 rows, 2048 / G at a time, or, where there are few tiles, one of
// 1 << parts_shift shares of it (512 x 512 at chunk 128 5.4 us, 8.0 with whole tiles; a share to each workgroup of a large
// matrix costs it half its speed again: 4096 x 4096 in units of 64 rows 14.0 us, 19.2 in shares).
template <int DT, bool POW2>
__device__ __forceinline__ void gemv_split_wg(const DequantBatch& B, const uint32_t wg, const uint32_t share, const int parts_shift,
                                              uint16_t* __restrict__ trits_of, double* part) {
    const int mi = batch_index(B.tile_start, B.n, wg);
    const DequantArgs& A = B.m[mi];
    const TileCoord tc = tile_coord(A.g, (int64_t)wg - B.tile_start[mi]);
    constexpr int EB = Elem<DT>::bytes;
    const int32_t G = A.g.chunk_w, lpr = G >> 3;
    const int32_t lpr_shift = 31 - __builtin_clz(lpr);          // POW2
    const int32_t rpp = POW2 ? GEMV_THREADS >> lpr_shift : GEMV_THREADS / lpr;      // rows of a pass
    const int32_t rsub = POW2 ? (int32_t)threadIdx.x >> lpr_shift : (int32_t)threadIdx.x / lpr, sub = (int32_t)threadIdx.x - rsub * lpr;
    const int32_t c = sub * 8;

    int a = A.action[tc.u];
    if (a >= WINDQ_N_ACTIONS) a = 0;
    const int64_t bpg = dq_bytes_per_group(a, G);
    const int64_t base = A.code_off[tc.u];
    if (base < 0 || (base & 15) != 0 || base > A.codes_bytes - bpg * A.g.R_u) a = 0;   // a malformed entry reads nothing; base + bytes could pass 2^63
    const int bits = a == 1 ? 8 : (a == 2 ? 4 : (a == 3 ? 3 : (a == 4 ? 2 : 1)));
    float xv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) xv[j] = A.x[tc.col0 + c + j];
    if (a == 5) {
        fill_trits(trits_of);
        __syncthreads();
    }
    double* __restrict__ out = A.gpart + (tc.col0 / G) * A.g.rows + tc.row0;
    for (int32_t r0 = (int32_t)share * rpp; r0 < tc.nrows; r0 += rpp << parts_shift) {
        const int32_t r = r0 + rsub;
        float dot = 0.0f;
        if ((POW2 || rsub < rpp) && r < tc.nrows) {
            float wh[8];
            uint32_t m = 0u;
            if (a == 0) {
                load8_global<DT>(static_cast<const char*>(A.W) + ((tc.row0 + r) * A.g.ld + tc.col0 + c) * EB, wh);
            } else {
                if (A.mask != nullptr) m = A.mask[(tc.row0 + r) * A.mask_ld + (tc.col0 >> 3) + sub];
                const int64_t gidx = tc.u * A.g.R_u + tc.lrow0 + r;
                decode8(a, bits, A.codes + base + (tc.lrow0 + r) * bpg, c, (int32_t)bpg, A.scale[gidx], A.offset[gidx], trits_of, wh);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) dot = fmaf(((m >> j) & 1u) != 0u ? 0.0f : wh[j], xv[j], dot);
        }
        // the row's 8-column runs summed in fp64
        double d = (double)dot;
        if (POW2) {
            for (int mk = 1; mk < lpr; mk <<= 1) d += __shfl_xor(d, mk, 64);
            if (sub == 0 && r < tc.nrows) out[r] = d;
        } else {
            __syncthreads();
            part[threadIdx.x] = d;
            __syncthreads();
            if ((int32_t)threadIdx.x < rpp && r0 + (int32_t)threadIdx.x < tc.nrows) {
                double t = 0.0;
                for (int32_t i = 0; i < lpr; ++i) t += part[(int32_t)threadIdx.x * lpr + i];
                out[r0 + (int32_t)threadIdx.x] = t;
            }
        }
    }
}
template <int DT, bool POW2>
__global__ __launch_bounds__(GEMV_THREADS) void gemv_split_kernel(const DequantBatch B, const int parts_shift) {
    __shared__ uint16_t trits_of[256];
    __shared__ double part[POW2 ? 1 : GEMV_THREADS];
    gemv_split_wg<DT, POW2>(B, blockIdx.x >> parts_shift, blockIdx.x & ((1u << parts_shift) - 1u), parts_shift, trits_of, part);
}

// A batch of both kinds, in one launch: the first n_rows matrices as gemv_kernel takes them, the others as gemv_split_kernel does.
// A launch of its own for those took 3.5 us of the host's time (six matrices of 0.1 to 34 M weights 29.4 us a call, so 25.8).  The
// split tiles come last: before the others, which are the longer, 0 to 2 us slower.
template <int DT, int RPT, bool MASKED>
__global__ __launch_bounds__(GEMV_THREADS, MASKED ? 4 : 6) void gemv_both_kernel(const DequantBatch B, const int n_rows, const int parts_shift,
                                                                                const int split_shift) {
    extern __shared__ __align__(16) char gemv_smem[];
    __shared__ double red[GEMV_THREADS / 64];
    const uint32_t wgs = (uint32_t)B.tile_start[n_rows], rows_blocks = wgs << parts_shift;
    if (blockIdx.x < rows_blocks) {
        gemv_rows_wg<DT, RPT, MASKED>(B, wgs, parts_shift, gemv_smem, red);
        return;
    }
    const uint32_t at = blockIdx.x - rows_blocks, wg = wgs + (at >> split_shift), share = at & ((1u << split_shift) - 1u);
    const int32_t G = B.m[0].g.chunk_w;
    double* part = reinterpret_cast<double*>(gemv_smem);                     // (GEMV_BOTH_LDS bytes)
    uint16_t* trits_of = reinterpret_cast<uint16_t*>(part + GEMV_THREADS);
    if ((G & (G - 1)) == 0) gemv_split_wg<DT, true>(B, wg, share, split_shift, trits_of, part);
    else gemv_split_wg<DT, false>(B, wg, share, split_shift, trits_of, part);
}

// y[row] = the row's chunk partials: 8 phases, phase p adds chunks p, p + 8, ..., the phases in order; fp64,
// rounded once.  32 rows to a workgroup, so that the short sums of a block's rows fill the chip.
constexpr int GEMV_FIN_ROWS = 32;
__global__ __launch_bounds__(256) void gemv_finalize_kernel(const DequantBatch B) {
    __shared__ double red[8][GEMV_FIN_ROWS];
    const int mi = batch_index(B.row_start, B.n, blockIdx.x);
    const DequantArgs& A = B.m[mi];
    const int rl = threadIdx.x & (GEMV_FIN_ROWS - 1), ph = threadIdx.x / GEMV_FIN_ROWS;
    const int64_t row = ((int64_t)blockIdx.x - B.row_start[mi]) * GEMV_FIN_ROWS + rl;
    double t = 0.0;
    if (row < A.g.rows) {
#pragma unroll 4
        for (int64_t c = ph; c < A.g.n_chunks; c += 8) t += A.gpart[c * A.g.rows + row];
    }
    red[ph][rl] = t;
    __syncthreads();
    if (threadIdx.x >= GEMV_FIN_ROWS || row >= A.g.rows) return;
#pragma unroll
    for (int p = 1; p < 8; ++p) t += red[p][rl];
    A.y[row] = (float)t;
}

// Numbers the tiles and units of the first B->n matrices.
static int64_t dequant_number(DequantBatch* B) {
    int64_t tiles = 0, units = 0, rows = 0;
    for (int32_t i = 0; i < B->n; ++i) {
        B->tile_start[i] = tiles;
        B->unit_start[i] = units;
        B->row_start[i] = rows;
        tiles += B->m[i].g.n_tiles;
        units += B->m[i].g.U;
        rows += B->m[i].g.rows;
    }
    for (int32_t i = B->n; i <= WINDQ_MAX_BATCH; ++i) {
        B->tile_start[i] = tiles;
        B->unit_start[i] = units;
        B->row_start[i] = rows;
    }
    for (int32_t i = B->n; i < WINDQ_MAX_BATCH; ++i) B->m[i] = B->m[0];
    return tiles;
}

}  // namespace windq

using namespace windq;

// One matrix of a launch as the entry points see it (the check call, or the product when x is set).
struct DequantItem {
    const windq_mat* W;
    const float* s;
    const uint8_t* mask;
    const uint8_t* action;
    const int64_t* code_off;
    const uint8_t* codes;
    size_t codes_bytes;
    const float* scale;
    const float* offset;
    float* err;
    float* w_hat;
    const float* x;
    float* y;
    void* ws;
    size_t ws_bytes;
};

static void dequant_args(const DequantItem& it, DequantArgs* A) {
    A->W = it.W->data;
    A->s = it.s;
    A->mask = it.mask;
    A->mask_ld = it.W->cols / 8;
    A->action = it.action;
    A->code_off = it.code_off;
    A->codes = it.codes;
    A->codes_bytes = (int64_t)it.codes_bytes;
    A->scale = it.scale;
    A->offset = it.offset;
    A->what = nullptr;
    A->what_ld = it.W->cols;
    A->part = static_cast<double*>(it.ws);
    A->err = nullptr;
    A->per_unit = 0;
    A->x = it.x;
    A->y = it.y;
    A->gpart = static_cast<double*>(it.ws);
}

// Matrices whose buffers are aligned go in one launch, the others in one of their own, exactly as each would alone.
static int dequant_launch(const DequantItem* items, int32_t n, int32_t chunk_w, int64_t unit_rows, void* stream) {
    if (items == nullptr || n < 1 || n > WINDQ_MAX_BATCH) return WINDQ_EINVAL;
    const int32_t passes = dequant_passes(chunk_w);
    DequantBatch L[2];          // aligned, not
    L[0].n = L[1].n = 0;
    bool any_err[2] = {false, false};
    for (int32_t i = 0; i < n; ++i) {
        const DequantItem& it = items[i];
        DequantArgs A;
        if (it.W == nullptr) return WINDQ_EINVAL;
        const int st = make_geometry(it.W, chunk_w, unit_rows, &A.g);
        if (st != WINDQ_OK) return st;
        if (it.action == nullptr || it.code_off == nullptr || it.scale == nullptr || it.offset == nullptr) return WINDQ_EINVAL;
        if (it.codes == nullptr && it.codes_bytes != 0) return WINDQ_EINVAL;
        if (it.s == nullptr || (it.err == nullptr && it.w_hat == nullptr)) return WINDQ_EINVAL;
        if (it.w_hat != nullptr && !aligned(it.w_hat, 4)) return WINDQ_EINVAL;
        if (!aligned(it.code_off, 8)) return WINDQ_EINVAL;
        if (it.W->dtype != items[0].W->dtype) return WINDQ_EINVAL;      // one kernel per launch
        if (it.ws == nullptr || it.ws_bytes < dequant_ws_bytes(A.g) || !aligned(it.ws, 256)) return WINDQ_EWORKSPACE;
        dequant_args(it, &A);
        A.what = it.w_hat;
        A.err = it.err;
        A.per_unit = A.g.tiles_per_unit * passes;
        const int un = (A.what == nullptr || aligned(A.what, 16)) && aligned(it.codes, 8) ? 0 : 1;
        L[un].m[L[un].n++] = A;
        any_err[un] = any_err[un] || A.err != nullptr;
    }
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const int32_t dtype = items[0].W->dtype;
    int lpr_shift = -1;         // chunk_w = 8 << lpr_shift
    for (int k = 0; k <= 6; ++k)
        if (chunk_w == (8 << k)) lpr_shift = k;
    int64_t wgs[2];
    for (int un = 0; un < 2; ++un) {
        wgs[un] = dequant_number(&L[un]) * passes;
        if (!fits_launch(wgs[un], DQ_THREADS)) return WINDQ_ESHAPE;
    }
    for (int un = 0; un < 2; ++un) {
        DequantBatch& B = L[un];
        if (B.n == 0) continue;
        const dim3 grid((unsigned)wgs[un]);
        if (un == 1) {
            if (dtype == WINDQ_BF16) hipLaunchKernelGGL((dequant_any_kernel<WINDQ_BF16, false>), grid, dim3(DQ_THREADS), 0, hs, B, chunk_w);
            else hipLaunchKernelGGL((dequant_any_kernel<WINDQ_F32, false>), grid, dim3(DQ_THREADS), 0, hs, B, chunk_w);
        } else if (lpr_shift >= 0) {
            if (dtype == WINDQ_BF16) hipLaunchKernelGGL(dequant_split_kernel<WINDQ_BF16>, grid, dim3(DQ_THREADS), 0, hs, B, lpr_shift);
            else hipLaunchKernelGGL(dequant_split_kernel<WINDQ_F32>, grid, dim3(DQ_THREADS), 0, hs, B, lpr_shift);
        } else {
            if (dtype == WINDQ_BF16) hipLaunchKernelGGL((dequant_any_kernel<WINDQ_BF16, true>), grid, dim3(DQ_THREADS), 0, hs, B, chunk_w);
            else hipLaunchKernelGGL((dequant_any_kernel<WINDQ_F32, true>), grid, dim3(DQ_THREADS), 0, hs, B, chunk_w);
        }
        if (any_err[un]) hipLaunchKernelGGL(dequant_finalize_kernel, dim3((unsigned)B.unit_start[B.n]), dim3(256), 0, hs, B);
    }
    return hipPeekAtLastError() == hipSuccess ? WINDQ_OK : WINDQ_EHIP;
}

// The product: which kernel a matrix takes.  It alone decides, so that a batch gives the bits of single calls.  Lanes that
// share a row (split) against a row to each lane (rows), us at a mixed 2-bit plan:
//   rows per unit, 4096 x 4096 bf16, chunk 128           32: 15.3 against 27.7   64: 14.0, 18.0   96: 15.2, 14.6   128: 14.1, 12.7
//   the same under a mask                               128: 15.3, 25.3         256: 15.3, 12.9
//   weights, whole columns, chunk 128    1024 x 1024: 5.6, 7.7   2048 x 768: 6.0, 7.7   1024 x 2048: 6.8, 8.1   (4096 x 4096: 14, 8.6)
//                      chunks 96 and 32  2048 x 768: 6.6, 7.2 and 6.6, 7.9   1024 x 2016: 8.1, 8.2 and 7.0, 7.4
//   under a mask                         2048 x 2048 at chunk 256: 9, 13, at chunk 32 (512 workgroups of 256 rows): 8.5, 7.9
constexpr int GEMV_SPLIT = 0, GEMV_ROWS = 1, GEMV_ROWS_MASKED = 2;
constexpr int64_t GEMV_SHORT_UNIT = 96, GEMV_SHORT_UNIT_MASKED = 256;     // rows
constexpr int64_t GEMV_SMALL = 3 << 19, GEMV_SMALL_MASKED = 1 << 22;      // weights
constexpr int64_t GEMV_FEW_WGS_MASKED = 256;
static int gemv_route(const Geometry& g, bool masked) {
    const int64_t wgs = g.U * ((g.R_u + GEMV_THREADS - 1) / GEMV_THREADS), n = g.rows * g.cols;
    if (g.R_u < (masked ? GEMV_SHORT_UNIT_MASKED : GEMV_SHORT_UNIT) || n <= GEMV_SMALL) return GEMV_SPLIT;
    if (masked && n <= GEMV_SMALL_MASKED && wgs <= GEMV_FEW_WGS_MASKED) return GEMV_SPLIT;
    return masked ? GEMV_ROWS_MASKED : GEMV_ROWS;
}
constexpr int64_t GEMV_SPLIT_WGS = 2048;    // up to which a tile's rows are spread over several workgroups: two rounds of a full chip at most

// How many workgroups (as a shift) share a tile's rows where lanes share a row.
static int gemv_split_shift(int64_t tiles, int32_t chunk_w) {
    int shift = 0;
    while ((1 << shift) < dequant_passes(chunk_w) && (tiles << shift) < GEMV_SPLIT_WGS) ++shift;
    return shift;
}

// The first n_rows matrices of B in `wgs` workgroups a part; the others, if any, in tiles.
template <int RPT, bool MASKED>
static void gemv_rows_launch(const DequantBatch& B, int32_t n_rows, int64_t wgs, int parts_shift, bool bf, size_t lds, hipStream_t hs) {
    const dim3 block(GEMV_THREADS);
    if (n_rows == B.n) {
        const dim3 grid((unsigned)(wgs << parts_shift));
        if (bf) hipLaunchKernelGGL((gemv_kernel<WINDQ_BF16, RPT, MASKED>), grid, block, lds, hs, B, parts_shift);
        else hipLaunchKernelGGL((gemv_kernel<WINDQ_F32, RPT, MASKED>), grid, block, lds, hs, B, parts_shift);
        return;
    }
    const int64_t tiles = B.tile_start[B.n] - wgs;
    const int split_shift = gemv_split_shift(tiles, B.m[0].g.chunk_w);
    const dim3 grid((unsigned)((wgs << parts_shift) + (tiles << split_shift)));
    if (lds < GEMV_BOTH_LDS) lds = GEMV_BOTH_LDS;
    if (bf) hipLaunchKernelGGL((gemv_both_kernel<WINDQ_BF16, RPT, MASKED>), grid, block, lds, hs, B, n_rows, parts_shift, split_shift);
    else hipLaunchKernelGGL((gemv_both_kernel<WINDQ_F32, RPT, MASKED>), grid, block, lds, hs, B, n_rows, parts_shift, split_shift);
}

// A workgroup takes 512 rows of a unit (two per thread, their loads in flight together) where that still
// makes four workgroups per CU, else 256.  1024 rows are as fast when all units have one bit-width, but the few units at
// 8 bits or skipped then outlast the others: 4096 x 11008 x 4 at a mixed plan 45 us against 35.
constexpr int64_t GEMV_MIN_WGS = 1024;
static int gemv_launch(const DequantItem* items, int32_t n, int32_t chunk_w, int64_t unit_rows, void* stream) {
    if (items == nullptr || n < 1 || n > WINDQ_MAX_BATCH) return WINDQ_EINVAL;
    DequantBatch L[3], All;
    All.n = n;
    for (int k = 0; k < 3; ++k) L[k].n = 0;
    int64_t fin = 0;
    for (int32_t i = 0; i < n; ++i) {
        const DequantItem& it = items[i];
        DequantArgs& A = All.m[i];
        if (it.W == nullptr) return WINDQ_EINVAL;
        const int st = make_geometry(it.W, chunk_w, unit_rows, &A.g);
        if (st != WINDQ_OK) return st;
        if (it.action == nullptr || it.code_off == nullptr || it.scale == nullptr || it.offset == nullptr) return WINDQ_EINVAL;
        if (it.codes == nullptr && it.codes_bytes != 0) return WINDQ_EINVAL;
        if (it.x == nullptr || it.y == nullptr || !aligned(it.code_off, 8)) return WINDQ_EINVAL;
        if (it.W->dtype != items[0].W->dtype) return WINDQ_EINVAL;      // one kernel per launch
        if (it.ws == nullptr || it.ws_bytes < dequant_gemv_ws_bytes(A.g) || !aligned(it.ws, 256)) return WINDQ_EWORKSPACE;
        dequant_args(it, &A);
        DequantBatch& B = L[gemv_route(A.g, A.mask != nullptr)];
        B.m[B.n++] = A;
    }
    dequant_number(&All);
    for (int32_t i = 0; i <= WINDQ_MAX_BATCH; ++i) {        // the finalize kernel's workgroups
        All.row_start[i] = fin;
        if (i < n) fin += (All.m[i].g.rows + GEMV_FIN_ROWS - 1) / GEMV_FIN_ROWS;
    }
    if (All.tile_start[n] > (int64_t)0x7fffffff || !fits_launch(fin, 256)) return WINDQ_ESHAPE;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const bool bf = items[0].W->dtype == WINDQ_BF16;
    DequantBatch& S = L[GEMV_SPLIT];
    const int64_t tiles = S.n > 0 ? dequant_number(&S) : 0;
    if (S.n == n) {
        const int parts_shift = gemv_split_shift(tiles, chunk_w);
        if (!fits_launch(tiles << parts_shift, GEMV_THREADS)) return WINDQ_ESHAPE;
        const dim3 grid((unsigned)(tiles << parts_shift)), block(GEMV_THREADS);
        const bool pow2 = (chunk_w & (chunk_w - 1)) == 0;
        if (bf && pow2) hipLaunchKernelGGL((gemv_split_kernel<WINDQ_BF16, true>), grid, block, 0, hs, S, parts_shift);
        else if (bf) hipLaunchKernelGGL((gemv_split_kernel<WINDQ_BF16, false>), grid, block, 0, hs, S, parts_shift);
        else if (pow2) hipLaunchKernelGGL((gemv_split_kernel<WINDQ_F32, true>), grid, block, 0, hs, S, parts_shift);
        else hipLaunchKernelGGL((gemv_split_kernel<WINDQ_F32, false>), grid, block, 0, hs, S, parts_shift);
    }
    for (int k = GEMV_ROWS; k <= GEMV_ROWS_MASKED; ++k) {
        DequantBatch& B = L[k];
        if (B.n == 0) continue;
        dequant_number(&B);
        int rpt = 4;
        int64_t wgs;
        do {
            rpt >>= 1;
            wgs = 0;
            for (int32_t i = 0; i <= WINDQ_MAX_BATCH; ++i) {
                B.tile_start[i] = wgs;
                if (i < B.n) wgs += B.m[i].g.U * ((B.m[i].g.R_u + rpt * GEMV_THREADS - 1) / (rpt * GEMV_THREADS));
            }
        } while (rpt > 1 && wgs < GEMV_MIN_WGS);
        // a skip unit's rows in parts, where there are fewer than two workgroups per CU (four under a mask, where 8-bit units share
        // too), each of at least four loads per thread: skip units of 4096 x 4096 at chunk 512 16.5 us, 38 in one part
        B.by_cost = k == GEMV_ROWS && wgs >= GEMV_MIN_WGS ? 1 : 0;
        int parts_shift = 0;
        while (parts_shift < 2 && (wgs << parts_shift) < (k == GEMV_ROWS ? GEMV_MIN_WGS / 2 : GEMV_MIN_WGS)) {
            const int64_t rows = rpt * GEMV_THREADS >> (parts_shift + 1);       // of a part
            if (rows >= B.m[0].g.R_u || rows * chunk_w < 4 * GEMV_THREADS * 8) break;
            ++parts_shift;
        }
        if (!fits_launch((wgs << parts_shift) + (S.n > 0 ? tiles << gemv_split_shift(tiles, chunk_w) : 0), GEMV_THREADS)) return WINDQ_ESHAPE;
        const int32_t n_rows = B.n;
        for (int32_t i = 0; i < S.n; ++i, ++B.n) {          // into the first launch of the other kind
            B.m[B.n] = S.m[i];
            B.tile_start[B.n] = wgs + S.tile_start[i];
        }
        for (int32_t i = B.n; i <= WINDQ_MAX_BATCH; ++i) B.tile_start[i] = wgs + (B.n > n_rows ? tiles : 0);
        S.n = 0;
        const size_t lds = k == GEMV_ROWS ? gemv_lds(chunk_w) : WINDQ_MAX_CHUNK * sizeof(float) + 256 * sizeof(uint16_t);   // tables: at most 41 KB
        if (k == GEMV_ROWS) {
            if (rpt == 2) gemv_rows_launch<2, false>(B, n_rows, wgs, parts_shift, bf, lds, hs);
            else gemv_rows_launch<1, false>(B, n_rows, wgs, parts_shift, bf, lds, hs);
        } else {
            if (rpt == 2) gemv_rows_launch<2, true>(B, n_rows, wgs, parts_shift, bf, lds, hs);
            else gemv_rows_launch<1, true>(B, n_rows, wgs, parts_shift, bf, lds, hs);
        }
    }
    hipLaunchKernelGGL(gemv_finalize_kernel, dim3((unsigned)fin), dim3(256), 0, hs, All);
    return hipPeekAtLastError() == hipSuccess ? WINDQ_OK : WINDQ_EHIP;
}

extern "C" int windq_dequant_plan(const windq_mat* W, const float* s, int32_t chunk_w, int64_t unit_rows,
                                  const uint8_t* mask, const uint8_t* action, const int64_t* code_off,
                                  const uint8_t* codes, size_t codes_bytes, const float* scale, const float* offset,
                                  float* err, float* w_hat, void* ws, size_t ws_bytes, void* stream) {
    const DequantItem it = {W, s, mask, action, code_off, codes, codes_bytes, scale, offset, err, w_hat, nullptr, nullptr, ws, ws_bytes};
    return dequant_launch(&it, 1, chunk_w, unit_rows, stream);
}

extern "C" int windq_dequant_plan_batch(const windq_dequant_item* items, int32_t n, int32_t chunk_w, int64_t unit_rows,
                                        void* stream) {
    if (items == nullptr || n < 1 || n > WINDQ_MAX_BATCH) return WINDQ_EINVAL;
    DequantItem its[WINDQ_MAX_BATCH];
    for (int32_t i = 0; i < n; ++i)
        its[i] = {items[i].W, items[i].s, items[i].mask, items[i].action, items[i].code_off, items[i].codes, items[i].codes_bytes,
                  items[i].scale, items[i].offset, items[i].err, items[i].w_hat, nullptr, nullptr, items[i].ws, items[i].ws_bytes};
    return dequant_launch(its, n, chunk_w, unit_rows, stream);
}

extern "C" int windq_dequant_gemv(const windq_mat* W, int32_t chunk_w, int64_t unit_rows, const uint8_t* mask,
                                  const uint8_t* action, const int64_t* code_off, const uint8_t* codes, size_t codes_bytes,
                                  const float* scale, const float* offset, const float* x, float* y, void* ws,
                                  size_t ws_bytes, void* stream) {
    const DequantItem it = {W, nullptr, mask, action, code_off, codes, codes_bytes, scale, offset, nullptr, nullptr, x, y, ws, ws_bytes};
    return gemv_launch(&it, 1, chunk_w, unit_rows, stream);
}

extern "C" int windq_dequant_gemv_batch(const windq_gemv_item* items, int32_t n, int32_t chunk_w, int64_t unit_rows,
                                        void* stream) {
    if (items == nullptr || n < 1 || n > WINDQ_MAX_BATCH) return WINDQ_EINVAL;
    DequantItem its[WINDQ_MAX_BATCH];
    for (int32_t i = 0; i < n; ++i)
        its[i] = {items[i].W, nullptr, items[i].mask, items[i].action, items[i].code_off, items[i].codes, items[i].codes_bytes,
                  items[i].scale, items[i].offset, nullptr, nullptr, items[i].x, items[i].y, items[i].ws, items[i].ws_bytes};
    return gemv_launch(its, n, chunk_w, unit_rows, stream);
}
