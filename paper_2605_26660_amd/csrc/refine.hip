// windq_refine_plan: windq_apply_plan with refined scales.  The paper fits each operator's
// scale by a short local optimisation of the reconstruction loss on the unit (App. "Per-unit
// Scale Optimization": ~10 optimiser steps, no model-wide backward pass).  The deterministic
// stand-in here: every group is seeded with its grid fit, then alternates
//     assign codes by the normative fp32 steps  |  solve the activation-weighted
//     least-squares problem for the group's parameters in closed form
// for n_iter rounds; neither half-step can raise the loss.  Uniform: minimise
// sum a_c (w - lo - q step)^2 over (lo, step) by the 2x2 normal equations; ternary:
// gamma = sum a q w / sum a q^2; binary (signs fixed): alpha = sum a |w| / sum a.
// The sums are fp64 in column order from plain multiplies and adds (this file is compiled
// with contraction off), the parameters are rounded to fp32 after every solve: the results
// are defined to the bit, so codes and stored parameters can be checked exactly.
//
// One wavefront per 64-row tile, one lane per group: a group's refinement is a lane-private sequence of
// passes over its row, fp64 arithmetic at 7 to 10 operations per weight and round: bound by the fp64
// ALU, not by HBM; it runs once per chosen plan.  A lane's row lies in registers (64 for 128 bf16 weights, up to
// 128), read eight weights at a time by register indexing: a tile staged in LDS (17 KB) leaves room for two wavefronts
// per SIMD, too few to fill the ALU.  LDS only turns the tile round on its way in, 128 bytes of every row at a
// time, and the packed codes on their way out.  Wider rows stay in LDS.  Refining a 7B-shaped block at 2 bits, three rounds:
// 225 us, dear units first (285 in the matrix's own order, see RF_ORDERED_TILES); 610 with the tile in LDS, a select per
// weight for a mask that is not there, and passes of their own for error and codes; then 303 with a code and a product
// by it per ternary weight, base-3 bytes by integer multiplies, and the sign in a binary weight's residual.  Five wavefronts
// per SIMD would spill (1.4 ms), an unrolled pair of blocks is 7 % slower, and s_c^2 read from LDS weight by weight
// between a ternary round's adds costs 13 us.
#include <float.h>

#include "windq_common.hpp"
#include "windq_group.hpp"
#include "windq_order.hpp"
#include "windq_ws.hpp"

namespace windq {

struct RefineArgs {
    const void* W;
    const float* s;
    const uint8_t* mask;       // or null
    int64_t mask_ld;
    const uint8_t* action;
    const uint8_t* clip_idx;   // or null
    const int64_t* code_off;
    uint8_t* codes;
    int64_t codes_bytes;
    float* scale;
    float* offset;
    double* part;              // [n_tiles]
    float* err;                // [U]
    Geometry g;
};

// A launch covers up to WINDQ_MAX_BATCH matrices (one chunk width, one element type, one clip
// grid and round count): their tiles and units are numbered one matrix after the other.
struct RefineBatch {
    int32_t n;
    int32_t K;
    int32_t n_iter;
    int32_t by_cost;           // tiles in the order of what their units cost (see RF_ORDERED_TILES)
    int64_t tile_start[WINDQ_MAX_BATCH + 1];
    int64_t unit_start[WINDQ_MAX_BATCH + 1];
    RefineArgs m[WINDQ_MAX_BATCH];
    ClipGrid grid;
};

// A lane's row of G weights in LDS, element type of the input.
template <int DT>
struct LdsRow {
    const char* p;
    // f(c, w): eight weights from column c, in column order
    template <typename F>
    __device__ __forceinline__ void blocks(int32_t G, F f) const {
        for (int32_t c = 0; c < G; c += 8) {
            float w[8];
            read8<DT>(p, c, w);
            f(c, w);
        }
    }
};

// A lane's row in NV x 32 registers (128 bytes each).
typedef uint32_t Regs32 __attribute__((ext_vector_type(32)));
template <int DT, int NV>
struct RegRow {
    Regs32 r[NV];
    template <typename F>
    __device__ __forceinline__ void blocks(int32_t G, F f) const {
        constexpr int PER = DT == WINDQ_BF16 ? 8 : 4;           // blocks of eight weights in 32 registers
        constexpr int DW = 32 / PER;
        const int nb = G >> 3;
#pragma unroll
        for (int h = 0; h < NV; ++h) {
            const int n = nb - h * PER < PER ? nb - h * PER : PER;
#pragma unroll 1
            for (int i = 0; i < n; ++i) {
                uint32_t d[DW];
#pragma unroll
                for (int k = 0; k < DW; ++k) d[k] = r[h][i * DW + k];
                float w[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (DT == WINDQ_BF16) w[j] = __uint_as_float((j & 1) != 0 ? d[j >> 1] & 0xffff0000u : d[j >> 1] << 16);
                    else w[j] = __uint_as_float(d[j < DW ? j : 0]);
                }
                f((h * PER + i) * 8, w);
            }
        }
    }
};

// The tile into its lanes' rows: 128 bytes of every row at a time through LDS (buf: 64 rows of 144 bytes).
constexpr int RF_THREADS = 64;
constexpr int RF_SLAB = 128, RF_SLAB_STRIDE = RF_SLAB + 16;
template <int DT, int NV>
__device__ __forceinline__ void load_rows(const RefineArgs& A, const TileCoord& tc, char* buf, RegRow<DT, NV>& row) {
    const int lane = threadIdx.x;
    const int32_t row_bytes = A.g.chunk_w * Elem<DT>::bytes;
    const char* __restrict__ src = static_cast<const char*>(A.W) + (tc.row0 * A.g.ld + tc.col0) * Elem<DT>::bytes;
    const int64_t ld = A.g.ld * Elem<DT>::bytes;
    uint4 raw[NV][8];
#pragma unroll
    for (int h = 0; h < NV; ++h) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int r = 8 * k + (lane >> 3), at = h * RF_SLAB + (lane & 7) * 16;
            raw[h][k] = make_uint4(0u, 0u, 0u, 0u);
            if (r < tc.nrows && at < row_bytes) raw[h][k] = *reinterpret_cast<const uint4*>(src + r * ld + at);
        }
    }
#pragma unroll
    for (int h = 0; h < NV; ++h) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; ++k) *reinterpret_cast<uint4*>(buf + (8 * k + (lane >> 3)) * RF_SLAB_STRIDE + (lane & 7) * 16) = raw[h][k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint4 q = *reinterpret_cast<const uint4*>(buf + lane * RF_SLAB_STRIDE + k * 16);
            row.r[h][4 * k] = q.x;
            row.r[h][4 * k + 1] = q.y;
            row.r[h][4 * k + 2] = q.z;
            row.r[h][4 * k + 3] = q.w;
        }
    }
    __syncthreads();
}

// Adds p to n and a to d in the lanes whose |t| is above 0.5 (or NaN), by a compare that writes the execution mask: three
// vector instructions where a select of two fp64 values takes seven.
__device__ __forceinline__ void add_where_above_half(float t, double p, double a, double& n, double& d) {
    uint64_t all;
    asm volatile("s_mov_b64 %2, exec\n\t"
                 "v_cmpx_nle_f32_e64 vcc, |%3|, 0.5\n\t"
                 "v_add_f64 %0, %0, %4\n\t"
                 "v_add_f64 %1, %1, %5\n\t"
                 "s_mov_b64 exec, %2"
                 : "+v"(n), "+v"(d), "=&s"(all)
                 : "v"(t), "v"(p), "v"(a)
                 : "vcc");
}

// bits = 2 bits + (w >= 0): a compare into the carry and an add with carry.
__device__ __forceinline__ void push_not_negative(uint32_t& bits, float w) {
    asm("v_cmp_le_f32_e32 vcc, 0, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(w) : "vcc");
}

// One group: its row, its protection bits (masked calls), s_c^2 of the columns.
template <int DT, bool MASKED, typename Row>
struct RefineGroup {
    Row row;
    const uint8_t* mrow;
    const double* acol;
    int32_t G;
    bool protects;              // MASKED: the item has a mask (else its mask bytes are zeros)
    bool finite;                // every s_c^2 of the chunk is

    __device__ __forceinline__ uint32_t bits(int32_t c) const { return MASKED ? mrow[c >> 3] : 0u; }
    __device__ __forceinline__ bool kept(uint32_t m, int j) const { return !MASKED || ((m >> j) & 1u) == 0u; }
    // s_c^2 of column c + j, zero for a protected weight
    __device__ __forceinline__ double weight(uint32_t m, int32_t c, int j) const { return kept(m, j) ? acol[c + j] : 0.0; }

    // min and max of the kept weights.  Under a mask 0, 0 when none is kept (or all that are kept are NaN); an item without
    // one gives NaN for a group of NaN, also in a masked launch
    __device__ __forceinline__ void min_max(float* mn_out, float* mx_out) const {
        float mn = INFINITY, mx = -INFINITY;
        row.blocks(G, [&](int32_t c, const float (&w)[8]) {
            const uint32_t m = bits(c);
            if (!(MASKED && protects) && c == 0) mn = mx = w[0];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                mn = fminf(mn, kept(m, j) ? w[j] : INFINITY);
                mx = fmaxf(mx, kept(m, j) ? w[j] : -INFINITY);
            }
        });
        if (MASKED && protects && mn > mx) mn = mx = 0.0f;
        *mn_out = mn;
        *mx_out = mx;
    }

    // mean |w| as stored: the fp64 sum in column order over the kept weights, rounded to fp32; 0 when none is kept
    __device__ __forceinline__ float abs_mean() const {
        double S1 = 0.0;
        int32_t n = G;
        row.blocks(G, [&](int32_t c, const float (&w)[8]) {
            const uint32_t m = bits(c);
            n -= __builtin_popcount(m);
#pragma unroll
            for (int j = 0; j < 8; ++j) S1 += kept(m, j) ? (double)fabsf(w[j]) : 0.0;
        });
        return n > 0 ? (float)(S1 / (double)n) : 0.0f;
    }

    // The sums of one round of the uniform refinement.  S0 = sum a and T0 = sum a w do not depend on the
    // codes: the first round computes them (FIRST), later rounds reuse them; the
    // order of every sum is the column order either way.
    // TWO: 2 bits.  s_c^2 has at most 48 significant bits, so s_c^2 q^2 is exact for q up to 3, and a fused multiply-add
    // rounds as the product and the sum do.
    template <bool FIRST, bool TWO>
    __device__ __forceinline__ void uniform_sums(float lo, float inv, float qmax, double& S0, double& T0, double& S1, double& S2,
                                                 double& T1) const {
        if (FIRST) S0 = T0 = 0.0;
        S1 = S2 = T1 = 0.0;
        row.blocks(G, [&](int32_t c, const float (&w)[8]) {
            const uint32_t m = bits(c);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float u = w[j] - lo;
                const float t = u * inv;
                const double q = (double)__builtin_amdgcn_fmed3f(__builtin_rintf(t), 0.0f, qmax);
                const double a = weight(m, c, j);             // a masked weight adds zeros
                const double wd = (double)w[j];
                const double aq = a * q;
                if (FIRST) {
                    S0 = S0 + a;
                    T0 = T0 + a * wd;
                }
                S1 = S1 + aq;
                S2 = TWO ? __builtin_fma(aq, q, S2) : S2 + aq * q;
                T1 = T1 + aq * wd;
            }
        });
    }

    template <bool TWO>
    __device__ __forceinline__ void uniform(float qmax, int n_iter, float* lo_io, float* d_io) const {
        float lo = *lo_io, d = *d_io;
        double S0 = 0.0, T0 = 0.0;
        for (int it = 0; it < n_iter; ++it) {
            if (!(d >= FLT_MIN)) break;
            const float inv = 1.0f / d;
            double S1, S2, T1;
            if (it == 0) uniform_sums<true, TWO>(lo, inv, qmax, S0, T0, S1, S2, T1);
            else uniform_sums<false, TWO>(lo, inv, qmax, S0, T0, S1, S2, T1);
            const double det = S0 * S2 - S1 * S1;
            if (!(det > 0.0)) break;
            const double d_new = (S0 * T1 - S1 * T0) / det;
            const double lo_new = (T0 - S1 * d_new) / S0;
            const float d32 = (float)d_new, lo32 = (float)lo_new;
            if (!(d32 >= FLT_MIN)) break;
            lo = lo32;
            d = d32;
        }
        *lo_io = lo;
        *d_io = d;
    }

    // q = clamp(rne(w / gamma)) is the sign of w where |w / gamma| > 0.5, else 0.  Without a mask the sums are
    // therefore those of s_c^2 |w| and of s_c^2 over these weights: the terms left out are zeros, the others have the same
    // bits as (s_c^2 q) w.  (A column whose s_c^2 is not finite makes both sums infinite or NaN, their quotient NaN: no round
    // changes gamma.)
    __device__ __forceinline__ float ternary(int n_iter, float gamma) const {
        if (!MASKED && !finite) return gamma;
        for (int it = 0; it < n_iter; ++it) {
            if (!(gamma >= FLT_MIN)) break;
            const float inv = 1.0f / gamma;
            double N1 = 0.0, D1 = 0.0;
            row.blocks(G, [&](int32_t c, const float (&w)[8]) {
                const uint32_t m = bits(c);
                if constexpr (!MASKED) {        // (all eight products first: the adds do not wait for LDS one by one)
                    double a[8], p[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) a[j] = acol[c + j];
#pragma unroll
                    for (int j = 0; j < 8; ++j) p[j] = a[j] * (double)fabsf(w[j]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < 8; ++j) add_where_above_half(w[j] * inv, p[j], a[j], N1, D1);
                    return;
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float t = w[j] * inv;
                    const double q = (double)__builtin_amdgcn_fmed3f(__builtin_rintf(t), -1.0f, 1.0f);
                    const double aq = weight(m, c, j) * q;
                    N1 = N1 + aq * (double)w[j];
                    D1 = D1 + fabs(aq);                       // a q^2: q is -1, 0 or 1
                }
            });
            if (!(D1 > 0.0)) break;
            const float g = (float)(N1 / D1);
            if (!(g >= FLT_MIN)) break;
            gamma = g;
        }
        return gamma;
    }

    // The seed (mean |w|) matters only where nothing is weighted.
    __device__ __forceinline__ float binary(int n_iter) const {
        if (n_iter <= 0) return abs_mean();
        double N1 = 0.0, D1 = 0.0;
        row.blocks(G, [&](int32_t c, const float (&w)[8]) {
            const uint32_t m = bits(c);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const double a = weight(m, c, j);
                N1 = N1 + a * (double)fabsf(w[j]);
                D1 = D1 + a;
            }
        });
        if (D1 > 0.0) return (float)(N1 / D1);
        return abs_mean();
    }

    // Codes under the final parameters, packed at dst (which may be the row's own LDS storage: behind the read position),
    // and the activation-weighted error (fp64; w_hat from the stored fp32 numbers, as everywhere).
    template <int BITS>
    __device__ __forceinline__ double uniform_finish(float sc, float of, uint8_t* dst) const {
        const float qmax = (float)((1 << BITS) - 1);
        const float inv = sc >= FLT_MIN ? 1.0f / sc : 0.0f;
        double e = 0.0;
        row.blocks(G, [&](int32_t c, const float (&w)[8]) {
            const uint32_t m = bits(c);
            uint32_t code[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float t = (w[j] - of) * inv;
                const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(t), 0.0f, qmax);
                const double what = __builtin_fma((double)q, (double)sc, (double)of);      // (the product is exact)
                const double d = (double)w[j] - what;
                e = e + weight(m, c, j) * d * d;
                code[j] = kept(m, j) ? (uint32_t)q : 0u;
            }
            store_codes8<BITS>(dst + (c >> 3) * BITS, code);
        });
        return e;
    }

    // Eight weights of which the first has place AT in its byte of five trits; sum: sum of q 3^place of the byte under way.
    template <int AT>
    __device__ __forceinline__ void ternary_block(int32_t c, const float (&w)[8], float sc, float inv, double& e, float& sum, uint8_t*& dst) const {
        constexpr float POW[5] = {1.0f, 3.0f, 9.0f, 27.0f, 81.0f};
        const uint32_t m = bits(c);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int at = (AT + j) % 5;
            const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(w[j] * inv), -1.0f, 1.0f);
            const double d = (double)w[j] - (double)(sc * q);                // sc q is exact
            e = e + weight(m, c, j) * d * d;
            const float trit = kept(m, j) ? q : -1.0f;                       // less one: a protected weight's trit is 0
            sum = at == 0 ? trit : __builtin_fmaf(trit, POW[at], sum);
            if (at == 4) *dst++ = (uint8_t)(uint32_t)(sum + 121.0f);
        }
    }
    __device__ __forceinline__ double ternary_finish(float sc, uint8_t* dst) const {
        const float inv = sc >= FLT_MIN ? 1.0f / sc : 0.0f;
        double e = 0.0;
        float sum = 0.0f;
        int at = 0;                                                          // the same in every lane
        row.blocks(G, [&](int32_t c, const float (&w)[8]) {
            switch (at) {
                case 0: ternary_block<0>(c, w, sc, inv, e, sum, dst); break;
                case 1: ternary_block<1>(c, w, sc, inv, e, sum, dst); break;
                case 2: ternary_block<2>(c, w, sc, inv, e, sum, dst); break;
                case 3: ternary_block<3>(c, w, sc, inv, e, sum, dst); break;
                default: ternary_block<4>(c, w, sc, inv, e, sum, dst); break;
            }
            at = at >= 2 ? at - 2 : at + 3;                                  // eight further, by fives
        });
        if (at != 0) *dst = (uint8_t)(uint32_t)(sum + (at == 1 ? 1.0f : (at == 2 ? 4.0f : (at == 3 ? 13.0f : 40.0f))));
        return e;
    }

    // (|w| - alpha is the residual of w but for its sign, which its square does not show)
    __device__ __forceinline__ double binary_finish(float sc, uint8_t* dst) const {
        double e = 0.0;
        row.blocks(G, [&](int32_t c, const float (&w)[8]) {
            const uint32_t m = bits(c);
            uint32_t byte = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const double d = (double)fabsf(w[j]) - (double)sc;
                e = e + weight(m, c, j) * d * d;
            }
#pragma unroll
            for (int j = 7; j >= 0; --j) push_not_negative(byte, w[j]);
            dst[c >> 3] = (uint8_t)(byte & ~m);
        });
        return e;
    }
};

// LDS of a tile: its rows (NV = 0), or what turns them round and stages the codes; s_c^2 of the columns; the mask bytes.
__host__ __device__ inline int32_t refine_pack_stride(int32_t G) { return G + 16; }       // 8-bit codes of a row
static size_t refine_lds(int32_t dtype, int32_t G, int nv, bool masked) {
    const size_t turn = (size_t)TILE_ROWS * RF_SLAB_STRIDE, pack = (size_t)TILE_ROWS * (size_t)refine_pack_stride(G);
    return (nv == 0 ? raw_tile_lds_bytes(dtype, G) : (turn > pack ? turn : pack)) + (size_t)G * sizeof(double) +
           (masked ? mask_tile_lds_bytes(G) : 0);
}

template <int DT, int NV>
struct RefineRowOf {
    using type = RegRow<DT, NV>;
};
template <int DT>
struct RefineRowOf<DT, 0> {
    using type = LdsRow<DT>;
};

// A tile of a uniform unit takes four times as long as one of a binary unit (at three rounds), and a launch of more
// tiles than the chip holds at once (4096 at chunk 128, bf16) ends with what came last: in the matrix's own order, where every band
// of rows has units of each kind, a 7B-shaped block took 285 us, dear units first 225.  Launches that fit keep that order:
// with 500 tiles the look at the actions costs 1 us of 20.  Skipped units come last, and one workgroup takes 16 of such a unit's
// tiles: where each looked for its own, a plan of nothing else took 18.4 us (7B-shaped block) and 17.0 (28672 x 8192), 14.4 and
// 12.7 so, 14.7 and 13.2 in the matrix's own order; 8192 x 28672, with four loads of actions per look, 20.8, 15.7 and 13.0.
constexpr int64_t RF_ORDERED_TILES = 2048;
// action:        skip      8, 4, 3, 2 bits   ternary        binary         outside the plan's
constexpr uint32_t RF_CLASSES = 3u | 0u | (1u << 10) | (2u << 12) | (3u << (2 * WINDQ_N_ACTIONS));

// Tiles of a skipped unit that one workgroup of an ordered launch takes.
constexpr int32_t RF_SKIP_TILES = 16;
// A tile of a skipped unit: scales, offsets and error are zeros.
__device__ __forceinline__ void skip_tile(const RefineArgs& A, const TileCoord& tc) {
    const int lane = threadIdx.x;
    if (lane < tc.nrows) {
        const int64_t gidx = tc.u * A.g.R_u + tc.lrow0 + lane;
        A.scale[gidx] = 0.0f;
        A.offset[gidx] = 0.0f;
    }
    if (lane == 0) A.part[(size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)tc.t] = 0.0;
}

// NV: registers of a row / 32; 0: the row in LDS.  128 VGPRs (four wavefronts per SIMD) for NV = 2.
template <int DT, int NV, bool MASKED>
__global__ __launch_bounds__(RF_THREADS, NV == 2 ? 4 : 2) void refine_plan_kernel(const RefineBatch B) {
    extern __shared__ __align__(16) char smem[];
    const int mi = batch_index(B.tile_start, B.n, blockIdx.x);
    const RefineArgs& A = B.m[mi];
    const uint32_t local = (uint32_t)((int64_t)blockIdx.x - B.tile_start[mi]);
    TileCoord tc;
    if (B.by_cost != 0 && A.g.U <= ORDER_MAX_UNITS) {
        const int32_t tiles = (int32_t)A.g.tiles_per_unit, per_skipped = (tiles + RF_SKIP_TILES - 1) / RF_SKIP_TILES;
        const OrderedItem o = item_by_cost<true>(A.action, (int32_t)A.g.U, tiles, per_skipped, (int32_t)local, RF_CLASSES);
        if (o.cls == 3) {               // zeros for every per_skipped'th tile of a skipped unit; the others have nothing to do
            if (o.unit < 0) return;
            for (int32_t t = o.item; t < tiles; t += per_skipped) skip_tile(A, tile_coord_of_unit(A.g, o.unit, t));
            return;
        }
        tc = tile_coord_of_unit(A.g, o.unit, o.item);
    } else {
        tc = tile_coord(A.g, (int64_t)local);
    }
    const int32_t G = A.g.chunk_w;
    const int lane = threadIdx.x;
    const bool valid = lane < tc.nrows;
    const int64_t gidx = tc.u * A.g.R_u + tc.lrow0 + lane;
    const size_t tile_idx = (size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)tc.t;

    int a = A.action[tc.u];
    if (a >= WINDQ_N_ACTIONS) a = 0;
    const int64_t bpg = dev_bytes_per_group(a, G);
    const int64_t base = A.code_off[tc.u];
    const int64_t payload = bpg * A.g.R_u;
    const int64_t padded = (payload + 15) & ~(int64_t)15;
    if (base < 0 || (base & 15) != 0 || base > A.codes_bytes - padded) a = 0;     // (base + padded could pass 2^63)
    if (a == 0) {
        skip_tile(A, tc);
        return;
    }

    double* acol = reinterpret_cast<double*>(smem);                              // s_c^2 of the chunk's columns
    char* tile = smem + (size_t)G * sizeof(double);
    const int32_t stride = NV == 0 ? G * Elem<DT>::bytes + 16 : refine_pack_stride(G);
    const int32_t turn = TILE_ROWS * (NV == 0 || stride > RF_SLAB_STRIDE ? stride : RF_SLAB_STRIDE);
    uint8_t* mtile = reinterpret_cast<uint8_t*>(tile + turn);                    // the tile's mask bytes (masked calls)
    RefineGroup<DT, MASKED, typename RefineRowOf<DT, NV>::type> g;
    bool finite = true;
    for (int32_t c = lane; c < G; c += RF_THREADS) {
        const double sv = (double)A.s[tc.col0 + c];
        acol[c] = sv * sv;
        finite = finite && sv * sv < (double)INFINITY;
    }
    g.finite = __all(finite);
    if (MASKED) {
        if (A.mask != nullptr) {
            load_mask_tile(A.mask, A.mask_ld, tc, G, mtile);
        } else {                                                                 // an item without one in a masked launch
            for (int32_t i = lane; i < TILE_ROWS * mask_row_stride(G); i += RF_THREADS) mtile[i] = 0;
        }
    }
    if constexpr (NV == 0) {
        load_tile_raw<DT>(A.W, A.g.ld, tc, G, tile);
        g.row.p = tile + lane * stride;
        __syncthreads();
    } else {
        load_rows<DT, NV>(A, tc, tile, g.row);
    }
    g.mrow = MASKED ? mtile + lane * mask_row_stride(G) : nullptr;
    g.acol = acol;
    g.G = G;
    g.protects = MASKED && A.mask != nullptr;

    double err = 0.0;
    if (valid) {
        uint8_t* dst = reinterpret_cast<uint8_t*>(tile + lane * stride);
        float sc = 0.0f, of = 0.0f;
        if (a <= 4) {
            float p = 1.0f;
            if (A.clip_idx != nullptr) {
                int k = A.clip_idx[tc.u * 4 + (a - 1)];
                k = k < B.K ? k : B.K - 1;
                p = B.grid.p[k];
            }
            const int bits = a == 1 ? 8 : (a == 2 ? 4 : (a == 3 ? 3 : 2));
            const float qmax = (float)((1 << bits) - 1);
            float mn, mx;
            g.min_max(&mn, &mx);
            uniform_params(mn, mx, p, qmax, &of, &sc);
            if (a == 4) g.template uniform<true>(qmax, B.n_iter, &of, &sc);
            else g.template uniform<false>(qmax, B.n_iter, &of, &sc);
            switch (a) {
                case 1: err = g.template uniform_finish<8>(sc, of, dst); break;
                case 2: err = g.template uniform_finish<4>(sc, of, dst); break;
                case 3: err = g.template uniform_finish<3>(sc, of, dst); break;
                default: err = g.template uniform_finish<2>(sc, of, dst); break;
            }
        } else if (a == 5) {
            sc = g.abs_mean();
            sc = sc >= FLT_MIN ? sc : 0.0f;
            sc = g.ternary(B.n_iter, sc);
            err = g.ternary_finish(sc, dst);
        } else {
            sc = g.binary(B.n_iter);
            err = g.binary_finish(sc, dst);
        }
        A.scale[gidx] = sc;
        A.offset[gidx] = of;
    }
    // rows of the tile in order (lane 0 first): a fixed-order fp64 sum
    err = wave_sum(err);
    if (lane == 0) A.part[tile_idx] = err;
    __syncthreads();
    copy_out_rows(tile, stride, (int32_t)bpg, tc.nrows, A.codes + base + tc.lrow0 * bpg, lane, RF_THREADS);
    if (padded != payload && tc.t == A.g.tiles_per_unit - 1 && lane < padded - payload)
        A.codes[base + payload + lane] = 0;
}

// err[u] = the sum of unit u's tile partials; one workgroup per unit.
__global__ __launch_bounds__(256) void refine_finalize_kernel(const RefineBatch B) {
    __shared__ double red[4];
    const int mi = batch_index(B.unit_start, B.n, blockIdx.x);
    const RefineArgs& A = B.m[mi];
    const int64_t u = (int64_t)blockIdx.x - B.unit_start[mi];
    const double t = unit_partial_sum<256>(A.part + (size_t)u * (size_t)A.g.tiles_per_unit, A.g.tiles_per_unit, red);
    if (threadIdx.x == 0) A.err[u] = (float)t;
}

}  // namespace windq

using namespace windq;

template <int DT, int NV, bool MASKED>
static int refine_launch_kernel(const RefineBatch& B, int32_t chunk_w, dim3 grid, hipStream_t hs) {
    const size_t lds = refine_lds(DT, chunk_w, NV, MASKED);
    const int st = ensure_lds(reinterpret_cast<const void*>(&refine_plan_kernel<DT, NV, MASKED>), lds);
    if (st != WINDQ_OK) return st;
    hipLaunchKernelGGL((refine_plan_kernel<DT, NV, MASKED>), grid, dim3(RF_THREADS), lds, hs, B);
    return WINDQ_OK;
}

// Rows of up to 256 bytes in 64 registers, up to 512 bytes in 128, wider ones in LDS.
template <int DT>
static int refine_launch_rows(const RefineBatch& B, int32_t chunk_w, bool masked, dim3 grid, hipStream_t hs) {
    const int32_t row_bytes = chunk_w * Elem<DT>::bytes;
    if (row_bytes <= 2 * RF_SLAB)
        return masked ? refine_launch_kernel<DT, 2, true>(B, chunk_w, grid, hs) : refine_launch_kernel<DT, 2, false>(B, chunk_w, grid, hs);
    if (row_bytes <= 4 * RF_SLAB)
        return masked ? refine_launch_kernel<DT, 4, true>(B, chunk_w, grid, hs) : refine_launch_kernel<DT, 4, false>(B, chunk_w, grid, hs);
    return masked ? refine_launch_kernel<DT, 0, true>(B, chunk_w, grid, hs) : refine_launch_kernel<DT, 0, false>(B, chunk_w, grid, hs);
}

static int refine_launch(const windq_refine_item* items, int32_t n, int32_t chunk_w, int64_t unit_rows,
                         const float* clip_grid, int32_t K, int32_t n_iter, void* stream) {
    if (items == nullptr || n < 1 || n > WINDQ_MAX_BATCH) return WINDQ_EINVAL;
    if (n_iter < 0 || n_iter > 64) return WINDQ_EINVAL;
    bool any_idx = false, any_mask = false;
    for (int32_t i = 0; i < n; ++i) {
        any_idx = any_idx || items[i].clip_idx != nullptr;
        any_mask = any_mask || items[i].mask != nullptr;
    }
    int st;
    if (any_idx || clip_grid != nullptr) {
        st = check_clip_grid(clip_grid, K);
        if (st != WINDQ_OK) return st;
    } else {
        K = 1;
    }
    RefineBatch B;
    B.n = n;
    B.K = K;
    B.n_iter = n_iter;
    for (int k = 0; k < WINDQ_MAX_CLIP; ++k) B.grid.p[k] = clip_grid != nullptr ? clip_grid[k < K ? k : K - 1] : 1.0f;
    int64_t tiles = 0, units = 0;
    for (int32_t i = 0; i < n; ++i) {
        const windq_refine_item& it = items[i];
        RefineArgs& A = B.m[i];
        if (it.W == nullptr) return WINDQ_EINVAL;
        st = make_geometry(it.W, chunk_w, unit_rows, &A.g);
        if (st != WINDQ_OK) return st;
        if (it.s == nullptr || it.action == nullptr || it.code_off == nullptr || it.scale == nullptr ||
            it.offset == nullptr || it.err == nullptr)
            return WINDQ_EINVAL;
        if (it.codes == nullptr && it.codes_bytes != 0) return WINDQ_EINVAL;
        if (it.codes != nullptr && !aligned(it.codes, 16)) return WINDQ_EINVAL;
        if (!aligned(it.code_off, 8)) return WINDQ_EINVAL;
        if (it.W->dtype != items[0].W->dtype) return WINDQ_EINVAL;      // one kernel per launch
        if (it.ws == nullptr || it.ws_bytes < unit_saliency_ws_bytes(A.g) || !aligned(it.ws, 256)) return WINDQ_EWORKSPACE;
        A.W = it.W->data;
        A.s = it.s;
        A.mask = it.mask;
        A.mask_ld = it.W->cols / 8;
        A.action = it.action;
        A.clip_idx = clip_grid != nullptr ? it.clip_idx : nullptr;
        A.code_off = it.code_off;
        A.codes = it.codes;
        A.codes_bytes = (int64_t)it.codes_bytes;
        A.scale = it.scale;
        A.offset = it.offset;
        A.part = static_cast<double*>(it.ws);
        A.err = it.err;
        B.tile_start[i] = tiles;
        B.unit_start[i] = units;
        tiles += A.g.n_tiles;
        units += A.g.U;
    }
    for (int32_t i = n; i <= WINDQ_MAX_BATCH; ++i) {
        B.tile_start[i] = tiles;
        B.unit_start[i] = units;
    }
    for (int32_t i = n; i < WINDQ_MAX_BATCH; ++i) B.m[i] = B.m[0];
    if (!fits_launch(tiles, RF_THREADS) || !fits_launch(units, 256)) return WINDQ_ESHAPE;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const int32_t dtype = items[0].W->dtype;
    B.by_cost = tiles > RF_ORDERED_TILES ? 1 : 0;
    const dim3 grid((unsigned)tiles);
    st = dtype == WINDQ_BF16 ? refine_launch_rows<WINDQ_BF16>(B, chunk_w, any_mask, grid, hs) : refine_launch_rows<WINDQ_F32>(B, chunk_w, any_mask, grid, hs);
    if (st != WINDQ_OK) return st;
    hipLaunchKernelGGL(refine_finalize_kernel, dim3((unsigned)units), dim3(256), 0, hs, B);
    return hipPeekAtLastError() == hipSuccess ? WINDQ_OK : WINDQ_EHIP;
}

extern "C" int windq_refine_plan(const windq_mat* W, const float* s, int32_t chunk_w, int64_t unit_rows,
                                 const uint8_t* mask, const uint8_t* action, const uint8_t* clip_idx,
                                 const float* clip_grid, int32_t K, int32_t n_iter, const int64_t* code_off,
                                 uint8_t* codes, size_t codes_bytes, float* scale, float* offset, float* err, void* ws,
                                 size_t ws_bytes, void* stream) {
    const windq_refine_item it = {W, s, mask, action, clip_idx, code_off, codes, codes_bytes, scale, offset, err, ws, ws_bytes};
    return refine_launch(&it, 1, chunk_w, unit_rows, clip_grid, K, n_iter, stream);
}

extern "C" int windq_refine_plan_batch(const windq_refine_item* items, int32_t n, int32_t chunk_w, int64_t unit_rows,
                                       const float* clip_grid, int32_t K, int32_t n_iter, void* stream) {
    return refine_launch(items, n, chunk_w, unit_rows, clip_grid, K, n_iter, stream);
}
