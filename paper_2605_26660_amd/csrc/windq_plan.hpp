// fit+score heavy columns first (part of fit_score.hip).
//
// Activation scales differ so much between channels that a few of a chunk's columns hold most of the sum of s_c^2, and with it of
// every candidate's error.  What a candidate's heaviest columns add up to is a lower bound on its error, and most candidates'
// bounds already pass the least error of their bit-width.  So the columns are put in the order of their weight, the tiles
// score every candidate on the heavy ones (fit_heavy_kernel), and per unit a plan says which candidates go on, and to how many
// columns (fit_plan_kernel); the main kernel scores those (score_list) beside its other work.
//   The plan estimates the light columns' part of an error from a sample of the tiles.  The finalize step proves the choice as it
// does for the 8-bit candidates that are left out: the sum of every candidate that has not taken all columns exceeds the
// chosen error, or the unit is listed and its open candidates are scored on all columns (fit_score_redo_kernel).  So the
// estimate decides speed, never the result.
#pragma once

namespace windq {

// Which matrices: bf16, no mask, 2048 tiles or more, units of 1024 rows (16 tiles) or more, chunks of 64, 128, 192 or 256 columns, and clip
// ratios times columns 2560 or more.  The tiles are read and set up a second time (the heavy columns' kernel: 2948 vector instructions a
// wavefront and tile at chunk 128, 20 ratios, two thirds of them in its sweeps) and the call has two launches more, which
// large matrices and large chunks' sweeps pay for.  Features and fit of one matrix a call, us in one piece, then what heavy columns first
// changes for scales that are (a) log-normal of sigma 1 with one column in a hundred 30 times larger, (b) log-normal of sigma 1, (c) of 0.7, and
// (d) flat (0.3: scored in one piece all the same, the two launches, 8.6 us and 0.35 for a thousand tiles, find nothing to do):
//                                                 tiles   us   (a)   (b)   (c)   (d) %
//   chunk 128, 20 ratios   2816 x 4096             1408  103    +4   +13   +23    +9     not so
//                          3584 x 4096             1792  115    +4    +9   +21    +8     not so
//                          4096 x 4096             2048  131    -6    +1   +13    +7
//                          5120 x 5120             3200  187   -13    -8    +1    +5
//                          8192 x 4096             4096  228   -16   -11    +1    +4
//                          8192 x 8192             8192  437   -31   -20    -7    +3
//   chunk 64, 40 ratios    1024 x 6144             1536  104    +3   +26   +50    +9     not so
//                          1024 x 8192             2048  131    -6    +2    +6    +7
//                          2048 x 8192             4096  227   -16   -11    +1    +4
//   chunk 256, 20 ratios   4096 x 4096             1024  150    +7   +15   +25    +6     not so
//                          8192 x 8192             4096  493   -30   -17    -8    +3
//   chunk 128, 20, in one call: four 4096 x 4096   8192  418   -25   -17    -6    +3
//                               7B-shaped block   24704 1222   -29   -22   -10    +1
//   chunk 64, 40, in one call: two 1024 x 8192     4096  230   -16   -11    -1    +4
// So the line of 2048 tiles is where a matrix by itself breaks even on (a); in a batch, whose matrices share the launches, it gains on all but
// flat scales from there.  (The matrix alone decides, so that a batch has the bits of its single calls: a line for single calls would be one for batches.)
//   Fewer rows: 512 rows (8 tiles, of which 3 are probed) 512 x 32768 132 +6 -1 +11 +7; 768 x 24576 147 -9 -3 +9 +6: the line could lie at 768.
//   Less work: chunk 128 with 16 ratios 4096 x 4096 129 -9 -3 +36 +7 and 8192 x 8192 433 -32 -23 +4 +3; 18 ratios 130 -7 0 +9 +7 and 435 -32 -21 -6
// +3; chunk 64 with 30 ratios 4096 x 4096 193 -6 +3 +21 +5 and 8192 x 8192 655 -25 -13 +9 +2, with 20 ratios 456 -2 +8 +5 +4.  There scales like (c) leave
// a quarter of the chunks in one piece by their cost, and chunks of both kinds side by side are the slowest: to let 16 to 19 ratios
// in (which take longer than 20 on steep scales) the rule on steep scales would have to be stricter for less work.
//   Other chunks: steep_matrix reads 64 scales at a time.  Chunk 96 (with a bound there) at 40 ratios, 4096 x 6144 319 -26 -18 -2 +3, at 20 ratios
// 181 -9 -2 +22 +5; chunk 160, 20 ratios, 4096 x 7680 215 -16 -8 +4 +4.  Not open yet.
//   Seen on the first version of these kernels only (half as many probed tiles): fp32, whose tiles leave three workgroups a CU, 203 -> 223 us; under a mask, which
// takes the largest products out and the columns' difference with them, 451 -> 620 us, 296 of them for units scored again.
constexpr int64_t PLAN_MIN_TILES = 2048;
constexpr int32_t PLAN_MIN_WORK = 2560;
constexpr int64_t PLAN_MIN_ROWS = 1024;
constexpr int64_t PLAN_MAX_UNITS = 1 << 18;       // of a matrix: eight of them stay within a launch
// What a chunk's scoring costs per candidate and row, in instructions of the fast kind: a heavy column COST_HEAVY; a light one
// COST_LIGHT (1 - share)^0.3, six for each candidate that goes on, whose number falls so with the heavy columns' share of the weight; a tile
// COST_TILE for its second load and the second set of parameters and sums.  A chunk is scored heavy columns first where that is less than in one piece.
// (COST_LIGHT 3.8 or 5.5: a 7B-shaped block within 1 %; 2.6: 8 % slower, its light columns leave twice as many candidates.)
constexpr float COST_HEAVY = 4.85f, COST_LIGHT = 4.8f, COST_TILE = 8000.0f;
// Tiles that are asked for the light columns' part of the least errors too: every second one of a unit of fewer than 32 tiles, every fourth below 64, every
// eighth from there, and not the first two, whose noise slots are in use (a probed tile has it there: three sums, then the heavy columns' errors
// that they belong to): 7 of 16 tiles, 15 of 31, 8 of 32, 8 of 64, 22 of 172.  (Units of 16 tiles with four probed: one in fifty scored again,
// 1024 x 8192 at chunk 64, 40 ratios 143 us; with seven, one in four hundred, 124; in one piece 131.)
constexpr int PROBE_FIRST = 2;
__device__ __forceinline__ int probe_every(int64_t tiles_per_unit) { return tiles_per_unit >= 64 ? 8 : (tiles_per_unit >= 32 ? 4 : 2); }
__device__ __forceinline__ bool probe_tile(int64_t t, int64_t tiles_per_unit) { return t >= PROBE_FIRST && (int)(t - PROBE_FIRST) % probe_every(tiles_per_unit) == 0; }
constexpr int PREP_ROWS = 32;                     // sampled for the columns' weight

static bool by_plan(const Geometry& g, int32_t dtype, bool masked, int32_t K) {
    return dtype == WINDQ_BF16 && !masked && K >= FS_PLAN_MIN_K && K * g.chunk_w >= PLAN_MIN_WORK && g.chunk_w % 64 == 0 &&
           g.chunk_w <= FS_PLAN_MAX_CHUNK && g.R_u >= PLAN_MIN_ROWS && g.n_tiles >= PLAN_MIN_TILES && g.U <= PLAN_MAX_UNITS;
}
// Workgroups of the preparing kernel that make a matrix's records.
__host__ __device__ __forceinline__ int64_t prepare_groups(const FitScoreMat& M) {
    return M.planned != 0 ? M.g.n_chunks : (M.g.n_chunks + FS_PREP_CHUNKS - 1) / FS_PREP_CHUNKS;
}
__device__ __forceinline__ int32_t chunk_heavy(const FitScoreMat& A, int64_t j) {
    return heavy_columns(__builtin_amdgcn_readfirstlane(__float_as_int(A.colsel[(size_t)j * (size_t)colsel_words(A.g.chunk_w) + A.g.chunk_w + FS_HMAX])));
}
// The share of a chunk's weight that the columns up to each step of PLAN_STEPS hold, and then the heavy ones: with the chunk's first unit.
__device__ __forceinline__ float* chunk_shares(const FitScoreMat& A, int32_t K, int64_t j) {
    return fit_listed(A.partial + (size_t)j * (size_t)A.g.tiles_per_unit * (size_t)fit_score_ncand(K), K)->shares;
}
static_assert(PLAN_MIN_ROWS > PROBE_FIRST * TILE_ROWS, "a second tile, and one that is probed");

// Whether a matrix's scales are steep enough: (sum s)^2 <= STEEP G sum s^2 in at least three quarters of sixteen chunks spread over it (all, where it has
// fewer).  Chunks in one piece and chunks heavy columns first do not mix well in a launch, and a matrix of which only a few chunks gain
// is slower by the other kernels' time.  Two 4096 x 4096 and one 11008 x 4096, chunk 128, 20 ratios, us in one piece / by the chunks' costs alone / with
// this rule: log-normal scales of sigma 0.3 485 / 544 / 495, 0.7 486 / 468 / 469, 1.0 488 / 416 / 417; sigma 0.3 with 2 % of them x5
// 487 / 559 / 497, 0.1 % x30 489 / 537 / 497, 5 % x10 491 / 410 / 414; chunk 64, 40 ratios, sigma 0.7 929 / 854 / 853 (933 with STEEP 0.69).
// What is left above one piece is the two further launches, which find nothing to do.  A stricter rule for small matrices gives single calls
// with scales of sigma 0.7 some of their loss back (STEEP 0.5 below 3072 tiles: 4096 x 4096 +14 -> +7 % over one piece) and takes more from batches (a
// 7B-shaped block -10 -> -6 %, two 1024 x 8192 with scales of sigma 1 -11 -> 0).  The weights are not looked at here: flat scales over columns of
// very different weights are scored in one piece.
constexpr int STEEP_SAMPLE = 16;
constexpr float STEEP = 0.75f;
__device__ __forceinline__ bool steep_matrix(const FitScoreMat& A) {
    __shared__ int32_t steep[FS_WAVES];
    constexpr int PER = STEEP_SAMPLE / FS_WAVES;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int32_t G = A.g.chunk_w, n = A.g.n_chunks < STEEP_SAMPLE ? (int32_t)A.g.n_chunks : STEEP_SAMPLE;
    float s1[PER], s2[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int32_t at = i * FS_WAVES + wave;
        const float* __restrict__ sc = A.s + ((int64_t)at * A.g.n_chunks / n) * G;
        s1[i] = s2[i] = 0.0f;
#pragma unroll
        for (int32_t c = 0; c < FS_PLAN_MAX_CHUNK; c += 64) {
            const float v = at < n && c < G ? sc[c + lane] : 0.0f;
            s1[i] += v;
            s2[i] = fmaf(v, v, s2[i]);
        }
    }
    int32_t count = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const float t1 = wave_sum_f32(s1[i]), t2 = wave_sum_f32(s2[i]);
        count += t1 * t1 < STEEP * (float)G * t2 ? 1 : 0;
    }
    if (lane == 0) steep[wave] = count;
    __syncthreads();
    return 4 * (steep[0] + steep[1] + steep[2] + steep[3]) >= 3 * n;
}
static_assert(FS_WAVES == 4, "steep_matrix adds four counts");

// The record of chunk j, by a workgroup, a column a thread; false (and nothing written) where scoring in one piece is expected to cost
// less.  A column's weight is s_c^2 times the root mean square of its weights, from a few rows: a column of large weights
// has larger residuals, but not by as much (clipping, and the range it gives to all columns, see to that).
__device__ __forceinline__ bool prepare_planned(const FitScoreArgs& B, const FitScoreMat& A, int64_t j) {
    __shared__ __align__(16) float keys[FS_PLAN_MAX_CHUNK];
    __shared__ float sorted[FS_PLAN_MAX_CHUNK], run[FS_PLAN_MAX_CHUNK / 8], upto[FS_PLAN_MAX_CHUNK / 8], ss_part[FS_WAVES];
    __shared__ int32_t heavy_sh;
    static_assert(FS_THREADS >= FS_PLAN_MAX_CHUNK, "a column a thread");
    if (!steep_matrix(A)) return false;                                                     // (the same for every chunk)
    const int32_t G = A.g.chunk_w, c = threadIdx.x, runs = G >> 3;
    const bool in = c < G;
    const float sv = in ? A.s[j * G + c] : 0.0f;
    float w2 = 0.0f;
    if (in) {
        const uint16_t* __restrict__ col = static_cast<const uint16_t*>(A.W) + j * G + c;
#pragma unroll 16
        for (int i = 0; i < PREP_ROWS; ++i) {
            const float w = bf16_bits_to_f32(col[(((int64_t)i * A.g.rows) / PREP_ROWS) * A.g.ld]);
            w2 = fmaf(w, w, w2);
        }
    }
    const float key = sv * sv * sqrtf(w2);
    keys[c] = key;
    sorted[c] = 0.0f;
    const float ss = wave_sum_f32(sv * sv);
    if ((c & 63) == 0) ss_part[c >> 6] = ss;
    if (__syncthreads_or(key == key && key <= FLT_MAX ? 0 : 1) != 0) return false;         // (the same for the whole workgroup)
    int at = 0;
    for (int32_t o = 0; o < G; o += 4) {
        const float4 k = *reinterpret_cast<const float4*>(keys + o);
        at += (k.x > key || (k.x == key && o < c) ? 1 : 0) + (k.y > key || (k.y == key && o + 1 < c) ? 1 : 0) +
              (k.z > key || (k.z == key && o + 2 < c) ? 1 : 0) + (k.w > key || (k.w == key && o + 3 < c) ? 1 : 0);
    }
    if (in) sorted[at] = key;
    __syncthreads();
    if (c < runs) {
        float sum = 0.0f;
#pragma unroll
        for (int t = 0; t < 8; ++t) sum += sorted[8 * c + t];
        run[c] = sum;
    }
    __syncthreads();
    if (c < 64) {
        float sum = 0.0f, whole = 0.0f;
        for (int32_t r = 0; r < runs; ++r) {
            whole += run[r];
            if (r <= c) sum += run[r];
        }
        if (c < runs) upto[c] = sum;
        // the cost of taking the columns up to here as heavy, per candidate and row (in fast instructions)
        const float n = 8.0f * (float)(c + 1), share = sum / whole;
        float cost = 2 * (c + 1) <= runs && share >= 0.5f ? n * COST_HEAVY + ((float)G - n) * COST_LIGHT * powf(fmaxf(1.0f - share, 0.0f), 0.3f) : INFINITY;
        if (!(whole > 0.0f && whole <= FLT_MAX)) cost = INFINITY;
        int best = c;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const float oc = __shfl_xor(cost, m, 64);
            const int ob = __shfl_xor(best, m, 64);
            if (oc < cost || (oc == cost && ob < best)) {
                cost = oc;
                best = ob;
            }
        }
        if (c == 0) heavy_sh = cost + COST_TILE / (float)(3 * B.K) < COST_HEAVY * (float)G ? 8 * (best + 1) : 0;
    }
    __syncthreads();
    const int32_t heavy = heavy_sh;
    if (heavy == 0) return false;
    float* __restrict__ rec = A.colsel + (size_t)j * (size_t)colsel_words(G);
    if (in) {
        rec[at] = sv;
        reinterpret_cast<uint8_t*>(rec + G)[c] = (uint8_t)at;
    }
    if (c <= PLAN_STEPS) chunk_shares(A, B.K, j)[c] = upto[(c < PLAN_STEPS ? plan_columns(G, c) : heavy) / 8 - 1] / upto[runs - 1];
    if (c == 0) {
        reinterpret_cast<int32_t*>(rec)[G + FS_HMAX] = -1 - heavy;
        rec[G + FS_HMAX + 1] = 0.0f;
        rec[G + FS_HMAX + 2] = ((ss_part[0] + ss_part[1]) + ss_part[2]) + ss_part[3];
    }
    return true;
}

// ---- tiles
// Loads rows with their columns in the plan's order.  src_row(r): first column of the tile's row r, or null.
template <typename ROW>
__device__ __forceinline__ void load_rows_placed(const ROW& src_row, int32_t G, const uint8_t* __restrict__ place, char* __restrict__ tile) {
    constexpr int NB = 4;
    const int32_t pieces = G >> 3, row_bytes = G * 2 + 16, total = TILE_ROWS * pieces;
    if ((pieces & (pieces - 1)) == 0 && pieces >= 4) {
        // a thread's pieces lie below one another: its columns' places once
        const int32_t r0 = (int32_t)((uint32_t)threadIdx.x / (uint32_t)pieces), pc = (int32_t)threadIdx.x - r0 * pieces, dr = FS_THREADS / pieces;
        const uint2 places = *reinterpret_cast<const uint2*>(place + pc * 8);
        int32_t to[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) to[j] = (int32_t)(((j < 4 ? places.x : places.y) >> (8 * (j & 3))) & 0xffu) * 2;
        for (int32_t r = r0; r < TILE_ROWS; r += NB * dr) {
            uint4 v[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                v[k] = make_uint4(0u, 0u, 0u, 0u);
                if (r + k * dr < TILE_ROWS) {
                    const char* src = src_row(r + k * dr);
                    if (src != nullptr) v[k] = *reinterpret_cast<const uint4*>(src + pc * 16);
                }
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                if (r + k * dr < TILE_ROWS) {
                    char* __restrict__ row = tile + (r + k * dr) * row_bytes;
                    const uint32_t x[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
                    for (int j = 0; j < 8; ++j) *reinterpret_cast<uint16_t*>(row + to[j]) = (uint16_t)(j & 1 ? x[j >> 1] >> 16 : x[j >> 1]);
                }
            }
        }
        return;
    }
    PieceWalk at((int32_t)threadIdx.x, FS_THREADS, pieces);
    for (int32_t i = threadIdx.x; i < total; i += FS_THREADS) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        const char* src = src_row(at.r);
        if (src != nullptr) v = *reinterpret_cast<const uint4*>(src + at.pc * 16);
        scatter_piece(tile + at.r * row_bytes, v, place + at.pc * 8);
        at.next();
    }
}
// (min, max) of a wavefront's quarter of the columns, to gstat; called by all threads, ends before a barrier.
__device__ __forceinline__ void quarter_ranges(const char* __restrict__ wrow, int32_t G, int wave, int lane, float2* __restrict__ gstat) {
    const int32_t runs = G >> 3;
    float mn = INFINITY, mx = -INFINITY;
    for (int32_t c = ((wave * runs) >> 2) << 3; c < (((wave + 1) * runs) >> 2) << 3; c += 8) {
        float w[8];
        read8<WINDQ_BF16>(wrow, c, w);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            mn = fminf(mn, w[t]);
            mx = fmaxf(mx, w[t]);
        }
    }
    gstat[wave * TILE_ROWS + lane] = make_float2(mn, mx);
}
__device__ __forceinline__ float2 row_range(const float2* __restrict__ gstat, int lane) {
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < FS_WAVES; ++q) {
        const float2 st = gstat[q * TILE_ROWS + lane];
        mn = fminf(mn, st.x);
        mx = fmaxf(mx, st.y);
    }
    return make_float2(mn, mx);
}

// ---- scoring by a list
// The list as the wavefronts read it: per entry the clip ratio and (columns << 8) | (bit-width << 6) | ratio.
__device__ __forceinline__ int plan_entries(const uint8_t (&n)[PLAN_STEPS]) {
    int sum = 0;
#pragma unroll
    for (int s = 0; s < PLAN_STEPS; ++s) sum += n[s];
    return sum;
}
__device__ __forceinline__ void plan_table(const float* __restrict__ grid, const FitPlan* __restrict__ plan, int32_t G, float2* __restrict__ table) {
    const int n_low = plan_entries(plan->low), n = n_low + plan_entries(plan->high);
    const int i = threadIdx.x;
    static_assert(FS_THREADS >= 4 * WINDQ_MAX_CLIP, "an entry a thread");
    if (i >= n) return;
    const bool high = i >= n_low;
    int left = high ? i - n_low : i, cols = 8;
    bool found = false;
#pragma unroll
    for (int s = PLAN_STEPS - 1; s >= 0; --s) {
        const int here = high ? plan->high[s] : plan->low[s];
        if (!found && left < here) {
            cols = plan_columns(G, s);
            found = true;
        }
        left -= here;
    }
    const uint32_t e = plan->list[i];
    table[i] = make_float2(grid[e & 63u], __uint_as_float((uint32_t)cols << 8 | e));
}

constexpr int LIST_MOST = 6;             // low candidates of a sweep (5 or 4: the same time within 1 %)

struct LowParams {
    float rinv, h;     // x = clamp01(w rinv + h): the position in the clipped range
    float codes;       // 2^b - 1
    float nlo, nd;     // -lo, -step
};
__device__ __forceinline__ LowParams low_params(float p, int b, float mn, float mx) {
    LowParams L;
    const float lo = p * mn, rg = p * mx - lo;
    const float rinv = rg >= FLT_MIN ? __builtin_amdgcn_rcpf(rg) : 0.0f;
    // (the correctly rounded quotient, as in fit_score_tile)
    float d = (float)((double)rg * (b == 1 ? 1.0 / 15.0 : (b == 2 ? 1.0 / 7.0 : 1.0 / 3.0)));
    d = d >= FLT_MIN ? d : 0.0f;
    L.rinv = pin_vgpr(rinv);
    L.h = pin_vgpr(-lo * rinv);
    L.codes = pin_vgpr(b == 1 ? 15.0f : (b == 2 ? 7.0f : 3.0f));
    L.nlo = pin_vgpr(-lo);
    L.nd = pin_vgpr(-d);
    return L;
}
struct Params8 {
    float rinv, h, nc, Mq, nd;      // as in KParams
};

// The first P of the candidates at 4 bits or less over columns c .. c1, 6 instructions a weight each.
// They form the reconstruction first, v = -(lo + code step), and then s_c (w - what) = s_c w + s_c v: with a range and a
// bit-width of its own for each candidate this is as short as the steps of score_low_bits, whose shared parts it has not.
// Stage by stage over the candidates (and, where they are few, over weights side by side), as in score_weight_short.
template <int P, bool ANCHORED, int MOST>
__device__ __forceinline__ void low_sweep(const char* __restrict__ wrow, const float* __restrict__ ss, int32_t& c, const int32_t c1,
                                          const LowParams (&L)[MOST], const float M, float (&acc)[MOST]) {
    constexpr int SIDE = P >= 4 ? 1 : (P >= 2 ? 2 : 4);
    for (; c < c1; c += 8) {
        float w[8];
        read8<WINDQ_BF16>(wrow, c, w);
        const float4 sa = *reinterpret_cast<const float4*>(ss + c);
        const float4 sb = *reinterpret_cast<const float4*>(ss + c + 4);
        const float s8[8] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
#pragma unroll
        for (int g = 0; g < 8; g += SIDE) {
            float t[SIDE][P], w1[SIDE];
#pragma unroll
            for (int a = 0; a < SIDE; ++a) {
                w1[a] = w[g + a] * s8[g + a];
#pragma unroll
                for (int i = 0; i < P; ++i)
                    t[a][i] = ANCHORED ? fma_clamp01(w[g + a], L[i].rinv, L[i].h) : mul_clamp01(w[g + a] + L[i].nlo, L[i].rinv);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < SIDE; ++a) {
#pragma unroll
                for (int i = 0; i < P; ++i) t[a][i] = fmaf(t[a][i], L[i].codes, M);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < SIDE; ++a) {
#pragma unroll
                for (int i = 0; i < P; ++i) t[a][i] = t[a][i] - M;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < SIDE; ++a) {
#pragma unroll
                for (int i = 0; i < P; ++i) t[a][i] = fmaf(t[a][i], L[i].nd, L[i].nlo);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < SIDE; ++a) {
#pragma unroll
                for (int i = 0; i < P; ++i) t[a][i] = fmaf(t[a][i], s8[g + a], w1[a]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < SIDE; ++a) {
#pragma unroll
                for (int i = 0; i < P; ++i) acc[i] = fmaf(t[a][i], t[a][i], acc[i]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// One candidate at 8 bits, on the exact route (exact_residual8), four weights side by side.
template <bool ANCHORED>
__device__ __forceinline__ float high_sweep(const char* __restrict__ wrow, const float* __restrict__ ss, const int32_t c0, const int32_t c1, const Params8& X) {
    const float M = pin_vgpr(RNE_POS), Q8 = pin_vgpr(255.0f);
    KParams P;
    P.rinv = X.rinv;
    P.h = X.h;
    P.nc = X.nc;
    P.Mq = X.Mq;
    P.nd[0] = X.nd;
    float acc = 0.0f;
    for (int32_t c = c0; c < c1; c += 8) {
        float w[8];
        read8<WINDQ_BF16>(wrow, c, w);
        const float4 sa = *reinterpret_cast<const float4*>(ss + c);
        const float4 sb = *reinterpret_cast<const float4*>(ss + c + 4);
        const float s8[8] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
        if (!ANCHORED) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                float x;
                const float r = exact_residual8<false, false>(w[t], s8[t], P, Q8, M, x);
                acc = fmaf(r, r, acc);
            }
            continue;
        }
#pragma unroll
        for (int g = 0; g < 8; g += 4) {
            float t[4];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < 4; ++a) t[a] = fma_clamp01(w[g + a], X.rinv, X.h);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < 4; ++a) t[a] = fmaf(t[a], Q8, M);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < 4; ++a) t[a] = t[a] - X.Mq;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < 4; ++a) t[a] = fmaf(t[a], X.nd, w[g + a]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < 4; ++a) t[a] = t[a] + X.nc;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < 4; ++a) t[a] = t[a] * s8[g + a];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < 4; ++a) acc = fmaf(t[a], t[a], acc);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return acc;
}

// A tile by its unit's list.  Entries go to the wavefronts by turns, back and forth (0 1 2 3 3 2 1 0 ...; the 8-bit ones from the other
// end), so that all get as many columns; a wavefront takes up to MOST of its low ones in a sweep, which goes on with fewer as
// the shorter ones end.  From column c0 on; the sums are added to the tile's.  PAST: they take the place of the tile's, stored past
// the L2s (another workgroup of the launch adds them up).
// collected(lane, total): called once, with the sums of the first collection (its last columns hold what the tile has laid down before).
template <bool PAST, int NROW, int MOST, typename F>
__device__ __forceinline__ void score_list(const FitScoreArgs& B, const FitPlan* __restrict__ plan, const float2* __restrict__ table, const char* __restrict__ tile,
                                           int32_t row_bytes, const float* __restrict__ ss, int32_t c0, int nrows,
                                           float mn, float mx, int wave, int rot, float* __restrict__ red, double* __restrict__ out, const F& collected) {
    const int32_t K = B.K;
    const bool anchored = __builtin_amdgcn_ballot_w64(!(mn <= 0.0f && mx >= 0.0f)) == 0;
    const int n_low = __builtin_amdgcn_readfirstlane(plan_entries(plan->low)), n_high = __builtin_amdgcn_readfirstlane(plan_entries(plan->high));
    const int q = (wave + rot) & (FS_WAVES - 1);
    const auto turn = [](int r, int w) -> int { return FS_WAVES * r + ((r & 1) != 0 ? FS_WAVES - 1 - w : w); };
    const auto turns = [&](int n, int w) -> int { return n / FS_WAVES + (turn(n / FS_WAVES, w) < n ? 1 : 0); };
    const auto code = [&](int i) -> uint32_t { return __builtin_amdgcn_readfirstlane(__float_as_uint(table[i].y)); };
    const auto store = [&](int i, double tot) {
        const uint32_t e = __float_as_uint(table[i].y);
        double* slot = out + ((e >> 6) & 3u) * K + (e & 63u);
        if (PAST) __hip_atomic_store(slot, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else *slot += tot;
    };
    using std::integral_constant;
    int ncollect = NROW;
    const auto collect = [&](int lane, int n) -> double {
        const double tot = rows_collect<NROW>(red, lane, ncollect > n ? ncollect : n);
        if (ncollect != 0) collected(lane, tot);
        ncollect = 0;
        return tot;
    };

    const int my_low = turns(n_low, q);
    for (int r0 = 0; r0 < my_low;) {
        const int left = my_low - r0, rounds = anchored ? (left + MOST - 1) / MOST : left;
        const int p = (left + rounds - 1) / rounds;
        LowParams L[MOST];
        float acc[MOST];
        int32_t c1[MOST];
#pragma unroll
        for (int i = 0; i < MOST; ++i) {
            acc[i] = 0.0f;
            c1[i] = 0;
            if (i < p) {
                const int at = turn(r0 + i, q);
                const float pr = table[at].x;
                const uint32_t e = code(at);
                const int b = (int)((e >> 6) & 3u);
                c1[i] = (int32_t)(e >> 8);
                L[i] = low_params(pr, b, mn, mx);
            }
        }
        const float M = pin_vgpr(RNE_POS);
        __builtin_amdgcn_s_setprio(0);
        const int lane_v = fresh_lane();
        const char* __restrict__ wrow = tile + lane_v * row_bytes;
        int32_t c = c0;
        if (!anchored) {           // no group of real weights: one candidate at a time
            low_sweep<1, false, MOST>(wrow, ss, c, c1[0], L, M, acc);
        } else {
            if constexpr (MOST >= 6) { if (p >= 6) low_sweep<6, true, MOST>(wrow, ss, c, c1[5], L, M, acc); }
            if constexpr (MOST >= 5) { if (p >= 5) low_sweep<5, true, MOST>(wrow, ss, c, c1[4], L, M, acc); }
            if constexpr (MOST >= 4) { if (p >= 4) low_sweep<4, true, MOST>(wrow, ss, c, c1[3], L, M, acc); }
            if constexpr (MOST >= 3) { if (p >= 3) low_sweep<3, true, MOST>(wrow, ss, c, c1[2], L, M, acc); }
            if (p >= 2) low_sweep<2, true, MOST>(wrow, ss, c, c1[1], L, M, acc);
            low_sweep<1, true, MOST>(wrow, ss, c, c1[0], L, M, acc);
        }
        __builtin_amdgcn_s_setprio(3);
        const int lane = fresh_lane();
        if (lane >= nrows) {
#pragma unroll
            for (int i = 0; i < MOST; ++i) acc[i] = 0.0f;
        }
        rows_deposit<NROW>(acc, red, lane, 0);
        const double tot = collect(lane, MOST);
        if (lane < p) store(turn(r0 + lane, q), tot);
        r0 += p;
    }
    const int my_high = turns(n_high, FS_WAVES - 1 - q);
    for (int r = 0; r < my_high; ++r) {
        const int at = n_low + turn(r, FS_WAVES - 1 - q);
        const float pr = table[at].x;
        const int32_t c1 = (int32_t)(code(at) >> 8);
        const float lo = pr * mn, hi = pr * mx, rg = hi - lo;
        const float rinv = rg >= FLT_MIN ? __builtin_amdgcn_rcpf(rg) : 0.0f;
        float d = (float)((double)rg * (1.0 / 255.0));
        d = d >= FLT_MIN ? d : 0.0f;
        float q0 = 0.0f;
        if (lo <= 0.0f && hi >= 0.0f) q0 = __builtin_amdgcn_fmed3f(__builtin_rintf(-lo * rinv * 255.0f), 0.0f, 255.0f);
        const float cc = fmaf(q0, d, lo);
        Params8 X;
        X.rinv = pin_vgpr(rinv);
        X.h = pin_vgpr((anchored ? -lo : cc - lo) * rinv);
        X.nc = pin_vgpr(-cc);
        X.Mq = pin_vgpr(RNE_POS + q0);
        X.nd = pin_vgpr(-d);
        __builtin_amdgcn_s_setprio(0);
        const int lane = fresh_lane();
        const char* __restrict__ wrow = tile + lane * row_bytes;
        float acc[1];
        acc[0] = anchored ? high_sweep<true>(wrow, ss, c0, c1, X) : high_sweep<false>(wrow, ss, c0, c1, X);
        __builtin_amdgcn_s_setprio(3);
        if (lane >= nrows) acc[0] = 0.0f;
        rows_deposit<NROW>(acc, red, lane, 0);
        const double tot = collect(lane, 1);
        if (lane == 0) store(at, tot);
    }
}

// ---- the heavy columns
constexpr int HEAVY_NROW = FS_KB * 4;
inline size_t heavy_lds_bytes(int32_t chunk_w) {
    return raw_tile_lds_bytes(WINDQ_BF16, chunk_w) + (size_t)chunk_w * sizeof(float) + (size_t)FS_WAVES * TILE_ROWS * sizeof(float2) +
           (size_t)FS_WAVES * 16 * HEAVY_NROW * sizeof(float) + (size_t)FS_WAVES * sizeof(float);
}

// Every candidate on a tile's heavy columns, the 8-bit ones on the exact route or left out as in fit_score_tile (by the clipping
// error of the heavy columns), a sweep over FS_KB ratios a wavefront.  The sums lie where the tile's sums do: the main kernel adds the light columns'.
__global__ __launch_bounds__(FS_THREADS, 5) void fit_heavy_kernel(const FitScoreArgs B) {
    extern __shared__ char smem[];
    const int mi = batch_index(B.heavy_start, B.n, blockIdx.x);
    const FitScoreMat& A = B.m[mi];
    const TileCoord tc = tile_coord(A.g, (int64_t)blockIdx.x - B.heavy_start[mi], true);
    const int32_t K = B.K, G = A.g.chunk_w;
    const int64_t j = tc.col0 / G;
    const int32_t heavy = chunk_heavy(A, j);
    if (heavy == 0) return;
    const int32_t row_bytes = G * 2 + 16;
    char* __restrict__ tile = smem;
    float* __restrict__ ss = reinterpret_cast<float*>(smem + TILE_ROWS * row_bytes);
    float2* __restrict__ gstat = reinterpret_cast<float2*>(ss + G);
    float* __restrict__ red_all = reinterpret_cast<float*>(gstat + FS_WAVES * TILE_ROWS);
    float* __restrict__ ctab = red_all + FS_WAVES * 16 * HEAVY_NROW;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const float* __restrict__ rec = A.colsel + (size_t)j * (size_t)colsel_words(G);
    const uint8_t* __restrict__ place = reinterpret_cast<const uint8_t*>(rec + G);
    __builtin_amdgcn_s_setprio(3);
    load_rows_placed([&](int r) -> const char* { return r < tc.nrows ? static_cast<const char*>(A.W) + ((tc.row0 + r) * A.g.ld + tc.col0) * 2 : nullptr; },
                         G, place, tile);
    for (int32_t c = threadIdx.x; c < G; c += FS_THREADS) ss[c] = rec[c];
    const float s2 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(rec[G + FS_HMAX + 2])));
    __syncthreads();
    quarter_ranges(tile + lane * row_bytes, G, wave, lane, gstat);
    __syncthreads();
    const float2 range = row_range(gstat, lane);
    const float mn = range.x, mx = range.y;
    double* __restrict__ out = A.partial + ((size_t)tc.u * (size_t)A.g.tiles_per_unit + (size_t)tc.t) * (size_t)fit_score_ncand(K);

    // the heavy columns' clipping error at skip8_p
    float tile_clip, s2_rg2;
    {
        const float clo = pin_vgpr(B.skip8_p * mn), chi = pin_vgpr(B.skip8_p * mx);
        float sums[2] = {0.0f, (mx - mn) * (mx - mn)}, none[1] = {0.0f};
        const char* __restrict__ wrow = tile + lane * row_bytes;
        for (int32_t c = 8 * wave; c < heavy; c += 8 * FS_WAVES) {
            float w[8];
            read8<WINDQ_BF16>(wrow, c, w);
            const float4 sa = *reinterpret_cast<const float4*>(ss + c);
            const float4 sb = *reinterpret_cast<const float4*>(ss + c + 4);
            const float s8[8] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float rc = (w[t] - __builtin_amdgcn_fmed3f(w[t], clo, chi)) * s8[t];
                sums[0] = fmaf(rc, rc, sums[0]);
            }
        }
        wave_sums_maxes(sums, none);
        if (lane == 0) ctab[wave] = sums[0];
        __syncthreads();
        tile_clip = ((ctab[0] + ctab[1]) + ctab[2]) + ctab[3];
        s2_rg2 = s2 * sums[1];
        tile_clip = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(tile_clip)));
        s2_rg2 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s2_rg2)));
    }
    const float skip8_above = s2_rg2 * ((A.g.tiles_per_unit <= SKIP8_FEW_TILES ? SKIP8_MARGIN_FEW : SKIP8_MARGIN) / (12.0f * 65025.0f)) * B.skip8_q +
                              tile_clip * B.skip8_last;
    const bool anchored = __builtin_amdgcn_ballot_w64(!(mn <= 0.0f && mx >= 0.0f)) == 0;
    const bool probe = probe_tile(tc.t, A.g.tiles_per_unit);
    double* __restrict__ etab = reinterpret_cast<double*>(gstat);         // (the ranges have been read)
    static_assert(FS_WAVES * TILE_ROWS * sizeof(float2) >= 4 * WINDQ_MAX_CLIP * sizeof(double), "a tile's sums in the place of the ranges");
    float* __restrict__ red = red_all + wave * 16 * HEAVY_NROW;
    const float Q[4] = {pin_vgpr(255.0f), pin_vgpr(15.0f), pin_vgpr(7.0f), pin_vgpr(3.0f)};
    const float M = pin_vgpr(RNE_POS), nM = pin_vgpr(-RNE_POS);
    for (int v = (wave - (int)blockIdx.x) & (FS_WAVES - 1); v < B.shares; v += FS_WAVES) {
        const int32_t k0 = share_ratio(K, B.shares, 0, v), dk = B.shares;
        int32_t skip_here = 0;
#pragma unroll
        for (int i = 0; i < FS_KB; ++i) {
            const int k = k0 + dk * i;
            skip_here += tile_clip * B.skip8_f.p[k > 0 ? k : 0] > skip8_above ? 1 : 0;
        }
        const int32_t s8 = !anchored || skip_here < FS_KB - 2 ? 0 : skip_here;
        KParams P[FS_KB];
        float acc[FS_KB][4];
#pragma unroll
        for (int i = 0; i < FS_KB; ++i) {
            int k = k0 + dk * i;
            k = k > 0 ? k : 0;
            const float p = B.grid.p[k];
            const float flo = p * mn, fhi = p * mx, frg = fhi - flo;
            const float rinv = frg >= FLT_MIN ? __builtin_amdgcn_rcpf(frg) : 0.0f;
            // step: the correctly rounded quotient, as in fit_score_tile
            const auto step = [&](double rq) -> float {
                const float d = (float)((double)frg * rq);
                return d >= FLT_MIN ? d : 0.0f;
            };
            P[i].nd[1] = pin_vgpr(-step(1.0 / 15.0));
            P[i].nd[2] = pin_vgpr(-step(1.0 / 7.0));
            P[i].nd[3] = pin_vgpr(-step(1.0 / 3.0));
            P[i].rinv = rinv;
            P[i].h = pin_vgpr(-flo * rinv);
            P[i].nlo = pin_vgpr(-flo);
            if (i >= s8) {             // the 8-bit candidate's anchor
                const float d8 = step(1.0 / 255.0);
                float q0 = 0.0f;
                if (flo <= 0.0f && fhi >= 0.0f) q0 = __builtin_amdgcn_fmed3f(__builtin_rintf(-flo * rinv * 255.0f), 0.0f, 255.0f);
                const float c = fmaf(q0, d8, flo);
                P[i].nd[0] = pin_vgpr(-d8);
                P[i].nc = pin_vgpr(-c);
                P[i].Mq = pin_vgpr(RNE_POS + q0);
                if (!anchored) P[i].h = pin_vgpr((c - flo) * rinv);
            }
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[i][b] = 0.0f;
        }
        __builtin_amdgcn_s_setprio(0);
        const auto sweep = [&](auto anchored_t, auto s8_t) {
            const int lane_v = fresh_lane();
            const char* __restrict__ wrow = tile + lane_v * row_bytes;
            for (int32_t c = 0; c < heavy; c += 4) {
                float w[4];
                read4<WINDQ_BF16>(wrow, c, w);
                const float4 sa = *reinterpret_cast<const float4*>(ss + c);
                const float s4[4] = {sa.x, sa.y, sa.z, sa.w};
#pragma unroll
                for (int t = 0; t < 4; ++t) score_weight_staged<decltype(anchored_t)::value, false, decltype(s8_t)::value>(w[t], s4[t], P, Q, M, nM, acc);
            }
        };
        using std::integral_constant;
        if (!anchored) sweep(std::false_type{}, integral_constant<int, 0>{});
        else if (s8 == FS_KB) sweep(std::true_type{}, integral_constant<int, FS_KB>{});
        else if (s8 == FS_KB - 1) sweep(std::true_type{}, integral_constant<int, FS_KB - 1>{});
        else if (s8 == FS_KB - 2) sweep(std::true_type{}, integral_constant<int, FS_KB - 2>{});
        else sweep(std::true_type{}, integral_constant<int, 0>{});
        __builtin_amdgcn_s_setprio(3);
        float flat[FS_KB * 4];
        const int lane_r = fresh_lane();
#pragma unroll
        for (int i = 0; i < FS_KB; ++i) {
#pragma unroll
            for (int b = 0; b < 4; ++b) flat[i * 4 + b] = lane_r < tc.nrows ? acc[i][b] : 0.0f;
        }
        rows_deposit<HEAVY_NROW>(flat, red, lane_r, 0);
        double tot = rows_collect<HEAVY_NROW>(red, lane_r, FS_KB * 4);
        const int i = lane_r >> 2, k = k0 + dk * i;
        if (lane_r < FS_KB * 4 && k >= 0) {
            if ((lane_r & 3) == 0 && i < s8) tot = plan_bound((double)(tile_clip * B.skip8_f.p[k]));
            out[(lane_r & 3) * K + k] = tot;
            if (probe) etab[(lane_r & 3) * K + k] = tot;
        }
    }
    if (!probe) return;
    // what the light columns add to the least error of a bit-width, a wavefront each
    __syncthreads();
    if (wave == 0) return;
    const int b = wave;
    double least = lane < K ? etab[b * K + lane] : INFINITY;
    int at = lane;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const double other = __shfl_xor(least, m, 64);
        const int oat = __shfl_xor(at, m, 64);
        if (other < least || (other == least && oat < at)) {
            least = other;
            at = oat;
        }
    }
    LowParams L[1];
    L[0] = low_params(B.grid.p[__builtin_amdgcn_readfirstlane(at < K ? at : 0)], b, mn, mx);
    float acc[1] = {0.0f};
    int32_t c = heavy;
    const char* __restrict__ wrow = tile + lane * row_bytes;
    if (anchored) low_sweep<1, true, 1>(wrow, ss, c, G, L, M, acc);
    else low_sweep<1, false, 1>(wrow, ss, c, G, L, M, acc);
    if (lane >= tc.nrows) acc[0] = 0.0f;
    rows_deposit<HEAVY_NROW>(acc, red, lane, 0);
    const double light = rows_collect<HEAVY_NROW>(red, lane, 1);
    if (lane == 0) {
        double* to = out + fit_score_noise_slot(K);
        to[b - 1] = light;
        to[3 + b - 1] = least;
    }
}

// ---- the plan
// The light columns' part of an error is taken to be the heavy columns' times the ratio that the probed tiles show for the least errors
// (at 8 bits, where residuals do not depend on the column: the ratio of the sums of s_c^2): PLAN_HIGH of that for the least error,
// with PLAN_MARGIN on the whole; PLAN_LOW of that, dealt to the columns by their weight, for what is left out.  With these one unit in
// five hundred of a 7B-shaped block is scored again (40 draws of scales as (a) above: 4096 x 4096 one in 320, 11008 x 4096 none of 1280, 4096 x 11008 one in
// 570; 1024 x 8192 at chunk 64 one in 390; 8192 x 8192 at chunk 256 one in 53); half the margins list three times as many, in the same time.  (A ratio taken from the columns'
// weights alone is off by up to four times where a column of heavy-tailed weights is a light one: one unit in ten again.)
constexpr int PLAN_THREADS = 1024;
constexpr double PLAN_LOW = 0.8, PLAN_HIGH = 1.12, PLAN_MARGIN = 1.01;

inline size_t fit_plan_lds_bytes(int32_t K) { return (size_t)(FIN_PHASES + 1) * 4 * (size_t)K * sizeof(double) + PLAN_LIST_WORDS * sizeof(uint64_t); }

// One workgroup per unit.
__global__ __launch_bounds__(PLAN_THREADS) void fit_plan_kernel(const FitScoreArgs B) {
    extern __shared__ char smem[];
    const int mi = batch_index(B.plan_start, B.n, blockIdx.x);
    const FitScoreMat& A = B.m[mi];
    const int64_t u = (int64_t)blockIdx.x - B.plan_start[mi];
    const int32_t K = B.K, G = A.g.chunk_w, ncand = fit_score_ncand(K);
    const int64_t j = (int64_t)((uint32_t)u % (uint32_t)A.g.n_chunks);
    const int32_t heavy = chunk_heavy(A, j);
    if (heavy == 0) return;
    double* __restrict__ phases = reinterpret_cast<double*>(smem);
    double* __restrict__ E = phases + FIN_PHASES * 4 * K;
    uint64_t* __restrict__ lists = reinterpret_cast<uint64_t*>(E + 4 * K);
    double* unit = A.partial + (size_t)u * (size_t)A.g.tiles_per_unit * (size_t)ncand;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const float* __restrict__ shares = chunk_shares(A, K, j);
    float share[PLAN_STEPS + 1];
#pragma unroll
    for (int s = 0; s <= PLAN_STEPS; ++s) share[s] = shares[s];
    static_assert(PLAN_THREADS / 64 == FIN_PHASES, "a wavefront per phase");
    __shared__ double ratio_sh[4];
    if (wave < 4) {          // bit-width wave
        double part[2] = {0.0, 0.0};         // light, heavy
        if (wave == 0) {
            const float* __restrict__ rec = A.colsel + (size_t)j * (size_t)colsel_words(G);
            for (int32_t c = lane; c < G; c += 64) part[c < heavy ? 1 : 0] += (double)rec[c] * (double)rec[c];
        } else {
            const int every = probe_every(A.g.tiles_per_unit);
            for (int64_t t = PROBE_FIRST + every * lane; t < A.g.tiles_per_unit; t += every * 64) {
                const double* __restrict__ from = unit + (size_t)t * (size_t)ncand + fit_score_noise_slot(K);
                part[0] += from[wave - 1];
                part[1] += from[3 + wave - 1];
            }
        }
        const double light = wave_sum(part[0]), kept = wave_sum(part[1]);
        if (lane == 0) ratio_sh[wave] = light / kept;
    }
    for (int32_t cand = lane; cand < 4 * K; cand += 64) {
        double sum[1];
        fit_phase_sums<1, false>(unit, A.g.tiles_per_unit, ncand, cand, wave, 0, sum);
        phases[wave * 4 * K + cand] = sum[0];
    }
    __syncthreads();
    if (tid < 4 * K) E[tid] = fit_phases_total(phases, 4 * K, tid);
    __syncthreads();
    int step = -1;
    if (tid < 4 * K) {
        const int b = tid / K;
        double best, bound;
        fit_least(E + b * K, K, &best, &bound);
        const double whole = share[PLAN_STEPS], ratio = ratio_sh[b], need = best * (1.0 + PLAN_HIGH * ratio) * PLAN_MARGIN, e = E[tid];
        step = PLAN_STEPS - 1;          // (also where a number is not finite)
        if (need > 0.0 && need < INFINITY) {
#pragma unroll
            for (int s = PLAN_STEPS - 2; s >= 0; --s) {
                if (plan_columns(G, s) > heavy && e * (1.0 + PLAN_LOW * ratio * ((double)share[s] - whole) / (1.0 - whole)) >= need) step = s;
            }
            if (e >= need) step = -1;
        }
        if (e < 0.0) step = -1;         // an 8-bit candidate that a tile has left out stays a bound
    }
    fit_plan_list(fit_plan(unit, K), lists, step, K, tid);
}

// A tile of a listed unit: its list (the open candidates, on all columns).  With few tiles the launch waits for memory most of the time: what the
// tile needs is asked for at once.
constexpr int LISTED_NROW = 8;
constexpr int LISTED_PIECES = 4;          // 16-byte pieces a thread keeps in registers
__device__ __forceinline__ void fit_listed_tile(const FitScoreArgs& B, const FitScoreMat& A, const TileCoord& tc, const int rot, char* __restrict__ smem) {
    const int32_t K = B.K, G = A.g.chunk_w, ncand = fit_score_ncand(K);
    const float* __restrict__ rec = A.colsel + (size_t)(tc.col0 / G) * (size_t)colsel_words(G);
    double* __restrict__ unit = A.partial + (size_t)tc.u * (size_t)A.g.tiles_per_unit * (size_t)ncand;
    const int32_t row_bytes = G * 2 + 16;
    char* __restrict__ tile = smem;
    float* __restrict__ ss = reinterpret_cast<float*>(smem + TILE_ROWS * row_bytes);           // the chunk's record, as in memory
    const uint8_t* __restrict__ place = reinterpret_cast<const uint8_t*>(ss + G);
    float2* __restrict__ gstat = reinterpret_cast<float2*>(ss + G + FS_PLAN_MAX_CHUNK / 4);
    float2* __restrict__ table = gstat + FS_WAVES * TILE_ROWS;
    float* __restrict__ grid = reinterpret_cast<float*>(table + 4 * WINDQ_MAX_CLIP);
    FitPlan* __restrict__ plan = reinterpret_cast<FitPlan*>(grid + WINDQ_MAX_CLIP);
    float* __restrict__ red_all = reinterpret_cast<float*>(plan + 1);
    static_assert(sizeof(FitPlan) % 8 == 0, "");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int32_t pieces = G >> 3, total = TILE_ROWS * pieces;
    PieceWalk at((int32_t)threadIdx.x, FS_THREADS, pieces);
    const char* __restrict__ src = static_cast<const char*>(A.W) + (tc.row0 * A.g.ld + tc.col0) * 2;
    for (int32_t i0 = threadIdx.x; i0 - (int32_t)threadIdx.x < total; i0 += LISTED_PIECES * FS_THREADS) {
        uint4 v[LISTED_PIECES];
        int32_t r[LISTED_PIECES], pc[LISTED_PIECES];
#pragma unroll
        for (int k = 0; k < LISTED_PIECES; ++k) {
            v[k] = make_uint4(0u, 0u, 0u, 0u);
            r[k] = at.r;
            pc[k] = at.pc;
            if (i0 + k * FS_THREADS < total && at.r < tc.nrows) v[k] = *reinterpret_cast<const uint4*>(src + (int64_t)at.r * A.g.ld * 2 + at.pc * 16);
            at.next();
        }
        if (i0 == (int32_t)threadIdx.x) {
            const int32_t words = G + FS_PLAN_MAX_CHUNK / 4;
            for (int32_t c = threadIdx.x; c < words; c += FS_THREADS) ss[c] = rec[c];
            if (threadIdx.x < WINDQ_MAX_CLIP) grid[threadIdx.x] = B.grid.p[threadIdx.x];
            const uint32_t plan_words = (uint32_t)(sizeof(FitPlan) - 4 * WINDQ_MAX_CLIP + 4 * K) / 4;
            if (threadIdx.x < plan_words) reinterpret_cast<uint32_t*>(plan)[threadIdx.x] = reinterpret_cast<const uint32_t*>(fit_plan(unit, K))[threadIdx.x];
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < LISTED_PIECES; ++k)
            if (i0 + k * FS_THREADS < total) scatter_piece(tile + r[k] * row_bytes, v[k], place + pc[k] * 8);
    }
    plan_table(grid, plan, G, table);
    __syncthreads();
    quarter_ranges(tile + lane * row_bytes, G, wave, lane, gstat);
    __syncthreads();
    const float2 range = row_range(gstat, lane);
    score_list<true, LISTED_NROW, 2>(B, plan, table, tile, row_bytes, ss, 0, tc.nrows, range.x, range.y, wave, rot,
                                                 red_all + wave * 16 * LISTED_NROW, unit + (size_t)tc.t * (size_t)ncand, [](int, double) {});
}
static_assert(FS_PLAN_MAX_CHUNK + 4 * WINDQ_MAX_CLIP * sizeof(float2) + WINDQ_MAX_CLIP * sizeof(float) + sizeof(FitPlan) + FS_WAVES * 16 * LISTED_NROW * sizeof(float) <=
                  FS_WAVES * 16 * fs_nrow(true) * sizeof(float),
              "within the LDS of the launch that scores listed units again (fit_score_lds_bytes)");

// The end of a listed unit: its open candidates' sums, in the finalize step's order, against the least errors so far.  By the workgroup that has scored
// the unit's last tile; all the tiles' sums are asked for at once, as many candidates at a time as LDS holds (lds: LISTED_SUMS doubles).
constexpr int LISTED_SUMS = 1536;
__device__ __forceinline__ void fit_listed_end(const FitScoreMat& A, int64_t u, double* __restrict__ unit, int32_t K, double* __restrict__ lds) {
    const int32_t ncand = fit_score_ncand(K);
    const int64_t tpu = A.g.tiles_per_unit;
    FitPlan* __restrict__ plan = fit_plan(unit, K);
    FitListed* __restrict__ listed = fit_listed(unit, K);
    const int n = plan_entries(plan->low) + plan_entries(plan->high), tid = threadIdx.x;
    double* __restrict__ phase = lds + LISTED_SUMS;             // [candidates at a time][FIN_PHASES]
    const int fit = (int)(LISTED_SUMS / tpu), many = fit > FS_THREADS / FIN_PHASES ? FS_THREADS / FIN_PHASES : fit;
    double best[4];
    int32_t bk[4];
    if (tid == 0) {
        for (int b = 0; b < 4; ++b) {
            best[b] = listed->best[b];
            bk[b] = listed->at[b];
        }
    }
    for (int first = 0; first < n; first += many > 0 ? many : 1) {
        const int now = many > 0 ? (n - first < many ? n - first : many) : 1;
        if (many > 0) {
            for (int i = tid; i < now * (int)tpu; i += FS_THREADS) {
                const int c = i / (int)tpu, t = i - c * (int)tpu;
                const uint32_t e = plan->list[first + c];
                lds[i] = __hip_atomic_load(unit + (size_t)t * ncand + (e >> 6) * K + (e & 63u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
        }
        if (tid < now * FIN_PHASES) {
            const int c = tid / FIN_PHASES, p = tid - c * FIN_PHASES;
            double sum = 0.0;
            if (many > 0) {
                for (int64_t t = p; t < tpu; t += FIN_PHASES) sum += fabs(lds[c * tpu + t]);
            } else {             // a unit of more tiles than LDS holds
                const uint32_t e = plan->list[first];
                double one[1];
                fit_phase_sums<1, true>(unit, tpu, ncand, (int32_t)((e >> 6) * K + (e & 63u)), p, 0, one);
                sum = fabs(one[0]);
            }
            phase[c * FIN_PHASES + p] = sum;
        }
        __syncthreads();
        if (tid == 0) {
            for (int c = 0; c < now; ++c) {
                const uint32_t e = plan->list[first + c];
                double sum = 0.0;
                for (int p = 0; p < FIN_PHASES; ++p) sum += phase[c * FIN_PHASES + p];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    if ((int)(e >> 6) != b) continue;
                    const int k = (int)(e & 63u);
                    // as fit_least over all of them: ties to the largest ratio; a first error that is no number stays
                    const bool first_nan = bk[b] == 0 && best[b] != best[b];
                    const bool take = k == 0 && sum != sum ? true : !first_nan && (best[b] != best[b] ? sum == sum : sum < best[b] || (sum == best[b] && k > bk[b]));
                    if (take) {
                        best[b] = sum;
                        bk[b] = k;
                    }
                }
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        for (int b = 0; b < 4; ++b) {
            A.err[u * WINDQ_N_ERR + b] = (float)best[b];
            A.clip_idx[u * 4 + b] = (uint8_t)bk[b];
        }
    }
}

}  // namespace windq
