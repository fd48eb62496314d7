// windq_calib_stats: per input channel activation scale from calibration activations
// (App. "Salient Weight Protection": per-channel activation scale from a calibration
// forward pass).  s_absmean[c] = mean_t |x_tc|, s_rms[c] = sqrt(mean_t x_tc^2).
//
// Pure streaming reduction over the token axis, bound by HBM.  A workgroup owns a strip of
// 8 L channels (L lanes side by side, 8 channels = 16 or 32 bytes each) and a slab of tokens;
// its 256 / L lane groups take every (256 / L)-th token, eight (or four) loads in flight per lane.
// fp64 sums, combined in a fixed order: lane groups through LDS, slabs by the finalize kernel.
//
// How a matrix is cut (calib_cut; its own size alone decides, so that a batch gives the bits of single calls):
//   few tokens (the calibration sets of the benchmark configurations: 512): ONE slab and narrow
//     strips (L = 8, 64 channels), so that the workgroup writes the result itself: two dependent
//     launches cost more than a few MB do.  Always below 2048 tokens, and up to 4096 where a token's bytes are more than
//     1.5 per token, since then the strips (and the other inputs of a batch) fill enough of the chip.  us, one slab against
//     several, alone and four in a batch, bf16:
//       1536 x 1024: 5.3, 6.0 and 5.8, 8.0       2048 x 1024: 6.4, 5.6 and 6.9, 7.9     2048 x 4096: 6.6, 7.5 and 12.2, 16.8
//       3072 x 2048: 8.4, 7.4 and 11.8, 14.2     4096 x 2048: 10.3, 7.4 and 14.6, 16.9  4096 x 4096: 11.5, 10.5 and 21, 28.5
//   more: L = 64 (512 channels, a wavefront reads 1 KB of a token; less for narrow matrices) and
//     as many slabs as give the chip about 1024 workgroups, four for each of its 256 CUs (what
//     the 33 KB of LDS allow; 2048 measured 14 % slower): more slabs only mean more partial sums
//     to write and read back.  16384 x 4096 bf16, both statistics: 33 us = 4.0 TB/s (162 us with
//     32-token slabs, whose 33 MB of partial sums one thread per channel then added in a chain);
//     a large copy moves 5.1 TB/s.
// All matrices of a batch share the launch (and the finalize launch, where any needs it) but those whose slab sums would
// lie in the same memory.
#include "windq_common.hpp"
#include "windq_ws.hpp"

namespace windq {

constexpr int CALIB_THREADS = 256;
constexpr int CALIB_CPL = 8;                        // channels per lane
constexpr int CALIB_INFLIGHT = 8;                   // loads in flight per lane; 4 for fp32 inputs in one slab each and 128 workgroups or more,
constexpr int64_t CALIB_FEWER_WGS = 128;            // whose registers cost more (3072 x 8192: 17.7 us with 8, 16.0 with 4; 1024 x 5120: 5.1, 5.3)
constexpr int64_t CALIB_DIRECT_ROWS = 2047, CALIB_DIRECT_ROWS_WIDE = 4096;
constexpr int64_t CALIB_TARGET_WGS = 1024;
constexpr int64_t CALIB_MAX_SLABS = 65535;          // of 32 tokens: the interface's limit on one input (no kernel here needs it)

// One activation matrix of a launch; a launch covers up to WINDQ_MAX_BATCH of them, their
// workgroups (and the finalize kernel's) numbered one matrix after the other.
struct CalibMat {
    const void* X;
    int64_t rows, cols, ld;
    float* s_absmean;
    float* s_rms;
    double* partial;        // [slabs][2][cols]: sum |x|, sum x^2
    int64_t slab_rows;
    int32_t slabs, strips;
    int32_t lane_shift;     // L = 1 << lane_shift
    int32_t reserved;
};
struct CalibBatch {
    int32_t n;
    int64_t wg_start[WINDQ_MAX_BATCH + 1];
    CalibMat m[WINDQ_MAX_BATCH];
};

// Eight consecutive activations as they lie in memory.
template <int DT>
struct Raw8 {
    uint4 q[DT == WINDQ_BF16 ? 1 : 2];
    __device__ __forceinline__ void load(const char* __restrict__ p) {
#pragma unroll
        for (int h = 0; h < (DT == WINDQ_BF16 ? 1 : 2); ++h) q[h] = reinterpret_cast<const uint4*>(p)[h];
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int h = 0; h < (DT == WINDQ_BF16 ? 1 : 2); ++h) q[h] = make_uint4(0u, 0u, 0u, 0u);
    }
};

template <int DT, bool RMS>
__device__ __forceinline__ void calib_add(const Raw8<DT>& raw, double (&sa)[CALIB_CPL], double (&sq)[CALIB_CPL]) {
    float v[CALIB_CPL];
    const uint4 a = raw.q[0];
    if (DT == WINDQ_BF16) {
        v[0] = bf16_bits_to_f32(a.x & 0xffffu); v[1] = __uint_as_float(a.x & 0xffff0000u);
        v[2] = bf16_bits_to_f32(a.y & 0xffffu); v[3] = __uint_as_float(a.y & 0xffff0000u);
        v[4] = bf16_bits_to_f32(a.z & 0xffffu); v[5] = __uint_as_float(a.z & 0xffff0000u);
        v[6] = bf16_bits_to_f32(a.w & 0xffffu); v[7] = __uint_as_float(a.w & 0xffff0000u);
    } else {
        const uint4 b = raw.q[DT == WINDQ_BF16 ? 0 : 1];
        v[0] = __uint_as_float(a.x); v[1] = __uint_as_float(a.y); v[2] = __uint_as_float(a.z); v[3] = __uint_as_float(a.w);
        v[4] = __uint_as_float(b.x); v[5] = __uint_as_float(b.y); v[6] = __uint_as_float(b.z); v[7] = __uint_as_float(b.w);
    }
#pragma unroll
    for (int j = 0; j < CALIB_CPL; ++j) {
        const double x = (double)v[j];
        sa[j] += fabs(x);
        if (RMS) sq[j] = fma(x, x, sq[j]);
    }
}

template <int DT, bool RMS, int INFLIGHT>      // (INFLIGHT changes no sum: a lane adds its tokens in order)
__global__ __launch_bounds__(CALIB_THREADS) void calib_sum_kernel(const CalibBatch B) {
    constexpr int NV = RMS ? 2 * CALIB_CPL : CALIB_CPL;
    // [value][thread]; the odd row length spreads the eight values of a lane over the banks
    __shared__ double red[NV][CALIB_THREADS + 1];
    const int mi = batch_index(B.wg_start, B.n, blockIdx.x);
    const CalibMat& M = B.m[mi];
    const uint32_t at = (uint32_t)((int64_t)blockIdx.x - B.wg_start[mi]);
    const uint32_t slab = at / (uint32_t)M.strips;
    const uint32_t strip = at - slab * (uint32_t)M.strips;
    const int L = 1 << M.lane_shift;
    const int groups = CALIB_THREADS >> M.lane_shift;
    const int cl = threadIdx.x & (L - 1);
    const int tg = threadIdx.x >> M.lane_shift;
    const int64_t cols = M.cols;
    const int64_t strip0 = (int64_t)strip * (int64_t)(L * CALIB_CPL);
    const int64_t c0 = strip0 + cl * CALIB_CPL;
    const int64_t r_end = (int64_t)(slab + 1) * M.slab_rows < M.rows ? (int64_t)(slab + 1) * M.slab_rows : M.rows;
    double sa[CALIB_CPL], sq[CALIB_CPL];
#pragma unroll
    for (int j = 0; j < CALIB_CPL; ++j) sa[j] = sq[j] = 0.0;
    if (c0 < cols) {
        constexpr int EB = Elem<DT>::bytes;
        const char* __restrict__ src = static_cast<const char*>(M.X) + c0 * EB;
        const int64_t step = M.ld * EB;
        int64_t r = (int64_t)slab * M.slab_rows + tg;
        // whole batches of loads without a bounds check between them; then the rest, four at a time: a token past
        // the end is read from the slab's last one and added as zeros
        for (; r + (int64_t)groups * (INFLIGHT - 1) < r_end; r += (int64_t)groups * INFLIGHT) {
            Raw8<DT> raw[INFLIGHT];
#pragma unroll
            for (int k = 0; k < INFLIGHT; ++k) raw[k].load(src + (r + (int64_t)k * groups) * step);
#pragma unroll
            for (int k = 0; k < INFLIGHT; ++k) calib_add<DT, RMS>(raw[k], sa, sq);
        }
        for (; r < r_end; r += (int64_t)groups * 4) {
            Raw8<DT> raw[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t rr = r + (int64_t)k * groups;
                raw[k].load(src + (rr < r_end ? rr : r_end - 1) * step);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (r + (int64_t)k * groups >= r_end) raw[k].clear();
                calib_add<DT, RMS>(raw[k], sa, sq);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < CALIB_CPL; ++j) {
        red[j][threadIdx.x] = sa[j];
        if (RMS) red[CALIB_CPL + j][threadIdx.x] = sq[j];
    }
    __syncthreads();
    // channel by channel, lane groups in order
    for (int q = threadIdx.x; q < L * NV; q += CALIB_THREADS) {
        const int which = q >> (M.lane_shift + 3);                            // 0: sum |x|, 1: sum x^2
        const int col = q & (L * CALIB_CPL - 1);
        const double* __restrict__ row = red[which * CALIB_CPL + (col & (CALIB_CPL - 1))] + (col >> 3);
        double t = 0.0;
        if (groups == 32) {                                                   // all reads in flight, added in order
#pragma unroll
            for (int g = 0; g < 32; ++g) t += row[g << 3];
        } else {
            for (int g = 0; g < groups; g += 4) {                             // four
                const double t0 = row[g << M.lane_shift], t1 = row[(g + 1) << M.lane_shift];
                const double t2 = row[(g + 2) << M.lane_shift], t3 = row[(g + 3) << M.lane_shift];
                t = (((t + t0) + t1) + t2) + t3;
            }
        }
        const int64_t c = strip0 + col;
        if (c >= cols) continue;
        if (M.slabs > 1) {
            M.partial[((size_t)slab * 2 + (size_t)which) * (size_t)cols + (size_t)c] = t;
        } else if (which == 0) {
            M.s_absmean[c] = (float)(t / (double)M.rows);
        } else if (M.s_rms != nullptr) {
            M.s_rms[c] = (float)sqrt(t / (double)M.rows);
        }
    }
}

// The slabs of 16 channels by a workgroup: 16 phases, phase p adds slabs p, p + 16, ..., the phases in order.
constexpr int CALIB_FIN_COLS = 16;
template <bool RMS>
__global__ __launch_bounds__(256) void calib_finalize_kernel(const CalibBatch B) {
    constexpr int PH = 256 / CALIB_FIN_COLS;
    __shared__ double red[2][PH][CALIB_FIN_COLS + 1];
    const int mi = batch_index(B.wg_start, B.n, blockIdx.x);
    const CalibMat& M = B.m[mi];
    const int cl = threadIdx.x & (CALIB_FIN_COLS - 1);
    const int ph = threadIdx.x / CALIB_FIN_COLS;
    const int64_t c = ((int64_t)blockIdx.x - B.wg_start[mi]) * CALIB_FIN_COLS + cl;
    double a = 0.0, q = 0.0;
    if (c < M.cols) {
        const double* __restrict__ src = M.partial + c;
#pragma unroll 4
        for (int32_t s = ph; s < M.slabs; s += PH) {
            a += src[(size_t)s * 2 * (size_t)M.cols];
            if (RMS) q += src[((size_t)s * 2 + 1) * (size_t)M.cols];
        }
    }
    red[0][ph][cl] = a;
    red[1][ph][cl] = q;
    __syncthreads();
    if (threadIdx.x >= 2 * CALIB_FIN_COLS) return;
    const int which = threadIdx.x / CALIB_FIN_COLS;
    if (c >= M.cols) return;
    double t = 0.0;
#pragma unroll
    for (int p = 0; p < PH; ++p) t += red[which][p][cl];
    if (which == 0) M.s_absmean[c] = (float)(t / (double)M.rows);
    else if (RMS && M.s_rms != nullptr) M.s_rms[c] = (float)sqrt(t / (double)M.rows);
}

}  // namespace windq

using namespace windq;

static int calib_check(const windq_mat* X, const float* s_absmean, const void* ws, size_t ws_bytes) {
    const int st = check_matrix(X);
    if (st != WINDQ_OK) return st;
    if (s_absmean == nullptr) return WINDQ_EINVAL;
    const size_t need = calib_ws_bytes(X->rows, X->cols);
    if (ws == nullptr || ws_bytes < need || !aligned(ws, 256)) return WINDQ_EWORKSPACE;
    if (calib_slabs(X->rows) > CALIB_MAX_SLABS) return WINDQ_ESHAPE;
    return WINDQ_OK;
}

// How a matrix is cut into strips and slabs (the rule and its reasons: top of the file).  A slab has
// at least 32 tokens: the workspace holds one pair of sums per channel and 32 tokens.
static void calib_cut(CalibMat* M, int elem_bytes) {
    const bool direct = M->rows <= CALIB_DIRECT_ROWS || (M->rows <= CALIB_DIRECT_ROWS_WIDE && 2 * M->cols * elem_bytes > 3 * M->rows);
    M->lane_shift = direct ? 3 : 6;
    while (M->lane_shift > 3 && (int64_t)(CALIB_CPL << (M->lane_shift - 1)) >= M->cols) --M->lane_shift;
    const int64_t strip = (int64_t)CALIB_CPL << M->lane_shift;
    M->strips = (int32_t)((M->cols + strip - 1) / strip);
    int64_t slabs = 1;
    if (!direct) {
        slabs = (CALIB_TARGET_WGS + M->strips - 1) / M->strips;
        if (slabs > calib_slabs(M->rows)) slabs = calib_slabs(M->rows);
    }
    M->slab_rows = ((M->rows + slabs - 1) / slabs + CALIB_SLAB_ROWS - 1) / CALIB_SLAB_ROWS * CALIB_SLAB_ROWS;
    M->slabs = (int32_t)((M->rows + M->slab_rows - 1) / M->slab_rows);
}

// The matrices of one launch (two, where slabs are to be added).
static int calib_launch(const CalibMat* mats, int32_t n, int32_t dtype, hipStream_t hs) {
    CalibBatch B, F;            // all matrices; those whose slabs are still to be added
    B.n = n;
    F.n = 0;
    int64_t wgs = 0, fin = 0;
    bool rms = false;
    for (int32_t i = 0; i < n; ++i) {
        const CalibMat& M = mats[i];
        B.m[i] = M;
        rms = rms || M.s_rms != nullptr;
        B.wg_start[i] = wgs;
        wgs += (int64_t)M.strips * M.slabs;
        if (M.slabs > 1) {
            F.wg_start[F.n] = fin;
            fin += (M.cols + CALIB_FIN_COLS - 1) / CALIB_FIN_COLS;
            F.m[F.n++] = M;
        }
    }
    for (int32_t i = n; i <= WINDQ_MAX_BATCH; ++i) B.wg_start[i] = wgs;
    for (int32_t i = n; i < WINDQ_MAX_BATCH; ++i) B.m[i] = B.m[0];
    const dim3 grid((unsigned)wgs), block(CALIB_THREADS);
    if (dtype == WINDQ_BF16) {
        if (rms) hipLaunchKernelGGL((calib_sum_kernel<WINDQ_BF16, true, CALIB_INFLIGHT>), grid, block, 0, hs, B);
        else hipLaunchKernelGGL((calib_sum_kernel<WINDQ_BF16, false, CALIB_INFLIGHT>), grid, block, 0, hs, B);
    } else if (wgs < CALIB_FEWER_WGS || F.n > 0) {
        if (rms) hipLaunchKernelGGL((calib_sum_kernel<WINDQ_F32, true, CALIB_INFLIGHT>), grid, block, 0, hs, B);
        else hipLaunchKernelGGL((calib_sum_kernel<WINDQ_F32, false, CALIB_INFLIGHT>), grid, block, 0, hs, B);
    } else {
        if (rms) hipLaunchKernelGGL((calib_sum_kernel<WINDQ_F32, true, 4>), grid, block, 0, hs, B);
        else hipLaunchKernelGGL((calib_sum_kernel<WINDQ_F32, false, 4>), grid, block, 0, hs, B);
    }
    if (F.n > 0) {
        for (int32_t i = F.n; i <= WINDQ_MAX_BATCH; ++i) F.wg_start[i] = fin;
        for (int32_t i = F.n; i < WINDQ_MAX_BATCH; ++i) F.m[i] = F.m[0];
        if (rms) hipLaunchKernelGGL(calib_finalize_kernel<true>, dim3((unsigned)fin), dim3(256), 0, hs, F);
        else hipLaunchKernelGGL(calib_finalize_kernel<false>, dim3((unsigned)fin), dim3(256), 0, hs, F);
    }
    return hipPeekAtLastError() == hipSuccess ? WINDQ_OK : WINDQ_EHIP;
}

// Do two matrices write slab sums to the same memory?
static bool calib_share(const CalibMat& a, const CalibMat& b) {
    if (a.slabs == 1 || b.slabs == 1) return false;
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a.partial), b0 = reinterpret_cast<uintptr_t>(b.partial);
    const uintptr_t a1 = a0 + (uintptr_t)a.slabs * 2 * (uintptr_t)a.cols * sizeof(double);
    const uintptr_t b1 = b0 + (uintptr_t)b.slabs * 2 * (uintptr_t)b.cols * sizeof(double);
    return a0 < b1 && b0 < a1;
}

// One launch for all matrices whose slab sums do not meet; an item is a call of its own, so that several may name one
// workspace: those wait for a later launch.
extern "C" int windq_calib_stats_batch(const windq_calib_item* items, int32_t n, void* stream) {
    if (items == nullptr || n < 1 || n > WINDQ_MAX_BATCH) return WINDQ_EINVAL;
    CalibMat mats[WINDQ_MAX_BATCH];
    int64_t wgs = 0;
    for (int32_t i = 0; i < n; ++i) {
        const windq_mat* X = items[i].X;
        if (X == nullptr) return WINDQ_EINVAL;
        const int st = calib_check(X, items[i].s_absmean, items[i].ws, items[i].ws_bytes);
        if (st != WINDQ_OK) return st;
        if (X->dtype != items[0].X->dtype) return WINDQ_EINVAL;      // one kernel per launch
        CalibMat& M = mats[i];
        M.X = X->data;
        M.rows = X->rows;
        M.cols = X->cols;
        M.ld = X->ld;
        M.s_absmean = items[i].s_absmean;
        M.s_rms = items[i].s_rms;
        M.partial = static_cast<double*>(items[i].ws);
        M.reserved = 0;
        calib_cut(&M, X->dtype == WINDQ_BF16 ? 2 : 4);
        wgs += (int64_t)M.strips * M.slabs;
    }
    if (!fits_launch(wgs, CALIB_THREADS)) return WINDQ_ESHAPE;
    int32_t left = n;
    while (left > 0) {
        CalibMat now[WINDQ_MAX_BATCH];
        int32_t n_now = 0, n_later = 0;
        for (int32_t i = 0; i < left; ++i) {
            bool meets = false;
            for (int32_t k = 0; k < n_now; ++k) meets = meets || calib_share(now[k], mats[i]);
            if (meets) mats[n_later++] = mats[i];
            else now[n_now++] = mats[i];
        }
        left = n_later;
        const int st = calib_launch(now, n_now, items[0].X->dtype, static_cast<hipStream_t>(stream));
        if (st != WINDQ_OK) return st;
    }
    return WINDQ_OK;
}

extern "C" int windq_calib_stats(const windq_mat* X, float* s_absmean, float* s_rms, void* ws, size_t ws_bytes,
                                 void* stream) {
    const windq_calib_item it = {X, s_absmean, s_rms, ws, ws_bytes};
    if (X == nullptr) return WINDQ_EINVAL;
    return windq_calib_stats_batch(&it, 1, stream);
}
