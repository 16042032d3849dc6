// warmstart.hip -- kernels of the per-projection temporal-weight fit and of its learned warm start.
//
// The plain fit finds, for each view t, the rank-R weights w_t of the low-rank motion model
// (Sec. 3.3, Eq. 9) that minimise the projection residual 1/2 ||I(w_t) - P_t||^2 by
// Levenberg-Marquardt; k_lm_normal_eq forms its normal equations from rendered images. The learned
// warm start is a small MLP (downsampled projection and gantry angle in, w_t out) whose matrix
// products run on the gfx950 matrix cores: BF16 operands, FP32 accumulation (k_gemm_bf16), with
// FP32 master weights updated by Adam.
#include <algorithm>

#include "kernels.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------------------------------------
// C[M][N] = epilogue(A . B) with op(A) [M][K] and op(B) [K][N] read from FP32 memory, rounded to
// BF16 in registers and multiplied on v_mfma_f32_16x16x32_bf16 with FP32 accumulation. A is stored
// [M][K] (lda) or, with TA, [K][M]; B is stored [K][N] (ldb) or, with TB, [N][K]. Epilogue, in
// order: + C (accumulate), + bias[col], max(., 0) (relu), zero where gate[row][col] <= 0 (gate has
// the leading dimension ldc).
//
// A wave computes 16 rows by 16 TN columns, from operands that its lanes load straight into the
// matrix cores' layout: the products of the warm-start network are latency-bound, with few tiles
// of C or few steps of K, so there is little reuse for a staged tile to serve and no barrier in
// the loop. Column TN * (l % 16) + j of the wave's tile is column l % 16 of its j-th matrix, which
// makes a lane's TN columns adjacent in memory. KW waves of a workgroup share a tile, wave w
// taking the 32-wide steps w, w + KW, ... of K, and their sums are added in wave order; with
// KW == 1 the workgroup's four waves take neighbouring tiles. Tiles go along the rows of C, or down its
// columns where those are more and the rows either many or one row of tiles enough to fill the chip: B
// is then used again while it is in the caches (256x65536x1024: 568 us along, 310 down; 4096x8192x4096:
// 2549 and 2006, with A transposed 3575 and 2151; but 64x16384x512: 13 and 22).
// Measured against 64x64 tiles of C staged through LDS, a workgroup each (M x N x K): 267 -> 9 us
// (32x256x4098), 558 -> 21 (256x512x4098), 50 -> 4 (186x128x578), 20 -> 3 (32x256x256), gradients of
// the weights 7.3 -> 4.4 (4098x256x32) and 41 -> 17 (4098x512x256).
#define GT_ROWS 16
#define GT_K 32

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // any float's alignment

// Eight values k .. k+7 of a row, contiguous (KC) or ld apart with TN adjacent ones each; those at
// k >= K read the last value in range and are zero if GUARD
template <bool KC, int TN, bool GUARD>
__device__ __forceinline__ void gemm_load(const float *const (&p)[TN], size_t ld, int k, int K,
                                          float (&v)[TN][8])
{
    if constexpr (GUARD) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float x = p[t][(KC ? (size_t)1 : ld) * (size_t)min(k + j, K - 1)];
                v[t][j] = k + j < K ? x : 0.0f;
            }
    } else if constexpr (KC) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int j = 0; j < 8; j += 4) {
                const f32x4u x = *(const f32x4u *)(p[t] + k + j);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[t][j + i] = x[i];
            }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float *q = p[0] + ld * (size_t)(k + j);
            if constexpr (TN == 4) {
                const f32x4u x = *(const f32x4u *)q;
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t][j] = x[t];
            } else {
                v[0][j] = *q;
            }
        }
    }
}

__device__ __forceinline__ bf16x8 pack_bf16(const float (&v)[8])
{
    bf16x8 b;
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = (__bf16)v[j];   // rounds to nearest even
    return b;
}

// Rows and columns beyond the matrix repeat its last ones and are not stored; TN == 4 needs N >= 4.
template <bool TA, bool TB, int TN, int KW>
__global__ __launch_bounds__(KW == 16 ? 1024 : 256) void k_gemm_bf16(
    int M, int N, int K, const float *__restrict__ A, int lda, const float *__restrict__ B, int ldb,
    float *__restrict__ C, int ldc, const float *__restrict__ bias,
    const float *__restrict__ gate, int relu, int accumulate)
{
    constexpr int COLS = 16 * TN, NT = KW == 1 ? 4 : 1;   // tiles per workgroup
    __shared__ __attribute__((aligned(16))) float red[KW == 1 ? 1 : KW * GT_ROWS * COLS];
    const int wave = threadIdx.x / DIGS_WAVE, lane = lane_id();
    const int ntn = (N + COLS - 1) / COLS, ntm = (M + GT_ROWS - 1) / GT_ROWS;
    // (launch_gemm: fewer than 2^26 tiles)
    const uint32_t tile = blockIdx.x * NT + (KW == 1 ? wave : 0);
    const bool have = tile < (uint32_t)ntn * (uint32_t)ntm;   // (false only with KW == 1)
    const bool down = N > M && (M >= 1024 || N >= 65536);
    const uint32_t line = have ? tile / (uint32_t)(down ? ntm : ntn) : 0u;
    const uint32_t step = have ? tile - line * (uint32_t)(down ? ntm : ntn) : 0u;
    const int m0 = (int)(down ? step : line) * GT_ROWS, n0 = (int)(down ? line : step) * COLS;
    const int kw = KW == 1 ? 0 : wave, kl = 8 * (lane >> 4);
    const float *pa[1], *pb[TN];
    const int row = min(m0 + (lane & 15), M - 1);
    pa[0] = A + (TA ? (size_t)row : (size_t)row * lda);
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int col = min(n0 + TN * (lane & 15), N - TN) + t;
        pb[t] = B + (TB ? (size_t)col * ldb : (size_t)col);
    }
    f32x4 acc[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](const float (&a)[1][8], const float (&b)[TN][8]) {
        const bf16x8 fa = pack_bf16(a[0]);
#pragma unroll
        for (int t = 0; t < TN; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, pack_bf16(b[t]), acc[t], 0, 0, 0);
    };
    const int steps = K / GT_K;
    if (kw < steps) {
        // the next step's operands are loaded before this one's are used
        float a[1][8], b[TN][8], an[1][8], bn[TN][8];
        gemm_load<!TA, 1, false>(pa, lda, kw * GT_K + kl, K, a);
        gemm_load<TB, TN, false>(pb, ldb, kw * GT_K + kl, K, b);
        for (int s = kw; s < steps; s += KW) {
            const int k = min(s + KW, steps - 1) * GT_K + kl;
            gemm_load<!TA, 1, false>(pa, lda, k, K, an);
            gemm_load<TB, TN, false>(pb, ldb, k, K, bn);
            multiply(a, b);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                a[0][j] = an[0][j];
#pragma unroll
                for (int t = 0; t < TN; ++t) b[t][j] = bn[t][j];
            }
        }
    }
    if (K % GT_K != 0 && kw == steps % KW) {
        float a[1][8], b[TN][8];
        gemm_load<!TA, 1, true>(pa, lda, steps * GT_K + kl, K, a);
        gemm_load<TB, TN, true>(pb, ldb, steps * GT_K + kl, K, b);
        multiply(a, b);
    }
    // row r of the tile and the TN columns of lane l % 16 == l
    auto store = [&](int r, int l, const float (&v)[TN]) {
        const int rw = m0 + r, first = n0 + TN * l, col = min(first, N - TN);
        if (rw >= M || first >= N) return;
        const size_t o = (size_t)rw * ldc + col;
        float x[TN];
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            x[t] = v[t];
            if (accumulate) x[t] += C[o + t];
            if (bias) x[t] += bias[col + t];
            if (relu) x[t] = fmaxf(x[t], 0.0f);
            if (gate && !(gate[o + t] > 0.0f)) x[t] = 0.0f;
        }
        if (TN == 4 && first == col) {
            *(f32x4u *)(C + o) = f32x4u{x[0], x[1 % TN], x[2 % TN], x[3 % TN]};
        } else {   // (columns before `first` are another lane's)
#pragma unroll
            for (int t = 0; t < TN; ++t)
                if (col + t >= first) C[o + t] = x[t];
        }
    };
    // result lane layout: element r of lane l is row 4 (l / 16) + r, column l % 16
    if constexpr (KW == 1) {
        if (have)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float v[TN];
#pragma unroll
                for (int t = 0; t < TN; ++t) v[t] = acc[t][r];
                store(4 * (lane >> 4) + r, lane & 15, v);
            }
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < TN; ++t)
                red[(wave * GT_ROWS + 4 * (lane >> 4) + r) * COLS + TN * (lane & 15) + t] =
                    acc[t][r];
        __syncthreads();
        if (threadIdx.x < 16 * GT_ROWS) {   // (row, lane of the row)
            float v[TN];
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const float *e = red + TN * threadIdx.x + t;
                v[t] = e[0];
#pragma unroll
                for (int w = 1; w < KW; ++w) v[t] += e[w * GT_ROWS * COLS];
            }
            store(threadIdx.x >> 4, threadIdx.x & 15, v);
        }
    }
}

// The same from tiles of 64 x 64, a workgroup each (four waves, a 32 x 32 block each on
// v_mfma_f32_32x32x16_bf16), K staged through LDS 32 at a time: each operand is read once per 64 rows
// or columns of C, coalesced also where K is the contiguous index.
#define GT_TILE 64
#define GT_LDS 40   // bf16 per LDS row: 80 bytes, so every 8-element fragment is 16-byte aligned

template <bool TA, bool TB>
__global__ __launch_bounds__(256) void k_gemm_bf16_staged(
    int M, int N, int K, const float *__restrict__ A, int lda, const float *__restrict__ B, int ldb,
    float *__restrict__ C, int ldc, const float *__restrict__ bias,
    const float *__restrict__ gate, int relu, int accumulate)
{
    __shared__ __attribute__((aligned(16))) __bf16 As[GT_TILE * GT_LDS];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[GT_TILE * GT_LDS];
    const int m0 = blockIdx.y * GT_TILE, n0 = blockIdx.x * GT_TILE;
    const int tid = threadIdx.x, wave = tid / DIGS_WAVE, lane = lane_id();
    const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    for (int k0 = 0; k0 < K; k0 += GT_K) {
        for (int e = tid; e < GT_TILE * GT_K; e += 256) {
            const int r = TA ? e % GT_TILE : e / GT_K, c = TA ? e / GT_TILE : e % GT_K;
            const int m = m0 + r, k = k0 + c;
            float v = 0.0f;
            if (m < M && k < K) v = TA ? A[(size_t)k * lda + m] : A[(size_t)m * lda + k];
            As[r * GT_LDS + c] = (__bf16)v;
        }
        for (int e = tid; e < GT_TILE * GT_K; e += 256) {
            const int r = TB ? e / GT_K : e % GT_TILE, c = TB ? e % GT_K : e / GT_TILE;
            const int nn = n0 + r, k = k0 + c;
            float v = 0.0f;
            if (nn < N && k < K) v = TB ? B[(size_t)nn * ldb + k] : B[(size_t)k * ldb + nn];
            Bs[r * GT_LDS + c] = (__bf16)v;
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < GT_K; s += 16) {
            const int kk = s + 8 * (lane >> 5);
            const bf16x8 a = *(const bf16x8 *)&As[(wm + (lane & 31)) * GT_LDS + kk];
            const bf16x8 b = *(const bf16x8 *)&Bs[(wn + (lane & 31)) * GT_LDS + kk];
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
        }
        __syncthreads();
    }
    // result lane layout: element r of lane l is row 8(r/4) + 4(l/32) + r%4, column l%32
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = m0 + wm + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const int col = n0 + wn + (lane & 31);
        if (row < M && col < N) {
            const size_t o = (size_t)row * ldc + col;
            float v = acc[r];
            if (accumulate) v += C[o];
            if (bias) v += bias[col];
            if (relu) v = fmaxf(v, 0.0f);
            if (gate && !(gate[o] > 0.0f)) v = 0.0f;
            C[o] = v;
        }
    }
}

// out[j] = sum_i X[i][j] (bias gradients), a thread per column, rows in order
__global__ __launch_bounds__(256) void k_colsum_few(int M, int N, const float *__restrict__ X, int ldx,
                                                    float *__restrict__ out)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= N) return;
    float s = 0.0f;
    for (int i = 0; i < M; ++i) s += X[(size_t)i * ldx + j];
    out[j] = s;
}

// The same with the rows split: a workgroup takes 64 columns, its 16 waves every 16th row each, and
// their sums are added in wave order.
#define COLSUM_WAVES 16
__global__ __launch_bounds__(COLSUM_WAVES * DIGS_WAVE) void k_colsum(int M, int N,
                                                                     const float *__restrict__ X,
                                                                     int ldx,
                                                                     float *__restrict__ out)
{
    __shared__ float part[COLSUM_WAVES][DIGS_WAVE];
    const int wave = threadIdx.x / DIGS_WAVE, lane = lane_id();
    const int64_t j = (int64_t)blockIdx.x * DIGS_WAVE + lane;
    float s = 0.0f;
    if (j < N)
#pragma unroll 4
        for (int i = wave; i < M; i += COLSUM_WAVES) s += X[(size_t)i * ldx + j];
    part[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && j < N) {
#pragma unroll
        for (int w = 1; w < COLSUM_WAVES; ++w) s += part[w][lane];
        out[j] = s;
    }
}

// Mean squared error against standardised targets, (pred - (target - mean)/std)^2 averaged over
// the B x R entries: dpred = its gradient; loss[0] = its value. One workgroup, fixed order.
__global__ __launch_bounds__(256) void k_mse(int B, int R, const float *__restrict__ pred,
                                             const float *__restrict__ target,
                                             const float *__restrict__ mean,
                                             const float *__restrict__ stdv,
                                             float *__restrict__ dpred, float *__restrict__ loss)
{
    __shared__ float part[256];
    const int m = B * R;
    const float inv = 1.0f / (float)m;
    float s = 0.0f;
    for (int i = threadIdx.x; i < m; i += 256) {
        const int r = i % R;
        const float d = pred[i] - (target[i] - mean[r]) / stdv[r];
        dpred[i] = 2.0f * d * inv;
        s = fmaf(d, d, s);
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0 && loss) loss[0] = part[0] * inv;
}

// Adam on FP32 master weights (bias-corrected moments; c1 = 1 - b1^t, c2 = 1 - b2^t)
__global__ __launch_bounds__(256) void k_adam(int n, float *__restrict__ w,
                                              const float *__restrict__ g, float *__restrict__ m,
                                              float *__restrict__ v, float lr, float b1, float b2,
                                              float eps, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = fmaf(b1, m[i], (1.0f - b1) * gi);
    const float vi = fmaf(b2, v[i], (1.0f - b2) * gi * gi);
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Network input of view t: the projection averaged over fy x fx pixel blocks (row-major,
// (nv/fy) x (nu/fx) values) times `scale`, standardised per feature if fmean/fistd are given
// ((x - fmean[i]) * fistd[i]), then sin and cos of the gantry angle.
__global__ __launch_bounds__(256) void k_downsample(int T, int nv, int nu, int fy, int fx,
                                                    const float *__restrict__ proj,
                                                    const float *__restrict__ angles,
                                                    float scale, const float *__restrict__ fmean,
                                                    const float *__restrict__ fistd,
                                                    float *__restrict__ out, int ld_out)
{
    const int oy = nv / fy, ox = nu / fx;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int t = blockIdx.y;
    if (t >= T) return;
    float *o = out + (size_t)t * ld_out;
    if (i < oy * ox) {
        const int Y = i / ox, X = i % ox;
        const float *src = proj + ((size_t)t * nv + (size_t)Y * fy) * nu + (size_t)X * fx;
        float s = 0.0f;
        for (int a = 0; a < fy; ++a)
            for (int b = 0; b < fx; ++b) s += src[(size_t)a * nu + b];
        float v = s * scale / (float)(fy * fx);
        if (fmean) v = (v - fmean[i]) * fistd[i];
        o[i] = v;
    } else if (i == oy * ox && angles) {
        float sn, cs;
        sincosf(angles[t], &sn, &cs);
        o[i] = sn;
        o[i + 1] = cs;
    }
}

// X[i][j] = (X[i][j] - mean[j]) * istd[j] for the first N columns of M rows (in place)
__global__ __launch_bounds__(256) void k_standardize(int M, int N, float *__restrict__ X, int ldx,
                                                     const float *__restrict__ mean,
                                                     const float *__restrict__ istd)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)M * N) return;
    const int i = (int)(idx / N), j = (int)(idx % N);
    float *x = X + (size_t)i * ldx + j;
    *x = (*x - mean[j]) * istd[j];
}

// ------------------------------------------------------------------------------------------
// Normal equations of one Levenberg-Marquardt step per view. imgs holds, per view t, R + 1
// rendered images (base weights, then the base with w_r raised by h[r]), each npix long; meas the
// measured image. With J_r = (I_r - I_0)/h_r and res = I_0 - P:
//   out[t] = (JtJ upper triangle, row-major (R(R+1)/2), Jt res (R), res.res (1)).
// One workgroup per view and slice of LM_SLICE pixels (or, without a workspace for the slices'
// sums, per view), four pixels per thread at a time; fixed-order sums, which depend on npix alone.
// Memory-bound: each image is read once. A workgroup per view keeps at most T of the 256 CUs
// busy, each at what one CU can draw from memory.
// Measured against a workgroup per view, 64 views of 196608 pixels, R = 3: 267 -> 41 us (6.1 TB/s),
// with every image read for the first time 397 -> 47; one such view 119 -> 7.3 us.
#define LM_SLICE 4096

__device__ __forceinline__ float lm_wave_sum(float v)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, DIGS_WAVE);
    return v;
}

// dst[t][k][s]: term k of slice s of view t (nsl slices of `per` pixels)
template <int R>
__global__ __launch_bounds__(256) void k_lm_normal_eq(int npix, int per, int nsl,
                                                      const float *__restrict__ imgs,
                                                      const float *__restrict__ meas,
                                                      const float *__restrict__ h,
                                                      float *__restrict__ dst)
{
    constexpr int NOUT = R * (R + 1) / 2 + R + 1;
    __shared__ float red[4][NOUT];
    const int t = blockIdx.x / nsl, sl = blockIdx.x % nsl;
    const int begin = sl * per, end = min(npix - begin, per) + begin;
    const float *base = imgs + (size_t)t * (R + 1) * npix;
    const float *P = meas + (size_t)t * npix;
    float acc[NOUT];
#pragma unroll
    for (int k = 0; k < NOUT; ++k) acc[k] = 0.0f;
    float ih[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ih[r] = 1.0f / h[r];
    auto pixel = [&](float i0, float p, const float (&ir)[R]) {
        const float res = i0 - p;
        float J[R];
#pragma unroll
        for (int r = 0; r < R; ++r) J[r] = (ir[r] - i0) * ih[r];
        int k = 0;
#pragma unroll
        for (int a = 0; a < R; ++a)
#pragma unroll
            for (int b = a; b < R; ++b) acc[k++] += J[a] * J[b];
#pragma unroll
        for (int a = 0; a < R; ++a) acc[k++] += J[a] * res;
        acc[k] += res * res;
    };
    const int quads = (end - begin) / 4;
#pragma unroll 2
    for (int q = threadIdx.x; q < quads; q += 256) {
        const int p = begin + 4 * q;
        const f32x4u m = *(const f32x4u *)(P + p), i0 = *(const f32x4u *)(base + p);
        f32x4u ir[R];
#pragma unroll
        for (int r = 0; r < R; ++r) ir[r] = *(const f32x4u *)(base + (size_t)(r + 1) * npix + p);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v[R];
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = ir[r][i];
            pixel(i0[i], m[i], v);
        }
    }
    const int p = begin + 4 * quads + (int)threadIdx.x;
    if (p < end) {
        float v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = base[(size_t)(r + 1) * npix + p];
        pixel(base[p], P[p], v);
    }
#pragma unroll
    for (int k = 0; k < NOUT; ++k) {
        const float v = lm_wave_sum(acc[k]);
        if (lane_id() == 0) red[threadIdx.x / DIGS_WAVE][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < NOUT)
        dst[((size_t)t * NOUT + threadIdx.x) * nsl + sl] =
            (red[0][threadIdx.x] + red[1][threadIdx.x]) +
            (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// out[i] = sum over the slices of part[i][..], a wave per i
__global__ __launch_bounds__(256) void k_lm_sum(int64_t m, int nsl, const float *__restrict__ part,
                                                float *__restrict__ out)
{
    for (int64_t i = (int64_t)blockIdx.x * 4 + threadIdx.x / DIGS_WAVE; i < m;
         i += (int64_t)gridDim.x * 4) {
        float s = 0.0f;
        for (int k = lane_id(); k < nsl; k += DIGS_WAVE) s += part[i * nsl + k];
        s = lm_wave_sum(s);
        if (lane_id() == 0) out[i] = s;
    }
}

// ------------------------------------------------------------------------------------------
static int wrc(hipError_t e) { return e == hipSuccess ? DIGS_OK : digs_set_hip_error(e); }

struct GemmArgs {
    int M, N, K;
    const float *A;
    int lda;
    const float *B;
    int ldb;
    float *C;
    int ldc;
    const float *bias, *gate;
    int relu, accumulate;
    hipStream_t s;
};

template <bool TA, bool TB, int TN, int KW>
static void launch_gemm_tiles(const GemmArgs &g, int64_t tiles)
{
    const int64_t wgs = KW == 1 ? (tiles + 3) / 4 : tiles;
    hipLaunchKernelGGL((k_gemm_bf16<TA, TB, TN, KW>), dim3((unsigned)wgs),
                       dim3((KW == 1 ? 4 : KW) * DIGS_WAVE), 0, g.s, g.M, g.N, g.K, g.A, g.lda, g.B,
                       g.ldb, g.C, g.ldc, g.bias, g.gate, g.relu, g.accumulate);
}

// Where the lines lie (times in us, both ways measured at each):
// - Waves over K, so that one has at most a few steps of 32 to take in turn (16 from K = 993 on, 4 from
//   225 on), but only while the tiles leave the chip idle: at most 4 from 1024 tiles on (1024x1024x1024:
//   29 with 16, 21 with 4, 41 with 1), one from 2048 on (4096x512x1024: 57 with 16, 41 with 4, 35 with
//   1; 4096x2048x1024: 209, 140, 128).
// - Wide tiles read A a quarter as often, but there are a quarter as many of them: they are taken
//   where that leaves two waves per SIMD (256x512x4098: 24 narrow, 21 wide; 4098x512x256: 29 and 17),
//   not below (32x256x4098: 9 on 32 narrow tiles, 16 on 8 wide ones; 4098x256x32: 4.4 and 5.5).
// - Staged tiles where B is transposed (a lane's eight values of K are 32 bytes of a row there, and the
//   rows are far apart) and C large enough for the longer way to them: 2048x2048x64 18 direct and 11
//   staged, 3072x2048x1024 216 and 180, but 2048x2048x1024 145 and 170, 4096x512x256 24 and 36; and for
//   the shortest K (3072x2048x32: 11 and 9; 3072x2048x128: 12 and 13). Also where the direct tiles'
//   threads do not fit one dimension of a launch.
template <bool TA, bool TB>
static void launch_gemm(const GemmArgs &g)
{
    const int64_t rows = (g.M + GT_ROWS - 1) / GT_ROWS, cols = ((int64_t)g.N + 63) / 64;
    const int64_t wide = rows * cols, narrow = rows * (((int64_t)g.N + 15) / 16);
    const int steps = (g.K + GT_K - 1) / GT_K;
    int kw = steps >= 32 ? 16 : steps >= 8 ? 4 : 1;
    const bool use_wide = g.N >= 64 && wide * kw >= 2048;
    const int64_t tiles = use_wide ? wide : narrow;
    if (tiles >= 1024) kw = std::min(kw, 4);
    if (tiles >= 2048) kw = 1;
    const int64_t blocks = (rows + 3) / 4 * cols;   // of 64 x 64
    int64_t from = INT64_MAX;   // staged from so many blocks on
    if (TB) from = g.K <= 128 ? 512 : g.K <= 256 ? 768 : g.K <= 512 ? 1024 : 1536;
    else if (!TA && g.K <= 64) from = g.K <= 32 ? 1024 : 1536;
    if ((std::min(g.M, g.N) >= 64 && blocks >= from) || tiles >= (1 << 26)) {
        hipLaunchKernelGGL((k_gemm_bf16_staged<TA, TB>), dim3((unsigned)cols, (unsigned)((rows + 3) / 4)),
                           dim3(256), 0, g.s, g.M, g.N, g.K, g.A, g.lda, g.B, g.ldb, g.C, g.ldc,
                           g.bias, g.gate, g.relu, g.accumulate);
    } else if (use_wide) {
        if (kw == 16) launch_gemm_tiles<TA, TB, 4, 16>(g, wide);
        else if (kw == 4) launch_gemm_tiles<TA, TB, 4, 4>(g, wide);
        else launch_gemm_tiles<TA, TB, 4, 1>(g, wide);
    } else {
        if (kw == 16) launch_gemm_tiles<TA, TB, 1, 16>(g, narrow);
        else if (kw == 4) launch_gemm_tiles<TA, TB, 1, 4>(g, narrow);
        else launch_gemm_tiles<TA, TB, 1, 1>(g, narrow);
    }
}

extern "C" int digs_gemm_bf16(int M, int N, int K, const float *A, int lda, int transA,
                              const float *B, int ldb, int transB, float *C, int ldc,
                              const float *bias, const float *gate, int relu, int accumulate,
                              void *stream)
{
    if (M < 0 || N < 0 || K < 0 || M > (1 << 24) || N > (1 << 24) || K > (1 << 24))
        return DIGS_EINVAL;
    if (M == 0 || N == 0) return DIGS_OK;
    if (!A || !B || !C || lda <= 0 || ldb <= 0 || ldc < N) return DIGS_EINVAL;
    if ((transA ? lda < M : lda < K) || (transB ? ldb < K : ldb < N)) return DIGS_EINVAL;
    GemmArgs g{M, N, K, A, lda, B, ldb, C, ldc, bias, gate, relu, accumulate, (hipStream_t)stream};
    if (!transA && !transB) launch_gemm<false, false>(g);
    else if (transA && !transB) launch_gemm<true, false>(g);
    else if (!transA && transB) launch_gemm<false, true>(g);
    else launch_gemm<true, true>(g);
    return wrc(hipGetLastError());
}

extern "C" int digs_colsum(int M, int N, const float *X, int ldx, float *out, void *stream)
{
    if (M < 0 || N < 0 || (N > 0 && (!X || !out || ldx < N))) return DIGS_EINVAL;
    if (N == 0) return DIGS_OK;
    // Few rows over many columns leave most of the 16 waves with one row or none, and the launch of
    // the waves is what takes the time: 16 x 2^20 13 us a thread per column, 31 split, 1 x 2^24 28 and
    // 379, 32 x 2^18 8 and 11; but 64 x 2^18 19 and 13, 32 x 2^16 8.5 and 7.6, 256 x 512 25 and 8. (A
    // launch has fewer than 2^32 threads.)
    if ((M < 64 && N > (1 << 16)) || N >= (1 << 28))
        hipLaunchKernelGGL(k_colsum_few, dim3((unsigned)(((int64_t)N + 255) / 256)), dim3(256), 0,
                           (hipStream_t)stream, M, N, X, ldx, out);
    else
        hipLaunchKernelGGL(k_colsum, dim3((N + DIGS_WAVE - 1) / DIGS_WAVE),
                           dim3(COLSUM_WAVES * DIGS_WAVE), 0, (hipStream_t)stream, M, N, X, ldx, out);
    return wrc(hipGetLastError());
}

extern "C" int digs_mse(int B, int R, const float *pred, const float *target, const float *mean,
                        const float *stdv, float *dpred, float *loss, void *stream)
{
    if (B <= 0 || R <= 0 || !pred || !target || !mean || !stdv || !dpred) return DIGS_EINVAL;
    hipLaunchKernelGGL(k_mse, dim3(1), dim3(256), 0, (hipStream_t)stream, B, R, pred, target,
                       mean, stdv, dpred, loss);
    return wrc(hipGetLastError());
}

extern "C" int digs_adam(int n, float *w, const float *g, float *m, float *v, float lr, float b1,
                         float b2, float eps, int step, void *stream)
{
    if (n < 0 || step < 1 || !(lr >= 0.0f) || (n > 0 && (!w || !g || !m || !v)))
        return DIGS_EINVAL;
    if (n == 0) return DIGS_OK;
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, n, w, g,
                       m, v, lr, b1, b2, eps, c1, c2);
    return wrc(hipGetLastError());
}

extern "C" int digs_downsample(int T, int nv, int nu, int fy, int fx, const float *proj,
                               const float *angles, float scale, const float *fmean,
                               const float *fistd, float *out, int ld_out, void *stream)
{
    if (T < 0 || nv <= 0 || nu <= 0 || fy <= 0 || fx <= 0 || nv % fy || nu % fx) return DIGS_EINVAL;
    const int nfeat = (nv / fy) * (nu / fx);
    if (T == 0) return DIGS_OK;
    if (!proj || !out || ld_out < nfeat + (angles ? 2 : 0) || (!fmean != !fistd))
        return DIGS_EINVAL;
    hipLaunchKernelGGL(k_downsample, dim3((nfeat + 2 + 255) / 256, T), dim3(256), 0,
                       (hipStream_t)stream, T, nv, nu, fy, fx, proj, angles, scale, fmean, fistd,
                       out, ld_out);
    return wrc(hipGetLastError());
}

extern "C" int digs_standardize(int M, int N, float *X, int ldx, const float *mean,
                                const float *istd, void *stream)
{
    if (M < 0 || N < 0 || (M > 0 && N > 0 && (!X || !mean || !istd || ldx < N)))
        return DIGS_EINVAL;
    const size_t m = (size_t)M * N;
    if (m == 0) return DIGS_OK;
    hipLaunchKernelGGL(k_standardize, dim3((unsigned)((m + 255) / 256)), dim3(256), 0,
                       (hipStream_t)stream, M, N, X, ldx, mean, istd);
    return wrc(hipGetLastError());
}

// Slices per view (a function of R and npix alone, but for results past 2^31 slices). Views of up to
// 73728 pixels in their R + 2 images go whole: the second launch and the workspace cost more there than
// the slices save (one view, R = 1, 16384 pixels: 4.0 us whole, 6.8 in slices, 32768 5.7 and 6.9, 65536
// 9.0 and 6.7; R = 4, 8192 pixels 6.7 and 7.6, 16384 8.8 and 7.6).
#define LM_WHOLE 73728

static int64_t lm_slices(int T, int R, int npix)
{
    const int64_t s = ((int64_t)npix + LM_SLICE - 1) / LM_SLICE;
    return (int64_t)npix * (R + 2) <= LM_WHOLE || s * T > INT32_MAX ? 1 : s;
}

static int launch_lm(int T, int R, int npix, const float *imgs, const float *meas, const float *h,
                     float *out, float *part, hipStream_t s)
{
    const int nsl = part ? (int)lm_slices(T, R, npix) : 1, per = nsl > 1 ? LM_SLICE : npix;
    float *dst = nsl > 1 ? part : out;
    switch (R) {
#define LM_CASE(r)                                                                               \
    case r:                                                                                      \
        hipLaunchKernelGGL(k_lm_normal_eq<r>, dim3((unsigned)T * (unsigned)nsl), dim3(256), 0,   \
                           s, npix, per, nsl, imgs, meas, h, dst);                               \
        break;
        LM_CASE(1) LM_CASE(2) LM_CASE(3) LM_CASE(4) LM_CASE(5) LM_CASE(6) LM_CASE(7) LM_CASE(8)
#undef LM_CASE
    }
    if (nsl > 1) {
        const int64_t m = (int64_t)T * (R * (R + 1) / 2 + R + 1);
        hipLaunchKernelGGL(k_lm_sum, dim3((unsigned)std::min<int64_t>((m + 3) / 4, 1 << 20)),
                           dim3(256), 0, s, m, nsl, part, out);
    }
    return wrc(hipGetLastError());
}

extern "C" int digs_lm_normal_eq(int T, int R, int npix, const float *imgs, const float *meas,
                                 const float *h, float *out, void *stream)
{
    if (T < 0 || R < 1 || R > DIGS_MAX_RANK || npix < 0) return DIGS_EINVAL;
    if (T == 0) return DIGS_OK;
    if (!imgs || !meas || !h || !out) return DIGS_EINVAL;
    return launch_lm(T, R, npix, imgs, meas, h, out, nullptr, (hipStream_t)stream);
}

extern "C" size_t digs_lm_workspace_size(int T, int R, int npix)
{
    if (T <= 0 || R < 1 || R > DIGS_MAX_RANK || npix < 0) return 0;
    const int64_t nsl = lm_slices(T, R, npix);
    return nsl > 1 ? (size_t)T * (R * (R + 1) / 2 + R + 1) * (size_t)nsl * sizeof(float) : 0;
}

extern "C" int digs_lm_normal_eq_ws(int T, int R, int npix, const float *imgs, const float *meas,
                                    const float *h, float *out, void *ws, size_t ws_bytes,
                                    void *stream)
{
    if (T < 0 || R < 1 || R > DIGS_MAX_RANK || npix < 0) return DIGS_EINVAL;
    if (T == 0) return DIGS_OK;
    if (!imgs || !meas || !h || !out) return DIGS_EINVAL;
    const size_t need = digs_lm_workspace_size(T, R, npix);
    if (need > 0 && (!ws || ws_bytes < need)) return DIGS_ENOWS;
    return launch_lm(T, R, npix, imgs, meas, h, out, need > 0 ? (float *)ws : nullptr,
                     (hipStream_t)stream);
}
