// fk_mlp.hip -- kernels of the launch-configuration cost model: a small
// fully connected ReLU network trained and run on the GPU.
//
//   gemm      C[M x N] = op(A) * op(B)  (+ bias[n], ReLU) or (* [mask > 0])
//             64x64 output tile per 256-thread block, 4x4 outputs per
//             thread, K-panels of 16 staged through LDS.  Each output sums
//             its K terms in a fixed order, so results are deterministic.
//   colsum    db[n] = sum over rows of dY[:, n]   (fixed row order)
//   mse       loss and dY = 2 (Y - T) / (rows * cols)
//   adam      one Adam step over a flat parameter array
//   gather    rows of a matrix by an index list (mini-batch assembly)
//   forward, delta, grad   the passes of networks of up to 128 hidden units
//             in one launch each, on the fp32 matrix instruction
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "fk_mlp.hpp"

namespace fk {

constexpr int kTile = 64;
constexpr int kPanel = 16;
constexpr int kThreads = 256;

// element (r, c) of a row-major matrix with `ld` columns, optionally read
// transposed
template <bool T>
__device__ __forceinline__ float at(const float *m, int ld, int r, int c)
{
    return T ? m[(int64_t)c * ld + r] : m[(int64_t)r * ld + c];
}

// op(A) is M x K: A row-major M x K (TA = false) or K x M (TA = true).
// op(B) is K x N: B row-major K x N (TB = false) or N x K (TB = true).
template <bool TA, bool TB>
__global__ __launch_bounds__(kThreads) void k_gemm(const float *__restrict__ A,
                                                   const float *__restrict__ B,
                                                   float *__restrict__ C, int M, int N, int K,
                                                   const float *__restrict__ bias,
                                                   const float *__restrict__ mask, int epilogue)
{
    __shared__ float As[kPanel][kTile + 1];
    __shared__ float Bs[kPanel][kTile + 1];
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const int row0 = blockIdx.y * kTile, col0 = blockIdx.x * kTile;
    const int lda = TA ? M : K;
    const int ldb = TB ? K : N;
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i][j] = 0.0f;
    for (int k0 = 0; k0 < K; k0 += kPanel) {
        // stage op(A)[row0.., k0..] and op(B)[k0.., col0..]: 1024 values each
        for (int e = threadIdx.x; e < kPanel * kTile; e += kThreads) {
            const int kk = e / kTile, mm = e % kTile;
            const int r = row0 + mm, k = k0 + kk;
            As[kk][mm] = (r < M && k < K) ? at<TA>(A, lda, r, k) : 0.0f;
            const int c = col0 + mm;
            Bs[kk][mm] = (c < N && k < K) ? at<TB>(B, ldb, k, c) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kPanel; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = As[kk][ty + 16 * i];
                b[i] = Bs[kk][tx + 16 * i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = row0 + ty + 16 * i;
        if (r >= M)
            continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = col0 + tx + 16 * j;
            if (c >= N)
                continue;
            float v = acc[i][j];
            if (epilogue == EPI_BIAS || epilogue == EPI_BIAS_RELU)
                v += bias[c];
            if (epilogue == EPI_BIAS_RELU)
                v = v > 0.0f ? v : 0.0f;
            if (epilogue == EPI_RELU_MASK)
                v = mask[(int64_t)r * N + c] > 0.0f ? v : 0.0f;
            C[(int64_t)r * N + c] = v;
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_colsum(const float *__restrict__ X, int rows, int cols,
                                                     float *__restrict__ out)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cols)
        return;
    float s = 0.0f;
    for (int r = 0; r < rows; ++r)
        s += X[(int64_t)r * cols + c];
    out[c] = s;
}

// One block: loss = mean((Y - T)^2) over rows x cols, dY = 2 (Y - T) / count.
__global__ __launch_bounds__(1024) void k_mse(const float *__restrict__ Y, const float *__restrict__ T,
                                              int64_t count, float *__restrict__ dY,
                                              float *__restrict__ loss)
{
    __shared__ float part[1024];
    float s = 0.0f;
    const float scale = 2.0f / (float)count;
#pragma unroll 8
    for (int64_t i = threadIdx.x; i < count; i += blockDim.x) {
        const float d = Y[i] - T[i];
        s = fmaf(d, d, s);
        dY[i] = scale * d;
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w /= 2) {
        if ((int)threadIdx.x < w)
            part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        loss[0] = part[0] / (float)count;
}

__global__ __launch_bounds__(kThreads) void k_adam(float *__restrict__ p, const float *__restrict__ g,
                                                   float *__restrict__ m, float *__restrict__ v,
                                                   int64_t n, float lr, float b1, float b2, float eps,
                                                   float c1, float c2)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1;  // bias corrections c1 = 1 - b1^t, c2 = 1 - b2^t
    const float vh = vi / c2;
    p[i] = p[i] - lr * mh / (sqrtf(vh) + eps);
}

__global__ __launch_bounds__(kThreads) void k_gather(const float *__restrict__ src, int cols,
                                                     const int32_t *__restrict__ idx, int rows,
                                                     float *__restrict__ dst)
{
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= (int64_t)rows * cols)
        return;
    const int r = (int)(e / cols), c = (int)(e % cols);
    dst[e] = src[(int64_t)idx[r] * cols + c];
}

// Per-column mean and standard deviation of a rows x cols matrix: sums of
// x and x^2 in fp64 over the rows in order; var = max(0, s2/n - mu^2); a
// column with var <= 1e-12 gets std 1.  One thread per column.
__global__ __launch_bounds__(kThreads) void k_colstats(const float *__restrict__ X, int rows,
                                                       int cols, float *__restrict__ mean,
                                                       float *__restrict__ stdv)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cols)
        return;
    double s1 = 0.0, s2 = 0.0;
    for (int r = 0; r < rows; ++r) {
        const double v = X[(int64_t)r * cols + c];
        s1 += v;
        s2 += v * v;
    }
    const double mu = s1 / rows;
    double var = s2 / rows - mu * mu;
    var = var > 0.0 ? var : 0.0;
    mean[c] = (float)mu;
    stdv[c] = var > 1e-12 ? (float)sqrt(var) : 1.0f;
}

// out = (X - mean[c]) / std[c], one fp32 subtraction and one IEEE division.
__global__ __launch_bounds__(kThreads) void k_standardize(const float *__restrict__ X, int64_t rows,
                                                          int cols, const float *__restrict__ mean,
                                                          const float *__restrict__ stdv,
                                                          float *__restrict__ out)
{
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= rows * cols)
        return;
    const int c = (int)(e % cols);
    out[e] = (X[e] - mean[c]) / stdv[c];
}

// out[0] = mean of x[0..n) (fp64 sum in order, one thread).
__global__ void k_mean(const float *__restrict__ x, int n, float *__restrict__ out)
{
    double acc = 0.0;
    for (int i = 0; i < n; ++i)
        acc += x[i];
    out[0] = (float)(acc / n);
}

// ------------------------------------------------ fused passes, H <= 128 --
// The whole network over a block's rows in one launch, on the fp32 matrix
// instruction (v_mfma_f32_16x16x4: lane l holds A[l % 16][l / 16],
// B[l / 16][l % 16] and D[4 (l / 16) + r][l % 16], r < 4; it adds its four
// products in order, so the forward pass has k_gemm's bits).
//
// Bound by latency at a training batch: 512 rows are 0.12 GFLOP and 0.5 MB.
// One launch per product, four dW products of 4 to 16 blocks that walked
// all rows (93 us each) and four column sums of one thread per column (96 us
// each) took 880 us for forward, loss and backward.  Here a pass is one
// launch (two for the backward), 16 rows a block, all weights fetched at
// once, and the reductions over rows split over the waves of a block:
// 40 us (12.7 forward, 4.3 loss, 6.2 deltas, 18 gradients; the last has 152
// blocks, of which the 8 of layer 0 walk all rows through two products).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kRows = 16;         // rows of a block: one tile
constexpr int kWaves = 8;         // one 16-column tile of a 128-wide layer each
constexpr int kLd = kMlpMaxH + 4; // LDS row: 4 (l % 16) + l / 16 are distinct banks
constexpr int kSteps = kMlpMaxH / 4;

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// One lane's B operands of a layer: element (k, col) at p[k * sk + col * sc],
// zero outside K x N.
__device__ __forceinline__ void load_b(const float *p, int sk, int sc, int K, int N, int col, int g,
                                       float (&b)[kSteps])
{
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
        // a load of every lane (element 0 outside), then a select: no branch per load
        const int k = 4 * s + g;
        const bool in = k < K && col < N;
        float v = 0.0f;
        if (4 * s < K)  // uniform
            v = p[in ? k * sk + col * sc : 0];
        b[s] = in ? v : 0.0f;
    }
}

// The 4 x 4 transpose of (lane / 16, register): register q of lane group g
// takes what register g of lane group q held.
__device__ __forceinline__ void transpose4(float &r0, float &r1, float &r2, float &r3)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    auto swap32 = [](float &a, float &b) {  // a.hi <-> b.lo (halves of the wave)
        const u2 t = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a),
                                                      __builtin_bit_cast(unsigned, b), false, false);
        const unsigned x = t.x, y = t.y;  // (bit_cast of an element takes element 0)
        a = __builtin_bit_cast(float, x);
        b = __builtin_bit_cast(float, y);
    };
    auto swap16 = [](float &a, float &b) {  // a's odd 16-lane rows <-> b's even ones
        const u2 t = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a),
                                                      __builtin_bit_cast(unsigned, b), false, false);
        const unsigned x = t.x, y = t.y;  // (bit_cast of an element takes element 0)
        a = __builtin_bit_cast(float, x);
        b = __builtin_bit_cast(float, y);
    };
    swap32(r0, r2);
    swap32(r1, r3);
    swap16(r0, r1);
    swap16(r2, r3);
}

// B operands of a layer y = x W^T: element (k, col) = W[col][k].  Full (K a
// multiple of 16, rows 16-byte aligned): 16 bytes a lane along k, in the
// order of the products after turn_w; columns past N repeat the last one
// (their results are not stored).
template <bool Full>
__device__ __forceinline__ void load_w(const float *w, int K, int N, int col, int g, float (&b)[kSteps])
{
    if constexpr (Full) {
        const float *p = w + (int64_t)(col < N ? col : N - 1) * K + 4 * g;
#pragma unroll
        for (int t = 0; t < kSteps / 4; ++t) {
            f32x4 q = {0.0f, 0.0f, 0.0f, 0.0f};
            if (16 * t < K)  // uniform
                q = *(const f32x4 *)(p + 16 * t);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                b[4 * t + c] = q[c];
        }
    } else {
        load_b(w, 1, K, K, N, col, g, b);
    }
}
template <bool Full>
__device__ __forceinline__ void turn_w(float (&b)[kSteps])
{
    if constexpr (Full) {
#pragma unroll
        for (int t = 0; t < kSteps / 4; ++t)
            transpose4(b[4 * t], b[4 * t + 1], b[4 * t + 2], b[4 * t + 3]);
    }
}

// A 16 x 16 tile of A (16 x K in LDS) times the lane's B operands.
__device__ __forceinline__ f32x4 tile_product(const float (*act)[kLd], const float (&b)[kSteps], int K,
                                              int i, int g)
{
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
        if (4 * s < K)  // uniform
            acc = mfma(act[i][4 * s + g], b[s], acc);
    return acc;
}

// 16 rows of src (n x cols) into LDS, zero past n and cols (up to a multiple of 4).
__device__ __forceinline__ void stage_rows(const float *src, int cols, int row0, int n, float (*act)[kLd])
{
    const int wide = (cols + 3) & ~3;
    for (int e = threadIdx.x; e < kRows * wide; e += kWaves * 64) {
        const int r = e / wide, c = e % wide;
        act[r][c] = row0 + r < n && c < cols ? src[(int64_t)(row0 + r) * cols + c] : 0.0f;
    }
}

template <bool Full>
__global__ __launch_bounds__(kWaves * 64) void k_mlp_forward(const MlpNet net, const float *__restrict__ x,
                                                             float *__restrict__ h0, float *__restrict__ h1,
                                                             float *__restrict__ h2, float *__restrict__ y,
                                                             int n)
{
    __shared__ float act[2][kRows][kLd];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int i = lane % 16, g = lane / 16;
    const int row0 = blockIdx.x * kRows, H = net.H;
    const int col = wave * 16 + i;
    // every layer's weights at once: one wait for memory instead of four
    float b[4][kSteps], bias[4];
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const int N = l == 3 ? kMlpOut : H;
        load_w<Full>(net.w[l], l == 0 ? kMlpIn : H, N, col, g, b[l]);
        bias[l] = net.b[l][col < N ? col : 0];
    }
    stage_rows(x, kMlpIn, row0, n, act[0]);
    __syncthreads();
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const int K = l == 0 ? kMlpIn : H, N = l == 3 ? kMlpOut : H;
        const bool on = wave * 16 < N;  // uniform over the wave
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        if (on) {
            turn_w<Full>(b[l]);
            acc = tile_product(act[l & 1], b[l], K, i, g);
            float *out = l == 0 ? h0 : l == 1 ? h1 : l == 2 ? h2 : y;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * g + r;
                float v = acc[r] + bias[l];
                if (l < 3)
                    v = v > 0.0f ? v : 0.0f;
                if (l < 3)
                    act[(l + 1) & 1][row][col] = col < N ? v : 0.0f;
                if (row0 + row < n && col < N)
                    out[(int64_t)(row0 + row) * N + col] = v;
            }
        }
        __syncthreads();
    }
}

// The loss gradient through layers 3 and 2: d2 = dy W3 masked by h2 > 0,
// d1 = d2 W2 masked by h1 > 0.
__global__ __launch_bounds__(kWaves * 64) void k_mlp_delta(const MlpNet net, const float *__restrict__ dy,
                                                           const float *__restrict__ h1,
                                                           const float *__restrict__ h2,
                                                           float *__restrict__ d1, float *__restrict__ d2,
                                                           int n)
{
    __shared__ float act[2][kRows][kLd];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int i = lane % 16, g = lane / 16;
    const int row0 = blockIdx.x * kRows, H = net.H;
    const int col = wave * 16 + i;
    const bool on = wave * 16 < H;  // uniform over the wave
    float b[2][kSteps], m[2][4];
    load_b(net.w[3], H, 1, kMlpOut, H, col, g, b[0]);
    load_b(net.w[2], H, 1, H, H, col, g, b[1]);
#pragma unroll
    for (int l = 0; l < 2; ++l)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool ok = row0 + 4 * g + r < n && col < H;
            const float v = (l == 0 ? h2 : h1)[ok ? (int64_t)(row0 + 4 * g + r) * H + col : 0];
            m[l][r] = ok ? v : 0.0f;
        }
    stage_rows(dy, kMlpOut, row0, n, act[0]);
    __syncthreads();
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        float *out = l == 0 ? d2 : d1;
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        if (on)
            acc = tile_product(act[l], b[l], l == 0 ? kMlpOut : H, i, g);
        if (on) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * g + r;
                const float v = m[l][r] > 0.0f ? acc[r] : 0.0f;
                if (l == 0)
                    act[1][row][col] = v;
                if (row0 + row < n && col < H)
                    out[(int64_t)(row0 + row) * H + col] = v;
            }
        }
        __syncthreads();
    }
}

// Every weight and bias gradient: a block per 16 x 16 tile of a dW (and the
// bias sums of its first tile column), its waves over the rows, combined in
// wave order.  dW0 = d0^T x needs d0 = d1 W1 masked by h0 > 0, which its
// blocks (a 16-wide tile of d0's columns each) compute 16 rows at a time:
// the product's D registers are the next product's A operands as they
// stand, with row 4 (l / 16) + r at step r.
template <bool Full>
__global__ __launch_bounds__(kWaves * 64) void k_mlp_grad(const MlpNet net, const float *__restrict__ x,
                                                          const float *__restrict__ h0,
                                                          const float *__restrict__ h1,
                                                          const float *__restrict__ h2,
                                                          const float *__restrict__ d1,
                                                          const float *__restrict__ d2,
                                                          const float *__restrict__ dy, MlpGrad out, int n)
{
    __shared__ float red[2][kWaves][4][64];
    __shared__ float red_b[kWaves][64];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int i = lane % 16, g = lane / 16;
    const int H = net.H, nt = (H + 15) / 16;
    int job = blockIdx.x, l = 0, to = 0, ti = 0;
    if (job < nt) {
        to = job;
    } else if ((job -= nt) < 2 * nt * nt) {
        l = 1 + job / (nt * nt);
        to = job % (nt * nt) / nt;
        ti = job % nt;
    } else {
        l = 3;
        job -= 2 * nt * nt;
        to = job / nt;
        ti = job % nt;
    }
    const int NO = l == 3 ? kMlpOut : H, NI = l == 0 ? kMlpIn : H;
    const int o = to * 16 + i, in = ti * 16 + i;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, acc2 = {0.0f, 0.0f, 0.0f, 0.0f};
    float sum = 0.0f;
    if (l > 0) {
        const float *d = l == 3 ? dy : l == 2 ? d2 : d1;
        const float *a = l == 3 ? h2 : l == 2 ? h1 : h0;
        // 32 rows a round, the next round's operands in flight
        constexpr int S = 8;
        float av[S], bv[S];
        auto fetch = [&](int r0, float (&pa)[S], float (&pb)[S]) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int row = r0 + 4 * s + g;
                const int64_t q = row < n ? row : n - 1;
                const float va = d[q * NO + (o < NO ? o : NO - 1)];
                const float vb = a[q * NI + (in < NI ? in : NI - 1)];
                pa[s] = row < n && o < NO ? va : 0.0f;
                pb[s] = row < n && in < NI ? vb : 0.0f;
            }
        };
        int r0 = wave * 4 * S;
        fetch(r0, av, bv);
        while (r0 < n) {
            float an[S], bn[S];
            r0 += kWaves * 4 * S;
            fetch(r0, an, bn);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                if (s % 2)
                    acc2 = mfma(av[s], bv[s], acc2);
                else
                    acc = mfma(av[s], bv[s], acc);
                sum += av[s];
                av[s] = an[s];
                bv[s] = bn[s];
            }
        }
        acc += acc2;
        acc2 = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    } else {
        // the product's k index in the order of the loads of d1's rows: any
        // order serves, as long as both operands take the same (Full: 16
        // bytes a lane, step 4 t + c at k = 16 t + 4 (l / 16) + c)
        float b[kSteps];
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int k = Full ? s / 4 * 16 + 4 * g + s % 4 : 4 * s + g;
            const bool ok = k < H && o < H;
            const float v = net.w[1][ok ? k * H + o : 0];
            b[s] = ok ? v : 0.0f;
        }
        struct Chunk {
            float a[kSteps], m[4], x[2][4];
        };
        auto fetch = [&](int r0, Chunk &q) {
            const int64_t ra = r0 + i < n ? r0 + i : n - 1;
#pragma unroll
            for (int s = 0; s < kSteps; s += 4) {
                if constexpr (Full) {
                    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
                    if (4 * s < H)  // uniform
                        v = *(const f32x4 *)(d1 + ra * H + 4 * s + 4 * g);
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        q.a[s + c] = v[c];
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int k = 4 * (s + c) + g;
                        const float v = d1[ra * H + (k < H ? k : 0)];
                        q.a[s + c] = k < H ? v : 0.0f;
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = r0 + 4 * g + r;
                const int64_t rc = row < n ? row : n - 1;
                const float h = h0[rc * H + (o < H ? o : 0)];
                const float x0 = x[rc * kMlpIn + i], x1 = x[rc * kMlpIn + 16 + i];
                q.m[r] = row < n && o < H ? h : 0.0f;
                q.x[0][r] = row < n ? x0 : 0.0f;
                q.x[1][r] = row < n ? x1 : 0.0f;
            }
        };
        Chunk cur;
        int r0 = wave * kRows;
        fetch(r0, cur);
        while (r0 < n) {
            Chunk nxt;
            r0 += kWaves * kRows;
            fetch(r0, nxt);
            f32x4 dd = {0.0f, 0.0f, 0.0f, 0.0f}, de = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < kSteps; s += 2)
                if (4 * s < H) {
                    dd = mfma(cur.a[s], b[s], dd);
                    de = mfma(cur.a[s + 1], b[s + 1], de);
                }
            dd += de;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool on = cur.m[r] > 0.0f;
                const float v = on ? dd[r] : 0.0f;
                acc = mfma(v, cur.x[0][r], acc);
                acc2 = mfma(v, cur.x[1][r], acc2);
                sum += v;
            }
            cur = nxt;
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        red[0][wave][r][lane] = acc[r];
        red[1][wave][r][lane] = acc2[r];
    }
    red_b[wave][lane] = sum;
    __syncthreads();
    // 256 sums of the tile (twice for dW0's two column tiles), then 16 of the bias
    for (int e = threadIdx.x; e < (l == 0 ? 512 : 256); e += kWaves * 64) {
        const int t = e / 256, r = e % 256 / 64, ln = e % 64;
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            s += red[t][w][r][ln];
        const int oo = to * 16 + 4 * (ln / 16) + r, ii = (ti + t) * 16 + ln % 16;
        if (oo < NO && ii < NI)
            out.w[l][(int64_t)oo * NI + ii] = s;
    }
    if (ti == 0 && threadIdx.x < 16 && to * 16 + (int)threadIdx.x < NO) {
        float s = 0.0f;
        for (int w = 0; w < kWaves; ++w)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                s += red_b[w][16 * q + threadIdx.x];
        out.b[l][to * 16 + threadIdx.x] = s;
    }
}

// ------------------------------------------------------------- launchers --

hipError_t mlp_gemm(bool ta, bool tb, const float *A, const float *B, float *C, int M, int N, int K,
                    const float *bias, const float *mask, int epilogue, hipStream_t s)
{
    if (M <= 0 || N <= 0)
        return hipSuccess;
    dim3 grid((N + kTile - 1) / kTile, (M + kTile - 1) / kTile);
    if (!ta && !tb)
        k_gemm<false, false><<<grid, kThreads, 0, s>>>(A, B, C, M, N, K, bias, mask, epilogue);
    else if (!ta && tb)
        k_gemm<false, true><<<grid, kThreads, 0, s>>>(A, B, C, M, N, K, bias, mask, epilogue);
    else if (ta && !tb)
        k_gemm<true, false><<<grid, kThreads, 0, s>>>(A, B, C, M, N, K, bias, mask, epilogue);
    else
        k_gemm<true, true><<<grid, kThreads, 0, s>>>(A, B, C, M, N, K, bias, mask, epilogue);
    return hipGetLastError();
}

hipError_t mlp_colsum(const float *X, int rows, int cols, float *out, hipStream_t s)
{
    k_colsum<<<(cols + kThreads - 1) / kThreads, kThreads, 0, s>>>(X, rows, cols, out);
    return hipGetLastError();
}

hipError_t mlp_mse(const float *Y, const float *T, int64_t count, float *dY, float *loss,
                   hipStream_t s)
{
    k_mse<<<1, 1024, 0, s>>>(Y, T, count, dY, loss);
    return hipGetLastError();
}

hipError_t mlp_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1,
                    float b2, float eps, int step, hipStream_t s)
{
    const float c1 = 1.0f - powf(b1, (float)step);
    const float c2 = 1.0f - powf(b2, (float)step);
    k_adam<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(p, g, m, v, n, lr, b1, b2,
                                                                         eps, c1, c2);
    return hipGetLastError();
}

hipError_t mlp_gather(const float *src, int cols, const int32_t *idx, int rows, float *dst,
                      hipStream_t s)
{
    const int64_t n = (int64_t)rows * cols;
    if (n == 0)
        return hipSuccess;
    k_gather<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(src, cols, idx, rows, dst);
    return hipGetLastError();
}

hipError_t mlp_colstats(const float *X, int rows, int cols, float *mean, float *stdv, hipStream_t s)
{
    k_colstats<<<(cols + kThreads - 1) / kThreads, kThreads, 0, s>>>(X, rows, cols, mean, stdv);
    return hipGetLastError();
}

hipError_t mlp_standardize(const float *X, int64_t rows, int cols, const float *mean,
                           const float *stdv, float *out, hipStream_t s)
{
    const int64_t n = rows * cols;
    if (n == 0)
        return hipSuccess;
    k_standardize<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(X, rows, cols, mean,
                                                                               stdv, out);
    return hipGetLastError();
}

hipError_t mlp_mean(const float *x, int n, float *out, hipStream_t s)
{
    k_mean<<<1, 1, 0, s>>>(x, n, out);
    return hipGetLastError();
}

hipError_t mlp_forward(const MlpNet &net, const float *x, float *const h[3], float *y, int n, hipStream_t s)
{
    const dim3 grid((n + kRows - 1) / kRows), block(kWaves * 64);
    if (net.H % 16 == 0)  // weights start 16-byte aligned: every offset is a multiple of H or 16 floats
        k_mlp_forward<true><<<grid, block, 0, s>>>(net, x, h[0], h[1], h[2], y, n);
    else
        k_mlp_forward<false><<<grid, block, 0, s>>>(net, x, h[0], h[1], h[2], y, n);
    return hipGetLastError();
}

hipError_t mlp_backward(const MlpNet &net, const float *x, const float *const h[3], const float *dy, float *d1,
                        float *d2, const MlpGrad &out, int n, hipStream_t s)
{
    k_mlp_delta<<<(n + kRows - 1) / kRows, kWaves * 64, 0, s>>>(net, dy, h[1], h[2], d1, d2, n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const int nt = (net.H + 15) / 16, no = (kMlpOut + 15) / 16;
    const dim3 grid(nt + 2 * nt * nt + no * nt), block(kWaves * 64);
    if (net.H % 16 == 0 && (uintptr_t)d1 % 16 == 0)
        k_mlp_grad<true><<<grid, block, 0, s>>>(net, x, h[0], h[1], h[2], d1, d2, dy, out, n);
    else
        k_mlp_grad<false><<<grid, block, 0, s>>>(net, x, h[0], h[1], h[2], d1, d2, dy, out, n);
    return hipGetLastError();
}

}  // namespace fk
