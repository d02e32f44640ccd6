// fk_mlp.hpp -- launchers of the cost-model network kernels (fk_mlp.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "../../include/fk.h"

namespace fk {

constexpr int kMlpIn = FK_MODEL_FEATURES, kMlpOut = FK_MODEL_OUTPUTS;
static_assert(kMlpIn == 32 && kMlpOut <= 32, "the fused passes' input and output tiles");
// Networks of at most this many hidden units take the fused passes: a layer
// is then one 16-column tile per wave of a block and its weights fit a
// wave's registers; wider ones take one product per launch.
constexpr int kMlpMaxH = 128;

// Whether the forward pass of `rows` rows takes the fused kernel (H <=
// kMlpMaxH).  It costs about the same whatever H below 128, a block of 8 waves
// for 16 rows, so on many rows of a narrow network one product a launch is the
// faster form; the two give the same bits.  Fused and by layers, in us:
// 65,536 rows of H = 16 39 and 36, 32 48 and 53; 262,144 of H = 48 199 and 203,
// 64 233 and 251, 128 476 and 720; 16,384 of H = 8 26 and 20, 24 29 and 28, 60
// 39 and 46, and 32,768 of H = 24 55 and 34, 60 75 and 58, 120 170 and 135
// (widths that are no multiple of 16 load their weights value by value).  The
// products' grids count blocks of 64 rows in y, at most 65,535 of them.
constexpr bool mlp_forward_fused(int H, int rows)
{
    return (H % 16 == 0 ? H >= 64 || rows <= 2048 * H : rows <= 12288) || rows > 64 * 65535;
}

// Parameters (or gradients) of the layers in -> H -> H -> H -> out, weights
// row-major [outputs][inputs].
struct MlpNet {
    const float *w[4], *b[4];
    int H;
};
struct MlpGrad {
    float *w[4], *b[4];
};
// x (n x in) -> hidden layers h[0..2] (n x H each) and y (n x out)
hipError_t mlp_forward(const MlpNet &net, const float *x, float *const h[3], float *y, int n, hipStream_t s);
// every gradient from dy (n x out); d1, d2: n x H each, written
hipError_t mlp_backward(const MlpNet &net, const float *x, const float *const h[3], const float *dy, float *d1,
                        float *d2, const MlpGrad &out, int n, hipStream_t s);

enum : int { EPI_NONE = 0, EPI_BIAS = 1, EPI_BIAS_RELU = 2, EPI_RELU_MASK = 3 };

// C[M x N] = op(A) op(B), then the epilogue: + bias[c] (and ReLU), or keep
// C only where mask[r][c] > 0 (ReLU backward).  op(X) = X^T when t* is set;
// all matrices row-major.
hipError_t mlp_gemm(bool ta, bool tb, const float *A, const float *B, float *C, int M, int N, int K,
                    const float *bias, const float *mask, int epilogue, hipStream_t s);
hipError_t mlp_colsum(const float *X, int rows, int cols, float *out, hipStream_t s);
hipError_t mlp_mse(const float *Y, const float *T, int64_t count, float *dY, float *loss,
                   hipStream_t s);
hipError_t mlp_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1,
                    float b2, float eps, int step, hipStream_t s);
hipError_t mlp_gather(const float *src, int cols, const int32_t *idx, int rows, float *dst,
                      hipStream_t s);
// per-column mean and std (fp64 sums; std 1 for a constant column)
hipError_t mlp_colstats(const float *X, int rows, int cols, float *mean, float *stdv, hipStream_t s);
// (X - mean[c]) / std[c]
hipError_t mlp_standardize(const float *X, int64_t rows, int cols, const float *mean,
                           const float *stdv, float *out, hipStream_t s);
// out[0] = mean of x[0..n)
hipError_t mlp_mean(const float *x, int n, float *out, hipStream_t s);

}  // namespace fk
