// Temperature-guess surrogate: MLP 6 -> 64 -> 64 -> 64 -> 1 with tanh,
// BF16 MFMA operands and FP32 accumulation, FP32 master weights and Adam.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

namespace dgx {

constexpr int kSurIn = 6;
constexpr int kSurH = 64;
// W1[64][6] b1[64] W2[64][64] b2[64] W3[64][64] b3[64] W4[64] b4[1]
constexpr int kSurParams = kSurH * kSurIn + kSurH + 2 * (kSurH * kSurH + kSurH) + kSurH + 1;
constexpr int kSurNorm = 14;  // feature mean[6], std[6], T mean, T std
// BF16 copies of W1, W2, W3, W2^T, W3^T in matrix-unit operand order:
// fragments of 64 lanes x 4 values (surrogate.hip)
constexpr int kSurFrags = 4 + 4 * 16;
constexpr int kSurPacked = kSurFrags * 64 * 4;
constexpr int kSurParamsRoom = (kSurParams + kSurNorm + 63) / 64 * 64;  // floats before the packed copy

constexpr size_t kSurKeepBytes = (size_t)64 << 20;

struct Surrogate {
    bool ready = false;
    float *params = nullptr;  // device [kSurParams + kSurNorm] FP32 master copy
    unsigned short *packed = nullptr;  // [kSurPacked] behind them, always the rounding of params
    float *adam_m = nullptr, *adam_v = nullptr, *grads = nullptr;
    // training workspace, kept between calls up to kSurKeepBytes: the waves'
    // partial gradients, the sample order and the loss accumulator
    float *partial = nullptr, *loss = nullptr;
    int *order = nullptr;
    size_t partial_rows = 0, order_n = 0;
    int64_t step = 0;  // Adam steps taken
    std::string err;
};

int surrogate_set(Surrogate &S, const float *host_params);
int surrogate_get(Surrogate &S, float *host_params);
int surrogate_predict(Surrogate &S, int dim, const double *states, int64_t count, double *Tg, hipStream_t s);
int surrogate_train(Surrogate &S, int dim, const double *states, const double *T, int64_t count, int epochs,
                    int batch, float lr, uint64_t seed, float *loss_host, hipStream_t s);
int surrogate_grad(Surrogate &S, int dim, const double *states, const double *T, int64_t count, float *grad_host,
                   float *loss_host, hipStream_t s);
int surrogate_init(Surrogate &S, int dim, const double *states, const double *T, int64_t count, uint64_t seed,
                   hipStream_t s);
void surrogate_free(Surrogate &S);

}  // namespace dgx
