// Temperature-guess surrogate: a 6 -> 64 -> 64 -> 64 -> 1 tanh MLP on the
// BF16 matrix cores of gfx950 (v_mfma_f32_16x16x16_bf16, FP32 accumulation),
// FP32 master weights, Adam.  It supplies the initial guess of the per-node
// T(e) Newton iteration (Appendix, Thermodynamics; the Introduction's
// requirement that the iterative thermochemistry be cheap).
//
// Wave-level tiling: a wave processes 16 samples.  With the MFMA operand
// layout (lane l, group g = l/16, row r = l%16)
//   A[m = r][k = 4g + j],  B[k = 4g + j][n = r],  D[m = 4g + j][n = r]  (j = 0..3)
// weights are the A operand (neurons x inputs) and activations the B operand
// (inputs x samples); a layer's FP32 result D, after bias + tanh and rounding
// to BF16, is exactly the B operand of the next layer (K block = output block).
// Weight gradients dW = dz . h^T contract over samples and take their
// operands through a per-wave LDS transpose.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <random>
#include <vector>

#include "surrogate.h"

namespace dgx {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int H = kSurH;
// parameter offsets
constexpr int oW1 = 0, ob1 = oW1 + H * kSurIn, oW2 = ob1 + H, ob2 = oW2 + H * H, oW3 = ob2 + H,
              ob3 = oW3 + H * H, oW4 = ob3 + H, ob4 = oW4 + H, oNorm = ob4 + 1;
static_assert(oNorm == kSurParams, "parameter layout");

// FP32 -> BF16, round to nearest even: the conversion instruction of gfx950
// (v_cvt_pk_bf16_f32, which also packs pairs)
__device__ __forceinline__ unsigned short to_bf16(float f) {
    return __builtin_bit_cast(unsigned short, (__bf16)f);
}
__device__ __forceinline__ float from_bf16(unsigned short h) { return __uint_as_float(((unsigned)h) << 16); }

typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef unsigned u32x2v __attribute__((ext_vector_type(2)));

// Four floats to BF16 (round to nearest even) in two paired conversions, one
// per dword, so that no byte shuffles are needed to assemble the fragment.
__device__ __forceinline__ bf16x4 pack4(float a, float b, float c, float d) {
    const f32x2v lo = {a, b}, hi = {c, d};
    const u32x2v w = {__builtin_bit_cast(unsigned, __builtin_convertvector(lo, bf16x2v)),
                      __builtin_bit_cast(unsigned, __builtin_convertvector(hi, bf16x2v))};
    return __builtin_bit_cast(bf16x4, w);
}

// tanh(x) = 1 - 2 / (exp(2x) + 1) with the hardware exp and reciprocal
// estimates (v_exp_f32, v_rcp_f32: FP32, about one ulp each; the activations
// are rounded to BF16 right after, or feed the FP32 output layer).
__device__ __forceinline__ float tanh_fast(float x) {
    const float t = __expf(2.0f * x);
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(t + 1.0f);
}

__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Standardised features of sample i (packed states [nvar][count]):
// log10 max(rho_s, 1e-30) for the 5 species and the specific internal energy.
template <int DIM>
__device__ __forceinline__ void features(const double *st, int64_t count, int64_t i, const float *nrm,
                                         float *x) {
    double rs[5], rho = 0.0;
#pragma unroll
    for (int s = 0; s < 5; ++s) {
        rs[s] = st[s * count + i];
        rho += rs[s];
    }
    double m2 = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        const double m = st[(5 + c) * count + i];
        m2 += m * m;
    }
    // the specific energy in FP64 (kinetic energy can dominate E); the
    // logarithms and the standardisation in FP32, which the features are
    // rounded to (and then to BF16 for the matrix unit)
    const double e = (st[(5 + DIM) * count + i] - 0.5 * m2 / rho) / rho;
#pragma unroll
    for (int s = 0; s < 5; ++s) x[s] = (log10f(fmaxf((float)rs[s], 1e-30f)) - nrm[s]) / nrm[6 + s];
    x[5] = (float)((e - (double)nrm[5]) / (double)nrm[11]);
}

// Weight fragments (A operands), kept beside the FP32 parameters as BF16 in
// the order in which lanes take them, so that a kernel reads two fragments
// with one 16-byte load per lane instead of gathering and rounding eight
// floats: pairs of fragments, then lanes, then the two fragments' 4 values.
// Forward fragment (mt, kc) of W: lane (r, g) holds W[16 mt + r][16 kc + 4 g +
// j], transposed one W[16 kc + 4 g + j][16 mt + r].  Order: W1 (4, columns 6
// and up zero), W2, W3, W2^T, W3^T (16 each, mt major).
constexpr int kF1 = 0, kF2 = 4, kF3 = 20, kT2 = 36, kT3 = 52;
static_assert(kT3 + 16 == kSurFrags, "fragment order");

__host__ __device__ __forceinline__ int packed_at(int frag, int r, int g, int j) {
    return ((frag >> 1) * 64 + 16 * g + r) * 8 + (frag & 1) * 4 + j;
}

// The places of parameter i in the packed copy: none, one (W1) or two.
__device__ __forceinline__ int packed_places(int i, int at[2]) {
    if (i < ob1) {
        const int row = i / kSurIn, col = i - row * kSurIn;
        at[0] = packed_at(kF1 + row / 16, row % 16, col / 4, col % 4);
        return 1;
    }
    const bool w2 = i >= oW2 && i < ob2, w3 = i >= oW3 && i < ob3;
    if (!w2 && !w3) return 0;
    const int k = i - (w2 ? oW2 : oW3), row = k / H, col = k % H;
    at[0] = packed_at((w2 ? kF2 : kF3) + 4 * (row / 16) + col / 16, row % 16, (col % 16) / 4, col % 4);
    at[1] = packed_at((w2 ? kT2 : kT3) + 4 * (col / 16) + row / 16, col % 16, (row % 16) / 4, row % 4);
    return 2;
}

// Fragments f0 .. f0 + n - 1 (f0 and n even) of the packed copy.
template <int n>
__device__ __forceinline__ void load_frags(const unsigned short *pk, int f0, int lane, bf16x4 *out) {
    typedef short bf16x8 __attribute__((ext_vector_type(8)));
#pragma unroll
    for (int i = 0; i < n; i += 2) {
        const bf16x8 v = *reinterpret_cast<const bf16x8 *>(pk + ((size_t)((f0 + i) >> 1) * 64 + lane) * 8);
        out[i] = bf16x4{v[0], v[1], v[2], v[3]};
        out[i + 1] = bf16x4{v[4], v[5], v[6], v[7]};
    }
}

struct Fwd {
    float h1[4][4], h2[4][4], h3[4][4];  // FP32 activations, D layout
    bf16x4 hb1[4], hb2[4];               // BF16 B-operands of layers 2 and 3
    bf16x4 xb;                           // BF16 features (B operand of layer 1)
    float y;                             // output before b4 (summed over groups)
};

// W: the forward fragments W1 (4), W2 (16), W3 (16)
__device__ __forceinline__ void forward(const float *P, const bf16x4 *W, const float *x, int g, Fwd &F) {
    {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 4 * g + j;
            v[j] = k < 6 ? x[k] : 0.0f;
        }
        F.xb = pack4(v[0], v[1], v[2], v[3]);
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma(W[kF1 + mt], F.xb, acc);
#pragma unroll
        for (int j = 0; j < 4; ++j) F.h1[mt][j] = tanh_fast(acc[j] + P[ob1 + 16 * mt + 4 * g + j]);
        F.hb1[mt] = pack4(F.h1[mt][0], F.h1[mt][1], F.h1[mt][2], F.h1[mt][3]);
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) acc = mfma(W[kF2 + 4 * mt + kc], F.hb1[kc], acc);
#pragma unroll
        for (int j = 0; j < 4; ++j) F.h2[mt][j] = tanh_fast(acc[j] + P[ob2 + 16 * mt + 4 * g + j]);
        F.hb2[mt] = pack4(F.h2[mt][0], F.h2[mt][1], F.h2[mt][2], F.h2[mt][3]);
    }
    float yp = 0.0f;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) acc = mfma(W[kF3 + 4 * mt + kc], F.hb2[kc], acc);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            F.h3[mt][j] = tanh_fast(acc[j] + P[ob3 + 16 * mt + 4 * g + j]);
            yp = fmaf(P[oW4 + 16 * mt + 4 * g + j], F.h3[mt][j], yp);
        }
    }
    yp += __shfl_xor(yp, 16);
    yp += __shfl_xor(yp, 32);
    F.y = yp;
}

// ------------------------------------------------------------ inference
// Weight fragments stay in registers for the whole kernel; biases and W4 sit
// in LDS; the features of 64 samples are computed one sample per lane and
// shared through LDS by the four 16-sample tiles.
template <int DIM>
__global__ void __launch_bounds__(256) k_mlp_predict(const float *__restrict__ P,
                                                     const unsigned short *__restrict__ pk,
                                                     const double *__restrict__ st, int64_t count,
                                                     double *__restrict__ Tg) {
    __shared__ float sx[4][64][8];         // per wave: features of 64 samples
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const float *nrm = P + oNorm;
    bf16x4 W1f[4], W2f[4][4], W3f[4][4];
    load_frags<4>(pk, kF1, lane, W1f);
    load_frags<16>(pk, kF2, lane, &W2f[0][0]);
    load_frags<16>(pk, kF3, lane, &W3f[0][0]);
    // this lane's biases (rows 16 mt + 4 g + j) start the accumulators, and
    // its output weights W4
    f32x4 bias1[4], bias2[4], bias3[4], w4[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = 16 * mt + 4 * g + j;
            bias1[mt][j] = P[ob1 + row];
            bias2[mt][j] = P[ob2 + row];
            bias3[mt][j] = P[ob3 + row];
            w4[mt][j] = P[oW4 + row];
        }
    const float b4 = P[ob4];
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t s0 = wave * 64; s0 < count; s0 += nwaves * 64) {
        {
            float x[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (s0 + lane < count) features<DIM>(st, count, s0 + lane, nrm, x);
#pragma unroll
            for (int k = 0; k < 6; ++k) sx[w][lane][k] = x[k];
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        // two independent 16-sample tiles per pass: the matrix unit works on
        // one while the vector ALU evaluates the other's tanh
#pragma unroll 1
        for (int tt = 0; tt < 4; tt += 2) {
            bf16x4 xb[2];
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = 4 * g + j;
                    v[j] = k < 6 ? sx[w][16 * (tt + t2) + r][k] : 0.0f;
                }
                xb[t2] = pack4(v[0], v[1], v[2], v[3]);
            }
            bf16x4 hb[2][4], hc[2][4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {
                    const f32x4 acc = mfma(W1f[mt], xb[t2], bias1[mt]);
                    float h[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) h[j] = tanh_fast(acc[j]);
                    hb[t2][mt] = pack4(h[0], h[1], h[2], h[3]);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {
                    f32x4 acc = bias2[mt];
#pragma unroll
                    for (int kc = 0; kc < 4; ++kc) acc = mfma(W2f[mt][kc], hb[t2][kc], acc);
                    float h[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) h[j] = tanh_fast(acc[j]);
                    hc[t2][mt] = pack4(h[0], h[1], h[2], h[3]);
                }
            }
            float yp[2] = {0.0f, 0.0f};
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {
                    f32x4 acc = bias3[mt];
#pragma unroll
                    for (int kc = 0; kc < 4; ++kc) acc = mfma(W3f[mt][kc], hc[t2][kc], acc);
#pragma unroll
                    for (int j = 0; j < 4; ++j) yp[t2] = fmaf(w4[mt][j], tanh_fast(acc[j]), yp[t2]);
                }
            }
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
                float y = yp[t2];
                y += __shfl_xor(y, 16);
                y += __shfl_xor(y, 32);
                const int64_t n = s0 + 16 * (tt + t2) + r;
                if (g == 0 && n < count) Tg[n] = (double)(y + b4) * (double)nrm[13] + (double)nrm[12];
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ------------------------------------------------------------ training
// Sum of v over the 16 lanes of a row (the samples of a tile), on every lane:
// the butterfly over lane distances 1, 2, 4, 8.  Once the lanes of a group of
// four (eight) agree, the mirrored lane of the other group holds the same
// value as the butterfly's partner, so all four steps are additions with a
// cross-lane operand, without LDS permutes.
template <int CTRL>
__device__ __forceinline__ float row_add(float v) {
    // (v is rounded before it is summed: no contraction of its last product)
#pragma clang fp contract(off)
    const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(float, o);
}
__device__ __forceinline__ float rowsum(float v) {
    v = row_add<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v = row_add<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v = row_add<0x141>(v);  // row_half_mirror
    return row_add<0x140>(v);  // row_mirror
}

// A row of partial results: the gradient in parameter order, then the sum of
// the squared residuals.
constexpr int kRowLoss = kSurParams;
constexpr int kRow = (kSurParams + 1 + 63) / 64 * 64;

// Partial gradients of the mean squared error over the samples idx[start ..
// start + nbatch): one wave per workgroup, a 16-sample tile each (tile tile0 +
// block, row = block).
//
// What bounds it: latency.  A minibatch of 4096 is 256 tiles, one per CU, and
// each is a chain of gathers, three layers forward and three back.  With four
// tiles per workgroup, the weights gathered and rounded per use and the four
// waves' sums taken in turn through LDS it took 34 us; with a workgroup per
// tile, the packed weights loaded ahead and no sum inside, 12 us.
template <int DIM>
__global__ void __launch_bounds__(64) k_mlp_grad(const float *__restrict__ P, const unsigned short *__restrict__ pk,
                                                 const double *__restrict__ st, const double *__restrict__ T,
                                                 int64_t count, const int *__restrict__ idx, int64_t start,
                                                 int64_t nbatch, int64_t tile0, float *__restrict__ partial) {
    __shared__ __align__(16) unsigned short sA[H][16];  // dz, neuron x sample (BF16)
    __shared__ __align__(16) unsigned short sB[H][16];  // activation, neuron x sample (BF16)
    const int lane = threadIdx.x;
    const int r = lane & 15, g = lane >> 4;
    const float *nrm = P + oNorm;
    const float inv_b = 2.0f / (float)nbatch;
    bf16x4 W[36];
    load_frags<36>(pk, kF1, lane, W);

    const int64_t pos = (tile0 + blockIdx.x) * 16 + r;
    const bool valid = pos < nbatch;
    const int64_t n = valid ? (int64_t)idx[start + pos] : 0;
    float x[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float tgt = 0.0f;
    if (valid) {
        features<DIM>(st, count, n, nrm, x);
        tgt = (float)((T[n] - (double)nrm[12]) / (double)nrm[13]);
    }
    Fwd F;
    forward(P, W, x, g, F);
    const float res = valid ? (F.y + P[ob4] - tgt) : 0.0f;
    const float dy = inv_b * res;
    const float l2 = g == 0 ? res * res : 0.0f, d4 = g == 0 ? dy : 0.0f;
    // output layer and dz3 (D layout)
    float dz[4][4], gb1[4][4], gb2[4][4], gb3[4][4], gW4[4][4];
    f32x4 dW3[4][4], dW2[4][4], dW1[4];
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 16 * mt + 4 * g + j;
            gW4[mt][j] = dy * F.h3[mt][j];
            dz[mt][j] = P[oW4 + k] * dy * (1.0f - F.h3[mt][j] * F.h3[mt][j]);
            gb3[mt][j] = dz[mt][j];
        }
    // ---- layer 3: dW3 = dz3 . h2^T ; dz2 = (W3^T dz3) * (1 - h2^2); then layers 2 and 1
#pragma unroll
    for (int layer = 3; layer >= 1; --layer) {
        bf16x4 Wt[16];
        if (layer > 1) load_frags<16>(pk, layer == 3 ? kT3 : kT2, lane, Wt);
        // stage dz (A) and the layer input (B) transposed through LDS
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = 16 * mt + 4 * g + j;
                sA[k][r] = to_bf16(dz[mt][j]);
                if (layer == 3) sB[k][r] = to_bf16(F.h2[mt][j]);
                if (layer == 2) sB[k][r] = to_bf16(F.h1[mt][j]);
            }
        if (layer == 1 && g == 0) {
#pragma unroll
            for (int k = 0; k < 16; ++k) sB[k][r] = k < 6 ? to_bf16(x[k]) : (unsigned short)0;
        }
        __syncthreads();
        bf16x4 Af[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) Af[mt] = *reinterpret_cast<const bf16x4 *>(&sA[16 * mt + r][4 * g]);
        if (layer == 1) {
            const bf16x4 b = *reinterpret_cast<const bf16x4 *>(&sB[r][4 * g]);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) dW1[mt] = mfma(Af[mt], b, zero);
        } else {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const bf16x4 b = *reinterpret_cast<const bf16x4 *>(&sB[16 * nt + r][4 * g]);
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    if (layer == 3) dW3[mt][nt] = mfma(Af[mt], b, zero);
                    else dW2[mt][nt] = mfma(Af[mt], b, zero);
                }
            }
        }
        __syncthreads();
        if (layer == 1) break;
        // back-propagate: dh = W^T dz (B operand = dz in D layout), dz_prev = dh * (1 - h^2)
        bf16x4 dzb[4];
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) dzb[kc] = pack4(dz[kc][0], dz[kc][1], dz[kc][2], dz[kc][3]);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            f32x4 acc = zero;
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) acc = mfma(Wt[4 * mt + kc], dzb[kc], acc);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float h = layer == 3 ? F.h2[mt][j] : F.h1[mt][j];
                dz[mt][j] = acc[j] * (1.0f - h * h);
                if (layer == 3) gb2[mt][j] = dz[mt][j];
                else gb1[mt][j] = dz[mt][j];
            }
        }
    }
    // biases and output weights: sums over the tile's samples
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            gb1[mt][j] = rowsum(gb1[mt][j]);
            gb2[mt][j] = rowsum(gb2[mt][j]);
            gb3[mt][j] = rowsum(gb3[mt][j]);
            gW4[mt][j] = rowsum(gW4[mt][j]);
        }
    const float g4 = rowsum(d4), ls = rowsum(l2);
    float *out = partial + (size_t)blockIdx.x * kRow;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 16 * mt + 4 * g + j;
            if (r < kSurIn) out[oW1 + k * kSurIn + r] = dW1[mt][j];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                out[oW3 + k * H + 16 * nt + r] = dW3[mt][nt][j];
                out[oW2 + k * H + 16 * nt + r] = dW2[mt][nt][j];
            }
            if (r == 0) {
                out[ob1 + k] = gb1[mt][j];
                out[ob2 + k] = gb2[mt][j];
                out[ob3 + k] = gb3[mt][j];
                out[oW4 + k] = gW4[mt][j];
            }
        }
    if (lane == 0) {
        out[ob4] = g4;
        out[kRowLoss] = ls;
    }
}

struct AdamC {
    float lr, c1, c2;
};

// Sums the partial rows in a fixed order (groups of four rows, a group's rows
// in turn, then the groups in turn) onto grad[i] (from 0 in the first part
// of a batch), grad[kRowLoss] likewise the loss; in the last part the loss is
// accumulated and with ADAM the parameters and their packed copy are updated.
// A workgroup takes 64 parameters:
// its four waves read and sum the groups of a chunk side by side into LDS,
// and one adds them in order.  (One thread per parameter walking 64 rows took
// 18 us, waiting for one load after another, and the update was a launch of
// its own, 5 us; now 256 rows and the update take 4 us.)
template <bool ADAM>
__global__ void __launch_bounds__(256) k_mlp_reduce(const float *__restrict__ partial, int rows, int first, int last,
                                                    float *__restrict__ grad, float *__restrict__ loss_acc,
                                                    float *__restrict__ P, unsigned short *__restrict__ pk,
                                                    float *__restrict__ m, float *__restrict__ v, AdamC A) {
    constexpr int CH = 64;  // groups per chunk
    __shared__ float sh[CH][64];
    const int p = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + p;  // < kRow
    const int ngroups = (rows + 3) / 4;
    float s = first || w != 0 ? 0.0f : grad[i];
    for (int c0 = 0; c0 < ngroups; c0 += CH) {
        // all rows of this wave's groups are loaded before the first sum;
        // rows past the end count as zero
        const int r0 = (c0 + w * (CH / 4)) * 4;
        const float *q = partial + (size_t)r0 * kRow + i;
        float b[CH];
        if (r0 + CH <= rows) {
#pragma unroll
            for (int x = 0; x < CH; ++x) b[x] = q[(size_t)x * kRow];
        } else {
#pragma unroll
            for (int x = 0; x < CH; ++x) b[x] = r0 + x < rows ? q[(size_t)x * kRow] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < CH / 4; ++k)
            sh[w * (CH / 4) + k][p] = ((b[4 * k] + b[4 * k + 1]) + b[4 * k + 2]) + b[4 * k + 3];
        __syncthreads();
        if (w == 0) {
            if (ngroups - c0 >= CH) {
#pragma unroll
                for (int k = 0; k < CH; ++k) s += sh[k][p];
            } else {
                for (int k = 0; k < ngroups - c0; ++k) s += sh[k][p];
            }
        }
        __syncthreads();
    }
    if (w != 0) return;
    grad[i] = s;
    if (!last) return;
    if (i == kRowLoss) loss_acc[0] += s;
    if (i >= kSurParams) return;
    if constexpr (ADAM) {
        const float mi = 0.9f * m[i] + 0.1f * s;
        const float vi = 0.999f * v[i] + 0.001f * s * s;
        m[i] = mi;
        v[i] = vi;
        const float pn = P[i] - A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + 1e-8f);
        P[i] = pn;
        int at[2];
        const int n = packed_places(i, at);
        for (int k = 0; k < n; ++k) pk[at[k]] = to_bf16(pn);
    }
}

int grid_for(int64_t count) {
    const int64_t waves = (count + 63) / 64;
    return (int)std::min<int64_t>((waves + 3) / 4, 2048);
}

}  // namespace

// FP32 -> BF16 on the host, round to nearest even, NaN kept (as the device's
// conversion).
static unsigned short host_bf16(float f) {
    unsigned u;
    std::memcpy(&u, &f, sizeof(u));
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)(u >> 16 | 0x40u);
    return (unsigned short)((u + 0x7fffu + (u >> 16 & 1u)) >> 16);
}

// The packed copy of the parameters P, fragment by fragment (the places of
// packed_places; asking it for every parameter took 43 us of a call's 58, the
// start of a program that sets its weights: now 16 in all).
static void pack_weights(const float *P, unsigned short *pk) {
    unsigned short b[kSurParams];
    for (int i = 0; i < kSurParams; ++i) b[i] = host_bf16(P[i]);
    for (int mt = 0; mt < 4; ++mt)
        for (int r = 0; r < 16; ++r)
            for (int col = 0; col < 16; ++col)
                pk[packed_at(kF1 + mt, r, col / 4, col % 4)] = col < kSurIn ? b[oW1 + (16 * mt + r) * kSurIn + col] : 0;
    for (int layer = 0; layer < 2; ++layer) {
        const unsigned short *W = b + (layer ? oW3 : oW2);
        const int f = layer ? kF3 : kF2, t = layer ? kT3 : kT2;
        for (int mt = 0; mt < 4; ++mt)
            for (int kc = 0; kc < 4; ++kc)
                for (int g = 0; g < 4; ++g)
                    for (int r = 0; r < 16; ++r) {
                        unsigned short *fw = pk + packed_at(f + 4 * mt + kc, r, g, 0);
                        unsigned short *tr = pk + packed_at(t + 4 * mt + kc, r, g, 0);
                        const unsigned short *row = W + (16 * mt + r) * H + 16 * kc + 4 * g;
                        const unsigned short *col = W + (16 * kc + 4 * g) * H + 16 * mt + r;
                        for (int j = 0; j < 4; ++j) {
                            fw[j] = row[j];
                            tr[j] = col[j * H];
                        }
                    }
    }
}

// (parameters and packed copy lie in one allocation and go there in one copy)
int surrogate_set(Surrogate &S, const float *host_params) {
    static thread_local struct {
        float params[kSurParamsRoom];
        unsigned short packed[kSurPacked];
    } block;
    std::memcpy(block.params, host_params, (kSurParams + kSurNorm) * sizeof(float));
    pack_weights(host_params, block.packed);
    if (!S.params && hipMalloc(&S.params, sizeof(block)) != hipSuccess) {
        S.params = nullptr;
        return -3;
    }
    S.packed = reinterpret_cast<unsigned short *>(S.params + kSurParamsRoom);
    S.ready = false;
    if (hipMemcpy(S.params, &block, sizeof(block), hipMemcpyHostToDevice) != hipSuccess) return -3;
    S.ready = true;
    return 0;
}

int surrogate_get(Surrogate &S, float *host_params) {
    return hipMemcpy(host_params, S.params, (kSurParams + kSurNorm) * sizeof(float), hipMemcpyDeviceToHost) ==
                   hipSuccess
               ? 0
               : -3;
}

int surrogate_predict(Surrogate &S, int dim, const double *states, int64_t count, double *Tg, hipStream_t s) {
    if (!S.ready) return -6;
    const int grid = grid_for(count);
    if (dim == 2) hipLaunchKernelGGL(k_mlp_predict<2>, dim3(grid), dim3(256), 0, s, S.params, S.packed, states, count, Tg);
    else hipLaunchKernelGGL(k_mlp_predict<3>, dim3(grid), dim3(256), 0, s, S.params, S.packed, states, count, Tg);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

static int ensure(float *&p, size_t n) {
    if (p) return 0;
    if (hipMalloc(&p, n * sizeof(float)) != hipSuccess) return -2;
    return hipMemset(p, 0, n * sizeof(float)) == hipSuccess ? 0 : -3;
}

// Partial rows per part of a minibatch: 16,384 samples, a wave for each SIMD
// of the chip, 36 MB.  Larger batches run part after part into the same rows,
// with the same sums.
constexpr int kPartRows = 1024;

// The training workspace: the partial rows of a batch of nb, room for n sample
// indices and the loss accumulator.
static int ensure_workspace(Surrogate &S, int64_t nb, size_t n) {
    const size_t rows = (size_t)std::min<int64_t>((nb + 15) / 16, kPartRows);
    if (!S.loss && hipMalloc(&S.loss, sizeof(float)) != hipSuccess) return -2;
    if (S.partial_rows < rows) {
        if (S.partial) (void)hipFree(S.partial);
        S.partial = nullptr;
        S.partial_rows = 0;
        if (hipMalloc(&S.partial, rows * kRow * sizeof(float)) != hipSuccess) return -2;
        S.partial_rows = rows;
    }
    if (S.order_n < n) {
        if (S.order) (void)hipFree(S.order);
        S.order = nullptr;
        S.order_n = 0;
        if (hipMalloc(&S.order, n * sizeof(int)) != hipSuccess) return -2;
        S.order_n = n;
    }
    return 0;
}

// Gives the sample order back where it is large (the stream has been waited
// for).
static void trim_workspace(Surrogate &S) {
    if (S.order_n * sizeof(int) > kSurKeepBytes) {
        (void)hipFree(S.order);
        S.order = nullptr;
        S.order_n = 0;
    }
}

// Gradient of the mean squared error over the samples order[start ..
// start+nb) into S.grads, the summed squared residual added to S.loss, and
// with adam the parameter update.
static int enqueue_grad(Surrogate &S, int dim, const double *states, const double *T, int64_t count, int64_t start,
                        int64_t nb, const AdamC *adam, hipStream_t s) {
    const int64_t tiles = (nb + 15) / 16;
    for (int64_t t0 = 0; t0 < tiles; t0 += kPartRows) {
        const int rows = (int)std::min<int64_t>(kPartRows, tiles - t0);
        const int first = t0 == 0, last = t0 + rows == tiles;
        auto grad = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(rows), dim3(64), 0, s, S.params, S.packed, states, T, count, S.order, start,
                               nb, t0, S.partial);
        };
        if (dim == 2) grad(k_mlp_grad<2>);
        else grad(k_mlp_grad<3>);
        auto reduce = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(kRow / 64), dim3(256), 0, s, S.partial, rows, first, last, S.grads, S.loss,
                               S.params, S.packed, S.adam_m, S.adam_v, adam ? *adam : AdamC{0.f, 1.f, 1.f});
        };
        if (adam) reduce(k_mlp_reduce<true>);
        else reduce(k_mlp_reduce<false>);
    }
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

int surrogate_grad(Surrogate &S, int dim, const double *states, const double *T, int64_t count, float *grad_host,
                   float *loss_host, hipStream_t s) {
    if (!S.ready) return -6;
    if (ensure(S.grads, kRow)) return -2;
    if (ensure_workspace(S, count, (size_t)count)) return -2;
    int rc = 0;
    std::vector<int> h(count);
    for (int64_t i = 0; i < count; ++i) h[i] = (int)i;
    if (hipMemcpyAsync(S.order, h.data(), count * sizeof(int), hipMemcpyHostToDevice, s) != hipSuccess) rc = -3;
    if (!rc && hipMemsetAsync(S.loss, 0, sizeof(float), s) != hipSuccess) rc = -3;
    if (!rc) rc = enqueue_grad(S, dim, states, T, count, 0, count, nullptr, s);
    if (!rc && hipMemcpyAsync(grad_host, S.grads, kSurParams * sizeof(float), hipMemcpyDeviceToHost, s) != hipSuccess)
        rc = -3;
    float l = 0.0f;
    if (!rc && hipMemcpyAsync(&l, S.loss, sizeof(float), hipMemcpyDeviceToHost, s) != hipSuccess) rc = -3;
    if (hipStreamSynchronize(s) != hipSuccess && !rc) rc = -3;
    if (!rc && loss_host) *loss_host = l / (float)count;
    trim_workspace(S);
    return rc;
}

int surrogate_train(Surrogate &S, int dim, const double *states, const double *T, int64_t count, int epochs, int batch,
                    float lr, uint64_t seed, float *loss_host, hipStream_t s) {
    if (!S.ready) {
        S.err = "set initial parameters (and normalisation) first";
        return -6;
    }
    if (ensure(S.grads, kRow) || ensure(S.adam_m, kSurParams) || ensure(S.adam_v, kSurParams)) return -2;
    if (ensure_workspace(S, std::min<int64_t>(batch, count), (size_t)count)) return -2;
    std::vector<int> order(count);
    for (int64_t i = 0; i < count; ++i) order[i] = (int)i;
    std::mt19937_64 rng(seed);
    int rc = 0;
    // cosine learning-rate decay over this call's steps, lr -> 0
    const int64_t per_epoch = (count + batch - 1) / batch;
    const double total = (double)epochs * (double)per_epoch;
    int64_t t = 0;
    for (int ep = 0; ep < epochs && !rc; ++ep) {
        std::shuffle(order.begin(), order.end(), rng);
        if (hipMemcpyAsync(S.order, order.data(), count * sizeof(int), hipMemcpyHostToDevice, s) != hipSuccess ||
            hipMemsetAsync(S.loss, 0, sizeof(float), s) != hipSuccess) {
            rc = -3;
            break;
        }
        for (int64_t b0 = 0; b0 < count && !rc; b0 += batch) {
            const int64_t nb = std::min<int64_t>(batch, count - b0);
            ++S.step;
            AdamC A;
            A.c1 = 1.0f - std::pow(0.9f, (float)S.step);
            A.c2 = 1.0f - std::pow(0.999f, (float)S.step);
            A.lr = (float)(0.5 * lr * (1.0 + std::cos(3.14159265358979323846 * (double)t / total)));
            ++t;
            rc = enqueue_grad(S, dim, states, T, count, b0, nb, &A, s);
        }
        float l = 0.0f;
        if (!rc && (hipMemcpyAsync(&l, S.loss, sizeof(float), hipMemcpyDeviceToHost, s) != hipSuccess ||
                    hipStreamSynchronize(s) != hipSuccess))
            rc = -3;
        if (!rc && loss_host) loss_host[ep] = l / (float)count;
    }
    (void)hipStreamSynchronize(s);
    trim_workspace(S);
    return rc;
}

// Normalisation (feature and temperature mean / standard deviation over the
// training set, host FP64) and Glorot-uniform initial weights from `seed`.
int surrogate_init(Surrogate &S, int dim, const double *states, const double *T, int64_t count, uint64_t seed,
                   hipStream_t s) {
    const int nvar = 5 + dim + 1;
    std::vector<double> h((size_t)nvar * count), ht(count);
    if (hipMemcpyAsync(h.data(), states, h.size() * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(ht.data(), T, count * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return -3;
    double sum[7] = {0}, sq[7] = {0};
    for (int64_t i = 0; i < count; ++i) {
        double rho = 0.0, m2 = 0.0, f[7];
        for (int k = 0; k < 5; ++k) rho += h[k * count + i];
        for (int c = 0; c < dim; ++c) m2 += h[(5 + c) * count + i] * h[(5 + c) * count + i];
        for (int k = 0; k < 5; ++k) f[k] = std::log10(std::max(h[k * count + i], 1e-30));
        f[5] = (h[(5 + dim) * count + i] - 0.5 * m2 / rho) / rho;
        f[6] = ht[i];
        for (int k = 0; k < 7; ++k) {
            sum[k] += f[k];
            sq[k] += f[k] * f[k];
        }
    }
    std::vector<float> prm(kSurParams + kSurNorm, 0.0f);
    std::mt19937_64 rng(seed);
    auto fill = [&](int off, int rows, int cols) {
        const double lim = std::sqrt(6.0 / (rows + cols));
        std::uniform_real_distribution<double> U(-lim, lim);
        for (int i = 0; i < rows * cols; ++i) prm[off + i] = (float)U(rng);
    };
    fill(oW1, H, kSurIn);
    fill(oW2, H, H);
    fill(oW3, H, H);
    fill(oW4, 1, H);
    for (int k = 0; k < 7; ++k) {
        const double mean = sum[k] / count;
        const double var = std::max(sq[k] / count - mean * mean, 0.0);
        const double sd = std::sqrt(var) > 1e-12 * std::max(1.0, std::fabs(mean)) ? std::sqrt(var) : 1.0;
        if (k < 6) {
            prm[oNorm + k] = (float)mean;
            prm[oNorm + 6 + k] = (float)sd;
        } else {
            prm[oNorm + 12] = (float)mean;
            prm[oNorm + 13] = (float)sd;
        }
    }
    S.step = 0;
    if (S.adam_m) (void)hipMemset(S.adam_m, 0, kSurParams * sizeof(float));
    if (S.adam_v) (void)hipMemset(S.adam_v, 0, kSurParams * sizeof(float));
    return surrogate_set(S, prm.data());
}

void surrogate_free(Surrogate &S) {
    if (S.params) (void)hipFree(S.params);
    if (S.adam_m) (void)hipFree(S.adam_m);
    if (S.adam_v) (void)hipFree(S.adam_v);
    if (S.grads) (void)hipFree(S.grads);
    if (S.partial) (void)hipFree(S.partial);
    if (S.loss) (void)hipFree(S.loss);
    if (S.order) (void)hipFree(S.order);
    S = Surrogate();
}

}  // namespace dgx
