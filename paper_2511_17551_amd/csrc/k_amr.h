// Dynamic AMR kernels: the refinement indicator per element and the
// solution transfer to an adapted octree mesh (3D, perfect gas).
//
// Sec. Results (AMR Taylor-Green case: Loehner's weighted second-derivative
// estimate or the Hennemann-Gassner modal-energy coefficient of a derived
// variable) and Sec. New Developments (interpolation from large to small
// elements, exact L2 projection back).
#pragma once

#include "k_rhs.h"

namespace dgx {

// Applies the 1D matrix M (N1 x N1, row-major [out][in]) along direction d
// of the element values in LDS src, writing dst (one thread per node).
template <int N1>
__device__ __forceinline__ void amr_apply_dir(const double *M, const double *src, double *dst, int node, int d) {
    const int stride = d == 0 ? 1 : d == 1 ? N1 : N1 * N1;
    const int a = (node / stride) % N1;
    const int base = node - a * stride;
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < N1; ++j) s = fma(M[a * N1 + j], src[base + j * stride], s);
    dst[node] = s;
}

// Indicator per element, one workgroup of (N+1)^3 threads per element.
// var: 0 rho, 1 p, 2 rho p, 3 |v|.  kind 0 (Loehner): the variable is
// sampled at N+1 equidistant points per direction (eq: [sample][node]) and
// the element takes the largest
//   |f+ - 2 f0 + f-| / (|f+ - f0| + |f0 - f-| + 0.2 (|f+| + 2|f0| + |f-|))
// over interior samples of all lines (0 where the denominator is 0).  kind
// 1 (Hennemann-Gassner): orthonormal Legendre modes of the variable, E =
// max((E_all - E_{<=N-1})/E_all, (E_{<=N-1} - E_{<=N-2})/E_{<=N-1}) and the
// coefficient 1/(1 + exp(-(s/T)(E - T))), T = 0.5 * 10^(-1.8 (N+1)^(1/4)),
// s = ln((1 - 1e-4)/1e-4), set to 0 below 1e-4.
template <int N>
__global__ void __launch_bounds__(128) k_amr_indicator(const double *__restrict__ u, int nelem, double gamma,
                                                        int kind, int var, const double *__restrict__ eq,
                                                        BasisC B, double *__restrict__ ind) {
    constexpr int N1 = N + 1, NN = N1 * N1 * N1;
    __shared__ double s0[NN], s1[NN], sm[N1 * N1];
    __shared__ double red[NN];
    const int e = blockIdx.x;
    const int node = threadIdx.x;
    if (node < N1 * N1) sm[node] = kind == 0 ? eq[node] : B.Vinv[node];
    if (node < NN) {
        const size_t stride = (size_t)nelem * NN, gi = (size_t)e * NN + node;
        const double rho = u[gi];
        double v[3], v2 = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c] = u[(1 + c) * stride + gi] / rho;
            v2 = fma(v[c], v[c], v2);
        }
        const double p = (gamma - 1.0) * (u[4 * stride + gi] - 0.5 * rho * v2);
        s0[node] = var == 0 ? rho : var == 1 ? p : var == 2 ? rho * p : sqrt(v2);
    }
    __syncthreads();
    // the three 1D transforms: s0 -> s1 -> s0 -> s1
    if (node < NN) amr_apply_dir<N1>(sm, s0, s1, node, 0);
    __syncthreads();
    if (node < NN) amr_apply_dir<N1>(sm, s1, s0, node, 1);
    __syncthreads();
    if (node < NN) amr_apply_dir<N1>(sm, s0, s1, node, 2);
    __syncthreads();
    if (node < NN) {
        double r = 0.0;
        if (kind == 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int stride = d == 0 ? 1 : d == 1 ? N1 : N1 * N1;
                const int a = (node / stride) % N1;
                if (a == 0 || a == N) continue;
                const double fm = s1[node - stride], f0 = s1[node], fp = s1[node + stride];
                const double num = fabs(fp - 2.0 * f0 + fm);
                const double den = fabs(fp - f0) + fabs(f0 - fm) + 0.2 * (fabs(fp) + 2.0 * fabs(f0) + fabs(fm));
                if (den > 0.0) r = fmax(r, num / den);
            }
        }
        red[node] = r;
    }
    __syncthreads();
    if (node == 0) {
        if (kind == 0) {
            double r = 0.0;
            for (int n = 0; n < NN; ++n) r = fmax(r, red[n]);
            ind[e] = r;
        } else {
            // mode energies by the largest mode index of each coefficient
            double ea = 0.0, e1 = 0.0, e2 = 0.0;
            for (int n = 0; n < NN; ++n) {
                const int a = n % N1, b = (n / N1) % N1, c = n / (N1 * N1);
                const int mx = max(a, max(b, c));
                const double m2 = s1[n] * s1[n];
                ea += m2;
                if (mx <= N - 1) e1 += m2;
                if (mx <= N - 2) e2 += m2;
            }
            const double E = fmax((ea - e1) / ea, (e1 - e2) / e1);
            const double T = 0.5 * pow(10.0, -1.8 * pow((double)(N + 1), 0.25));
            const double s = log((1.0 - 1e-4) / 1e-4);
            const double a = 1.0 / (1.0 + exp(-(s / T) * (E - T)));
            ind[e] = a < 1e-4 ? 0.0 : a;
        }
    }
}

// elements per workgroup of the transfer: 256 threads at N = 3, one element at
// N = 4 (its 125 nodes are no wave's multiple)
template <int N>
constexpr int kTransferElems = N == 3 ? 4 : 1;

// Transfer to the adapted mesh: a thread per (new element, node), the element's
// values in LDS.  Row tab[e] (kOctTab ints): kind 0 copies the old element,
// kind 1 interpolates the old element along the split path (per direction the
// composite of the half-interval interpolations I_0 / I_1), kind 2 sums the L2
// projections (P_0 / P_1 per direction) of the 8 old children; both apply
// their 1D operators one direction after the other.  ops: [I_0, I_1, P_0, P_1]
// as 25-wide [out][in] blocks.  The few merged elements bound the launch: as
// one sum over the 512 nodes of the children, read from memory by every
// thread and variable, their waves ran alone for most of it; an adaptation
// from 4,096 to 5,352 elements took 101 us, now 16.
template <int N>
__global__ void __launch_bounds__(256) k_amr_transfer(const double *__restrict__ uold, int nold,
                                                       double *__restrict__ unew, int nnew,
                                                       const int *__restrict__ tab, const double *__restrict__ ops) {
    constexpr int N1 = N + 1, NN = N1 * N1 * N1, TB = 12, NV = 5;
    constexpr bool WAVE = NN == 64;          // an element is a wave
    constexpr int EPB = kTransferElems<N>;   // elements per workgroup
    __shared__ double sops[100], sbuf[EPB][2][NV][NN];
    for (int i = threadIdx.x; i < 100; i += blockDim.x) sops[i] = ops[i];
    __syncthreads();
    const int el = WAVE ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64) : 0;
    const int node = WAVE ? (int)threadIdx.x & 63 : (int)threadIdx.x;
    const int e = blockIdx.x * EPB + el;
    if (e >= nnew) return;  // whole waves (EPB = 1: no workgroup)
    const bool own = node < NN;
    const int n = own ? node : 0;
    const int a = n % N1, b = (n / N1) % N1, c = n / (N1 * N1);
    const int *row = tab + (size_t)e * TB;
    const size_t so = (size_t)nold * NN, sn = (size_t)nnew * NN;
    const int kind = row[0];
    double out[NV], in[NV];
    auto load = [&](int src) {
        const size_t g = (size_t)src * NN + n;
#pragma unroll
        for (int v = 0; v < NV; ++v) in[v] = uold[v * so + g];
    };
    // out += (Mz x My x Mx) in, the rows of this node's position
    auto apply = [&](const double *Mx, const double *My, const double *Mz) {
        double(*A)[NN] = sbuf[el][0], (*B)[NN] = sbuf[el][1];
        if (own) {
#pragma unroll
            for (int v = 0; v < NV; ++v) A[v][n] = in[v];
        }
        element_sync<WAVE>();
        double s[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            s[v] = 0.0;
#pragma unroll
            for (int i = 0; i < N1; ++i) s[v] = fma(Mx[i], A[v][i + N1 * (b + N1 * c)], s[v]);
        }
        if (own) {
#pragma unroll
            for (int v = 0; v < NV; ++v) B[v][n] = s[v];
        }
        element_sync<WAVE>();
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            s[v] = 0.0;
#pragma unroll
            for (int j = 0; j < N1; ++j) s[v] = fma(My[j], B[v][a + N1 * (j + N1 * c)], s[v]);
        }
        if (own) {
#pragma unroll
            for (int v = 0; v < NV; ++v) A[v][n] = s[v];
        }
        element_sync<WAVE>();
#pragma unroll
        for (int v = 0; v < NV; ++v) {
#pragma unroll
            for (int k = 0; k < N1; ++k) out[v] = fma(Mz[k], A[v][a + N1 * (b + N1 * k)], out[v]);
        }
        element_sync<WAVE>();
    };
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v] = 0.0;
    load(row[3]);
    if (kind == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) out[v] = in[v];
    } else if (kind == 1) {
        // row pos[d] of I_{path[depth-1]} ... I_{path[0]} (first split applied first)
        const int depth = row[1], code = row[2];
        double M[3][N1];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int pos = d == 0 ? a : d == 1 ? b : c;
#pragma unroll
            for (int j = 0; j < N1; ++j) M[d][j] = j == pos ? 1.0 : 0.0;
            for (int q = depth - 1; q >= 0; --q) {
                const double *I = sops + ((code >> (3 * q + d)) & 1) * 25;
                double nr[N1];
#pragma unroll
                for (int j = 0; j < N1; ++j) {
                    nr[j] = 0.0;
#pragma unroll
                    for (int m = 0; m < N1; ++m) nr[j] = fma(M[d][m], I[m * N1 + j], nr[j]);
                }
#pragma unroll
                for (int j = 0; j < N1; ++j) M[d][j] = nr[j];
            }
        }
        apply(M[0], M[1], M[2]);
    } else {
#pragma unroll 1
        for (int ch = 0; ch < 8; ++ch) {
            double M[3][N1];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int pos = d == 0 ? a : d == 1 ? b : c;
#pragma unroll
                for (int j = 0; j < N1; ++j) M[d][j] = sops[50 + ((ch >> d) & 1) * 25 + pos * N1 + j];
            }
            double next[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) next[v] = ch < 7 ? uold[v * so + (size_t)row[ch < 7 ? 4 + ch : 3] * NN + n] : 0.0;
            apply(M[0], M[1], M[2]);
#pragma unroll
            for (int v = 0; v < NV; ++v) in[v] = next[v];
        }
    }
    if (own) {
#pragma unroll
        for (int v = 0; v < NV; ++v) unew[v * sn + (size_t)e * NN + n] = out[v];
    }
}

}  // namespace dgx
