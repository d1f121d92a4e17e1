// Auxiliary kernels of the right-hand side: BR1 gradients, mixture
// temperature, shock indicator, time-step bound.
#pragma once

#include "k_rhs.h"

namespace dgx {

// BR1 viscous terms, element-local part (Sec. Methodology, Viscous Fluxes,
// Eqs. auxil and auxstrongf; Appendix, Transport, Eq. stress; Sec. New
// Developments, gradient and viscous-flux patching across interfaces and
// mortars; Sec. Results, weak boundaries with the external state averaged
// with the interior one for the viscous terms).
//
// Per element: gradients q = (1/J) sum_d Ja^d [D_d W + lift(W* - W)] of
// W = (v, T = p/(rho R)), the nodal viscous flux F_v[c] = (tau_{.c},
// (tau v)_c + kappa dT/dx_c) and its contravariant form Ft^d = Ja^d . F_v.
// Interface values W*: (W_own + W_nbr)/2 on conforming faces; on a mortar
// face the small side's W*_s from the mortar gradient pass, the large side
// sum_s (P_a x P_b) W*_s; on a boundary face the mean with the external
// state (Dirichlet: the boundary state; outflow: W* = W; slip wall: the
// mirrored velocity), (0, T_wall) at an isothermal and (0, T) at an
// adiabatic no-slip wall.  The divergence with the interface flux F*,
//   (1/J) [ sum_d D_d Ft^d + (F* - Ft_own)/w_N |_{xi_d = 1} - (F* - Ft_own)/w_0 |_{xi_d = -1} ],
// is split into what this element knows (written to P.out, [dim+1][E][nn])
// and the face values Ft^d at its face nodes (written to P.grad as
// [E][2 dim][dim+1][nf]): on conforming and mortar faces F* is completed
// by the right-hand side kernel (the neighbour's half, or the mortar's
// averaged sub-face fluxes), on boundary faces F* = F_v(W*, q).n (viscosity
// at the temperature of W*; no heat flux at an adiabatic wall) is applied
// here.  CURV: nodal metric terms; OPEN: the mesh has boundary or mortar
// faces (the face values W* stay in LDS for the boundary fluxes).
// Memory bounds it on large meshes (15 doubles a node, 52 us at the copy rate
// for 32^3 elements, 67-77 us taken), the chain of its phases on small ones
// (8^3: 6.4 us as one workgroup of four elements that waited for indices, own
// data and traces in turn and met at four barriers, now 5.4).
template <int DIM, int N, bool OPEN = false>
struct GradShape {
    static constexpr int N1 = N + 1;
    static constexpr int NN = DIM == 2 ? N1 * N1 : N1 * N1 * N1;
    static constexpr int NF = NN / N1;
    static constexpr int NW = DIM + 1;
    static constexpr int NSF = 2 * DIM * NF;
    // own W and the neighbours' face traces of W (or the face values W*);
    // then the contravariant viscous fluxes of all directions, over the
    // traces, or after them when those are still needed
    static constexpr int SLOT0 = NW * NN + NW * NSF;
    static constexpr int OFF_T = OPEN ? SLOT0 : 0;
    static constexpr int SLOT = OPEN ? SLOT0 + DIM * NW * NN : (SLOT0 > DIM * NW * NN ? SLOT0 : DIM * NW * NN);
};

// Viscous flux F_v[c] (momentum, energy rows) of velocity v, gradients q,
// viscosity mu and conductivity kappa.
template <int DIM>
__device__ __forceinline__ void visc_flux(const double *v, const double (*q)[DIM + 1], double mu, double kappa,
                                          double (*Fv)[DIM + 1]) {
    double div = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) div += q[k][k];
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        double en = 0.0;
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            double t = mu * (q[c][k] + q[k][c]);
            if (k == c) t -= (2.0 / 3.0) * mu * div;
            en = fma(t, v[k], en);
            Fv[c][k] = t;
        }
        Fv[c][DIM] = en + kappa * q[c][DIM];
    }
}

// suthS > 0: Sutherland's law mu(T) = mu (T/T0)^(3/2) (T0 + S)/(T + S)
// (Eq. sutherland) at every node, the conductivity scaled alike (constant
// Pr); suthS = 0: constant mu.
template <int DIM, int N, bool CURV = false, bool OPEN = false>
__global__ void __launch_bounds__(512) k_grad(RhsParams P, double suthS, double suthT0) {
    using S = GradShape<DIM, N, OPEN>;
    constexpr int N1 = N + 1, NN = S::NN, NF = S::NF, NW = S::NW, NSF = S::NSF;
    constexpr int NV = DIM + 2;
    constexpr int GA = DIM * DIM + 1;
    constexpr int NSUB = DIM == 3 ? 4 : 2;
    extern __shared__ double smem[];
    __shared__ double sD[N1 * N1];  // read with per-lane indices
    const int tid = threadIdx.x;
    // 64 nodes: an element is a wave, its index uniform, and its threads take
    // its own faces, so that after the table's barrier the phases are ordered
    // by wave fences
    constexpr bool WAVE = NN % 64 == 0;
    const int NT = P.epb * NN;
    const int e0 = (P.xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x) * P.epb;
    const int nloc = min(P.epb, P.nelem - e0);
    int el = WAVE ? __builtin_amdgcn_readfirstlane(tid / NN) : tid / NN;
    const int node = tid - el * NN;
    const bool valid = el < nloc;
    const int e = e0 + (valid ? el : 0);
    if (el >= P.epb) el = 0;
    double *sw = smem + el * S::SLOT;
    double *sn = sw + NW * NN;
    const unsigned stride = (unsigned)P.nelem * NN;
    const unsigned gi = (unsigned)e * NN + node;
    const double iR = rcp(P.R);
    // this node's entry of row v of a nodal array
    auto own = [&](const double *x, int v) -> double {
        if constexpr (WAVE) return *(const GlobalDouble *)(scalar_base(x + ((size_t)v * stride + (size_t)e * NN)) + lane_bytes(node));
        else return (x + (size_t)v * stride)[gi];
    };

    auto prim = [&](const double *u, double *W) {
        const double ir = rcp(u[0]);
        double v2 = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            W[c] = u[1 + c] * ir;
            v2 = fma(W[c], W[c], v2);
        }
        const double p = (P.gamma - 1.0) * (u[1 + DIM] - 0.5 * u[0] * v2);
        W[DIM] = p * ir * iR;
    };
    auto transport = [&](double T, double &mu, double &kappa) {
        mu = P.mu;
        kappa = P.kappa;
        if (suthS > 0.0) {
            const double th = T / suthT0;
            const double f = th * sqrt(th) * (suthT0 + suthS) / (T + suthS);
            mu *= f;
            kappa *= f;
        }
    };
    // scaled normal Ja^d at node nd of element ee
    auto normal = [&](int ee, int d, int nd, double *n) {
#pragma unroll
        for (int c = 0; c < DIM; ++c)
            n[c] = CURV ? P.geo[(size_t)(d * DIM + c) * stride + (size_t)ee * NN + nd]
                        : P.geo[(size_t)ee * GA + d * DIM + c];
    };

    // Neighbour face traces (or, on an open mesh, the own trace at boundary
    // faces): one item per face node of every element of the workgroup,
    // spread over all threads (WAVE: of the own element).  The indices are
    // requested first, then what needs none, then the traces.
    constexpr int RF = (NSF + NN - 1) / NN;
    const Spread spf = spread_phase(tid, NT, P.epb * NSF, 0);
    double un[RF][NV], uo[NV];
    int slot[RF], code[RF], item[RF];
#pragma unroll
    for (int r = 0; r < RF; ++r) {
        const int it = WAVE ? el * NSF + r * NN + node : r * NT + spf.t;
        const bool has = WAVE ? valid && r * NN + node < NSF : tid < NT && it < nloc * NSF;
        const int ei = WAVE ? el : it / NSF;
        const int fi = it - ei * NSF;
        slot[r] = has ? ei * S::SLOT + NW * NN + fi : -1;
        item[r] = has ? it : 0;
        code[r] = 0;
        if (has) code[r] = P.nbr[(e0 + ei) * 2 * DIM + fi / NF];
    }
    const double tD = P.B.D[min(tid, N1 * N1 - 1)];
#pragma unroll
    for (int v = 0; v < NV; ++v) uo[v] = own(P.u, v);
    // (where an element is a wave its affine metric terms stay in scalar
    // registers)
    const int eu = WAVE ? __builtin_amdgcn_readfirstlane(e) : e;
    double Ja[DIM * DIM], J;
    if constexpr (CURV) {
#pragma unroll
        for (int k = 0; k < DIM * DIM; ++k) Ja[k] = own(P.geo, k);
        J = own(P.Jn, 0);
    } else {
        const double *g = P.geo + (size_t)eu * GA;
#pragma unroll
        for (int k = 0; k < DIM * DIM; ++k) Ja[k] = g[k];
        J = g[DIM * DIM];
    }
#pragma unroll
    for (int r = 0; r < RF; ++r) {
#pragma unroll
        for (int v = 0; v < NV; ++v) un[r][v] = 1.0;
        if (slot[r] < 0) continue;
        const int ei = WAVE ? el : item[r] / NSF;
        const int fi = item[r] - ei * NSF;
        const int f = fi / NF;
        const int q = fi - f * NF;
        const int d = f >> 1, side = f & 1;
        const int nb = code[r];
        unsigned gj;
        if (!OPEN || nb >= 0) {
            gj = (unsigned)nb * NN + face_node<N1, DIM>(d, side ? 0 : N, q);
        } else if (nb > kMortBase) {
            gj = (unsigned)(e0 + ei) * NN + face_node<N1, DIM>(d, side ? N : 0, q);
        } else {
            continue;  // mortar face: W* from the mortar gradient pass
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) un[r][v] = (P.u + (size_t)v * stride)[gj];
    }
    if (tid < N1 * N1) sD[tid] = tD;
    if (WAVE) __syncthreads();
    double Wo[NW];
    if (valid) {
        prim(uo, Wo);
#pragma unroll
        for (int w = 0; w < NW; ++w) sw[w * NN + node] = Wo[w];
    } else {
#pragma unroll
        for (int w = 0; w < NW; ++w) Wo[w] = 0.0;
    }
#pragma unroll
    for (int r = 0; r < RF; ++r) {
        if (slot[r] < 0) continue;
        double Wn[NW];
        const int nb = code[r];
        if (!OPEN || nb >= 0) {
            prim(un[r], Wn);
        } else {
            const int ei = item[r] / NSF;
            const int fi = item[r] - ei * NSF;
            const int f = fi / NF;
            const int q = fi - f * NF;
            const int d = f >> 1;
            if (nb > kMortBase) {
                // boundary face: W* from the own trace and the boundary kind
                const int bc = -1 - nb;
                const int kind = P.bc_kind[bc];
                double Wf[NW];
                prim(un[r], Wf);
                if (kind == 0) {
                    double ue[NV], We[NW];
#pragma unroll
                    for (int v = 0; v < NV; ++v) ue[v] = P.bc_state[bc * NV + v];
                    prim(ue, We);
#pragma unroll
                    for (int w = 0; w < NW; ++w) Wn[w] = 0.5 * (Wf[w] + We[w]);
                } else if (kind == 1) {
#pragma unroll
                    for (int w = 0; w < NW; ++w) Wn[w] = Wf[w];
                } else if (kind == 2) {
                    double n[DIM];
                    normal(e0 + ei, d, line_node<N1, DIM>(d, (f & 1) ? N : 0, q), n);
                    const double vn = dotn<DIM>(Wf, n) / dotn<DIM>(n, n);
#pragma unroll
                    for (int c = 0; c < DIM; ++c) Wn[c] = Wf[c] - vn * n[c];
                    Wn[DIM] = Wf[DIM];
                } else {
#pragma unroll
                    for (int c = 0; c < DIM; ++c) Wn[c] = 0.0;
                    Wn[DIM] = kind == 3 ? P.bc_state[bc * NV] : Wf[DIM];
                }
            } else {
                const int mc = kMortBase - nb;
                const int m = mc >> 3, role = mc & 7;
                const double *mg = P.mgw + (size_t)m * NSUB * NW * NF;
                if (role < NSUB) {
#pragma unroll
                    for (int w = 0; w < NW; ++w) Wn[w] = mg[(role * NW + w) * NF + q];
                } else {
                    // large side: sum_s (P_a x P_b) W*_s (four nodes' loads at
                    // a time: waiting for each of the 64 took k_grad 25 us on
                    // the wall channel of 904 elements, now 15; its fewer
                    // waves cost the meshes without mortars nothing, 54.5 us
                    // on 21,952 elements either way)
#pragma unroll
                    for (int w = 0; w < NW; ++w) Wn[w] = 0.0;
                    const int qa = q % N1, qb = q / N1;
#pragma unroll 1
                    for (int sb = 0; sb < NSUB; ++sb) {
                        const int a = sb & 1, bsel = sb >> 1;
#pragma unroll 4
                        for (int j = 0; j < NF; ++j) {
                            const int ja = j % N1, jb = j / N1;
                            double wt = P.mops[50 + a * 25 + qa * N1 + ja];
                            if (DIM == 3) wt *= P.mops[50 + bsel * 25 + qb * N1 + jb];
#pragma unroll
                            for (int w = 0; w < NW; ++w) Wn[w] = fma(wt, mg[(sb * NW + w) * NF + j], Wn[w]);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int w = 0; w < NW; ++w) smem[slot[r] + w * NSF] = Wn[w];
    }
    element_sync<WAVE>();
    const double iJ = rcp(J);
    // face codes of this node's faces (open meshes)
    int fcode[DIM];
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
        fcode[d] = 0;
        if constexpr (OPEN) {
            const int a = node_pos<N1>(node, d);
            if (valid && (a == 0 || a == N)) fcode[d] = P.nbr[(size_t)e * 2 * DIM + 2 * d + (a == N ? 1 : 0)];
        }
    }
    double q[DIM][NW];
#pragma unroll
    for (int c = 0; c < DIM; ++c)
#pragma unroll
        for (int w = 0; w < NW; ++w) q[c][w] = 0.0;
    if (valid) {
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
            const int a = node_pos<N1>(node, d);
            const int l = node_line<N1, DIM>(node, d);
            double dW[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) dW[w] = 0.0;
#pragma unroll
            for (int j = 0; j < N1; ++j) {
                const double Dj = sD[a * N1 + j];
                const int nj = line_node<N1, DIM>(d, j, l);
#pragma unroll
                for (int w = 0; w < NW; ++w) dW[w] = fma(Dj, sw[w * NN + nj], dW[w]);
            }
            if (a == 0 || a == N) {
                const int side = (a == N) ? 1 : 0;
                const int fi = (2 * d + side) * NF + l;
                const double sc = side ? P.B.iw0 : -P.B.iw0;
                const bool star = OPEN && fcode[d] < 0;  // the trace slot holds W* itself
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const double ws = star ? sn[w * NSF + fi] : 0.5 * (Wo[w] + sn[w * NSF + fi]);
                    dW[w] = fma(sc, ws - Wo[w], dW[w]);
                }
            }
#pragma unroll
            for (int c = 0; c < DIM; ++c)
#pragma unroll
                for (int w = 0; w < NW; ++w) q[c][w] = fma(Ja[d * DIM + c], dW[w], q[c][w]);
        }
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c)
#pragma unroll
        for (int w = 0; w < NW; ++w) q[c][w] *= iJ;
    // nodal viscous flux
    double Fv[DIM][NW];
    {
        double mu, kappa;
        transport(Wo[DIM], mu, kappa);
        visc_flux<DIM>(Wo, q, mu, kappa, Fv);
    }
    // divergence: volume part and the element's own half of the face terms.
    // All directions' contravariant fluxes go to LDS at once.
    double vis[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) vis[k] = 0.0;
    double *ff = P.out2;
    double *ft = smem + el * S::SLOT + S::OFF_T;  // [DIM][NW][NN]
    if (!OPEN) element_sync<WAVE>();  // the gradient's readers of sw and sn are done
    if (valid) {
#pragma unroll
        for (int d = 0; d < DIM; ++d)
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                double s = 0.0;
#pragma unroll
                for (int c = 0; c < DIM; ++c) s = fma(Ja[d * DIM + c], Fv[c][k], s);
                ft[(d * NW + k) * NN + node] = s;
            }
    }
    element_sync<WAVE>();
    if (valid) {
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
            const int a = node_pos<N1>(node, d);
            const int l = node_line<N1, DIM>(node, d);
#pragma unroll
            for (int j = 0; j < N1; ++j) {
                const double Dj = sD[a * N1 + j];
                const int nj = line_node<N1, DIM>(d, j, l);
#pragma unroll
                for (int k = 0; k < NW; ++k) vis[k] = fma(Dj, ft[(d * NW + k) * NN + nj], vis[k]);
            }
            if (a == 0 || a == N) {
                const int side = (a == N) ? 1 : 0;
                // row k of the face's values Ft
                const size_t f0 = ((size_t)e * 2 * DIM + 2 * d) * NW * NF;
                auto put_face = [&](int k, double x) {
                    if constexpr (WAVE)
                        ((GlobalDouble *)(scalar_base(ff + f0) + lane_bytes(side * NW * NF + l)))[k * NF] = x;
                    else (ff + f0 + side * NW * NF + l)[k * NF] = x;
                };
                if (OPEN && fcode[d] < 0 && fcode[d] > kMortBase) {
                    // boundary face: F* = F_v(W*, q).n, applied in full here
                    const int bc = -1 - fcode[d];
                    const int kind = P.bc_kind[bc];
                    const int fi = (2 * d + side) * NF + l;
                    double Wb[NW], mu, kappa, Fb[DIM][NW];
#pragma unroll
                    for (int w = 0; w < NW; ++w) Wb[w] = sn[w * NSF + fi];
                    transport(Wb[DIM], mu, kappa);
                    visc_flux<DIM>(Wb, q, mu, kind == 4 ? 0.0 : kappa, Fb);
                    const double sc = side ? P.B.iw0 : -P.B.iw0;
#pragma unroll
                    for (int k = 0; k < NW; ++k) {
                        double Fs = 0.0;
#pragma unroll
                        for (int c = 0; c < DIM; ++c) Fs = fma(Ja[d * DIM + c], Fb[c][k], Fs);
                        if (kind == 4 && k == DIM) Fs = 0.0;
                        const double Ftk = ft[(d * NW + k) * NN + node];
                        vis[k] = fma(sc, Fs - Ftk, vis[k]);
                        put_face(k, Ftk);
                    }
                } else {
                    const double sc = side ? -0.5 * P.B.iw0 : 0.5 * P.B.iw0;
#pragma unroll
                    for (int k = 0; k < NW; ++k) {
                        const double Ftk = ft[(d * NW + k) * NN + node];
                        vis[k] = fma(sc, Ftk, vis[k]);
                        put_face(k, Ftk);
                    }
                }
            }
        }
    }
    if (valid) {
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if constexpr (WAVE)
                *(GlobalDouble *)(scalar_base(P.out + ((size_t)k * stride + (size_t)e * NN)) + lane_bytes(node)) = vis[k] * iJ;
            else (P.out + (size_t)k * stride)[gi] = vis[k] * iJ;
        }
    }
}

// Mortar gradient pass (BR1 on 2:1 meshes): one thread per small-face node
// of every mortar sub-face.  The large element's conserved trace is
// interpolated to the node (I_a x I_b), W* = (W_small + W(I u_large))/2 is
// written to P.out as [nm][2^(dim-1)][dim+1][nf] for the gradient kernel
// (the small side reads it, the large side projects it back).  Perfect gas,
// affine elements.
template <int DIM, int N>
__global__ void __launch_bounds__(256) k_mortar_grad(RhsParams P, int nmort) {
    constexpr int N1 = N + 1;
    constexpr int NN = DIM == 2 ? N1 * N1 : N1 * N1 * N1;
    constexpr int NF = NN / N1;
    constexpr int NV = DIM + 2, NW = DIM + 1;
    constexpr int NSUB = DIM == 3 ? 4 : 2;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nmort * NSUB * NF) return;
    const int m = t / (NSUB * NF);
    const int r = t - m * NSUB * NF;
    const int s = r / NF, q = r - s * NF;
    const int *row = P.mort + (size_t)m * (3 + NSUB);
    const int eL = row[0], fL = row[1], es = row[2 + s], fS = row[2 + NSUB];
    const int d = fL >> 1, sideL = fL & 1;
    const size_t stride = (size_t)P.nelem * NN;
    const int a = s & 1, bsel = s >> 1;
    const int qa = q % N1, qb = q / N1;
    double ui[NV], us[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) ui[v] = 0.0;
    for (int j = 0; j < NF; ++j) {
        const int ja = j % N1, jb = j / N1;
        double w = P.mops[a * 25 + qa * N1 + ja];
        if (DIM == 3) w *= P.mops[bsel * 25 + qb * N1 + jb];
        const size_t gj = (size_t)eL * NN + line_node<N1, DIM>(d, sideL ? N : 0, j);
#pragma unroll
        for (int v = 0; v < NV; ++v) ui[v] = fma(w, P.u[v * stride + gj], ui[v]);
    }
    const size_t gs = (size_t)es * NN + line_node<N1, DIM>(d, (fS & 1) ? N : 0, q);
#pragma unroll
    for (int v = 0; v < NV; ++v) us[v] = P.u[v * stride + gs];
    double Wi[NW], Ws[NW];
    auto prim = [&](const double *u, double *W) {
        const double ir = rcp(u[0]);
        double v2 = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            W[c] = u[1 + c] * ir;
            v2 = fma(W[c], W[c], v2);
        }
        const double p = (P.gamma - 1.0) * (u[1 + DIM] - 0.5 * u[0] * v2);
        W[DIM] = p * ir / P.R;
    };
    prim(ui, Wi);
    prim(us, Ws);
    double *o = P.out + (size_t)m * NSUB * NW * NF;
#pragma unroll
    for (int w = 0; w < NW; ++w) o[(s * NW + w) * NF + q] = 0.5 * (Ws[w] + Wi[w]);
}

// The per-node T(e) solve (Appendix, Thermodynamics) of the conserved state
// uo of one node (species first): Newton from t (T0 when t is not a positive
// number); a failed warm start (warm != 0) is retried from T0.  Returns the
// iteration count, < 0 on failure; rs, rho for the caller.
template <int DIM>
__device__ __forceinline__ int node_temperature_state(const double *uo, double &t, double T0, double tol, int maxit,
                                                      const MixC &M, int warm, double *rs, double &rho) {
    rho = 0.0;
#pragma unroll
    for (int s = 0; s < kNS; ++s) {
        rs[s] = uo[s];
        rho += rs[s];
    }
    double m2 = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) m2 = fma(uo[kNS + c], uo[kNS + c], m2);
    const double rhoe = uo[kNS + DIM] - 0.5 * m2 / rho;
    if (!(t > 0.0) || !isfinite(t)) t = T0;
    int it = mix_newton(M, rs, rhoe, t, tol, maxit);
    if (warm && (it < 0 || !isfinite(t) || !(t > 0.0))) {
        t = T0;
        it = mix_newton(M, rs, rhoe, t, tol, maxit);
    }
    return (it < 0 || !isfinite(t) || !(t > 0.0)) ? -1 : it;
}

// The same for node i of u ([nvar][count]).
template <int DIM>
__device__ __forceinline__ int node_temperature(const double *__restrict__ u, size_t count, size_t i, double &t,
                                                double T0, double tol, int maxit, const MixC &M, int warm,
                                                double *rs, double &rho) {
    double uo[kNS + DIM + 1];
#pragma unroll
    for (int v = 0; v < kNS + DIM + 1; ++v) uo[v] = u[v * count + i];
    return node_temperature_state<DIM>(uo, t, T0, tol, maxit, M, warm, rs, rho);
}

// Per-node T(e) Newton (Appendix, Thermodynamics).  Tguess may be null
// (use T0).  Writes T, optionally p, and the iteration count.
template <int DIM>
__global__ void __launch_bounds__(256) k_thermo(const double *__restrict__ u, int64_t count,
                                                const double *__restrict__ Tguess, double T0,
                                                double tol, int maxit, MixC M, double *__restrict__ T,
                                                double *__restrict__ pout, double *__restrict__ cout,
                                                int *__restrict__ iters, unsigned *flags, int warm) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    double rs[kNS], rho;
    // guess: the given one (a learned guess), or with warm != 0 the node's
    // previous T (the right-hand side's solves), else T0.  A failed warm
    // start, and a failed solve from a given guess, are retried from T0, so
    // the converged T never depends on how good the guess was; the
    // iteration count then includes both attempts, and the retry is marked
    // in the count (bit kItersFallback) for the statistics.
    double t = Tguess ? Tguess[i] : (warm ? T[i] : T0);
    int it = node_temperature<DIM>(u, (size_t)count, (size_t)i, t, T0, tol, maxit, M, warm, rs, rho);
    bool fell_back = false;
    if (Tguess && it < 0) {
        t = T0;
        const int it2 = node_temperature<DIM>(u, (size_t)count, (size_t)i, t, T0, tol, maxit, M, 0, rs, rho);
        it = it2 < 0 ? -1 : it2 + maxit;
        fell_back = true;
    }
    T[i] = t;
    if (pout) pout[i] = mix_rR(M, rs) * t;
    if (cout) cout[i] = mix_sound(M, rs, rho, t);
    if (iters) iters[i] = it < 0 ? -1 : (fell_back ? (it | kItersFallback) : it);
    if (it < 0) atomicOr(flags, FLAG_NOCONV);
}

// Modal shock indicator (Hennemann et al. type, as referenced in
// Sec. Methodology): eps = rho*p or p, orthonormal Legendre modes by V^-1
// along each direction, energy ratio of the top modes, logistic map to alpha.
// A chain of short phases bounds it: where an element's nodes lie in one wave
// (16 or 64) they are ordered by wave fences and summed by lane shifts, in the
// order of the LDS tree, and the map's constants come from the host (9.7 ->
// 7.3 us on 8,192 elements of 16 nodes).
template <int DIM, int N, bool MIX>
__global__ void __launch_bounds__(512) k_indicator(RhsParams P, int ind_var, double alpha_max,
                                                   double alpha_min, double *__restrict__ alpha,
                                                   double *__restrict__ alpha_raw, double *__restrict__ Tw,
                                                   double *__restrict__ cw, double T0, double tol, int maxit) {
    constexpr int N1 = N + 1;
    constexpr int NN = DIM == 2 ? N1 * N1 : N1 * N1 * N1;
    constexpr int NV = (MIX ? kNS : 1) + DIM + 1;
    constexpr bool WAVE = 64 % NN == 0;
    extern __shared__ double smem[];
    __shared__ double sV[N1 * N1];  // V^-1, read with per-lane indices
    const int tid = threadIdx.x;
    const double tV = P.B.Vinv[min(tid, N1 * N1 - 1)];
    int el = tid / NN;
    const int node = tid - el * NN;
    const int e = blockIdx.x * P.epb + el;
    const bool valid = (el < P.epb) && (e < P.nelem);
    if (el >= P.epb) el = 0;
    double *x = smem + el * 3 * NN;
    double *y = x + NN;
    double *z = y + NN;
    const size_t stride = (size_t)P.nelem * NN;
    const size_t gi = (size_t)(valid ? e : 0) * NN + node;
    if (valid) {
        double uo[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) uo[v] = P.u[v * stride + gi];
        double Tn = 0.0;
        if constexpr (MIX) {
            Tn = P.T[gi];
            if (Tw) {
                // the right-hand side's T(e) solve, fused (the same steps as
                // k_thermo with a warm start): T and the frozen sound speed
                double rs[kNS], rho;
                const int it = node_temperature_state<DIM>(uo, Tn, T0, tol, maxit, P.M, 1, rs, rho);
                Tw[gi] = Tn;
                cw[gi] = mix_sound(P.M, rs, rho, Tn);
                if (it < 0) atomicOr(P.flags, FLAG_NOCONV);
            }
        }
        St<DIM, MIX> s;
        make_state<DIM, MIX>(uo, Tn, P.gamma, P.M, s);
        x[node] = ind_var == 1 ? s.p : s.rho * s.p;
    }
    if (tid < N1 * N1) sV[tid] = tV;
    __syncthreads();
#pragma unroll 1
    for (int d = 0; d < DIM; ++d) {
        double m = 0.0;
        if (valid) {
            const int a = node_pos<N1>(node, d);
            const int l = node_line<N1, DIM>(node, d);
#pragma unroll
            for (int j = 0; j < N1; ++j) m = fma(sV[a * N1 + j], x[line_node<N1, DIM>(d, j, l)], m);
        }
        element_sync<WAVE>();
        if (valid) x[node] = m;
        element_sync<WAVE>();
    }
    // modal energies: all modes, modes of degree <= N-1, <= N-2 (degree = the
    // largest one-dimensional index), summed over the element in a fixed tree
    int mx = 0;
#pragma unroll
    for (int d = 0; d < DIM; ++d) mx = max(mx, node_pos<N1>(node, d));
    const double m2 = valid ? x[node] * x[node] : 0.0;
    double eall = m2, e1 = mx <= N - 1 ? m2 : 0.0, e2 = mx <= N - 2 ? m2 : 0.0;
    if constexpr (WAVE) {
#pragma unroll
        for (int h = NN / 2; h > 0; h >>= 1) {
            eall += __shfl_down(eall, h);
            e1 += __shfl_down(e1, h);
            e2 += __shfl_down(e2, h);
        }
    } else {
        if (valid) {
            x[node] = eall;
            y[node] = e1;
            z[node] = e2;
        }
        __syncthreads();
        constexpr int P2 = NN <= 32 ? 32 : 128;
#pragma unroll
        for (int h = P2 / 2; h > 0; h >>= 1) {
            if (valid && node < h && node + h < NN) {
                x[node] += x[node + h];
                y[node] += y[node + h];
                z[node] += z[node + h];
            }
            __syncthreads();
        }
        eall = x[0];
        e1 = y[0];
        e2 = z[0];
    }
    if (valid && node == 0) {
        const double E = fmax((eall - e1) / eall, (e1 - e2) / e1);
        const double a = 1.0 / (1.0 + exp(-P.B.ind_slope * (E - P.B.ind_thr)));
        alpha_raw[e] = a;
        alpha[e] = a < alpha_min ? 0.0 : fmin(a, alpha_max);
    }
}

// Zhang-Shu positivity-preserving scaling limiter, in place on u (see
// dgx_limit_positivity in the C ABI).  Means and minima are reduced over the
// element's nodes in a fixed order (deterministic), one thread for each: the
// chain of these reductions bounds the kernel (by one thread for all of them:
// 9.3 us on 8,192 elements of 16 nodes, now 7.2).
template <int DIM, bool MIX>
__device__ __forceinline__ double zs_psi(const double *u, const MixC &M) {
    constexpr int off = MIX ? kNS : 1;
    double rho = 0.0, lin = u[off + DIM];
    if constexpr (MIX) {
#pragma unroll
        for (int s = 0; s < kNS; ++s) {
            rho += u[s];
            lin -= M.e0[s] * u[s];
        }
    } else {
        rho = u[0];
    }
    double m2 = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) m2 = fma(u[off + c], u[off + c], m2);
    return lin - 0.5 * m2 / rho;
}

// LDS doubles per element of k_positivity
template <int NN, int NV, int ND>
constexpr int kPosSlot = (NV + 1 + ND) * NN + NV + ND;

template <int DIM, int N, bool MIX, bool CURV>
__global__ void __launch_bounds__(512) k_positivity(RhsParams P, double *__restrict__ u) {
    constexpr int N1 = N + 1;
    constexpr int NN = DIM == 2 ? N1 * N1 : N1 * N1 * N1;
    constexpr int NV = (MIX ? kNS : 1) + DIM + 1;
    constexpr int ND = MIX ? kNS : 1;  // density variables
    constexpr int GA = DIM * DIM + 1;
    constexpr int SL = kPosSlot<NN, NV, ND>;
    extern __shared__ double smem[];
    const int tid = threadIdx.x;
    int el = tid / NN;
    const int node = tid - el * NN;
    const int e = blockIdx.x * P.epb + el;
    const bool valid = (el < P.epb) && (e < P.nelem);
    if (el >= P.epb) el = 0;
    double *sw = smem + el * SL;         // [NV+1][NN] weighted values, then scratch
    double *sr = sw + (NV + 1) * NN;     // [ND][NN] densities
    double *sbar = sr + ND * NN;         // [NV] means
    double *smin = sbar + NV;            // [ND] smallest densities
    const size_t stride = (size_t)P.nelem * NN;
    const size_t gi = (size_t)(valid ? e : 0) * NN + node;
    double uo[NV];
    double wJ = 0.0;
    if (valid) {
#pragma unroll
        for (int v = 0; v < NV; ++v) uo[v] = u[v * stride + gi];
        double w = 1.0;
#pragma unroll
        for (int d = 0; d < DIM; ++d) w *= P.B.w[node_pos<N1>(node, d)];
        const double J = CURV ? P.Jn[gi] : P.geo[(size_t)e * GA + DIM * DIM];
        wJ = w * J;
#pragma unroll
        for (int v = 0; v < NV; ++v) sw[v * NN + node] = wJ * uo[v];
        sw[NV * NN + node] = wJ;
#pragma unroll
        for (int s = 0; s < ND; ++s) sr[s * NN + node] = uo[s];
    }
    __syncthreads();
    static_assert(NV + ND <= NN, "a thread per reduction");
    if (valid && node < NV) {
        double vol = 0.0, s = 0.0;
#pragma unroll 16
        for (int n = 0; n < NN; ++n) {
            vol += sw[NV * NN + n];
            s += sw[node * NN + n];
        }
        sbar[node] = s / vol;
    } else if (valid && node < NV + ND) {
        const double *r = sr + (node - NV) * NN;
        double mn = r[0];
#pragma unroll 16
        for (int n = 1; n < NN; ++n) mn = fmin(mn, r[n]);
        smin[node - NV] = mn;
    }
    __syncthreads();
    double ubar[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) ubar[v] = sbar[v];
    // 1. densities
    bool changed = false;
#pragma unroll
    for (int s = 0; s < ND; ++s) {
        const double mn = smin[s];
        const double eps = MIX ? 1e-14 * fmax(ubar[s], 0.0) : fmin(1e-13, ubar[s]);
        const double th = (mn < eps && ubar[s] > eps) ? (ubar[s] - eps) / (ubar[s] - mn) : 1.0;
        if (th < 1.0) {
            uo[s] = ubar[s] + th * (uo[s] - ubar[s]);
            changed = true;
        }
    }
    // 2. pressure
    double rho_bar = 0.0;
#pragma unroll
    for (int s = 0; s < ND; ++s) rho_bar += ubar[s];
    const double pb = zs_psi<DIM, MIX>(ubar, P.M);
    const double eps_p = fmin(1e-13 * rho_bar * (MIX ? 1e5 : 1.0), pb);
    double tn = 1.0;
    if (valid && pb > 0.0 && zs_psi<DIM, MIX>(uo, P.M) < eps_p) {
        double lo = 0.0, hi = 1.0, ut[NV];
        for (int it = 0; it < 64; ++it) {
            const double mid = 0.5 * (lo + hi);
#pragma unroll
            for (int v = 0; v < NV; ++v) ut[v] = ubar[v] + mid * (uo[v] - ubar[v]);
            if (zs_psi<DIM, MIX>(ut, P.M) >= eps_p) lo = mid;
            else hi = mid;
        }
        tn = lo;
    }
    if (valid && node == 0 && pb <= 0.0) atomicOr(P.flags, FLAG_NONPHYS);
    double thp = 1.0;
    if (__syncthreads_or(tn < 1.0)) {
        if (valid) sw[node] = tn;
        __syncthreads();
        for (int n = 0; n < NN; ++n) thp = fmin(thp, sw[n]);
    }
    if (thp < 1.0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) uo[v] = ubar[v] + thp * (uo[v] - ubar[v]);
        changed = true;
    }
    if (valid && changed) {
#pragma unroll
        for (int v = 0; v < NV; ++v) u[v * stride + gi] = uo[v];
    }
}

// alpha_k <- max(alpha_k, alpha_nbr / 2) over conforming neighbours.
template <int DIM>
__global__ void k_alpha_smooth(const int *__restrict__ nbr, int nelem, const double *__restrict__ ain,
                               double *__restrict__ aout) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nelem) return;
    double a = ain[e];
#pragma unroll
    for (int f = 0; f < 2 * DIM; ++f) {
        const int nb = nbr[(size_t)e * 2 * DIM + f];
        if (nb >= 0) a = fmax(a, 0.5 * ain[nb]);
    }
    aout[e] = a;
}

// max_n sum_d (|v.Ja^d| + c |Ja^d|)/J, as an ordered uint64 of a positive
// double; +inf where a node's value is no number (fmax would drop a NaN and the
// caller take a step from the other nodes).
// Atomics on the one result take about 10 ns each, so the grid is at most
// kMaxrateBlocks workgroups, each with one (one per wave of nodes: 64 us for
// 342,528 nodes, now 10).
constexpr int kMaxrateBlocks = 512;
template <int DIM, bool MIX, bool CURV>
__global__ void __launch_bounds__(256) k_maxrate(RhsParams P, unsigned long long *out) {
    constexpr int GA = DIM * DIM + 1;
    const int NN = P.epb;  // nodes per element passed in epb
    const int64_t total = (int64_t)P.nelem * NN;
    double best = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int e = (int)(i / NN);
        const size_t stride = (size_t)total;
        constexpr int NV = (MIX ? kNS : 1) + DIM + 1;
        double uo[NV];
        for (int v = 0; v < NV; ++v) uo[v] = P.u[v * stride + i];
        St<DIM, MIX> s;
        make_state<DIM, MIX>(uo, MIX ? P.T[i] : 0.0, P.gamma, P.M, s, MIX ? P.csnd + i : nullptr);
        const double J = CURV ? P.Jn[i] : P.geo[(size_t)e * GA + DIM * DIM];
        double rate = 0.0;
        for (int d = 0; d < DIM; ++d) {
            double n[DIM];
            for (int c = 0; c < DIM; ++c)
                n[c] = CURV ? P.geo[(d * DIM + c) * stride + i] : P.geo[(size_t)e * GA + d * DIM + c];
            rate += fabs(dotn<DIM>(s.v, n)) + s.c * wave_sqrt(dotn<DIM>(n, n));
        }
        rate /= fabs(J);
        best = fmax(best, rate >= 0.0 ? rate : (double)INFINITY);
    }
    for (int off = 32; off > 0; off >>= 1) best = fmax(best, __shfl_xor(best, off));
    __shared__ double wave[4];
    if ((threadIdx.x & 63) == 0) wave[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0)
        atomicMax(out, (unsigned long long)__double_as_longlong(fmax(fmax(wave[0], wave[1]), fmax(wave[2], wave[3]))));
}

}  // namespace dgx
