// Reverse mode of the explicit step: hand-written adjoints of G2P (with the
// Hencky / Drucker-Prager constitutive map), the grid update and P2G.
//
// Per step, with the forward recomputed from the step's input state:
//   k_g2p_adj      per particle (in G2P's output order): recomputes grad v and
//                  F_trial from the staged grid tile, back-propagates the
//                  output adjoints through the constitutive map (Daleckii-Krein
//                  form on the eigen-decomposition of F F^T, with closed-form
//                  divided differences), and writes x_bar (partial), F_bar, and
//                  the per-particle (x, v'_bar, B_bar, W_bar) that the grid
//                  needs; accumulates dL/dE and dL/dphi.
//   k_scatter_adj  v_bar_n = sum_p N v'_bar + N B_bar (x_n - x_p) + W_bar grad N,
//                  a workgroup per owner block, a lane per base cell and rank
//                  group, like P2G; the tiles go to the tile store.
//   k_gather_adj   sums the tiles that cover a node (as P2G's second pass does)
//                  and applies the adjoint of the grid update: u_bar = (boundary
//                  Jacobian) v_bar; p_bar = u_bar / m, m_bar = -u_bar . (u - dt g) / m.
//                  (On a dense grid the scatter adds to a cleared grid instead,
//                  and k_grid_adj follows.)
//   k_p2g_adj      per particle gather of (p_bar, m_bar): v_bar, C_bar, tau_bar
//                  and the position terms (shape-function gradient and Hessian).
//
// The gathers need sums over the stencil of the node vectors against N, its
// gradient and its Hessian.  All are products of one-dimensional factors, so
// they are formed an axis at a time (gather_moments), about 1000 fused
// multiply-adds per particle instead of 3500 with the factors of each node
// formed in full.
#include <math.h>

#include <algorithm>

#include "internal.h"
#include "particle.h"

namespace mpmx {

// 1 / x to about half an ulp: hardware reciprocal and one Newton step.
__device__ __forceinline__ float rcp_nr(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(fmaf(-x, r, 1.f), r, r);
}
// sinh(y) / y from y^2 <= 1 (the next term is below 2e-10)
__device__ __forceinline__ float shc(float y2) {
    return 1.f + y2 * (1.f / 6.f) * (1.f + y2 * (1.f / 20.f) * (1.f + y2 * (1.f / 42.f) * (1.f + y2 * (1.f / 72.f) *
           (1.f + y2 * (1.f / 110.f)))));
}
// x / sinh(x), and sinh(hb x) / sinh(x) for |hb| <= 1/2, smooth through 0
__device__ __forceinline__ void sinh_ratios(float hb, float x, float* x_over_sinh, float* ratio) {
    if (fabsf(x) <= 1.f) {
        *x_over_sinh = rcp_nr(shc(x * x));
        *ratio = hb * shc(hb * x * hb * x) * *x_over_sinh;
    } else {
        const float sh = sinhf(x);
        *x_over_sinh = x / sh;
        *ratio = sinhf(hb * x) / sh;
    }
}
// ln(1 + m): 2 atanh(m / (2 + m)) by its series near 0, where 1 + m would round
__device__ __forceinline__ float log1p_small(float m) {
    if (fabsf(m) > 0.3f) return logf(fmaxf(1.f + m, 1e-6f));
    const float z = m * rcp_nr(2.f + m), z2 = z * z;
    return 2.f * z * (1.f + z2 * (1.f / 3.f + z2 * (0.2f + z2 * (1.f / 7.f + z2 * (1.f / 9.f + z2 * (1.f / 11.f))))));
}

// Adjoint of (F^E, tau) = Z(F_trial).  Inputs: Ft (F_trial), Fe_bar (full),
// tau_bar as stored components; outputs: Ft_bar, dL/dE, dL/dalpha.
//
// In principal values the return map gives eps'_i = kappa eps_i + c0 for all i
// (elastic: kappa = 1, c0 = 0; apex: both 0; cone: the closed forms below), so
//   exp(eps'_i - eps_i) = h_i, exp(-eps_i) = q_i
// give every divided difference: for i != j, with x = eps_i - eps_j,
//   (tau_i - tau_j) / (lam_i - lam_j) = mu kappa q_i q_j x / sinh x,
//   (h_i - h_j) / (lam_i - lam_j) = sqrt(h_i h_j) q_i q_j sinh(beta x / 2) / sinh x
// (lam = exp(2 eps), beta = kappa - 1), and the Jacobian of the cone map is
// applied to a vector without being formed.
//
// Which branch of the return map a particle within rounding of a kink takes
// is settled by one fixed evaluation of F_trial (trial_by_nodes) and of the
// strains (NODES), not by the faster ones used elsewhere: the gradients jump
// there, so a particle that fell on the other side would move dL/dphi by its
// whole share (3e-4 of it, in one of 262,144 particles over 20 steps).  (It is
// not the forward pass's evaluation, which takes the branch from the matrix
// series: within rounding of a kink the two can differ.)
// The two evaluations of tr differ by 3e-8 rms (1 + M rounds in each strain).
// Deciding takes 7 us of 48 at 262,144 particles of loaded material: 4 us for the
// registers of the second copy of the code, 3 us to run it.  Undeformed
// particles are all in doubt (F = I is the kink): a rollout from rest, 61 us.
//
// Error of the gradients against 64 bits over 80 calibration passes of 1,000 to
// 60,000 particles (the same with expf, sqrtf and divisions in these maps, in
// brackets): dL/dE median 1.6e-7 (1.7e-7), dL/dphi 2.4e-6 (2.4e-6).
constexpr float KINK_TOL = 2.5e-7f;
struct Principal {
    float U[3][3];                 // eigenvectors of F_trial F_trial^T
    float q[3] = {1.f, 1.f, 1.f};  // exp(-eps)
    float eps[3] = {0.f, 0.f, 0.f}, dev[3] = {0.f, 0.f, 0.f};
    float tr = 0.f, nd = 0.f;  // trace of eps, norm of dev
    int branch = 0;            // 0 elastic, 1 apex, 2 cone
};
// Whether the branch is in doubt (never with NODES).
template <int DIM, bool NODES>
__device__ __forceinline__ bool principal_strains(const DevParams& P, const float (*Ft)[3], Principal& S) {
    float M[3][3];
    const float ca = P.dp_coef * P.alpha;
    {
        float Hm[3][3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) Hm[a][b] = (a < DIM && b < DIM) ? Ft[a][b] - (a == b ? 1.f : 0.f) : 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = a; b < 3; ++b) {
                float s = Hm[a][b] + Hm[b][a];
#pragma unroll
                for (int c = 0; c < DIM; ++c) s += Hm[a][c] * Hm[b][c];
                M[a][b] = M[b][a] = s;
            }
    }
    jacobi_sym<DIM>(M, S.U);
    float wide = 1.f;
    S.tr = 0.f;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const float lam = fmaxf(1.f + M[a][a], 1e-6f);
        S.eps[a] = 0.5f * (NODES ? logf(lam) : log1p_small(M[a][a]));
        const float r = __builtin_amdgcn_rsqf(lam);
        S.q[a] = fmaf(0.5f * r, fmaf(-lam * r, r, 1.f), r);  // 1 / sqrt(lam), one Newton step
        wide = fmaxf(wide, S.q[a] * S.q[a]);
        S.tr += S.eps[a];
    }
    if (P.model != MPM_MODEL_DP) return false;
    float nd2 = 0.f;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        S.dev[a] = S.eps[a] - S.tr / (float)DIM;
        nd2 += S.dev[a] * S.dev[a];
    }
    S.nd = sqrtf(nd2);
    const float dg = S.nd + P.dp_coef * S.tr * P.alpha, tol = KINK_TOL * wide;
    S.branch = S.tr > 0.f ? 1 : dg > 0.f ? 2 : 0;
    if (NODES) {
        if (S.branch != 2)  // not needed any more in the form that decided
#pragma unroll
            for (int a = 0; a < DIM; ++a) S.eps[a] = 0.5f * log1p_small(M[a][a]);
        return false;
    }
    return !(fabsf(S.tr) > tol && (S.branch == 1 || fabsf(dg) > tol * (1.f + ca)));
}

// Adjoint of (F^E, tau) = Z(F_trial) from the strains of F_trial.
template <int DIM>
__device__ __forceinline__ void constitutive_adj(const DevParams& P, const Principal& pr, const float (*Ft)[3],
                                                 const float (*Fe_bar)[3], const float* tau_bar_c, float (*Ft_bar)[3],
                                                 float* E_bar, float* a_bar) {
    const float (*U)[3] = pr.U;
    const float *q = pr.q, *eps = pr.eps, *dev = pr.dev, tr = pr.tr, nd = pr.nd, ca = P.dp_coef * P.alpha;
    const int branch = pr.branch;
    float e2[3] = {eps[0], eps[1], eps[2]}, nh[3] = {0.f, 0.f, 0.f}, kappa = 1.f, rnd = 0.f;
    if (branch == 1) {
        kappa = 0.f;
        e2[0] = e2[1] = e2[2] = 0.f;
    } else if (branch == 2) {
        rnd = rcp_nr(nd);
        kappa = -ca * tr * rnd;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            nh[a] = dev[a] * rnd;
            e2[a] = tr / (float)DIM - ca * tr * nh[a];
        }
    }
    float tr2 = 0.f, h[3] = {1.f, 1.f, 1.f};
#pragma unroll
    for (int a = 0; a < DIM; ++a) tr2 += e2[a];
    if (branch != 0)
#pragma unroll
        for (int a = 0; a < DIM; ++a) h[a] = __builtin_amdgcn_exp2f((e2[a] - eps[a]) * 1.44269504f);
    // H = U diag(h) U^T: Ft_bar = H Fe_bar for now; H_bar = Fe_bar Ft^T
    float Hb[3][3];
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < DIM; ++c) s += Fe_bar[a][c] * Ft[b][c];
            Hb[a][b] = s;
        }
    {
        float Hmat[3][3];
#pragma unroll
        for (int a = 0; a < DIM; ++a)
#pragma unroll
            for (int b = a; b < DIM; ++b) {
                float s = 0.f;
#pragma unroll
                for (int c = 0; c < DIM; ++c) s += U[a][c] * h[c] * U[b][c];
                Hmat[a][b] = Hmat[b][a] = s;
            }
#pragma unroll
        for (int a = 0; a < DIM; ++a)
#pragma unroll
            for (int b = 0; b < DIM; ++b) {
                float s = 0.f;
#pragma unroll
                for (int c = 0; c < DIM; ++c) s += Hmat[a][c] * Fe_bar[c][b];
                Ft_bar[a][b] = s;
            }
    }
    // symmetric parts in the eigenbasis: Y = U^T sym(.) U (upper triangles)
    float Yt[3][3], Yh[3][3];
    {
        float ts[3][3], t1[3][3], t2[3][3];
        if (DIM == 3) {
            ts[0][0] = tau_bar_c[0];
            ts[1][1] = tau_bar_c[1];
            ts[2][2] = tau_bar_c[2];
            ts[0][1] = ts[1][0] = 0.5f * tau_bar_c[3];
            ts[1][2] = ts[2][1] = 0.5f * tau_bar_c[4];
            ts[0][2] = ts[2][0] = 0.5f * tau_bar_c[5];
        } else {
            ts[0][0] = tau_bar_c[0];
            ts[1][1] = tau_bar_c[1];
            ts[0][1] = ts[1][0] = 0.5f * tau_bar_c[2];
        }
#pragma unroll
        for (int a = 0; a < DIM; ++a)
#pragma unroll
            for (int b = 0; b < DIM; ++b) {
                float s1 = 0.f, s2 = 0.f;
#pragma unroll
                for (int c = 0; c < DIM; ++c) {
                    s1 += ts[a][c] * U[c][b];
                    s2 += 0.5f * (Hb[a][c] + Hb[c][a]) * U[c][b];
                }
                t1[a][b] = s1;
                t2[a][b] = s2;
            }
#pragma unroll
        for (int a = 0; a < DIM; ++a)
#pragma unroll
            for (int b = a; b < DIM; ++b) {
                float s1 = 0.f, s2 = 0.f;
#pragma unroll
                for (int c = 0; c < DIM; ++c) {
                    s1 += U[c][a] * t1[c][b];
                    s2 += U[c][a] * t2[c][b];
                }
                Yt[a][b] = s1;
                Yh[a][b] = s2;
            }
    }
    // diagonal: S_jj = (sum_i J_ij z_i - h_j Yh_jj) / (2 lam_j) with J = d eps'/d eps
    // and z_i = 2 mu Yt_ii + lambda tr(Yt) + h_i Yh_ii
    float trY = 0.f, z[3] = {0.f, 0.f, 0.f}, Z = 0.f, nz = 0.f, eb = 0.f;
#pragma unroll
    for (int i = 0; i < DIM; ++i) trY += Yt[i][i];
#pragma unroll
    for (int i = 0; i < DIM; ++i) {
        z[i] = 2.f * P.mu * Yt[i][i] + P.lam * trY + h[i] * Yh[i][i];
        Z += z[i];
        nz += nh[i] * z[i];
        eb += Yt[i][i] * (2.f * P.mu * e2[i] + P.lam * tr2);
    }
    float S[3][3];
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
        float Jz = branch == 0 ? z[j] : 0.f;
        if (branch == 2)
            Jz = Z / (float)DIM - ca * (nz + tr * rnd * (z[j] - Z / (float)DIM - nz * nh[j]));
        S[j][j] = 0.5f * q[j] * q[j] * (Jz - h[j] * Yh[j][j]);
    }
    const float hb = 0.5f * (kappa - 1.f);
#pragma unroll
    for (int i = 0; i < DIM; ++i)
#pragma unroll
        for (int j = i + 1; j < DIM; ++j) {
            float xs, sr;
            sinh_ratios(hb, eps[i] - eps[j], &xs, &sr);
            const float qq = q[i] * q[j];
            S[i][j] = S[j][i] = qq * (P.mu * kappa * xs * Yt[i][j] + sqrtf(h[i] * h[j]) * sr * Yh[i][j]);
        }
    // b_bar = U S U^T; Ft_bar += 2 b_bar Ft
    float t1[3][3], bb[3][3];
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < DIM; ++c) s += S[a][c] * U[b][c];
            t1[a][b] = s;
        }
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int b = a; b < DIM; ++b) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < DIM; ++c) s += U[a][c] * t1[c][b];
            bb[a][b] = bb[b][a] = s;
        }
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < DIM; ++c) s += bb[a][c] * Ft[c][b];
            Ft_bar[a][b] += 2.f * s;
        }
    // parameters: tau is proportional to E; alpha enters eps' on the cone,
    // d eps'/d alpha = -dp_coef tr nh
    *E_bar = eb * rcp_nr(P.E);
    *a_bar = -P.dp_coef * tr * nz;
}

// Sums over a particle's stencil, of the tile's node vectors v and (MASS) their
// fourth component m, with d = x_n - x_p:
//   V_a = sum N v_a, W_ab = sum v_a dN/dx_b, S_c = sum dN/dx_c (v . U d),
//   FULL_Y:  Y_a(bc) = sum v_a d2N/dx_b dx_c, (bc) = xx, yy, zz, xy, yz, xz
//            (2D: xx, yy, xy);
//   !FULL_Y: T_c = sum_b d2N/dx_b dx_c (Q v)_b for a symmetric Q known beforehand;
//   ND:      D_ab = sum N v_a d_b;   MASS: G_c = sum m dN/dx_c.
template <int DIM, bool FULL_Y, bool ND, bool MASS>
struct Moments {
    float V[3] = {0, 0, 0}, W[3][3] = {{0}}, S[3] = {0, 0, 0};
    float Y[FULL_Y ? 3 : 1][6] = {{0}}, T[3] = {0, 0, 0};
    float D[ND ? 3 : 1][3] = {{0}}, G[3] = {0, 0, 0};
};

// padded float4 tile in LDS: row and plane strides (as k_g2p's)
constexpr int ADJ_SY = 20;
template <int DIM>
constexpr int adj_sz() { return DIM == 3 ? 120 : 0; }
template <int DIM>
constexpr int adj_tile() { return DIM == 3 ? 6 * 120 : 6 * ADJ_SY; }

template <int DIM, bool FULL_Y, bool ND, bool MASS>
__device__ __forceinline__ void gather_moments(const float4* vt, const int* lb, const float* t, const float* u,
                                               float dx, float inv_dx, const float (*U)[3], const float (*Q)[3],
                                               Moments<DIM, FULL_Y, ND, MASS>& O) {
    float w[3][3], dw[3][3];
    bspline<DIM>(t, u, inv_dx, w, dw);
    const float i2 = inv_dx * inv_dx;
    auto off = [&](int a, int k) { return ((float)k - 0.5f - t[a]) * dx; };
    const float4* base = vt + lb[0] + ADJ_SY * lb[1] + (DIM == 3 ? adj_sz<DIM>() * lb[2] : 0);
    // column a of a matrix with the plane sums of one kind
    auto dot = [](const float (*m)[3], int col, const float* v) {
        float r = m[0][col] * v[0];
#pragma unroll
        for (int a = 1; a < DIM; ++a) r = fmaf(m[a][col], v[a], r);
        return r;
    };
#pragma unroll 1
    for (int kz = 0; kz < (DIM == 3 ? 3 : 1); ++kz) {
        // sums over the plane, factors along x and y: N N, N' N, N N', N'' N,
        // N' N', N N'', (N d) N, N (N d), (N' d) N, N' (N d), (N d) N', N (N' d)
        float A0[3] = {0, 0, 0}, A1[3] = {0, 0, 0}, A2[3] = {0, 0, 0}, A3[3] = {0, 0, 0}, A4[3] = {0, 0, 0},
              A5[3] = {0, 0, 0}, A6[3] = {0, 0, 0}, A7[3] = {0, 0, 0}, A8[3] = {0, 0, 0}, A9[3] = {0, 0, 0},
              Aa[3] = {0, 0, 0}, Ab[3] = {0, 0, 0};
        float B0 = 0, B1 = 0, B2 = 0;
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
            float r0[3] = {0, 0, 0}, r1[3] = {0, 0, 0}, r2[3] = {0, 0, 0}, r3[3] = {0, 0, 0}, r4[3] = {0, 0, 0};
            float m0 = 0, m1 = 0;
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                const float4 g = base[kx + ADJ_SY * ky];
                const float v[3] = {g.x, g.y, g.z};
                const float wx = w[0][kx], dwx = dw[0][kx], ox = off(0, kx), ddx = kx == 1 ? -2.f * i2 : i2;
                const float wdx = wx * ox, dwdx = dwx * ox;
#pragma unroll
                for (int a = 0; a < DIM; ++a) {
                    r0[a] = fmaf(wx, v[a], r0[a]);
                    r1[a] = fmaf(dwx, v[a], r1[a]);
                    r2[a] = fmaf(ddx, v[a], r2[a]);
                    r3[a] = fmaf(wdx, v[a], r3[a]);
                    r4[a] = fmaf(dwdx, v[a], r4[a]);
                }
                if (MASS) {
                    m0 = fmaf(wx, g.w, m0);
                    m1 = fmaf(dwx, g.w, m1);
                }
            }
            const float wy = w[1][ky], dwy = dw[1][ky], oy = off(1, ky), ddy = ky == 1 ? -2.f * i2 : i2;
            const float wyd = wy * oy, dwyd = dwy * oy;
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                A0[a] = fmaf(wy, r0[a], A0[a]);
                A1[a] = fmaf(wy, r1[a], A1[a]);
                A2[a] = fmaf(dwy, r0[a], A2[a]);
                A3[a] = fmaf(wy, r2[a], A3[a]);
                A4[a] = fmaf(dwy, r1[a], A4[a]);
                A5[a] = fmaf(ddy, r0[a], A5[a]);
                A6[a] = fmaf(wy, r3[a], A6[a]);
                A7[a] = fmaf(wyd, r0[a], A7[a]);
                A8[a] = fmaf(wy, r4[a], A8[a]);
                A9[a] = fmaf(wyd, r1[a], A9[a]);
                Aa[a] = fmaf(dwy, r3[a], Aa[a]);
                Ab[a] = fmaf(dwyd, r0[a], Ab[a]);
            }
            if (MASS) {
                B0 = fmaf(wy, m0, B0);
                B1 = fmaf(wy, m1, B1);
                B2 = fmaf(dwy, m0, B2);
            }
            // one row of LDS reads in flight at a time, and the row's sums
            // finished here: left to itself the compiler sinks sums below
            // their last use and keeps all 27 node vectors live
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                asm volatile("" : "+v"(A0[a]), "+v"(A1[a]), "+v"(A2[a]), "+v"(A3[a]), "+v"(A4[a]), "+v"(A5[a]));
                asm volatile("" : "+v"(A6[a]), "+v"(A7[a]), "+v"(A8[a]), "+v"(A9[a]), "+v"(Aa[a]), "+v"(Ab[a]));
            }
            if (MASS) asm volatile("" : "+v"(B0), "+v"(B1), "+v"(B2));
        }
        base += adj_sz<DIM>();
        auto pick = [&](const float* f) { return kz == 0 ? f[0] : kz == 1 ? f[1] : f[2]; };
        const float wz = DIM == 3 ? pick(w[2]) : 1.f, dwz = DIM == 3 ? pick(dw[2]) : 0.f;
        const float oz = DIM == 3 ? off(2, kz) : 0.f, ddz = kz == 1 ? -2.f * i2 : i2;
        const float wzd = wz * oz, dwzd = dwz * oz;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            O.V[a] = fmaf(wz, A0[a], O.V[a]);
            O.W[a][0] = fmaf(wz, A1[a], O.W[a][0]);
            O.W[a][1] = fmaf(wz, A2[a], O.W[a][1]);
            if (DIM == 3) O.W[a][2] = fmaf(dwz, A0[a], O.W[a][2]);
            if (FULL_Y) {
                O.Y[a][0] = fmaf(wz, A3[a], O.Y[a][0]);
                O.Y[a][1] = fmaf(wz, A5[a], O.Y[a][1]);
                O.Y[a][DIM == 3 ? 3 : 2] = fmaf(wz, A4[a], O.Y[a][DIM == 3 ? 3 : 2]);
                if (DIM == 3) {
                    O.Y[a][2] = fmaf(ddz, A0[a], O.Y[a][2]);
                    O.Y[a][4] = fmaf(dwz, A2[a], O.Y[a][4]);
                    O.Y[a][5] = fmaf(dwz, A1[a], O.Y[a][5]);
                }
            }
            if (ND) {
                O.D[a][0] = fmaf(wz, A6[a], O.D[a][0]);
                O.D[a][1] = fmaf(wz, A7[a], O.D[a][1]);
                if (DIM == 3) O.D[a][2] = fmaf(wzd, A0[a], O.D[a][2]);
            }
        }
        O.S[0] = fmaf(wz, dot(U, 0, A8) + dot(U, 1, A9), O.S[0]);
        O.S[1] = fmaf(wz, dot(U, 0, Aa) + dot(U, 1, Ab), O.S[1]);
        if (DIM == 3) {
            O.S[0] = fmaf(wzd, dot(U, 2, A1), O.S[0]);
            O.S[1] = fmaf(wzd, dot(U, 2, A2), O.S[1]);
            O.S[2] = fmaf(dwz, dot(U, 0, A6) + dot(U, 1, A7), fmaf(dwzd, dot(U, 2, A0), O.S[2]));
        }
        if (!FULL_Y) {
            O.T[0] = fmaf(wz, dot(Q, 0, A3) + dot(Q, 1, A4), O.T[0]);
            O.T[1] = fmaf(wz, dot(Q, 0, A4) + dot(Q, 1, A5), O.T[1]);
            if (DIM == 3) {
                O.T[0] = fmaf(dwz, dot(Q, 2, A1), O.T[0]);
                O.T[1] = fmaf(dwz, dot(Q, 2, A2), O.T[1]);
                O.T[2] = fmaf(dwz, dot(Q, 0, A1) + dot(Q, 1, A2), fmaf(ddz, dot(Q, 2, A0), O.T[2]));
            }
        }
        if (MASS) {
            O.G[0] = fmaf(wz, B1, O.G[0]);
            O.G[1] = fmaf(wz, B2, O.G[1]);
            if (DIM == 3) O.G[2] = fmaf(dwz, B0, O.G[2]);
        }
    }
}

struct OutBar {
    const float* x;
    const float* v;
    const float* C;
    const float* F;
    const float* tau;
};

// Work of one workgroup of the per-particle reverse kernels: ADJ_WG positions of
// a work item (an item of up to `chunk` particles is shared by `parts`
// workgroups; small items in flight at once matter more here than the tile
// that each of them stages).
constexpr int ADJ_WG = 128;

// Stages the tile of work item `blk` from a node array into LDS; the origin of
// the block goes to org (every thread).  Ends with a barrier.
template <int DIM>
__device__ __forceinline__ void stage_tile(const DevParams& P, const float4* __restrict__ grid, int blk, float4* vt,
                                           int* org) {
    using T = Tile<DIM>;
    block_coords<DIM>(P, blk, org);
#pragma unroll
    for (int a = 0; a < 3; ++a) org[a] *= BLK;
#pragma unroll
    for (int r = 0; r < (T::N + ADJ_WG - 1) / ADJ_WG; ++r) {
        const int t = (int)threadIdx.x + r * ADJ_WG;
        if (t < T::N) {
            const int I = t % T::E, J = (t / T::E) % T::E, K = DIM == 3 ? t / (T::E * T::E) : 0;
            const int d = (I >> 2) | ((J >> 2) << 1) | ((K >> 2) << 2);
            const int phi = P.b_nbr[(size_t)blk * T::NB + d];
            const int l = (I & 3) + BLK * ((J & 3) + BLK * (K & 3));
            vt[I + ADJ_SY * J + adj_sz<DIM>() * K] =
                phi >= 0 ? grid[(size_t)phi * T::NPB + l] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
    __syncthreads();
}

// F_trial of input particle q with grad v summed node by node (rarely called:
// rolled, and everything is read again).
template <int DIM>
__device__ __forceinline__ void trial_by_nodes(const DevParams& P, const float4* vt, const int* org,
                                               const float* __restrict__ x, const float* __restrict__ F, size_t q,
                                               int n, float (*Ft)[3]) {
    float xp[3] = {0, 0, 0}, tt[3] = {0, 0, 0}, uu[3] = {1, 1, 1}, wt[3][3], dw[3][3], W[3][3] = {{0}};
    int lb[3] = {0, 0, 0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) xp[a] = x[(size_t)a * n + q];
    particle_frame<DIM>(P, xp, org, lb, tt, uu);
    bspline<DIM>(tt, uu, P.inv_dxf, wt, dw);
    const float4* base = vt + lb[0] + ADJ_SY * lb[1] + (DIM == 3 ? adj_sz<DIM>() * lb[2] : 0);
    auto pick = [](const float* f, int k) { return k == 0 ? f[0] : k == 1 ? f[1] : f[2]; };
#pragma unroll 1
    for (int k = 0; k < (DIM == 3 ? 27 : 9); ++k) {  // x fastest
        const int kk[3] = {k % 3, k / 3 % 3, k / 9};
        const float4 g4 = base[kk[0] + ADJ_SY * kk[1] + adj_sz<DIM>() * kk[2]];
        const float v[3] = {g4.x, g4.y, g4.z};
        float w[3] = {1.f, 1.f, 1.f}, d[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            w[a] = pick(wt[a], kk[a]);
            d[a] = pick(dw[a], kk[a]);
        }
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            float g = d[b];
#pragma unroll
            for (int e = 0; e < DIM; ++e)
                if (e != b) g *= w[e];
#pragma unroll
            for (int a = 0; a < DIM; ++a) W[a][b] += v[a] * g;
        }
    }
    float Fp[3][3];
#pragma unroll
    for (int k = 0; k < DIM * DIM; ++k) Fp[k / DIM][k % DIM] = F[(size_t)k * n + q];
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < DIM; ++c) s += W[a][c] * Fp[c][b];
            Ft[a][b] = Fp[a][b] + P.dt * s;
        }
}

// One particle of k_g2p_adj; false where its branch has to be settled by NODES
// (what was written up to there is written again).
template <int DIM, bool NODES>
__device__ __forceinline__ bool g2p_adj_particle(const DevParams& P, const float4* vt, const int* org,
                                                 const float* __restrict__ x, const float* __restrict__ F,
                                                 const OutBar& ob, float* __restrict__ x_bar,
                                                 float* __restrict__ F_bar, int n, int o, size_t q, const float* xp,
                                                 const float (*Bb)[3], float* accE, float* accA) {
    constexpr int NS = DIM == 3 ? 6 : 3;
    constexpr int DD = DIM * DIM;
    const float dt = P.dt, dx = P.dxf, inv_dx = P.inv_dxf;
    int lb[3] = {0, 0, 0};
    float tt[3] = {0, 0, 0}, uu[3] = {1, 1, 1};
    particle_frame<DIM>(P, xp, org, lb, tt, uu);
    Moments<DIM, true, false, false> Mo;
    gather_moments<DIM, true, false, false>(vt, lb, tt, uu, dx, inv_dx, Bb, Bb, Mo);
    __builtin_amdgcn_sched_barrier(0);
    float Fp[3][3], xbo[3] = {0, 0, 0}, vpb[3] = {0, 0, 0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        xbo[a] = ob.x[(size_t)a * n + o];
        vpb[a] = ob.v[(size_t)a * n + o] + dt * xbo[a];
    }
#pragma unroll
    for (int k = 0; k < DD; ++k) Fp[k / DIM][k % DIM] = F[(size_t)k * n + q];
    float* sc = P.adj_scratch;
    float xb[3];
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        // position adjoint through the weights of v_p and B_p
        xb[c] = xbo[c] + Mo.S[c];
#pragma unroll
        for (int a = 0; a < DIM; ++a) xb[c] += Mo.W[a][c] * vpb[a] - Bb[a][c] * Mo.V[a];
        sc[(size_t)c * n + o] = vpb[c];
        sc[(size_t)(DIM + 2 * DD + c) * n + o] = xp[c];
    }
#pragma unroll
    for (int k = 0; k < DD; ++k) sc[(size_t)(DIM + k) * n + o] = Bb[k / DIM][k % DIM];
    float Ft[3][3], Fbo[3][3] = {{0}}, tbo[6] = {0};
    Principal pr;
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            float s2 = 0.f;
#pragma unroll
            for (int c = 0; c < DIM; ++c) s2 += Mo.W[a][c] * Fp[c][b];
            Ft[a][b] = Fp[a][b] + dt * s2;
        }
#pragma unroll
    for (int k = 0; k < DD; ++k) Fbo[k / DIM][k % DIM] = ob.F[(size_t)k * n + o];
#pragma unroll
    for (int k = 0; k < NS; ++k) tbo[k] = ob.tau[(size_t)k * n + o];
    if (NODES) trial_by_nodes<DIM>(P, vt, org, x, F, q, n, Ft);
    if (principal_strains<DIM, NODES>(P, Ft, pr)) return false;
    float Ftb[3][3], eb, ab;
    constitutive_adj<DIM>(P, pr, Ft, Fbo, tbo, Ftb, &eb, &ab);
    *accE += eb;
    *accA += ab;
    // F_trial = (I + dt W) F
    float Wb[3][3];
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            float s1 = Ftb[a][b], s2 = 0.f;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                s1 += dt * Mo.W[c][a] * Ftb[c][b];
                s2 += Ftb[a][c] * Fp[b][c];
            }
            F_bar[(size_t)(a * DIM + b) * n + q] = s1;
            Wb[a][b] = dt * s2;
            sc[(size_t)(DIM + DD + a * DIM + b) * n + o] = Wb[a][b];
        }
    // and through the weights of grad v
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        if (DIM == 3) {
            xb[0] += Wb[a][0] * Mo.Y[a][0] + Wb[a][1] * Mo.Y[a][3] + Wb[a][2] * Mo.Y[a][5];
            xb[1] += Wb[a][0] * Mo.Y[a][3] + Wb[a][1] * Mo.Y[a][1] + Wb[a][2] * Mo.Y[a][4];
            xb[2] += Wb[a][0] * Mo.Y[a][5] + Wb[a][1] * Mo.Y[a][4] + Wb[a][2] * Mo.Y[a][2];
        } else {
            xb[0] += Wb[a][0] * Mo.Y[a][0] + Wb[a][1] * Mo.Y[a][2];
            xb[1] += Wb[a][0] * Mo.Y[a][2] + Wb[a][1] * Mo.Y[a][1];
        }
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c) x_bar[(size_t)c * n + q] = xb[c];
    return true;
}

// osrc[o]: the input particle that G2P stores at position o.  A work item's
// range of positions holds particles of its block whichever way the block's
// particles are listed, so the item's part is walked in output order: the
// output adjoints and the scratch are read and written contiguously.
// Bound by its arithmetic and registers (about 3000 instructions a particle at
// three waves per SIMD, for which it spills 24 bytes a lane; its bytes take 16
// us): 262,144 particles of loaded material in 48 us, 109 before (27 nodes times
// all Hessian factors, 283 registers, one wave per SIMD).
template <int DIM>
__global__ __launch_bounds__(ADJ_WG, 3) void k_g2p_adj(DevParams P, const float* __restrict__ x,
                                                    const float* __restrict__ F, OutBar ob, float* __restrict__ x_bar,
                                                    float* __restrict__ F_bar, int n, const uint32_t* __restrict__ osrc,
                                                    int parts) {
    constexpr int DD = DIM * DIM;
    __shared__ float4 vt[adj_tile<DIM>()];
    __shared__ float red[2][ADJ_WG / 64];
    const int n_work = min(P.ctr->n_work, P.work_cap) * parts;
    const float bscale = 4.f * P.inv_dxf * P.inv_dxf;
    float accE = 0.f, accA = 0.f;
    for (int w = blockIdx.x; w < n_work; w += gridDim.x) {
        const int it = w / parts;
        const int s = P.w_start[it] + (w % parts) * ADJ_WG, e = min(P.w_end[it], s + ADJ_WG);
        if (s >= e) continue;
        const int o = s + (int)threadIdx.x;
        // what the gather needs is loaded before the tile's barrier, the rest
        // after it (registers: three waves per SIMD)
        const int oc = min(o, e - 1);
        const size_t q = osrc[oc];
        float xp[3] = {0, 0, 0}, Bb[3][3] = {{0}};
#pragma unroll
        for (int a = 0; a < DIM; ++a) xp[a] = x[(size_t)a * n + q];
#pragma unroll
        for (int k = 0; k < DD; ++k) Bb[k / DIM][k % DIM] = ob.C[(size_t)k * n + oc];
        int org[3];
        stage_tile<DIM>(P, P.grid, P.w_block[it], vt, org);
        if (o < e) {
#pragma unroll
            for (int k = 0; k < DD; ++k) Bb[k / DIM][k % DIM] *= bscale;
            bool sure = g2p_adj_particle<DIM, false>(P, vt, org, x, F, ob, x_bar, F_bar, n, o, q, xp, Bb, &accE, &accA);
            if (!sure) {
                int o2 = o;
                asm volatile("" : "+v"(o2));  // nothing of the first attempt is kept for the second
                const size_t q2 = osrc[o2];
#pragma unroll
                for (int a = 0; a < DIM; ++a) xp[a] = x[(size_t)a * n + q2];
#pragma unroll
                for (int k = 0; k < DD; ++k) Bb[k / DIM][k % DIM] = bscale * ob.C[(size_t)k * n + o2];
                g2p_adj_particle<DIM, true>(P, vt, org, x, F, ob, x_bar, F_bar, n, o2, q2, xp, Bb, &accE, &accA);
            }
        }
        __syncthreads();
    }
    // parameter gradients: one partial sum per workgroup, added up by the
    // scatter that follows (adds to one address from many workgroups are
    // served one after another, 15 ns each)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        accE += __shfl_xor(accE, o);
        accA += __shfl_xor(accA, o);
    }
    if (__lane_id() == 0) {
        red[0][threadIdx.x >> 6] = accE;
        red[1][threadIdx.x >> 6] = accA;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float se = 0.f, sa = 0.f;
#pragma unroll
        for (int k = 0; k < ADJ_WG / 64; ++k) {
            se += red[0][k];
            sa += red[1][k];
        }
        P.adj_part[2 * blockIdx.x] = se;
        P.adj_part[2 * blockIdx.x + 1] = sa;
    }
}

// v_bar_n = sum_p N v'_bar + N B_bar (x_n - x_p) + W_bar grad N, organised like
// the forward P2G: a workgroup per owner block, a lane per base cell, register
// sums merged into an LDS tile offset by offset.  The workgroup's 64 NW / 4^d
// groups of 4^d lanes take the particles of a cell in turns, each group with a
// tile of its own, summed when the tiles are stored.  A block's walk is a
// serial chain of as many rounds as its fullest cell has particles for each
// group; several waves per block shorten it where the blocks leave SIMDs idle
// (launch_scatter_adj has the line).  Cells are read in G2P's output order, in
// which consecutive lanes hold consecutive addresses.
// The first workgroup also adds up the parameter gradients' partial sums.
// 262,144 particles: 19 us, with the clearing of a grid and atomics 45.
template <int DIM, int NW>
__global__ __launch_bounds__(64 * NW) void k_scatter_adj(DevParams P, int n, const uint32_t* __restrict__ skeys,
                                                         int n_part, int parts) {
    using T = Tile<DIM>;
    constexpr int NC = T::NPB;
    constexpr int NK = DIM == 3 ? 27 : 9;
    constexpr int DD = DIM * DIM;
    constexpr int TH = 64 * NW, SPL = TH / NC;
    __shared__ float tile[SPL][3][T::NP];
    __shared__ Interleave<DIM> il;
    const int lane = threadIdx.x, cell = lane % NC, grp = lane / NC;
    const int nb = min(P.ctr->nb, P.block_cap);
    const float dx = P.dxf, inv_dx = P.inv_dxf;
    const float* sc = P.adj_scratch;
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        n_part = min(n_part, min(P.ctr->n_work, P.work_cap) * parts);  // the rest had no item
        double se = 0.0, sa = 0.0;
        for (int i = threadIdx.x; i < n_part; i += 64) {
            se += (double)P.adj_part[2 * i];
            sa += (double)P.adj_part[2 * i + 1];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            se += __shfl_xor(se, o);
            sa += __shfl_xor(sa, o);
        }
        if (threadIdx.x == 0) {
            // (the accumulator is the caller's: several contexts may add to one)
            atomicAdd(&P.param_bar[0], (float)se);
            atomicAdd(&P.param_bar[1], (float)(sa * (double)P.dalpha_dphi));
        }
    }
    for (int b = blockIdx.x; b < nb; b += gridDim.x) {
        const int cnt = P.b_count[b], st = P.b_start[b];
        if (cnt <= 0) continue;
        for (int t = lane; t < SPL * 3 * T::NP; t += TH) (&tile[0][0][0])[t] = 0.f;
        int bc[3];
        block_coords<DIM>(P, b, bc);
        const int lb[3] = {cell & 3, (cell >> 2) & 3, DIM == 3 ? (cell >> 4) & 3 : 0};
        const double base[3] = {(double)(bc[0] * BLK + lb[0]), (double)(bc[1] * BLK + lb[1]),
                                (double)(bc[2] * BLK + lb[2])};
        interleave_setup<DIM>(il, skeys, st, st + cnt);
        float acc[NK][3];
#pragma unroll
        for (int k = 0; k < NK; ++k) acc[k][0] = acc[k][1] = acc[k][2] = 0.f;
        const int nj = il.ce[cell] - il.cs[cell];
        const bool has = nj > grp;
        struct Part {
            float x[3], v[3], A[9], W[9];
        };
        auto load_into = [&](Part& p, int j) {
            const size_t o = (size_t)interleave_pos_cj<DIM>(il, cell, j);
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                p.v[a] = sc[(size_t)a * n + o];
                p.x[a] = sc[(size_t)(DIM + 2 * DD + a) * n + o];
            }
#pragma unroll
            for (int k = 0; k < DD; ++k) {
                p.A[k] = sc[(size_t)(DIM + k) * n + o];
                p.W[k] = sc[(size_t)(DIM + DD + k) * n + o];
            }
        };
        auto process = [&](const Part& p) {
            float t[3] = {0, 0, 0}, u[3] = {1, 1, 1};
            particle_frame_at<DIM>(P, p.x, base, t, u);
            float wt[3][3], dw[3][3], dxn[3][3];
            bspline<DIM>(t, u, inv_dx, wt, dw);
#pragma unroll
            for (int a = 0; a < DIM; ++a)
#pragma unroll
                for (int k = 0; k < 3; ++k) dxn[a][k] = ((float)k - 0.5f - t[a]) * dx;
            // the P2G's factorisation: w_x b(ky, kz) + (w_z w_y) h(kx)
            float h[3][3];
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                for (int q = 0; q < DIM; ++q)
                    h[kx][q] = wt[0][kx] * dxn[0][kx] * p.A[q * DIM] + dw[0][kx] * p.W[q * DIM];
            if (DIM == 3) {
                float Z[3][3];
#pragma unroll
                for (int kz = 0; kz < 3; ++kz)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        Z[kz][q] = wt[2][kz] * dxn[2][kz] * p.A[q * DIM + 2] + dw[2][kz] * p.W[q * DIM + 2];
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) {
                    const float wy = wt[1][ky];
                    float Y[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        Y[q] = wy * (p.v[q] + p.A[q * DIM + 1] * dxn[1][ky]) + p.W[q * DIM + 1] * dw[1][ky];
#pragma unroll
                    for (int kz = 0; kz < 3; ++kz) {
                        const float wz = wt[2][kz], wzy = wz * wy;
                        float be[3];
#pragma unroll
                        for (int q = 0; q < 3; ++q) be[q] = wz * Y[q] + wy * Z[kz][q];
#pragma unroll
                        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                            for (int q = 0; q < 3; ++q) {
                                float& a = acc[kx + 3 * (ky + 3 * kz)][q];
                                a = fmaf(wt[0][kx], be[q], fmaf(wzy, h[kx][q], a));
                            }
                    }
                }
            } else {
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) {
                    const float wy = wt[1][ky];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const float Y = wy * (p.v[q] + p.A[q * DIM + 1] * dxn[1][ky]) + p.W[q * DIM + 1] * dw[1][ky];
#pragma unroll
                        for (int kx = 0; kx < 3; ++kx) {
                            float& a = acc[kx + 3 * ky][q];
                            a = fmaf(wt[0][kx], Y, fmaf(wy, h[kx][q], a));
                        }
                    }
                }
            }
        };
        // two register sets take turns: the loads of the next particle are in
        // flight while the current one is accumulated (as in P2G)
        Part pa, pb;
        if (has) load_into(pa, grp);
        for (int j = grp; j < nj; j += 2 * SPL) {
            load_into(pb, min(j + SPL, nj - 1));
            process(pa);
            load_into(pa, min(j + 2 * SPL, nj - 1));
            if (j + SPL < nj) process(pb);
        }
        // merge into the group's tile: for a fixed offset distinct cells
        // address distinct nodes; a group's cells are all in one wave, whose
        // LDS accesses are served in the order they are issued
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            const int kx = k % 3, ky = (k / 3) % 3, kz = DIM == 3 ? k / 9 : 0;
            const int idx = T::pad(lb[0] + kx, lb[1] + ky, DIM == 3 ? lb[2] + kz : 0);
            if (has) {
#pragma unroll
                for (int a = 0; a < DIM; ++a) tile[grp][a][idx] += acc[k][a];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        for (int t = lane; t < T::N; t += TH) {
            int I, J, K;
            T::store_node(t, &I, &J, &K);
            const int tp = T::pad(I, J, K);
            float g[3] = {0, 0, 0};
#pragma unroll
            for (int r = 0; r < SPL; ++r)
#pragma unroll
                for (int a = 0; a < DIM; ++a) g[a] += tile[r][a][tp];
            if (!P.dense) {
                P.tiles[(size_t)b * T::N + t] = make_float4(g[0], g[1], g[2], 0.f);
            } else if (g[0] != 0.f || g[1] != 0.f || g[2] != 0.f) {
                const int d = (I >> 2) | ((J >> 2) << 1) | ((K >> 2) << 2);
                const int phi = P.b_nbr[(size_t)b * T::NB + d];
                if (phi >= 0) {
                    const int l = (I & 3) + BLK * ((J & 3) + BLK * (K & 3));
                    float* o = reinterpret_cast<float*>(&P.grid_bar[(size_t)phi * T::NPB + l]);
                    atomicAdd(o + 0, g[0]);
                    atomicAdd(o + 1, g[1]);
                    if (DIM == 3) atomicAdd(o + 2, g[2]);
                }
            }
        }
        __syncthreads();
    }
}

// Adjoint of one node's update: gb = v_bar, gu = (u, m) from the forward pass;
// returns (p_bar, m_bar).
template <int DIM>
__device__ __forceinline__ float4 node_adj(const DevParams& P, const int* node, float4 gb, float4 gu) {
    const float m = gu.w;
    if (!(m > 0.f)) return make_float4(0.f, 0.f, 0.f, 0.f);
    float ub[3] = {gb.x, gb.y, gb.z};
    const float u[3] = {gu.x, gu.y, gu.z};
    // Jacobian of the wall projections (diagonal 0/1), applied to the adjoint
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const bool on = side == 0 ? node[a] < P.bound : node[a] > P.cells[a] - P.bound;
            if (!on) continue;
            const int kind = P.bc[a][side];
            if (kind == MPM_BC_STICKY) {
                ub[0] = ub[1] = ub[2] = 0.f;
            } else if (kind == MPM_BC_SLIP) {
                ub[a] = 0.f;
            } else if (kind == MPM_BC_SEPARATE) {
                if (side == 0 ? u[a] < 0.f : u[a] > 0.f) ub[a] = 0.f;
            }
        }
    }
    const float inv = 1.f / m;
    float mb = 0.f;
#pragma unroll
    for (int a = 0; a < DIM; ++a) mb -= ub[a] * (u[a] - P.dt * P.g[a]);
    return make_float4(ub[0] * inv, ub[1] * inv, DIM == 3 ? ub[2] * inv : 0.f, mb * inv);
}

// Sparse grids: the sum of the tiles that cover each node (k_p2g_gather's
// pattern, one wave per block), then the node's adjoint: 6.1 us for 262,144 particles
// (the adjoint alone, from a grid summed by atomics, took 4.8).
template <int DIM>
__global__ __launch_bounds__(WG) void k_gather_adj(DevParams P) {
    using T = Tile<DIM>;
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    const int nb = min(P.ctr->nb, P.block_cap);
    const int I = lane & 3, J = (lane >> 2) & 3, K = DIM == 3 ? (lane >> 4) & 3 : 0;
    for (int b = blockIdx.x * (WG / 64) + w; b < nb; b += gridDim.x * (WG / 64)) {
        int src[T::NB];
#pragma unroll
        for (int d = 0; d < T::NB; ++d) src[d] = P.b_lo[(size_t)b * T::NB + d];
        int bc[3];
        block_coords<DIM>(P, b, bc);
        const size_t s = (size_t)b * T::NPB + lane;
        const float4 gu = lane < T::NPB ? P.grid_u[s] : make_float4(0.f, 0.f, 0.f, 0.f);
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int d = 0; d < T::NB; ++d) {
            const int ex = d & 1, ey = (d >> 1) & 1, ez = (d >> 2) & 1;
            const bool reach = (!ex || I < 2) && (!ey || J < 2) && (DIM == 2 || !ez || K < 2);
            if (src[d] >= 0 && reach && lane < T::NPB) {
                const float4 g = P.tiles[(size_t)src[d] * T::N + T::store_index(I + 4 * ex, J + 4 * ey, K + 4 * ez)];
                sum.x += g.x;
                sum.y += g.y;
                sum.z += g.z;
            }
        }
        const int node[3] = {bc[0] * BLK + I, bc[1] * BLK + J, DIM == 3 ? bc[2] * BLK + K : 0};
        if (lane < T::NPB) P.grid_bar[s] = node_adj<DIM>(P, node, sum, gu);
    }
}

// Dense grids: the node's adjoint in place, after the scatter's atomics.
template <int DIM>
__global__ __launch_bounds__(WG) void k_grid_adj(DevParams P, long long n_nodes) {
    constexpr int NPB = Tile<DIM>::NPB;
    for (long long s = (long long)blockIdx.x * WG + threadIdx.x; s < n_nodes; s += (long long)gridDim.x * WG) {
        const int b = (int)(s / NPB), l = (int)(s % NPB);
        int bc[3];
        block_coords<DIM>(P, b, bc);
        const int node[3] = {bc[0] * BLK + (l & 3), bc[1] * BLK + ((l >> 2) & 3),
                             DIM == 3 ? bc[2] * BLK + (l >> 4) : 0};
        P.grid_bar[s] = node_adj<DIM>(P, node, P.grid_bar[s], P.grid_u[s]);
    }
}

struct PIn {
    const float* x;
    const float* v;
    const float* C;
    const float* tau;
};
struct PBar {
    float* x;
    float* v;
    float* C;
    float* tau;
};

// Input adjoints of P2G, a particle per lane in output order.  Bound like
// k_g2p_adj: 262,144 particles in 27 us, 44 before (node by node).
template <int DIM>
__global__ __launch_bounds__(ADJ_WG, 3) void k_p2g_adj(DevParams P, PIn in, PBar bar, int n,
                                                    const uint32_t* __restrict__ osrc, int parts) {
    constexpr int DD = DIM * DIM;
    constexpr int NS = DIM == 3 ? 6 : 3;
    __shared__ float4 vt[adj_tile<DIM>()];
    const int n_work = min(P.ctr->n_work, P.work_cap) * parts;
    const float mp = P.p_mass, dtv = P.dt * P.p_vol0;
    for (int w = blockIdx.x; w < n_work; w += gridDim.x) {
        const int it = w / parts;
        const int s = P.w_start[it] + (w % parts) * ADJ_WG, e = min(P.w_end[it], s + ADJ_WG);
        if (s >= e) continue;
        const int o = s + (int)threadIdx.x;
        // what the gather needs is loaded before the tile's barrier, the rest
        // after it (registers: three waves per SIMD)
        const size_t q = osrc[min(o, e - 1)];
        float xp[3] = {0, 0, 0}, C[3][3] = {{0}}, tc[NS];
#pragma unroll
        for (int a = 0; a < DIM; ++a) xp[a] = in.x[(size_t)a * n + q];
#pragma unroll
        for (int k = 0; k < DD; ++k) C[k / DIM][k % DIM] = in.C[(size_t)k * n + q];
#pragma unroll
        for (int k = 0; k < NS; ++k) tc[k] = in.tau[(size_t)k * n + q];
        int org[3];
        stage_tile<DIM>(P, P.grid_bar, P.w_block[it], vt, org);
        if (o < e) {
            float tau[3][3] = {{0}};
            if (DIM == 3) {
                tau[0][0] = tc[0];
                tau[1][1] = tc[1];
                tau[2][2] = tc[2];
                tau[0][1] = tau[1][0] = tc[3];
                tau[1][2] = tau[2][1] = tc[4];
                tau[0][2] = tau[2][0] = tc[5];
            } else {
                tau[0][0] = tc[0];
                tau[1][1] = tc[1];
                tau[0][1] = tau[1][0] = tc[2];
            }
            int lb[3] = {0, 0, 0};
            float tt[3] = {0, 0, 0}, uu[3] = {1, 1, 1};
            particle_frame<DIM>(P, xp, org, lb, tt, uu);
            Moments<DIM, false, true, true> Mo;
            gather_moments<DIM, false, true, true>(vt, lb, tt, uu, P.dxf, P.inv_dxf, C, tau, Mo);
            __builtin_amdgcn_sched_barrier(0);
            float vp[3] = {0, 0, 0}, xb[3] = {0, 0, 0};
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                vp[a] = in.v[(size_t)a * n + q];
                xb[a] = bar.x[(size_t)a * n + q];
            }
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                float g = Mo.G[c] + Mo.S[c];
#pragma unroll
                for (int a = 0; a < DIM; ++a) g += Mo.W[a][c] * vp[a] - C[a][c] * Mo.V[a];
                bar.x[(size_t)c * n + q] = xb[c] + (mp * g - dtv * Mo.T[c]);
                bar.v[(size_t)c * n + q] = mp * Mo.V[c];
            }
#pragma unroll
            for (int k = 0; k < DD; ++k) bar.C[(size_t)k * n + q] = mp * Mo.D[k / DIM][k % DIM];
            if (DIM == 3) {
                bar.tau[q] = -dtv * Mo.W[0][0];
                bar.tau[(size_t)n + q] = -dtv * Mo.W[1][1];
                bar.tau[2 * (size_t)n + q] = -dtv * Mo.W[2][2];
                bar.tau[3 * (size_t)n + q] = -dtv * (Mo.W[0][1] + Mo.W[1][0]);
                bar.tau[4 * (size_t)n + q] = -dtv * (Mo.W[1][2] + Mo.W[2][1]);
                bar.tau[5 * (size_t)n + q] = -dtv * (Mo.W[0][2] + Mo.W[2][0]);
            } else {
                bar.tau[q] = -dtv * Mo.W[0][0];
                bar.tau[(size_t)n + q] = -dtv * Mo.W[1][1];
                bar.tau[2 * (size_t)n + q] = -dtv * (Mo.W[0][1] + Mo.W[1][0]);
            }
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(WG) void k_grid_bar_clear(DevParams P, long long n_nodes) {
    for (long long s = (long long)blockIdx.x * WG + threadIdx.x; s < n_nodes; s += (long long)gridDim.x * WG)
        P.grid_bar[s] = make_float4(0.f, 0.f, 0.f, 0.f);
}

namespace {
// Workgroups of the per-particle kernels and parts per work item.
int adj_parts(const DevParams& P) { return (P.chunk + ADJ_WG - 1) / ADJ_WG; }
int adj_grid(const DevParams& P) { return (int)std::min<long long>((long long)P.work_cap * adj_parts(P), ADJ_MAX_WGS); }
}  // namespace

hipError_t launch_g2p_adj(const DevParams& P, const float* x, const float* F, const float* const* out_bar, float* x_bar,
                          float* F_bar, int n, const uint32_t* osrc, hipStream_t s) {
    OutBar ob{out_bar[0], out_bar[1], out_bar[2], out_bar[3], out_bar[4]};
    const auto k = P.dim == 3 ? k_g2p_adj<3> : k_g2p_adj<2>;
    k<<<adj_grid(P), ADJ_WG, 0, s>>>(P, x, F, ob, x_bar, F_bar, n, osrc, adj_parts(P));
    return hipGetLastError();
}

hipError_t launch_scatter_adj(const DevParams& P, int n, const uint32_t* skeys, int grid_blocks, hipStream_t s) {
    if (P.dense) {
        const long long nodes = (long long)P.block_cap * (P.dim == 3 ? 64 : 16);
        k_grid_bar_clear<<<(int)std::min<long long>((nodes + WG - 1) / WG, 65536), WG, 0, s>>>(P, nodes);
    }
    const int g = P.dense ? 65536 : grid_blocks * 4, np = adj_grid(P);
    // as many waves per block as keep every block's waves resident at once (two
    // per SIMD; 262,144 particles fill about 730 blocks)
    if (P.dim == 2)
        k_scatter_adj<2, 1><<<g, 64, 0, s>>>(P, n, skeys, np, adj_parts(P));
    else if (n <= (1 << 16))
        k_scatter_adj<3, 4><<<g, 256, 0, s>>>(P, n, skeys, np, adj_parts(P));
    else if (n <= (1 << 18))
        k_scatter_adj<3, 2><<<g, 128, 0, s>>>(P, n, skeys, np, adj_parts(P));
    else
        k_scatter_adj<3, 1><<<g, 64, 0, s>>>(P, n, skeys, np, adj_parts(P));
    return hipGetLastError();
}

hipError_t launch_grid_adj(const DevParams& P, hipStream_t s) {
    if (P.dense) {
        const long long nodes = (long long)P.block_cap * (P.dim == 3 ? 64 : 16);
        const auto k = P.dim == 3 ? k_grid_adj<3> : k_grid_adj<2>;
        k<<<(int)std::min<long long>((nodes + WG - 1) / WG, 65536), WG, 0, s>>>(P, nodes);
    } else {
        const auto k = P.dim == 3 ? k_gather_adj<3> : k_gather_adj<2>;
        k<<<(int)std::min<long long>(((long long)P.block_cap + 3) / 4, 16384), WG, 0, s>>>(P);
    }
    return hipGetLastError();
}

hipError_t launch_p2g_adj(const DevParams& P, const float* const* in, float* const* in_bar, int n,
                          const uint32_t* osrc, hipStream_t s) {
    PIn pin{in[0], in[1], in[2], in[3]};
    PBar pb{in_bar[0], in_bar[1], in_bar[2], in_bar[3]};
    const auto k = P.dim == 3 ? k_p2g_adj<3> : k_p2g_adj<2>;
    k<<<adj_grid(P), ADJ_WG, 0, s>>>(P, pin, pb, n, osrc, adj_parts(P));
    return hipGetLastError();
}

}  // namespace mpmx
