// Per-cell element arithmetic of the matrix-free operator (paper eq. (2.3)).
//
// A lattice cell holds 6 Kuhn simplices.  Given the 8 corner values U[k][c]
// (corner k = dx + 2 dy + 4 dz, component c) these routines add each simplex's
// contribution A_e u_e to the corner accumulators F[k][c].
//
// Scalar (-div nu grad u): the unit element matrix is (h/6) times the path
// Laplacian, so simplex s with path corners k0..k3 contributes the fluxes
// g_j = w (U[k_j] - U[k_{j-1}]), w = nu_e h / 6:  F[k_{j-1}] -= g_j, F[k_j] += g_j.
//
// Vector (-div 2 nu eps(u)): with path differences d_j = U[k_j] - U[k_{j-1}]
// (j = 1..3) the displacement gradient in the simplex's axis frame is
// G[i][j] = d_j[a_i] / h.  The stress 2 nu eps = nu (G + G^T) tested against the
// barycentric gradients g0 = -e_a1, g1 = e_a1 - e_a2, ... gives the same flux
// structure, now with vector fluxes q_j[a_i] = w (d_j[a_i] + d_i[a_j]).
//
// Compiled for the device and, in tests, for the host.
#pragma once

#include "kuhn.h"

#if defined(__HIPCC__)
#define AGCA_HD __host__ __device__ __forceinline__
#else
#include <cmath>
#define AGCA_HD inline
using std::fma;
#endif

namespace agca {

template <int S, int NC, typename T>
AGCA_HD void tet_dca(const T (&U)[8][NC], T w, T (&F)[8][NC]) {
    constexpr int a1 = axis1(S), a2 = axis2(S), a3 = axis3(S);
    constexpr int k0 = 0, k1 = 1 << a1, k2 = (1 << a1) | (1 << a2), k3 = 7;
    if constexpr (NC == 1) {
        const T d1 = U[k1][0] - U[k0][0];
        const T d2 = U[k2][0] - U[k1][0];
        const T d3 = U[k3][0] - U[k2][0];
        F[k0][0] = fma(-w, d1, F[k0][0]);
        F[k1][0] = fma(w, d1 - d2, F[k1][0]);
        F[k2][0] = fma(w, d2 - d3, F[k2][0]);
        F[k3][0] = fma(w, d3, F[k3][0]);
    } else {
        constexpr int A[3] = {a1, a2, a3};
        T d[3][3];  // d[j][c]
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            d[0][c] = U[k1][c] - U[k0][c];
            d[1][c] = U[k2][c] - U[k1][c];
            d[2][c] = U[k3][c] - U[k2][c];
        }
        // symmetric s[i][j] = d_j[a_i] + d_i[a_j]; the flux of path step j in component a_i
        // is w s[i][j]
        T sm[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) sm[i][i] = d[i][A[i]] + d[i][A[i]];
        sm[0][1] = sm[1][0] = d[1][A[0]] + d[0][A[1]];
        sm[0][2] = sm[2][0] = d[2][A[0]] + d[0][A[2]];
        sm[1][2] = sm[2][1] = d[2][A[1]] + d[1][A[2]];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int c = A[i];
            F[k0][c] = fma(-w, sm[i][0], F[k0][c]);
            F[k1][c] = fma(w, sm[i][0] - sm[i][1], F[k1][c]);
            F[k2][c] = fma(w, sm[i][1] - sm[i][2], F[k2][c]);
            F[k3][c] = fma(w, sm[i][2], F[k3][c]);
        }
    }
}

// all six simplices of a cell with coefficients w[s] (already multiplied by h/6)
template <int NC, typename T>
AGCA_HD void cell_dca(const T (&U)[8][NC], const T (&w)[6], T (&F)[8][NC]) {
    tet_dca<0, NC, T>(U, w[0], F);
    tet_dca<1, NC, T>(U, w[1], F);
    tet_dca<2, NC, T>(U, w[2], F);
    tet_dca<3, NC, T>(U, w[3], F);
    tet_dca<4, NC, T>(U, w[4], F);
    tet_dca<5, NC, T>(U, w[5], F);
}

// Fluxes of simplex S (vector form) on its three path steps: added to f (the cell edge from
// corner 0) and l (the cell edge into corner 7), which two simplices share (NF / NL: this
// one is the first of them), and stored to m (its middle edge, its own).  Each off-diagonal
// product w s[i][j] serves both steps it belongs to.
template <int S, bool NF, bool NL, typename T>
AGCA_HD void tet_flux(const T (&U)[8][3], T w, T (&f)[3], T (&m)[3], T (&l)[3]) {
    constexpr int a1 = axis1(S), a2 = axis2(S), a3 = axis3(S);
    constexpr int k1 = 1 << a1, k2 = (1 << a1) | (1 << a2);
    T d1[3], d2[3], d3[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        d1[c] = U[k1][c] - U[0][c];
        d2[c] = U[k2][c] - U[k1][c];
        d3[c] = U[7][c] - U[k2][c];
    }
    const T w2 = w + w;
    const T t12 = w * (d2[a1] + d1[a2]), t13 = w * (d3[a1] + d1[a3]), t23 = w * (d3[a2] + d2[a3]);
    m[a1] = t12;
    m[a2] = w2 * d2[a2];
    m[a3] = t23;
    f[a1] = NF ? w2 * d1[a1] : fma(w2, d1[a1], f[a1]);
    f[a2] = NF ? t12 : f[a2] + t12;
    f[a3] = NF ? t13 : f[a3] + t13;
    l[a1] = NL ? t13 : l[a1] + t13;
    l[a2] = NL ? t23 : l[a2] + t23;
    l[a3] = NL ? w2 * d3[a3] : fma(w2, d3[a3], l[a3]);
}

// The same contributions, F overwritten, with the vector form's fluxes summed on the 12 cell
// edges first (the edges at corners 0 and 7 belong to two simplices each, consecutive in
// the order below); every corner then takes its three edges' sums: 156 additions and
// products against cell_dca's 180.
template <int NC, typename T>
AGCA_HD void cell_flux(const T (&U)[8][NC], const T (&w)[6], T (&F)[8][NC]) {
    if constexpr (NC == 1) {
#pragma unroll
        for (int k = 0; k < 8; ++k) F[k][0] = T(0);
        cell_dca<NC, T>(U, w, F);
    } else {
        T fx[3], fy[3], fz[3], lx[3], ly[3], lz[3];
        T mxy[3], mxz[3], myx[3], myz[3], mzx[3], mzy[3];
        tet_flux<0, true, true>(U, w[0], fx, mxy, lz);
        tet_flux<1, false, true>(U, w[1], fx, mxz, ly);
        tet_flux<4, true, false>(U, w[4], fz, mzx, ly);
        tet_flux<5, false, true>(U, w[5], fz, mzy, lx);
        tet_flux<3, true, false>(U, w[3], fy, myz, lx);
        tet_flux<2, false, false>(U, w[2], fy, myx, lz);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            F[0][c] = -fx[c] - fy[c] - fz[c];
            F[1][c] = fx[c] - mxy[c] - mxz[c];
            F[2][c] = fy[c] - myx[c] - myz[c];
            F[4][c] = fz[c] - mzx[c] - mzy[c];
            F[3][c] = mxy[c] + myx[c] - lz[c];
            F[5][c] = mxz[c] + mzx[c] - ly[c];
            F[6][c] = myz[c] + mzy[c] - lx[c];
            F[7][c] = lx[c] + ly[c] + lz[c];
        }
    }
}

}  // namespace agca

namespace agca {

// Element energy form u_e^T K_e w_e of the unit-coefficient element matrix (without h/6):
// scalar: sum_j du_j dw_j; vector: sum_ij (G_u[i][j] + G_u[j][i]) G_w[i][j].
template <int S, int NC, typename T>
AGCA_HD T tet_energy(const T (&U)[8][NC], const T (&W)[8][NC]) {
    constexpr int a1 = axis1(S), a2 = axis2(S);
    constexpr int k[4] = {0, 1 << a1, (1 << a1) | (1 << a2), 7};
    if constexpr (NC == 1) {
        T acc = T(0);
#pragma unroll
        for (int j = 1; j < 4; ++j) acc += (U[k[j]][0] - U[k[j - 1]][0]) * (W[k[j]][0] - W[k[j - 1]][0]);
        return acc;
    } else {
        constexpr int A[3] = {axis1(S), axis2(S), axis3(S)};
        T du[3][3], dw[3][3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                du[j][c] = U[k[j + 1]][c] - U[k[j]][c];
                dw[j][c] = W[k[j + 1]][c] - W[k[j]][c];
            }
        T acc = T(0);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) acc += (du[j][A[i]] + du[i][A[j]]) * dw[j][A[i]];
        return acc;
    }
}

template <int NC, typename T>
AGCA_HD void cell_energy(const T (&U)[8][NC], const T (&W)[8][NC], T (&e)[6]) {
    e[0] = tet_energy<0, NC, T>(U, W);
    e[1] = tet_energy<1, NC, T>(U, W);
    e[2] = tet_energy<2, NC, T>(U, W);
    e[3] = tet_energy<3, NC, T>(U, W);
    e[4] = tet_energy<4, NC, T>(U, W);
    e[5] = tet_energy<5, NC, T>(U, W);
}

}  // namespace agca
