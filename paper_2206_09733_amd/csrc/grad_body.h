// grad_body.h -- Navier-Stokes pass A for one element (the body of grad_kernel and its batched entry).
#pragma once

#include <hip/hip_runtime.h>

#include "dg_device.h"

namespace dg {

// On the six faces, the contravariant viscous flux along the face normal direction of the face
// viscous flux scheme: Fvf[e][2d+side][c][face node] (BR1: from the lifted gradient of (v, T);
// BR2 and interior penalty: see face_viscous_br2_ip).  The stage kernel averages the two sides.
// XV: the BR2 / interior-penalty face fluxes (compiled apart, the BR1 kernels keep their registers).
// CART: plain boxes, whose metric terms are constants (BR1 reads none).  EW elements per workgroup,
// (NT lanes) starting at e0 = EW wg; the last workgroup repeats the last element in its spare places.
template <int N, typename T, bool XV, int EW>
struct GradLds {
  static constexpr int n = N + 1;
  double D[n * n];
  T G[4][EW * n * n * n];                   // g = (v, T)
  T J[EW * 6][4][n * n];                    // half jumps of g on the faces
  T Fb[XV ? EW * 6 : 1][4][XV ? n * n : 1];  // broken-gradient face fluxes
};

template <int N, typename T, bool XV, bool CART, int EW, int NT, typename VW>
__device__ __forceinline__ void grad_body(GradLds<N, T, XV, EW>& lds, const VW& v, const int wg, const int cur) {
  constexpr int n = N + 1, nn = n * n * n, nf = n * n, NN = EW * nn;
  constexpr int NFP = EW * 6 * nf;
  const int t = threadIdx.x;
  const bool act = t < NN;
  const int el = EW > 1 ? (act ? t / nn : 0) : 0;
  const int tl = EW > 1 ? t - el * nn : t;
  const int ti = tl % n, tj = (tl / n) % n, tk = tl / nf;
  const int e0 = wg * EW;
  auto elem_of = [&](int k) { return EW > 1 ? (e0 + k < v.E ? e0 + k : v.E - 1) : e0; };
  const int e = elem_of(el);
  const bool put = act && (EW == 1 || e0 + el < v.E);
  const double* __restrict__ Uin = v.U[cur];
  double* sD = lds.D;
  T(*sG)[NN] = lds.G;
  T(*sJ)[4][nf] = lds.J;
  const double Tref = sizeof(T) == 4 ? v.p_r / v.rho_r : 0.0;
  for (int x = t; x < n * n; x += NT) sD[x] = v.tab[2 * n + x];
  const long base = (long)e * nn;
  if (act) {
    double u[5];
#pragma unroll
    for (int c = 0; c < 5; c++) u[c] = Uin[base * 5 + c * nn + tl];
    T g[4];
    gvars(u, v.gamma, Tref, g);
#pragma unroll
    for (int c = 0; c < 4; c++) sG[c][t] = g[c];
  }
  __syncthreads();
  for (int x = t; x < NFP; x += NT) {
    const int ff = x / nf, q = x - ff * nf;  // ff = 6 (element of the workgroup) + face
    const int fe = EW > 1 ? ff / 6 : 0, f = EW > 1 ? ff - 6 * fe : ff;
    const int d = f >> 1, side = f & 1;
    const int p = q % n, r = q / n;
    const int io = fe * nn + face_node<n>(d, side ? N : 0, p, r);
    const int ne = v.nbr[(long)elem_of(fe) * 6 + f];
    const int inb = face_node<n>(d, side ? 0 : N, p, r);
    double un[5];
#pragma unroll
    for (int c = 0; c < 5; c++) un[c] = Uin[(long)ne * nn * 5 + c * nn + inb];
    T gn[4];
    gvars(un, v.gamma, Tref, gn);
#pragma unroll
    for (int c = 0; c < 4; c++) sJ[ff][c][q] = (T)0.5 * (gn[c] - sG[c][io]);
  }
  __syncthreads();
  const T iwN = (T)v.iwN, iw0 = (T)v.iw0;
  const T* const gp[4] = {sG[0], sG[1], sG[2], sG[3]};
  if constexpr (XV) {
    // BR2 / interior penalty: broken-gradient fluxes of the face nodes, then one lane per face point
    T(*sFb)[4][nf] = lds.Fb;
    if (act) {
      double ja[9];
#pragma unroll
      for (int c = 0; c < 9; c++) ja[c] = v.Ja[base * 9 + c * nn + tl];
      broken_face_fluxes<n, T>(t, ti, tj, tk, sD, gp, ja, v.invJ[base + tl], (T)v.mu, (T)v.kappa, sFb + 6 * el);
    }
    __syncthreads();
    for (int x = t; x < NFP; x += NT) {
      const int ff = x / nf, q = x - ff * nf;
      const int fe = EW > 1 ? ff / 6 : 0, f = EW > 1 ? ff - 6 * fe : ff;
      if (EW > 1 && e0 + fe >= v.E) continue;
      const int io = face_node<n>(f >> 1, (f & 1) ? N : 0, q % n, q / n);
      T Ff[4];
      face_viscous_br2_ip<n, T>(v, e0 + fe, cur, Tref, f, q, io, fe * nn, 6 * fe, iwN, iw0, gp, sJ, sFb, Ff);
      T* Fvf = reinterpret_cast<T*>(v.Fvf) + (long)(e0 + fe) * 6 * 4 * nf;
#pragma unroll
      for (int c = 0; c < 4; c++) Fvf[(f * 4 + c) * nf + q] = Ff[c];
    }
  } else if (put) {  // BR1: the lifted gradient's flux
    double ja[9], ij = v.cij;
    if constexpr (!CART) {
#pragma unroll
      for (int c = 0; c < 9; c++) ja[c] = v.Ja[base * 9 + c * nn + tl];
      ij = v.invJ[base + tl];
    }
    T Fvd[3][4];
    gradient_and_viscous_flux<n, T, CART>(t, ti, tj, tk, sD, iwN, iw0, gp, sJ + 6 * el, ja, ij, v, Fvd);
    T* Fvf = reinterpret_cast<T*>(v.Fvf) + (long)e * 6 * 4 * nf;
    const int ii[3] = {ti, tj, tk};
#pragma unroll
    for (int d = 0; d < 3; d++) {
      const int qd = d == 0 ? tj + n * tk : (d == 1 ? ti + n * tk : ti + n * tj);
      if (ii[d] == N) {
#pragma unroll
        for (int c = 0; c < 4; c++) Fvf[((2 * d + 1) * 4 + c) * nf + qd] = Fvd[d][c];
      }
      if (ii[d] == 0) {
#pragma unroll
        for (int c = 0; c < 4; c++) Fvf[((2 * d) * 4 + c) * nf + qd] = Fvd[d][c];
      }
    }
  }
}

}  // namespace dg
