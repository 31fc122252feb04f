// kernels_mixed.hip -- kernels for meshes whose elements carry their own anisotropic orders
// (N1, N2, N3) (section "Spatial p-adaptation": per-element and per-direction orders; mortar
// coupling of p-nonconforming faces).  Euler equations, FP64 and FP32-bulk.
//
// A face kernel, one wave per face, then one workgroup per element, in buckets of a work list
// sorted by node count (largest first) so that the long elements start early.  Faces whose two
// sides have equal tangential orders are evaluated pointwise; on the others both traces and
// the owner's normal are interpolated to the Lobatto grid of the larger tangential orders
// (the mortar), the numerical flux is evaluated there, and the result is L2-projected back onto
// both elements' face grids; the projections preserve its integral, so the totals are conserved.
#include <hip/hip_runtime.h>

#include <cmath>

#include "dg_device.h"

namespace dg {

constexpr int kMixN = kMixMaxOrder + 1;  // nodes per direction at most
constexpr int kMixNN = kMixN * kMixN * kMixN;
constexpr int kMixNF = kMixN * kMixN;

struct ElemInfo {
  int n[3];
  int nn;
  long off;
};

__device__ __forceinline__ ElemInfo elem_info(const View& v, int e) {
  const int4 q = v.elem[e];
  ElemInfo I;
  I.n[0] = q.x;
  I.n[1] = q.y;
  I.n[2] = q.z;
  I.nn = q.x * q.y * q.z;
  I.off = q.w;
  return I;
}

// Lobatto table pointers of order N (node count n = N + 1)
// (the member arrays of the kernel argument are read with constant indices and a select: a
// runtime index makes the compiler copy the whole argument to private memory)
__device__ __forceinline__ int tab_offset(const View& v, int n) {
  int o = v.tab_off[0];
#pragma unroll
  for (int k = 1; k < kMixN; k++) o = n - 1 == k ? v.tab_off[k] : o;
  return o;
}
__device__ __forceinline__ const double* tab_w(const View& v, int n) { return v.tab + tab_offset(v, n) + n; }
__device__ __forceinline__ const double* tab_D(const View& v, int n) { return v.tab + tab_offset(v, n) + 2 * n; }
__device__ __forceinline__ double* state(const View& v, int k) { return k ? v.U[1] : v.U[0]; }

// ------------------------------------------------------------------ geometry (FP64)
__global__ void __launch_bounds__(512) geometry_mixed_kernel(View v) {
  const int e = blockIdx.x;
  const ElemInfo I = elem_info(v, e);
  const int t = threadIdx.x;
  const bool act = t < I.nn;
  const int ti = t % I.n[0], tj = (t / I.n[0]) % I.n[1], tk = t / (I.n[0] * I.n[1]);
  const int ii[3] = {ti, tj, tk};
  __shared__ double sD[3][kMixNF + 15], sxi[3][8];
  __shared__ double sXl[3][512], sdX[9][512], sA[3][512];
  for (int d = 0; d < 3; d++) {
    const int n = I.n[d];
    const double* tab = v.tab + v.tab_off[n - 1];
    for (int x = t; x < n * n; x += blockDim.x) sD[d][x] = tab[2 * n + x];
    if (t < n) sxi[d][t] = tab[t];
  }
  __syncthreads();
  const int cell[3] = {e % v.ex, (e / v.ex) % v.ey, e / (v.ex * v.ey)};
  const long off = I.off, nn = I.nn;
  if (act) {
    double loc[3], xu[3], dx[3] = {0, 0, 0};
    for (int d = 0; d < 3; d++) {
      loc[d] = (1.0 + sxi[d][ii[d]]) * 0.5 * v.h[d];
      xu[d] = v.lo[d] + cell[d] * v.h[d] + loc[d];
    }
    if (v.deform) {
      dx[0] = v.amp * sin(xu[1]) * sin(xu[2]);
      dx[1] = v.amp * sin(xu[2]) * sin(xu[0]);
      dx[2] = v.amp * sin(xu[0]) * sin(xu[1]);
    }
    for (int d = 0; d < 3; d++) {
      v.X[off * 3 + d * nn + t] = xu[d] + dx[d];
      sXl[d][t] = loc[d] + dx[d];
    }
  }
  __syncthreads();
  auto dref = [&](const double* f, int d) {
    const int n = I.n[d];
    const int stride = d == 0 ? 1 : (d == 1 ? I.n[0] : I.n[0] * I.n[1]);
    const int b0 = t - ii[d] * stride;
    double s = 0.0;
    for (int m = 0; m < n; m++) s += sD[d][ii[d] * n + m] * f[b0 + m * stride];
    return s;
  };
  if (act)
    for (int m = 0; m < 3; m++)
      for (int d = 0; d < 3; d++) sdX[3 * m + d][t] = dref(sXl[m], d);
  __syncthreads();
  for (int c = 0; c < 3; c++) {
    const int m = (c + 1) % 3, l = (c + 2) % 3;
    if (act)
      for (int d = 0; d < 3; d++) sA[d][t] = sXl[l][t] * sdX[3 * m + d][t];
    __syncthreads();
    if (act) {
      const double c0 = dref(sA[2], 1) - dref(sA[1], 2);
      const double c1 = dref(sA[0], 2) - dref(sA[2], 0);
      const double c2 = dref(sA[1], 0) - dref(sA[0], 1);
      v.Ja[off * 9 + (3 * 0 + c) * nn + t] = -c0;
      v.Ja[off * 9 + (3 * 1 + c) * nn + t] = -c1;
      v.Ja[off * 9 + (3 * 2 + c) * nn + t] = -c2;
    }
    __syncthreads();
  }
  if (act) {
    auto X = [&](int m, int d) { return sdX[3 * m + d][t]; };
    const double J = X(0, 0) * (X(1, 1) * X(2, 2) - X(2, 1) * X(1, 2)) +
                     X(1, 0) * (X(2, 1) * X(0, 2) - X(0, 1) * X(2, 2)) +
                     X(2, 0) * (X(0, 1) * X(1, 2) - X(1, 1) * X(0, 2));
    v.J[off + t] = J;
    v.invJ[off + t] = 1.0 / J;
  }
}

// ------------------------------------------------------------------ initial conditions
__global__ void __launch_bounds__(512) ic_mixed_kernel(View v, int cur, int ic, IcParams P) {
  const int e = blockIdx.x;
  const ElemInfo I = elem_info(v, e);
  const long off = I.off, nn = I.nn;
  for (int q = threadIdx.x; q < I.nn; q += blockDim.x) {
    const double x = v.X[off * 3 + q], y = v.X[off * 3 + nn + q], z = v.X[off * 3 + 2 * nn + q];
    double u[5];
    ic_point(v, ic, P, x, y, z, u);
    for (int c = 0; c < 5; c++) {
      v.U[cur][off * 5 + c * nn + q] = u[c];
      v.dU[off * 5 + c * nn + q] = 0.0;
    }
  }
}

// lanes of a workgroup for elements of up to nnmax nodes, npl nodes per lane (whole waves)
__host__ __device__ constexpr int mix_lanes(int nnmax, int npl) { return ((nnmax + npl - 1) / npl + 63) / 64 * 64; }

// q / n for 0 <= q < 4096 and 1 <= n <= 64, from inv_n = 1.0f / n: (q + 1/2)/n lies at least
// 1/(2n) away from an integer, far more than the rounding error of the FP32 product (checked
// for every q and n in that range).
__device__ __forceinline__ int sdiv(int q, float inv_n) { return (int)(((float)q + 0.5f) * inv_n); }

// ------------------------------------------------------------------ stage: faces
// One 64-lane workgroup (a single wave) per face: the face normal to d between the owner L (its
// +xi_d side) and R = nbr(L, +d), with L's metric Ja^d as the scaled normal.  Traces are staged
// in LDS, interpolated to the mortar of the larger tangential orders (the identity where the
// orders agree), the numerical flux is evaluated at the mortar points, and it is L2-projected
// onto the face grids of both elements: Fs[e], packed in the order [f][c][p + n_a r], f = 2 d + side of
// element e, c = 0..4 the flux and (FP32-bulk) c = 5 its FP64 mass component, so that the stage kernel
// copies one contiguous block.  Each face is evaluated once.
// In each tangential direction at most one side has fewer nodes than the mortar: only that side
// is interpolated and projected along it (the other side's data already lies on the mortar
// grid and is used in place), so every loop has a trip count and branches that are uniform over
// the wave.
// XS: the extended surface fluxes (codes >= 4), compiled apart so that the others keep their
// registers
// CART: plain boxes: the scaled normal is cja[d] e_d, so only the two states are interpolated (with
// their velocity components in the rotated frame) and no metric term is read.
template <typename T, bool XS, bool CART>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(XS ? 3 : (CART ? 5 : 4))))
    mixed_face_kernel(View v, int cur) {
  constexpr bool DEV = sizeof(T) == 4;
  constexpr int NL = CART ? 5 : 8;  // L's fields: state, and its Ja^d
  constexpr int NC = DEV ? 6 : 5;
  static_assert(kMixNF <= 64, "a face grid, or a mortar matrix, fits one wave");
  const int fid = block_element(3 * v.E);
  const int e = fid / 3, d = fid - 3 * e;
  const int t = threadIdx.x;
  const double* __restrict__ Uin = v.U[cur];
  const Ref Rf = make_ref(v.rho_r, v.p_r, v.gamma);
  // the face's table entry: R, both elements' node counts and first nodes (one load, where the
  // neighbour and then its element entry would be two in sequence)
  const int4 fd = v.fdesc[fid];
  const int eR = fd.x;
  const int nL0 = fd.y & 7, nL1 = (fd.y >> 3) & 7, nL2 = (fd.y >> 6) & 7;
  const int nR0 = (fd.y >> 9) & 7, nR1 = (fd.y >> 12) & 7, nR2 = (fd.y >> 15) & 7;
  // node counts along a and b, and node strides (selected by d: an array indexed by a runtime
  // value would be kept in private memory)
  const int naL = d == 0 ? nL1 : nL0, nbL = d == 2 ? nL1 : nL2;
  const int naR = d == 0 ? nR1 : nR0, nbR = d == 2 ? nR1 : nR2;
  const int ma = naL > naR ? naL : naR, mb = nbL > nbR ? nbL : nbR;
  const float ima = 1.0f / (float)ma;
  // the side (0 = L, 1 = R, -1 = none) with fewer nodes than the mortar along a and along b
  const int sa = naL < ma ? 0 : (naR < ma ? 1 : -1);
  const int sb = nbL < mb ? 0 : (nbR < mb ? 1 : -1);
  // na_s, nb_a: the a-side's node counts along a and b; nb_s: the b-side's node count along b
  const int na_s = sa == 0 ? naL : naR, nb_a = sa == 0 ? nbL : nbR, nb_s = sb == 0 ? nbL : nbR;
  // sA: rows 0-4 L's state, 5-7 L's Ja^d (L's grid), rows 8-12 R's state (R's grid); later
  // rows 0-5 the flux on the mortar.  sB: the side interpolated along a (up to 8 rows), later
  // the flux projected along a onto that side's grid (up to 6 rows).
  // (CART: R's state in rows 5-9)
  __shared__ double sA[NL + 5][kMixNF], sB[NL > NC ? NL : NC][kMixNF];
  // interpolation to the mortar and projection back, along a and along b (only the sides
  // that need them)
  __shared__ double sIa[kMixNF], sPa[kMixNF], sIb[kMixNF], sPb[kMixNF];
  // Every operand is requested before any is stored (one lane per point or matrix entry, the
  // indices clamped so that no load waits on a branch): the traces on their own grids (index
  // p + n_a r) and the mortar matrices.
  const int sLa = d == 0 ? nL0 : 1, sLb = d == 2 ? nL0 : nL0 * nL1;
  const int sRa = d == 0 ? nR0 : 1, sRb = d == 2 ? nR0 : nR0 * nR1;
  const int baseL = d == 0 ? nL0 - 1 : (d == 1 ? (nL1 - 1) * nL0 : (nL2 - 1) * nL0 * nL1);
  const long offL = fd.z, offR = fd.w, nnL = nL0 * nL1 * nL2, nnR = nR0 * nR1 * nR2;
  double tL[NL], tR[5];
  // component of the rotated frame's axis k (CART), or k itself
  const int a0 = CART ? d : 0, a1 = CART ? (d == 2 ? 0 : d + 1) : 1, a2 = CART ? (d == 0 ? 2 : d - 1) : 2;
  {
    const int x = t < naL * nbL ? t : 0;
    const int r = sdiv(x, 1.0f / (float)naL), p = x - r * naL;
    const int q = baseL + p * sLa + r * sLb;
#pragma unroll
    for (int c = 0; c < 5; c++) {
      const int cc = c == 1 ? 1 + a0 : (c == 2 ? 1 + a1 : (c == 3 ? 1 + a2 : c));
      tL[c] = Uin[offL * 5 + cc * nnL + q];
    }
    if constexpr (!CART) {
#pragma unroll
      for (int c = 0; c < 3; c++) tL[5 + c] = v.Ja[offL * 9 + (3 * d + c) * nnL + q];
    }
  }
  {
    const int y = t < naR * nbR ? t : 0;
    const int r = sdiv(y, 1.0f / (float)naR), p = y - r * naR;
    const int q = p * sRa + r * sRb;
#pragma unroll
    for (int c = 0; c < 5; c++) {
      const int cc = c == 1 ? 1 + a0 : (c == 2 ? 1 + a1 : (c == 3 ? 1 + a2 : c));
      tR[c] = Uin[offR * 5 + cc * nnR + q];
    }
  }
  const double* mt = v.mtab;
  double tIa = 0.0, tPa = 0.0, tIb = 0.0, tPb = 0.0;
  if (sa >= 0) {
    const double* src = mt + v.mort_off[na_s - 1][ma - 1];
    const int x = t < ma * na_s ? t : 0;
    tIa = src[x];
    tPa = src[ma * na_s + x];
  }
  if (sb >= 0) {
    const double* src = mt + v.mort_off[nb_s - 1][mb - 1];
    const int x = t < mb * nb_s ? t : 0;
    tIb = src[x];
    tPb = src[mb * nb_s + x];
  }
  if (t < naL * nbL) {
#pragma unroll
    for (int c = 0; c < NL; c++) sA[c][t] = tL[c];
  }
  if (t < naR * nbR) {
#pragma unroll
    for (int c = 0; c < 5; c++) sA[NL + c][t] = tR[c];
  }
  if (sa >= 0 && t < ma * na_s) {
    sIa[t] = tIa;
    sPa[t] = tPa;
  }
  if (sb >= 0 && t < mb * nb_s) {
    sIb[t] = tIb;
    sPb[t] = tPb;
  }
  __syncthreads();
  // along a: the smaller side to the mortar (index pm + ma r); its fields are L's 8 or R's 5.
  // Each weight is read once and applied to every field (the sum over p of each field keeps its
  // order).
  if (sa >= 0) {
    const int c0 = sa == 0 ? 0 : NL, nc = sa == 0 ? NL : 5;
    for (int y = t; y < ma * nb_a; y += 64) {
      const int r = sdiv(y, ima), pm = y - r * ma;
      double s[NL] = {};
      for (int p = 0; p < na_s; p++) {
        const double w = sIa[pm * na_s + p];
        const int x = p + na_s * r;
#pragma unroll
        for (int c = 0; c < NL; c++)
          if (c < nc) s[c] += w * sA[c0 + c][x];
      }
#pragma unroll
      for (int c = 0; c < NL; c++)
        if (c < nc) sB[c][y] = s[c];
    }
  }
  __syncthreads();
  // along b, and the numerical flux at the mortar point (ma mb <= 49 points: one pass)
  {
    const int x = t;
    const bool on = x < ma * mb;
    const int rm = sdiv(x, ima), pm = x - rm * ma;
    double a[NL + 5];
    // L's fields (rows of sB if L was interpolated along a), then R's 5
    const double(*rowsL)[kMixNF] = sa == 0 ? sB : sA;
    const double(*rowsR)[kMixNF] = sa == 1 ? sB : sA + NL;
    if (nbL == mb) {
#pragma unroll
      for (int c = 0; c < NL; c++) a[c] = on ? rowsL[c][pm + ma * rm] : 0.0;
    } else {
#pragma unroll
      for (int c = 0; c < NL; c++) a[c] = 0.0;
      if (on)
        for (int r = 0; r < nbL; r++) {
          const double w = sIb[rm * nbL + r];
#pragma unroll
          for (int c = 0; c < NL; c++) a[c] += w * rowsL[c][pm + ma * r];
        }
    }
    if (nbR == mb) {
#pragma unroll
      for (int c = 0; c < 5; c++) a[NL + c] = on ? rowsR[c][pm + ma * rm] : 0.0;
    } else {
#pragma unroll
      for (int c = 0; c < 5; c++) a[NL + c] = 0.0;
      if (on)
        for (int r = 0; r < nbR; r++) {
          const double w = sIb[rm * nbR + r];
#pragma unroll
          for (int c = 0; c < 5; c++) a[NL + c] += w * rowsR[c][pm + ma * r];
        }
    }
    __syncthreads();  // every mortar point has read its data before the flux rows overwrite sA
    if (on) {
      const double uL[5] = {a[0], a[1], a[2], a[3], a[4]};
      const double uR[5] = {a[NL], a[NL + 1], a[NL + 2], a[NL + 3], a[NL + 4]};
      double S[3] = {d == 0 ? v.cja[0] : (d == 1 ? v.cja[1] : v.cja[2]), 0.0, 0.0};
      if constexpr (!CART) {
#pragma unroll
        for (int c = 0; c < 3; c++) S[c] = a[5 + c];
      }
      T F[5];
      if constexpr (DEV) {
        double F0d;
        face_flux_dev<T, CART>(v.surf, uL, uR, S, v.gamma, Rf, F, F0d);
        sA[5][x] = F0d;
      } else {
        face_flux<XS, CART>(v.surf, uL, uR, S, v.gamma, F, XS && v.surf == 8 ? v.adapt[3] : 0.0);
      }
#pragma unroll
      for (int c = 0; c < 5; c++) {
        const int cc = c == 1 ? 1 + a0 : (c == 2 ? 1 + a1 : (c == 3 ? 1 + a2 : c));
        sA[cc][x] = (double)F[c];
      }
    }
  }
  __syncthreads();
  // L2 projection along a onto the smaller side's grid (index po + na rm), into sB
  if (sa >= 0) {
    const float ina_s = 1.0f / (float)na_s;
    for (int y = t; y < na_s * mb; y += 64) {
      const int rm = sdiv(y, ina_s), po = y - rm * na_s;
      double s[NC];
#pragma unroll
      for (int c = 0; c < NC; c++) s[c] = 0.0;
      for (int pm = 0; pm < ma; pm++) {
        const double w = sPa[po * ma + pm];
#pragma unroll
        for (int c = 0; c < NC; c++) s[c] += w * sA[c][pm + ma * rm];
      }
#pragma unroll
      for (int c = 0; c < NC; c++) sB[c][y] = s[c];
    }
  }
  __syncthreads();
  // along b onto each side's face grid, into Fs
#pragma unroll
  for (int side = 0; side < 2; side++) {
    const int na = side ? naR : naL, nb = side ? nbR : nbL;
    const double(*src)[kMixNF] = sa == side ? sB : sA;  // the flux along a on this side's grid
    const int m0 = side ? nR0 : nL0, m1 = side ? nR1 : nL1, m2 = side ? nR2 : nL2, np = na * nb;
    // faces of the element before this one, components and points packed (L's +side, R's -side)
    const int before = d == 0 ? 0 : (d == 1 ? 2 * m1 * m2 : 2 * (m1 * m2 + m0 * m2));
    double* out = v.Fs + (long)(side ? eR : e) * kMixFaceDoubles + NC * (before + (side ? 0 : np));
    const float ina = 1.0f / (float)na;
    for (int y = t; y < na * nb; y += 64) {
      const int ro = sdiv(y, ina), po = y - ro * na;
      double s[NC];
      if (nb == mb) {
#pragma unroll
        for (int c = 0; c < NC; c++) s[c] = src[c][po + na * ro];
      } else {
#pragma unroll
        for (int c = 0; c < NC; c++) s[c] = 0.0;
        for (int rm = 0; rm < mb; rm++) {
          const double w = sPb[ro * mb + rm];
#pragma unroll
          for (int c = 0; c < NC; c++) s[c] += w * src[c][po + na * rm];
        }
      }
#pragma unroll
      for (int c = 0; c < NC; c++) out[c * np + y] = s[c];
    }
  }
}

// ------------------------------------------------------------------ stage: volume and update
// Elements are launched by bucket: bucket b holds the elements of 64 b < nn <= 64 (b + 1) nodes,
// a contiguous range of the work list (sorted by node count).  A lane holds NPL nodes (1 or 2,
// the autotuner's choice per bucket), so the workgroup has mix_lanes(NNMAX, NPL) lanes.  KEP
// selects the kinetic-energy-preserving volume fluxes (compiled apart, FP64 only).
// Bound on the face points of an element of at most nnmax nodes (sum over its six faces of the
// tangential node counts' products), for 1 <= n_d <= kMixN.
__host__ __device__ constexpr int mix_face_points(int nnmax) {
  int best = 0;
  for (int a = 1; a <= kMixN; a++)
    for (int b = 1; b <= kMixN; b++)
      for (int c = 1; c <= kMixN; c++)
        if (a * b * c <= nnmax) {
          const int f = 2 * (a * b + b * c + a * c);
          if (f > best) best = f;
        }
  return best;
}

// The volume term is that of the uniform-order stage kernel: a lane evaluates the two-point fluxes of
// its node with the nodes at cyclic distance o = 1 .. (n-1)/2 on its line and hands each flux to the
// partner through LDS (for even n the pairs at distance n/2 are evaluated by both nodes), so each
// pair is evaluated once; n is uniform over the workgroup, so the barriers of an exchange are too.
// CART: plain boxes, whose metric terms are constants: none is read and the fluxes are formed in a
// frame rotated to the direction.
// The loop over the directions is unrolled: the choices by direction disappear, and the RK register
// can be requested before the last direction without holding registers through the others (126 ->
// 116 VGPRs).  24^3, orders 2..6, RK3 step with the face pass, plain box: each pair from both nodes
// 819 us, once and CART 712, packed face fluxes 639-653, unrolled 609.
template <int NNMAX, int NPL, typename T, bool KEP, bool CART>
__global__ void __launch_bounds__(mix_lanes(NNMAX, NPL))
    mixed_stage_kernel(View v, int wbeg, int cur, double dt, double rkA, double rkB, int mode) {
  constexpr int BS = mix_lanes(NNMAX, NPL);
  constexpr bool DEV = sizeof(T) == 4;  // FP32-bulk: deviation form, FP64 mass flux
  constexpr int NC = DEV ? 6 : 5;       // face flux components read (FP32-bulk: + FP64 mass)
  constexpr int NFS = NC * mix_face_points(NNMAX);
  constexpr int KF = (NFS + BS - 1) / BS;  // face flux values per lane
  // two exchange buffers in turn need one barrier an exchange instead of two; the large buckets
  // take one, which keeps three workgroups in a CU's LDS
  constexpr int XB = NNMAX <= 192 ? 2 : 1;
  const int4 wi = v.work[wbeg + blockIdx.x];
  const int e = wi.x;
  const int n0 = wi.y & 7, n1 = (wi.y >> 3) & 7, n2 = (wi.y >> 6) & 7;
  const int t = threadIdx.x;
  const long off = wi.z, nn = wi.w;
  const int inn = wi.w;
  const double* __restrict__ Uin = state(v, cur);
  const double* __restrict__ Fs = v.Fs + (long)e * kMixFaceDoubles;
  const Ref Rf = make_ref(v.rho_r, v.p_r, v.gamma);
  const float inv0 = 1.0f / (float)n0, inv01 = 1.0f / (float)(n0 * n1);
  // face points of the faces normal to each direction, and where face f's fluxes start in sFs
  // (the element's faces packed: f = 2 d + side, component-major within a face)
  const int pt0 = n1 * n2, pt1 = n0 * n2, pt2 = n0 * n1;
  const int fo1 = NC * pt0, fo2 = 2 * NC * pt0, fo3 = fo2 + NC * pt1, fo4 = fo2 + 2 * NC * pt1,
            fo5 = fo4 + NC * pt2, fend = fo4 + 2 * NC * pt2;

  __shared__ double sD[3][kMixNF], sw[3][kMixN];
  __shared__ T sP[5][NNMAX];             // rho, v1, v2, v3, beta (FP32-bulk: deviations)
  constexpr int NV = DEV ? NNMAX : 1, NM = CART ? 1 : NNMAX;
  __shared__ double sVd[3][NV];          // FP32-bulk: FP64 velocities for the mass flux
  __shared__ double sJ3[3][NM];          // Ja^d of the direction in work
  __shared__ double sFs[NFS];            // the element's face fluxes
  __shared__ T sX[XB][DEV ? 4 : 5][NNMAX];  // the exchanged fluxes (FP32-bulk: 1..4, the FP64 mass flux in sX0)
  __shared__ double sX0[XB][NV];

  // Every operand of the element is requested before any is used: state, the first direction's
  // metric terms, the face fluxes and the tables (the tables with clamped indices, so that no
  // load waits on a branch).
  double u[NPL][5], jn[NPL][3];
#pragma unroll
  for (int s = 0; s < NPL; s++) {
    const int q = t + s * BS;
    const int qc = q < inn ? q : 0;
#pragma unroll
    for (int c = 0; c < 5; c++) u[s][c] = Uin[off * 5 + c * nn + qc];
    if constexpr (!CART) {
#pragma unroll
      for (int c = 0; c < 3; c++) jn[s][c] = v.Ja[off * 9 + c * nn + qc];
    }
  }
  double fv[KF];
#pragma unroll
  for (int k = 0; k < KF; k++) {
    const int x = t + k * BS;
    fv[k] = x < fend ? Fs[x] : 0.0;
  }
  double tD[3], tw[3];
#pragma unroll
  for (int d = 0; d < 3; d++) {
    const int n = d == 0 ? n0 : (d == 1 ? n1 : n2);
    tD[d] = tab_D(v, n)[t < n * n ? t : 0];
    tw[d] = tab_w(v, n)[t < n ? t : 0];
  }
  static_assert(BS >= kMixNF, "one table entry per lane");
#pragma unroll
  for (int d = 0; d < 3; d++) {
    const int n = d == 0 ? n0 : (d == 1 ? n1 : n2);
    if (t < n * n) sD[d][t] = tD[d];
    if (t < n) sw[d][t] = tw[d];
  }
#pragma unroll
  for (int k = 0; k < KF; k++)
    if (t + k * BS < fend) sFs[t + k * BS] = fv[k];

  int ii[NPL][3];
#pragma unroll
  for (int s = 0; s < NPL; s++) {
    const int q = t + s * BS;
    const int k = sdiv(q, inv01), rem = q - k * n0 * n1;
    const int j = sdiv(rem, inv0);
    ii[s][0] = rem - j * n0;
    ii[s][1] = j;
    ii[s][2] = k;
    if (q < inn) {
      const Prim<T> P = DEV ? make_prim_dev<T>(u[s], v.gamma, Rf) : make_prim<T>(u[s], v.gamma);
      sP[0][q] = P.rho; sP[1][q] = P.v1; sP[2][q] = P.v2; sP[3][q] = P.v3;
      sP[4][q] = P.beta;
      if (DEV) {
        const double ir = rcp(u[s][0]);
        sVd[0][DEV ? q : 0] = u[s][1] * ir;
        sVd[1][DEV ? q : 0] = u[s][2] * ir;
        sVd[2][DEV ? q : 0] = u[s][3] * ir;
      }
    }
  }

  // For each node and direction: sum over the line of D_im F#(U_i, U_m; Ja_i + Ja_m), then the
  // surface lift of the face fluxes.  Slot s of the lane holds node t + s BS.
  T acc[NPL][5];
  double accm[NPL];  // FP32-bulk: FP64 mass accumulators
  double du_in[NPL][5];
#pragma unroll
  for (int s = 0; s < NPL; s++) {
#pragma unroll
    for (int c = 0; c < 5; c++) acc[s][c] = 0;
    accm[s] = 0.0;
  }
  const T ce = (T)(0.5 / (v.gamma - 1.0)), gm1 = (T)(v.gamma - 1.0);
  const double cj0 = v.cja[0], cj1 = v.cja[1], cj2 = v.cja[2];
  int xb = 0;  // exchange buffer in use
  // (every per-direction choice is a select of values: an array indexed by the runtime d, or a select
  // between captured variables, would keep the kernel argument in private memory)
#pragma unroll
  for (int d = 0; d < 3; d++) {
    __syncthreads();  // primitives staged; the previous direction's LDS data is no longer read
    if constexpr (!CART) {
#pragma unroll
      for (int s = 0; s < NPL; s++)
        if (t + s * BS < inn)
#pragma unroll
          for (int c = 0; c < 3; c++) sJ3[c][CART ? 0 : t + s * BS] = jn[s][c];
      __syncthreads();
      if (d < 2) {  // the next direction's metric terms, in flight during this direction's sums
#pragma unroll
        for (int s = 0; s < NPL; s++) {
          const int q = t + s * BS;
          const int qc = q < inn ? q : 0;
#pragma unroll
          for (int c = 0; c < 3; c++) jn[s][c] = v.Ja[off * 9 + (3 * (d + 1) + c) * nn + qc];
        }
      }
    }
    if (d == 2 && mode != kModeResidual && rkA != 0.0) {  // the RK register, in flight during the last direction
#pragma unroll
      for (int s = 0; s < NPL; s++) {
        const int qc = t + s * BS < inn ? t + s * BS : 0;
#pragma unroll
        for (int c = 0; c < 5; c++) du_in[s][c] = v.dU[off * 5 + c * nn + qc];
      }
    }
    const int n = d == 0 ? n0 : (d == 1 ? n1 : n2), sd = d == 0 ? 1 : (d == 1 ? n0 : n0 * n1);
    const int pf = d == 0 ? pt0 : (d == 1 ? pt1 : pt2);
    const int flo = d == 0 ? 0 : (d == 1 ? fo2 : fo4), fhi = d == 0 ? fo1 : (d == 1 ? fo3 : fo5);
    const int c0 = CART ? d : 0, c1 = CART ? (d == 2 ? 0 : d + 1) : 1, c2 = CART ? (d == 0 ? 2 : d - 1) : 2;
    const double* Dd = sD[0] + d * kMixNF;
    // flux of node q (index id on its line) with the node qm
    auto pair_flux = [&](const int q, const int qm, T F[5], double& F0d) {
      Prim<T> A, B;
      A.rho = sP[0][q]; A.beta = sP[4][q];
      B.rho = sP[0][qm]; B.beta = sP[4][qm];
      double md[3] = {1.0, 0.0, 0.0};
      if constexpr (!CART) {
#pragma unroll
        for (int c = 0; c < 3; c++) md[c] = sJ3[c][CART ? 0 : q] + sJ3[c][CART ? 0 : qm];
      }
      if constexpr (DEV) {
        const double va[3] = {sVd[c0][DEV ? q : 0], sVd[c1][DEV ? q : 0], sVd[c2][DEV ? q : 0]};
        const double vb[3] = {sVd[c0][DEV ? qm : 0], sVd[c1][DEV ? qm : 0], sVd[c2][DEV ? qm : 0]};
        A.v1 = (T)va[0]; A.v2 = (T)va[1]; A.v3 = (T)va[2];
        B.v1 = (T)vb[0]; B.v2 = (T)vb[1]; B.v3 = (T)vb[2];
        if (v.vol == 0) {
          const double vn64 = 0.5 * dotn<CART>(va[0] + vb[0], va[1] + vb[1], va[2] + vb[2], md[0], md[1], md[2]);
          flux_ec_dev<CART>(A, B, (T)md[0], (T)md[1], (T)md[2], vn64, Rf, F, F0d);
        } else {
          flux_central_dev<CART>(A, B, (T)md[0], (T)md[1], (T)md[2], va, vb, md, Rf, F, F0d);
        }
      } else {
        A.v1 = sP[1 + c0][q]; A.v2 = sP[1 + c1][q]; A.v3 = sP[1 + c2][q];
        B.v1 = sP[1 + c0][qm]; B.v2 = sP[1 + c1][qm]; B.v3 = sP[1 + c2][qm];
        vol_flux<KEP, CART>(v.vol, A, B, (T)md[0], (T)md[1], (T)md[2], ce, gm1, F);
      }
    };
    T pa[NPL][5];
    double pm[NPL];
#pragma unroll
    for (int s = 0; s < NPL; s++) {
#pragma unroll
      for (int c = 0; c < 5; c++) pa[s][c] = 0;
      pm[s] = 0.0;
    }
    auto add = [&](const double D, const T F[5], const double F0d, T p[5], double& m) {
      if constexpr (DEV) m += D * F0d;
      else p[0] += (T)D * F[0];
#pragma unroll
      for (int c = 1; c < 5; c++) p[c] += (T)D * F[c];
    };
#pragma unroll 1
    for (int o = 1; 2 * o <= n; o++) {
      const bool half = 2 * o == n;
      if (XB == 1 && o > 1 && !half) __syncthreads();  // the buffer's previous readers are done
#pragma unroll
      for (int s = 0; s < NPL; s++) {
        const int q = t + s * BS;
        if (q >= inn) continue;
        const int id = d == 0 ? ii[s][0] : (d == 1 ? ii[s][1] : ii[s][2]);
        const int j = id + o < n ? id + o : id + o - n;
        T F[5];
        double F0d = 0.0;
        pair_flux(q, q + (j - id) * sd, F, F0d);
        add(Dd[id * n + j], F, F0d, pa[s], pm[s]);
        if (!half) {
          if constexpr (DEV) sX0[xb][DEV ? q : 0] = F0d;
#pragma unroll
          for (int c = DEV ? 1 : 0; c < 5; c++) sX[xb][c - (DEV ? 1 : 0)][q] = F[c];
        }
      }
      if (half) break;
      __syncthreads();
#pragma unroll
      for (int s = 0; s < NPL; s++) {
        const int q = t + s * BS;
        if (q >= inn) continue;
        const int id = d == 0 ? ii[s][0] : (d == 1 ? ii[s][1] : ii[s][2]);
        const int j = id - o >= 0 ? id - o : id - o + n;
        const int qm = q + (j - id) * sd;
        T F[5];
#pragma unroll
        for (int c = DEV ? 1 : 0; c < 5; c++) F[c] = sX[xb][c - (DEV ? 1 : 0)][qm];
        add(Dd[id * n + j], F, DEV ? sX0[xb][DEV ? qm : 0] : 0.0, pa[s], pm[s]);
      }
      xb = XB == 2 ? xb ^ 1 : 0;
    }
    const double s64 = CART ? 2.0 * (d == 0 ? cj0 : (d == 1 ? cj1 : cj2)) : 1.0;
#pragma unroll
    for (int s = 0; s < NPL; s++) {
      if (t + s * BS >= inn) continue;
      const int i0 = ii[s][0], i1 = ii[s][1], i2 = ii[s][2];
      const int id = d == 0 ? i0 : (d == 1 ? i1 : i2);
      // back from the rotated frame: component x of it is pa[1 + (x - d) mod 3]
      const T p1 = pa[s][1], p2 = pa[s][2], p3 = pa[s][3];
      T q[5] = {pa[s][0], p1, p2, p3, pa[s][4]};
      if constexpr (CART) {
        q[1] = d == 0 ? p1 : (d == 1 ? p3 : p2);
        q[2] = d == 0 ? p2 : (d == 1 ? p1 : p3);
        q[3] = d == 0 ? p3 : (d == 1 ? p2 : p1);
      }
      double qm = pm[s];
      if constexpr (CART) {
        qm *= s64;
#pragma unroll
        for (int c = 0; c < 5; c++) q[c] *= (T)s64;
      }
      // the node's point on the faces normal to d (tangential indices in increasing direction)
      const int qf = d == 0 ? i1 + n1 * i2 : (d == 1 ? i0 + n0 * i2 : i0 + n0 * i1);
      if (id == n - 1) {
        const double iw = rcp(sw[0][d * kMixN + n - 1]);
        const double* F = sFs + fhi;
#pragma unroll
        for (int c = 0; c < 5; c++) q[c] += (T)(iw * F[c * pf + qf]);
        if (DEV) qm += iw * F[5 * pf + qf];
      }
      if (id == 0) {
        const double iw = rcp(sw[0][d * kMixN]);
        const double* F = sFs + flo;
#pragma unroll
        for (int c = 0; c < 5; c++) q[c] -= (T)(iw * F[c * pf + qf]);
        if (DEV) qm -= iw * F[5 * pf + qf];
      }
#pragma unroll
      for (int c = 0; c < 5; c++) acc[s][c] += q[c];
      accm[s] += qm;
    }
  }
  auto node_update = [&](const int q, const T* acc, const double accm, const double* du_in) {
    const long o = off * 5 + q;
    const double ij = CART ? v.cij : v.invJ[off + q];
    double R[5];
#pragma unroll
    for (int c = 0; c < 5; c++) R[c] = -(double)acc[c] * ij;
    if (DEV) {  // FP64 mass; energy = H_r (mass) + deviation
      R[0] = -accm * ij;
      R[4] -= Rf.H * accm * ij;
    }
#pragma unroll
    for (int c = 0; c < 5; c++) {
      if (mode == kModeResidual) {
        v.R[o + c * nn] = R[c];
      } else {
        const double du = (rkA == 0.0 ? 0.0 : rkA * du_in[c]) + (v.dtp ? *v.dtp : dt) * R[c];
        v.dU[o + c * nn] = du;
        state(v, cur ^ 1)[o + c * nn] = Uin[o + c * nn] + rkB * du;
      }
    }
  };
#pragma unroll
  for (int s = 0; s < NPL; s++)
    if (t + s * BS < inn) node_update(t + s * BS, acc[s], accm[s], du_in[s]);
}

// ------------------------------------------------------------------ diagnostics (FP64)
// as the uniform-order kernel: a grid of at most kDiagBlocks workgroups walks over the elements,
// every lane adding its nodes to its own slots
constexpr int kMixDiagLanes = (kMixNN + 63) / 64 * 64;
__global__ void __launch_bounds__(kMixDiagLanes) diag_mixed_kernel(View v, int cur, int parts) {
  const int t = threadIdx.x;
  __shared__ double sD[2][3][kMixNF], sw[2][3][kMixN];
  __shared__ double sV[2][3][kMixNN];
  double s[kDiagUsed];
#pragma unroll
  for (int k = 0; k < kDiagUsed; k++) s[k] = diag_identity(k);
  int buf = 0;
  for (int e = blockIdx.x; e < v.E; e += gridDim.x, buf ^= 1) {
    const ElemInfo I = elem_info(v, e);
    const bool act = t < I.nn;
    const long off = I.off, nn = I.nn;
    const int ii[3] = {t % I.n[0], (t / I.n[0]) % I.n[1], t / (I.n[0] * I.n[1])};
    for (int d = 0; d < 3; d++) {
      const int n = I.n[d];
      if (t < n * n) sD[buf][d][t] = tab_D(v, n)[t];
      if (t < n) sw[buf][d][t] = tab_w(v, n)[t];
    }
    double u[5] = {0, 0, 0, 0, 0};
    if (act) {
      for (int c = 0; c < 5; c++) u[c] = v.U[cur][off * 5 + c * nn + t];
      for (int c = 0; c < 3; c++) sV[buf][c][t] = u[1 + c] / u[0];
    }
    __syncthreads();
    if (!act) continue;
    const double wq = sw[buf][0][ii[0]] * sw[buf][1][ii[1]] * sw[buf][2][ii[2]] * v.J[off + t];
    const double ij = v.invJ[off + t];
    double dv[3][3];
    for (int d = 0; d < 3; d++) {
      const int n = I.n[d];
      const int stride = d == 0 ? 1 : (d == 1 ? I.n[0] : I.n[0] * I.n[1]);
      const int b0 = t - ii[d] * stride;
      double a[3] = {0.0, 0.0, 0.0};
      for (int m = 0; m < n; m++)
        for (int c = 0; c < 3; c++) a[c] += sD[buf][d][ii[d] * n + m] * sV[buf][c][b0 + m * stride];
      for (int c = 0; c < 3; c++) dv[d][c] = a[c];
    }
    double gv[3][3];
    for (int c = 0; c < 3; c++)
      for (int x = 0; x < 3; x++) {
        double a = 0.0;
        for (int d = 0; d < 3; d++) a += v.Ja[off * 9 + (3 * d + x) * nn + t] * dv[d][c];
        gv[c][x] = a * ij;
      }
    diag_add(s, u, v.gamma, wq, gv[2][1] - gv[1][2], gv[0][2] - gv[2][0], gv[1][0] - gv[0][1]);
  }
  diag_store<kMixDiagLanes / 64>(s, v.part, parts, blockIdx.x);
}

// ------------------------------------------------------------------ launchers
hipError_t launch_geometry_mixed(const View& v, hipStream_t st) {
  hipLaunchKernelGGL(geometry_mixed_kernel, dim3(v.E), dim3(512), 0, st, v);
  return hipGetLastError();
}

hipError_t launch_ic_mixed(const View& v, int cur, int ic, const double* params, hipStream_t st) {
  IcParams P;
  for (int k = 0; k < 9; k++) P.p[k] = params ? params[k] : 0.0;
  hipLaunchKernelGGL(ic_mixed_kernel, dim3(v.E), dim3(512), 0, st, v, cur, ic, P);
  return hipGetLastError();
}

template <int NNMAX, int NPL, bool CART>
static hipError_t stage_bucket(const View& v, int b, int cur, double dt, double rkA, double rkB, int mode,
                               hipStream_t st) {
  const dim3 grid(v.mix_cnt[b]), block(mix_lanes(NNMAX, NPL));
  if (v.fp32)
    hipLaunchKernelGGL((mixed_stage_kernel<NNMAX, NPL, float, false, CART>), grid, block, 0, st, v, v.mix_beg[b],
                       cur, dt, rkA, rkB, mode);
  else if (flux_family(v.vol, v.surf) & 1)
    hipLaunchKernelGGL((mixed_stage_kernel<NNMAX, NPL, double, true, CART>), grid, block, 0, st, v, v.mix_beg[b],
                       cur, dt, rkA, rkB, mode);
  else
    hipLaunchKernelGGL((mixed_stage_kernel<NNMAX, NPL, double, false, CART>), grid, block, 0, st, v, v.mix_beg[b],
                       cur, dt, rkA, rkB, mode);
  return hipGetLastError();
}

template <int NNMAX>
static hipError_t stage_bucket_npl(const View& v, int b, int npl, int cur, double dt, double rkA, double rkB,
                                   int mode, hipStream_t st) {
  if (v.deform)
    return npl == 2 ? stage_bucket<NNMAX, 2, false>(v, b, cur, dt, rkA, rkB, mode, st)
                    : stage_bucket<NNMAX, 1, false>(v, b, cur, dt, rkA, rkB, mode, st);
  return npl == 2 ? stage_bucket<NNMAX, 2, true>(v, b, cur, dt, rkA, rkB, mode, st)
                  : stage_bucket<NNMAX, 1, true>(v, b, cur, dt, rkA, rkB, mode, st);
}

template <bool CART>
static hipError_t faces_mixed(const View& v, int cur, hipStream_t st) {
  if (v.fp32)
    hipLaunchKernelGGL((mixed_face_kernel<float, false, CART>), dim3(3 * v.E), dim3(64), 0, st, v, cur);
  else if (v.surf >= 4)
    hipLaunchKernelGGL((mixed_face_kernel<double, true, CART>), dim3(3 * v.E), dim3(64), 0, st, v, cur);
  else
    hipLaunchKernelGGL((mixed_face_kernel<double, false, CART>), dim3(3 * v.E), dim3(64), 0, st, v, cur);
  return hipGetLastError();
}

hipError_t launch_faces_mixed(const View& v, int cur, hipStream_t st) {
  return v.deform ? faces_mixed<false>(v, cur, st) : faces_mixed<true>(v, cur, st);
}

hipError_t launch_stage_mixed_bucket(const View& v, int b, int npl, int cur, double dt, double rkA, double rkB,
                                     int mode, hipStream_t st) {
  if (v.mix_cnt[b] <= 0) return hipSuccess;
  switch (b) {
    case 0: return stage_bucket_npl<64>(v, b, npl, cur, dt, rkA, rkB, mode, st);
    case 1: return stage_bucket_npl<128>(v, b, npl, cur, dt, rkA, rkB, mode, st);
    case 2: return stage_bucket_npl<192>(v, b, npl, cur, dt, rkA, rkB, mode, st);
    case 3: return stage_bucket_npl<256>(v, b, npl, cur, dt, rkA, rkB, mode, st);
    case 4: return stage_bucket_npl<320>(v, b, npl, cur, dt, rkA, rkB, mode, st);
    case 5: return stage_bucket_npl<384>(v, b, npl, cur, dt, rkA, rkB, mode, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_stage_mixed(const View& v, int cur, double dt, double rkA, double rkB, int mode, int tiles,
                              hipStream_t st, const MixStreams* ms) {
  hipError_t e = launch_faces_mixed(v, cur, st);
  if (e != hipSuccess) return e;
  int bk[kMixBuckets], nb = 0;
  for (int b = kMixBuckets - 1; b >= 0; b--)  // the work list starts with the largest elements
    if (v.mix_cnt[b] > 0) bk[nb++] = b;
  // the largest elements on st, up to kMixSide further buckets each on a side stream, the rest
  // after the largest on st
  const int ns = ms ? (nb - 1 < kMixSide ? nb - 1 : kMixSide) : 0;
  if (ns > 0) {
    e = hipEventRecord(ms->fork, st);
    if (e != hipSuccess) return e;
  }
  for (int i = 0; i < ns && e == hipSuccess; i++) {
    const int b = bk[1 + i];
    e = hipStreamWaitEvent(ms->side[i], ms->fork, 0);
    if (e == hipSuccess)
      e = launch_stage_mixed_bucket(v, b, (tiles >> b) & 1 ? 2 : 1, cur, dt, rkA, rkB, mode, ms->side[i]);
    if (e == hipSuccess) e = hipEventRecord(ms->join[i], ms->side[i]);
  }
  for (int i = 0; i < nb && e == hipSuccess; i++) {
    if (i >= 1 && i <= ns) continue;
    const int b = bk[i];
    e = launch_stage_mixed_bucket(v, b, (tiles >> b) & 1 ? 2 : 1, cur, dt, rkA, rkB, mode, st);
  }
  // the join, also after a failed launch: no side stream is left forked from st
  for (int i = 0; i < ns; i++) {
    const hipError_t ej = hipStreamWaitEvent(st, ms->join[i], 0);
    if (e == hipSuccess) e = ej;
  }
  return e;
}

hipError_t launch_diagnostics_mixed(const View& v, int cur, hipStream_t st) {
  const int parts = v.E < kDiagBlocks ? v.E : kDiagBlocks;
  hipLaunchKernelGGL(diag_mixed_kernel, dim3(parts), dim3(kMixDiagLanes), 0, st, v, cur, parts);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  return launch_diag_final(v, parts, st);
}

}  // namespace dg
