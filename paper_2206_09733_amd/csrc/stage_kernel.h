// stage_kernel.h -- the stage kernel (residual of one element and the fused low-storage RK
// update) and its batched entry, as templates over the order N, the arithmetic type T, the
// viscous terms, the flux family FX, the plain-box form CART and the shape of small meshes SMALL
// (small_mesh).  kernels.hip instantiates family
// 0 (and FP32-bulk), kernels_ext.hip the extended families 1..3, so the two compile in parallel.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "dg_device.h"

namespace dg {

// ------------------------------------------------------------------ stage kernel
// Residual of one element and, in RK mode, the low-storage update
//   dU <- A dU + dt R;  U_out <- U_in + B dU   (dU not read when A = 0).
//
// Volume term.  A lane holds one node.  Along each direction it evaluates the two-point fluxes
// with the nodes at cyclic distance o = 1 .. (n-1)/2 on its line: its own state and metric are in
// registers, the partner's come from LDS, and the flux is used twice, by this node at once and by
// the partner from LDS (each pair of a line is so evaluated once; for even n the pairs at distance
// n/2 are evaluated by both of their nodes instead of being exchanged).  Every lane has the same
// number of pairs and no pair list is decoded.  What it replaced: a pair list whose lanes read
// both nodes from LDS (20 values a pair, and 10 more to gather) behind three barriers a direction,
// and the viscous term's own three passes.
// CART (plain boxes): Ja^d = cja[d] e_d is a constant of the mesh, so no metric term is read from
// memory or LDS, and every flux is formed in a frame rotated to its direction, where the normal
// is (1, 0, 0).
//
// Bound by VALU issue and by the latency of an element's loads, not by HBM (the NS stage at 32^3,
// N = 4 moves 1.39 GB in 355-365 us).  Measured, RK3 step before -> now, microseconds: deformed
// NS 32^3 N = 4 FP64 1727 -> 1541, FP32-bulk 1460 -> 1312; deformed Euler RK4 20^3 N = 5 per
// step 809 -> 654; deformed NS residual 13x11x9 N = 7 191 -> 116; plain Euler 41x36x28 N = 2
// 322 -> 162; plain NS 18x23x20 N = 5 (Pirozzoli + ES) 823 -> 547.
//
// The plain-box FP32-bulk Euler kernels of orders 5 and 6 read the RK update's input state after the
// last direction (see stage_body): 100 -> 90 VGPRs, five waves per SIMD.
__host__ __device__ constexpr bool late_state(int N, bool fp32, bool visc, bool cart) {
  return fp32 && cart && !visc && (N == 5 || N == 6);
}
// occupancy target of the stage kernel: waves per SIMD the register allocation must allow.  Four
// for FP32-bulk (at order 3 with the filtered flux only) and for the plain-box Navier-Stokes kernels of orders 3
// and 4 without the filtered flux (24^3, N = 4: 511 -> 493 us per RK3 step; the extended surface
// fluxes would spill).  Spills cost more than the fourth wave gives: deformed Euler at four waves with
// 9 (N = 4) and 33 spilled (N = 5) took 364 -> 401 and 395 -> 657 us.  Order 1, whose wave evaluates three
// rounds of face points: two waves in FP64 and three in FP32-bulk, one more would spill 10-41 and 25-43.
// Spilled as it is: one VGPR, by the deformed FP32-bulk kernel of order 5 with the filtered flux.
__host__ __device__ constexpr int stage_waves_per_eu(int N, bool fp32, bool visc, int fx, bool sva, bool cart) {
  if (N == 1) return fp32 ? 3 : 2;
  if (late_state(N, fp32, visc, cart)) return 5;
  if (N > 5) return 2;
  if (fp32) return N != 3 || sva ? 4 : 3;
  return cart && visc && !sva && (fx & 2) == 0 && (N == 3 || N == 4) ? 4 : 3;
}
// The batched kernels hold a few registers more (the member's View and start).  FP64: three waves, four
// would spill 6-8 of the plain-box Navier-Stokes kernels.  Those that hold both metric forms: three, two at order 1
// (at one more, 6 to 12 VGPRs of FP32-bulk kernels spilled; as it is 6 of the FP64 Navier-Stokes kernel of order 4).
__host__ __device__ constexpr int batch_waves_per_eu(int N, bool fp32, bool visc, int fx, BoxForm form) {
  const int w = stage_waves_per_eu(N, fp32, visc, fx, false, form == BoxForm::plain);
  if (form == BoxForm::both) return N == 1 ? 2 : (w > 3 ? 3 : w);
  if (!fp32 && N == 2 && !visc && form == BoxForm::plain) return 4;  // (130 VGPRs without: 306 -> 336 us at 16 x 10^3)
  return !fp32 && w > 3 ? 3 : w;
}

// global operands of one face point of the stage kernel's face phase: the neighbour's and the
// element's traces, the face's scaled normal, and the sum of the two sides' face viscous fluxes
// (CART: vectors in the frame rotated to the face's direction)
template <typename T>
struct FaceIn {
  double un[5], uo[5], S[3];
  T fv[4];
};

constexpr int align16(int b) { return (b + 15) / 16 * 16; }
constexpr int imax(int a, int b) { return a > b ? a : b; }

// LDS of a stage workgroup (byte offsets):
//   D, Dhat; the primitive variables rho, v1, v2, v3, beta (FP32-bulk: deviations of rho, beta);
//   FP32-bulk: FP64 velocities for the mass flux;
//   FP32-bulk and orders 1 and 2: the face fluxes, lifted beside each direction's volume sum (the two
//   largely cancel; the other kernels take the lifts with phase A: see lifts_beside_volume);
//   one region that holds each phase's arrays in turn:
//     A (face phase): with viscosity temperature and half jumps of g; the face fluxes (FP32-bulk:
//       their FP64 mass components);
//     B (one direction of the volume phase): the direction's metric terms and contravariant
//       viscous flux, and the exchanged two-point fluxes (FP32-bulk: and their FP64 mass parts).
// Whether the lifts of the face fluxes join each direction's volume sum or are summed first.  With
// the lifts summed first the FP64 residual of random states was further from the long-double oracle's
// at low orders (central volume flux, deformed boxes, rms: order 1 1.12 and order 2 1.03 times that of
// lifts beside the volume from a pair list; so 1.07 and 1.02; below 1.005 from order 3 on).  The
// fluxes' LDS outlives phase A then: order 2 Euler 6.6 -> 10 KB, times within 3%.
__host__ __device__ constexpr bool lifts_beside_volume(int N, bool fp32) { return fp32 || N <= 2; }

template <int N, typename T, bool VISC, bool CART, int EW>
struct StageLds {
  static constexpr int n = N + 1, nf = n * n, NN = EW * n * n * n, K = (n - 1) / 2;
  static constexpr bool DEV = sizeof(T) == 4;
  static constexpr bool BESIDE = lifts_beside_volume(N, DEV);
  static constexpr int S = (int)sizeof(T);
  static constexpr int oD = 0;
  static constexpr int oDh = oD + nf * 8;
  static constexpr int oP = align16(oDh + (VISC ? nf * 8 : 0));
  static constexpr int oVd = align16(oP + 5 * NN * S);
  static constexpr int oFk = align16(oVd + (DEV ? 3 * NN * 8 : 0));
  static constexpr int oR = align16(oFk + (BESIDE ? EW * 30 * nf * S : 0));
  static constexpr int bT = VISC ? align16(NN * S) : 0;
  static constexpr int bJ = VISC ? align16(EW * 24 * nf * S) : 0;
  static constexpr int bytesA = bT + bJ + EW * (DEV ? 6 : (BESIDE ? 0 : 30)) * nf * 8;
  static constexpr int bM = CART ? 0 : 3 * NN * 8;
  static constexpr int bV = VISC ? align16(4 * NN * S) : 0;
  static constexpr int bX = DEV ? K * NN * 8 + 4 * K * NN * 4 : 5 * K * NN * 8;
  static constexpr int bytes = oR + imax(bytesA, bM + bV + bX);
};

// SVA (Navier-Stokes): the filtered spectral-vanishing-viscosity flux v.Fa (FP64; rounded to T
// as it is read) of the same state joins the viscous flux at the nodes, and on the faces the average of both sides'
// stored values (as the viscous face fluxes; a face node's lane lifts it, the sum taken in the same
// order from both sides), so the residual holds its term too
template <int N, typename T, bool VISC, int FX, bool SVA, bool CART, int EW, int NT, typename VW>
__device__ __forceinline__ void stage_body(char* lds, const VW& v, const int wg, const int cur, const double dt,
                                           const double rkA, const double rkB, const int mode) {
  static_assert(!SVA || VISC, "the folded SVV term needs the viscous kernel");
  constexpr int n = N + 1, nn = n * n * n, nf = n * n;
  constexpr int NN = EW * nn;  // EW elements and NT lanes per workgroup
  constexpr int K = (n - 1) / 2;           // cyclic distances whose fluxes are exchanged
  constexpr bool HALF = n % 2 == 0;        // the distance n/2, evaluated by both nodes
  constexpr int NFP = EW * 6 * nf;         // face points of the workgroup
  constexpr bool DEV = sizeof(T) == 4;     // FP32-bulk: deviation form, FP64 mass flux
  const int t = threadIdx.x;
  const bool act = t < NN;
  const int el = EW > 1 ? (act ? t / nn : 0) : 0;
  const int tl = EW > 1 ? t - el * nn : t;  // node of its element
  const int ti = tl % n, tj = (tl / n) % n, tk = tl / nf;
  const int ii[3] = {ti, tj, tk};
  // the last workgroup repeats the last element in its spare places (without storing it)
  const int e0 = wg * EW;
  const int e = EW > 1 ? (e0 + el < v.E ? e0 + el : v.E - 1) : e0;
  const bool put = act && (EW == 1 || e0 + el < v.E);
  const double* __restrict__ Uin = v.U[cur];
  const Ref Rf = make_ref(v.rho_r, v.p_r, v.gamma);
  const double Tref = DEV ? Rf.por : 0.0;

  // LDS (see StageLds)
  using L = StageLds<N, T, VISC, CART, EW>;
  double* sD = reinterpret_cast<double*>(lds + L::oD);
  double* sDh = reinterpret_cast<double*>(lds + L::oDh);
  T(*sP)[NN] = reinterpret_cast<T(*)[NN]>(lds + L::oP);
  double(*sVd)[NN] = reinterpret_cast<double(*)[NN]>(lds + L::oVd);
  T(*sFk)[5][nf] = reinterpret_cast<T(*)[5][nf]>(lds + L::oFk);
  T* sT = reinterpret_cast<T*>(lds + L::oR);
  T(*sJ)[4][nf] = reinterpret_cast<T(*)[4][nf]>(lds + L::oR + L::bT);
  double(*sFa)[5][nf] = reinterpret_cast<double(*)[5][nf]>(lds + (L::BESIDE ? L::oFk : L::oR + L::bT + L::bJ));
  double(*sF0)[nf] = reinterpret_cast<double(*)[nf]>(lds + L::oR + L::bT + L::bJ);
  double(*sM)[NN] = reinterpret_cast<double(*)[NN]>(lds + L::oR);
  T(*sFv)[NN] = reinterpret_cast<T(*)[NN]>(lds + L::oR + L::bM);
  // exchanged fluxes of distance o: components at sX[o - 1][c] (FP64: 5; FP32-bulk: 1..4 and the
  // FP64 mass flux in sX0)
  double(*sX0)[NN] = reinterpret_cast<double(*)[NN]>(lds + L::oR + L::bM + L::bV);
  T(*sX)[DEV ? 4 : 5][NN] =
      reinterpret_cast<T(*)[DEV ? 4 : 5][NN]>(lds + L::oR + L::bM + L::bV + (DEV ? K * NN * 8 : 0));

  // tables (every lane loads, the first n^2 store: no wait of their own before the other loads)
  static_assert(n * n <= NT, "one table entry per lane");
  const int tt = t < n * n ? t : 0;
  const double tD = v.tab[2 * n + tt], tDh = VISC ? v.tab[2 * n + n * n + tt] : 0.0;
  const long base = (long)e * nn;
  // The six neighbours (one element per workgroup: uniform, scalar loads), and the global operands
  // of this lane's first face point, issued before the node's own state so that the two memory
  // round trips overlap.
  int nb0 = 0, nb1 = 0, nb2 = 0, nb3 = 0, nb4 = 0, nb5 = 0;
  if constexpr (EW == 1) {
    const int* nb = v.nbr + (long)e * 6;
    nb0 = nb[0], nb1 = nb[1], nb2 = nb[2], nb3 = nb[3], nb4 = nb[4], nb5 = nb[5];
  }
  auto neighbour = [&](int ef, int f) {
    if constexpr (EW > 1) return v.nbr[(long)ef * 6 + f];
    return f < 3 ? (f == 0 ? nb0 : (f == 1 ? nb1 : nb2)) : (f == 3 ? nb3 : (f == 4 ? nb4 : nb5));
  };
  const T* FvfAll = VISC ? reinterpret_cast<const T*>(v.Fvf) : nullptr;
  auto face_load = [&](int x, FaceIn<T>& I) {
    const int fe = EW > 1 ? x / (6 * nf) : 0;
    const int f = EW > 1 ? x / nf - fe * 6 : x / nf, q = x % nf;
    const int d = f >> 1, side = f & 1;
    const int p = q % n, r = q / n;
    const int io = face_node<n>(d, side ? N : 0, p, r);
    const int inb = face_node<n>(d, side ? 0 : N, p, r);
    const int ef = EW > 1 ? (e0 + fe < v.E ? e0 + fe : v.E - 1) : e;
    const int ne = neighbour(ef, f);
    // component of the rotated frame's axis k (CART), or k itself
    const int a0 = CART ? d : 0, a1 = CART ? (d == 2 ? 0 : d + 1) : 1, a2 = CART ? (d == 0 ? 2 : d - 1) : 2;
    const double* un = Uin + (long)ne * nn * 5 + inb;
    const double* uo = Uin + (long)ef * nn * 5 + io;
    I.un[0] = un[0];
    I.un[1] = un[(1 + a0) * nn];
    I.un[2] = un[(1 + a1) * nn];
    I.un[3] = un[(1 + a2) * nn];
    I.un[4] = un[4 * nn];
    I.uo[0] = uo[0];
    I.uo[1] = uo[(1 + a0) * nn];
    I.uo[2] = uo[(1 + a1) * nn];
    I.uo[3] = uo[(1 + a2) * nn];
    I.uo[4] = uo[4 * nn];
    if constexpr (CART) {
      I.S[0] = d == 0 ? v.cja[0] : (d == 1 ? v.cja[1] : v.cja[2]);
      I.S[1] = I.S[2] = 0.0;
    } else {
#pragma unroll
      for (int c = 0; c < 3; c++) I.S[c] = v.Ja[(long)ef * nn * 9 + (3 * d + c) * nn + io];
    }
    if (VISC) {
      const T* fo = FvfAll + ((long)ef * 6 + f) * 4 * nf + q;
      const T* fn = FvfAll + ((long)ne * 6 + (f ^ 1)) * 4 * nf + q;
      I.fv[0] = fo[a0 * nf] + fn[a0 * nf];
      I.fv[1] = fo[a1 * nf] + fn[a1 * nf];
      I.fv[2] = fo[a2 * nf] + fn[a2 * nf];
      I.fv[3] = fo[3 * nf] + fn[3 * nf];
    }
  };
  FaceIn<T> face0;
  if (t < NFP) face_load(t, face0);
  if (t < n * n) {
    sD[t] = tD;
    if (VISC) sDh[t] = tDh;
  }
  double ja[9], ij = CART ? v.cij : 0.0;
  Prim<T> A;           // this node
  double va[3] = {0, 0, 0};  // FP32-bulk: its FP64 velocity
  if (act) {
    double u[5];
#pragma unroll
    for (int c = 0; c < 5; c++) u[c] = Uin[base * 5 + c * nn + tl];
    A = DEV ? make_prim_dev<T>(u, v.gamma, Rf) : make_prim<T>(u, v.gamma);
    sP[0][t] = A.rho; sP[1][t] = A.v1; sP[2][t] = A.v2; sP[3][t] = A.v3;
    sP[4][t] = A.beta;
    if (DEV) {
      const double ir = rcp(u[0]);
#pragma unroll
      for (int c = 0; c < 3; c++) {
        va[c] = u[1 + c] * ir;
        sVd[c][t] = va[c];
      }
    }
    // the extended surface fluxes, and the viscous terms, need the registers during the face
    // phase: those kernels load the metric terms after it
    if constexpr (!CART && (FX & 2) == 0 && !VISC) {
#pragma unroll
      for (int c = 0; c < 9; c++) ja[c] = v.Ja[base * 9 + c * nn + tl];
      ij = v.invJ[base + tl];
    }
    if (VISC) {
      T g[4];
      gvars(u, v.gamma, Tref, g);
      sT[t] = g[3];
    }
  }
  __syncthreads();

  // ---- faces: numerical flux (minus the BR1 viscous flux) on the 6 (N+1)^2 face grids.  Both
  // elements of a face evaluate it from the same global values in the same argument order, so
  // it is single-valued.
  const double lam_g = (FX & 2) != 0 && v.surf == 8 ? v.adapt[3] : 0.0;  // global Lax-Friedrichs
  auto face_eval = [&](int x, const FaceIn<T>& I) {
    const int fe = EW > 1 ? x / (6 * nf) : 0;
    const int ff = x / nf, f = EW > 1 ? ff - fe * 6 : ff, q = x - ff * nf;  // ff = 6 fe + f
    const int d = f >> 1, side = f & 1;
    const int p = q % n, r = q / n;
    const int io = (EW > 1 ? fe * nn : 0) + face_node<n>(d, side ? N : 0, p, r);
    double uL[5], uR[5];
#pragma unroll
    for (int c = 0; c < 5; c++) {
      uL[c] = side ? I.uo[c] : I.un[c];
      uR[c] = side ? I.un[c] : I.uo[c];
    }
    const int a0 = CART ? d : 0, a1 = CART ? (d == 2 ? 0 : d + 1) : 1, a2 = CART ? (d == 0 ? 2 : d - 1) : 2;
    T F[5];
    double F0d = 0.0;
    if constexpr (DEV) {
      face_flux_dev<T, CART>(v.surf, uL, uR, I.S, v.gamma, Rf, F, F0d);
      sF0[ff][q] = F0d;
    } else {
      face_flux<(FX & 2) != 0, CART>(v.surf, uL, uR, I.S, v.gamma, F, lam_g);
    }
    if (VISC) {
#pragma unroll
      for (int c = 0; c < 4; c++) F[1 + c] -= (T)0.5 * I.fv[c];
      T gn[4];
      gvars(I.un, v.gamma, Tref, gn);
      sJ[ff][a0][q] = (T)0.5 * (gn[0] - sP[1 + a0][io]);
      sJ[ff][a1][q] = (T)0.5 * (gn[1] - sP[1 + a1][io]);
      sJ[ff][a2][q] = (T)0.5 * (gn[2] - sP[1 + a2][io]);
      sJ[ff][3][q] = (T)0.5 * (gn[3] - sT[io]);
    }
    if constexpr (DEV) {
      sFk[ff][1 + a0][q] = F[1];
      sFk[ff][1 + a1][q] = F[2];
      sFk[ff][1 + a2][q] = F[3];
      sFk[ff][4][q] = F[4];
    } else {
      sFa[ff][0][q] = F[0];
      sFa[ff][1 + a0][q] = F[1];
      sFa[ff][1 + a1][q] = F[2];
      sFa[ff][1 + a2][q] = F[3];
      sFa[ff][4][q] = F[4];
    }
  };
  // the metric terms of the kernels that load them late: in FP64 with the standard surface fluxes
  // issued before the remaining face points, so that their latency overlaps that work; the others
  // issue them after the face points (issued early they would spill: FP32-bulk at 4 waves per
  // SIMD, the extended surface fluxes, and FP64 Navier-Stokes at order 3)
  auto load_metric = [&]() {
    if (act) {
#pragma unroll
      for (int c = 0; c < 9; c++) ja[c] = v.Ja[base * 9 + c * nn + tl];
      ij = v.invJ[base + tl];
    }
  };
  constexpr bool late_metric = !CART && ((FX & 2) != 0 || VISC);
  constexpr bool early = late_metric && !DEV && (FX & 2) == 0 && N != 3;
  if (t < NFP) face_eval(t, face0);
  if constexpr (early) load_metric();
#pragma unroll 1
  for (int x = t + NT; x < NFP; x += NT) {
    FaceIn<T> I;
    face_load(x, I);
    face_eval(x, I);
  }
  if constexpr (late_metric && !early) load_metric();
  __syncthreads();

  const T iwN = (T)v.iwN, iw0 = (T)v.iw0;
  T acc[5] = {0, 0, 0, 0, 0};
  double acc0d = 0.0;  // FP32-bulk mass accumulator
  T Fvd[3][4];         // contravariant viscous flux of this node
  if (act) {
    // lift of the face fluxes (FP32-bulk: of their FP64 mass components; the others beside the volume)
#pragma unroll
    for (int d = 0; d < 3; d++) {
      const int id = ii[d], ff = 6 * el + 2 * d;
      const int line = d == 0 ? tj + n * tk : (d == 1 ? ti + n * tk : ti + n * tj);
      if (id == N) {
        if constexpr (DEV) {
          acc0d += v.iwN * sF0[ff + 1][line];
        } else if constexpr (!L::BESIDE) {
#pragma unroll
          for (int c = 0; c < 5; c++) acc[c] += iwN * sFa[ff + 1][c][line];
        }
      }
      if (id == 0) {
        if constexpr (DEV) {
          acc0d -= v.iw0 * sF0[ff][line];
        } else if constexpr (!L::BESIDE) {
#pragma unroll
          for (int c = 0; c < 5; c++) acc[c] -= iw0 * sFa[ff][c][line];
        }
      }
    }
    if (VISC) {
      const T* const gp[4] = {sP[1], sP[2], sP[3], sT};
      gradient_and_viscous_flux<n, T, CART>(t, ti, tj, tk, sD, iwN, iw0, gp, sJ + 6 * el, ja, ij, v, Fvd);
    }
  }

  // ---- volume, one direction at a time
  constexpr bool kLateState = late_state(N, DEV, VISC, CART);
  const long o5 = base * 5 + tl;
  double u_in[5], du_in[5];
  const T ce = (T)(0.5 / (v.gamma - 1.0)), gm1 = (T)(v.gamma - 1.0);
#pragma unroll
  for (int d = 0; d < 3; d++) {
    constexpr int strides[3] = {1, n, nf};
    const int stride = strides[d], id = ii[d];
    const int c0 = CART ? d : 0, c1 = CART ? (d + 1) % 3 : 1, c2 = CART ? (d + 2) % 3 : 2;  // rotated axes
    T fa[4] = {0, 0, 0, 0}, fb[4] = {0, 0, 0, 0};  // SVA: this node's Fa^d, the neighbour's across a face
    const bool onf = SVA && act && (id == 0 || id == N);
    if (SVA && act) {
#pragma unroll
      for (int c = 0; c < 4; c++) fa[c] = (T)v.Fa[(base * 12) + (4 * d + c) * nn + tl];
    }
    if (onf) {
      const int side = id == N ? 1 : 0;
      const int ne = side ? neighbour(e, 2 * d + 1) : neighbour(e, 2 * d);
      const int inb = tl + (side ? -N : N) * stride;  // the matching node across the face
#pragma unroll
      for (int c = 0; c < 4; c++) fb[c] = (T)v.Fa[((long)ne * 12 + 4 * d + c) * nn + inb];
    }
    // the RK update's operands, requested before the last direction so that their latency hides
    // behind it (earlier they would add 20 registers to those that the first directions hold)
    if (d == 2 && act && mode != kModeResidual) {
#pragma unroll
      for (int c = 0; c < 5; c++) {
        if constexpr (!kLateState) u_in[c] = Uin[o5 + c * nn];
        du_in[c] = rkA == 0.0 ? 0.0 : v.dU[o5 + c * nn];
      }
    }
    __syncthreads();  // previous users of the region are done
    if constexpr (!CART || VISC) {
      if (act) {
        if constexpr (!CART) {
#pragma unroll
          for (int c = 0; c < 3; c++) sM[c][t] = ja[3 * d + c];
        }
        if (VISC) {
#pragma unroll
          for (int c = 0; c < 4; c++) sFv[c][t] = SVA ? Fvd[d][c] + fa[c] : Fvd[d][c];
        }
      }
      __syncthreads();
    }
    T pa[5] = {0, 0, 0, 0, 0};  // this direction's two-point sum (CART: along the unit normal, rotated)
    double pa0 = 0.0;
    // flux with the node at cyclic distance o; F rotated (CART)
    auto pair = [&](int o, T F[5], double& F0d) {
      int j = id + o;
      j = j >= n ? j - n : j;
      const int tb = t + (j - id) * stride;
      Prim<T> P, Q;
      P.rho = A.rho; P.beta = A.beta;
      const T av[3] = {A.v1, A.v2, A.v3};
      P.v1 = av[c0]; P.v2 = av[c1]; P.v3 = av[c2];
      Q.rho = sP[0][tb]; Q.beta = sP[4][tb];
      if constexpr (DEV) {
        const double vb[3] = {sVd[c0][tb], sVd[c1][tb], sVd[c2][tb]};
        const double vc[3] = {va[c0], va[c1], va[c2]};
        Q.v1 = (T)vb[0]; Q.v2 = (T)vb[1]; Q.v3 = (T)vb[2];
        double md[3] = {1.0, 0.0, 0.0};
        if constexpr (!CART) {
#pragma unroll
          for (int c = 0; c < 3; c++) md[c] = ja[3 * d + c] + sM[c][tb];
        }
        if (v.vol == 0) {
          const double vn64 = 0.5 * dotn<CART>(vc[0] + vb[0], vc[1] + vb[1], vc[2] + vb[2], md[0], md[1], md[2]);
          flux_ec_dev<CART>(P, Q, (T)md[0], (T)md[1], (T)md[2], vn64, Rf, F, F0d);
        } else {
          flux_central_dev<CART>(P, Q, (T)md[0], (T)md[1], (T)md[2], vc, vb, md, Rf, F, F0d);
        }
      } else {
        Q.v1 = sP[1 + c0][tb]; Q.v2 = sP[1 + c1][tb]; Q.v3 = sP[1 + c2][tb];
        T m1 = 1, m2 = 0, m3 = 0;
        if constexpr (!CART) {
          m1 = ja[3 * d] + sM[0][tb];
          m2 = ja[3 * d + 1] + sM[1][tb];
          m3 = ja[3 * d + 2] + sM[2][tb];
        }
        vol_flux<(FX & 1) != 0, CART>(v.vol, P, Q, m1, m2, m3, ce, gm1, F);
      }
      const double Dd = sD[id * n + j];
      if constexpr (DEV) {
        pa0 += Dd * F0d;
      } else {
        pa[0] += Dd * F[0];
      }
#pragma unroll
      for (int c = 1; c < 5; c++) pa[c] += (T)Dd * F[c];
    };
    if (act) {
#pragma unroll
      for (int o = 1; o <= K; o++) {
        T F[5];
        double F0d;
        pair(o, F, F0d);
        if constexpr (DEV) {
          sX0[o - 1][t] = F0d;
#pragma unroll
          for (int c = 1; c < 5; c++) sX[o - 1][c - 1][t] = F[c];
        } else {
#pragma unroll
          for (int c = 0; c < 5; c++) sX[o - 1][c][t] = F[c];
        }
      }
      if constexpr (HALF) {
        T F[5];
        double F0d;
        pair(n / 2, F, F0d);
      }
      if (VISC) {  // sum_m Dhat_im F~v^d_m
        const int b0 = t - id * stride;
#pragma unroll
        for (int m = 0; m < n; m++) {
          const T Dh = (T)sDh[id * n + m];
#pragma unroll
          for (int c = 0; c < 4; c++) acc[1 + c] -= Dh * sFv[c][b0 + m * stride];
        }
        if (onf) {  // lift of the face average of Fa (the own value's lift is in Dhat)
          const T wl = id == N ? -(T)0.5 * iwN : (T)0.5 * iw0;
#pragma unroll
          for (int c = 0; c < 4; c++) acc[1 + c] += wl * (fa[c] + fb[c]);  // (commutes: the same on both sides)
        }
      }
    }
    if constexpr (K > 0) {
      __syncthreads();
      if (act) {
#pragma unroll
        for (int o = 1; o <= K; o++) {
          int i = id - o;
          i = i < 0 ? i + n : i;
          const int tb = t + (i - id) * stride;
          const double Dd = sD[id * n + i];
          if constexpr (DEV) {
            pa0 += Dd * sX0[o - 1][tb];
#pragma unroll
            for (int c = 1; c < 5; c++) pa[c] += (T)Dd * sX[o - 1][c - 1][tb];
          } else {
#pragma unroll
            for (int c = 0; c < 5; c++) pa[c] += Dd * sX[o - 1][c][tb];
          }
        }
      }
    }
    if (act) {
      // CART: times twice the constant Ja^d (the pair sums of the general form hold Ja_i + Ja_m)
      const double s64 = CART ? 2.0 * v.cja[d] : 1.0;
      const T sc = (T)s64;
      if constexpr (DEV) {
        acc0d += s64 * pa0;
        const int ff = 6 * el + 2 * d;
        const int line = d == 0 ? tj + n * tk : (d == 1 ? ti + n * tk : ti + n * tj);
        T q[5] = {0, pa[1], pa[2], pa[3], pa[4]};
        if constexpr (CART) {
          q[1 + c0] = sc * pa[1];
          q[1 + c1] = sc * pa[2];
          q[1 + c2] = sc * pa[3];
          q[4] = sc * pa[4];
        }
        if (id == N) {
#pragma unroll
          for (int c = 1; c < 5; c++) q[c] += iwN * sFk[ff + 1][c][line];
        }
        if (id == 0) {
#pragma unroll
          for (int c = 1; c < 5; c++) q[c] -= iw0 * sFk[ff][c][line];
        }
#pragma unroll
        for (int c = 1; c < 5; c++) acc[c] += q[c];
      } else {
        acc[0] += CART ? sc * pa[0] : pa[0];
        acc[1 + c0] += CART ? sc * pa[1] : pa[1];
        acc[1 + c1] += CART ? sc * pa[2] : pa[2];
        acc[1 + c2] += CART ? sc * pa[3] : pa[3];
        acc[4] += CART ? sc * pa[4] : pa[4];
        if constexpr (L::BESIDE) {
          const int ff = 6 * el + 2 * d;
          const int line = d == 0 ? tj + n * tk : (d == 1 ? ti + n * tk : ti + n * tj);
          if (id == N) {
#pragma unroll
            for (int c = 0; c < 5; c++) acc[c] += iwN * sFa[ff + 1][c][line];
          }
          if (id == 0) {
#pragma unroll
            for (int c = 0; c < 5; c++) acc[c] -= iw0 * sFa[ff][c][line];
          }
        }
      }
    }
  }
  if (!put) return;
  double R[5];
#pragma unroll
  for (int c = 0; c < 5; c++) R[c] = -(double)acc[c] * ij;
  if (DEV) {  // FP64 mass; energy = H_r (mass) + deviation
    R[0] = -acc0d * ij;
    R[4] -= Rf.H * acc0d * ij;
  }
  if (mode == kModeResidual) {
#pragma unroll
    for (int c = 0; c < 5; c++) v.R[o5 + c * nn] = R[c];
    return;
  }
  if constexpr (kLateState) {
#pragma unroll
    for (int c = 0; c < 5; c++) u_in[c] = Uin[o5 + c * nn];
  }
  double* __restrict__ Uout = v.U[cur ^ 1];
  const double h = v.dtp ? *v.dtp : dt;
#pragma unroll
  for (int c = 0; c < 5; c++) {
    const double du = (rkA == 0.0 ? 0.0 : rkA * du_in[c]) + h * R[c];
    v.dU[o5 + c * nn] = du;
    Uout[o5 + c * nn] = u_in[c] + rkB * du;
  }
}

// FX: the flux family (see flux_family); each family is compiled as separate kernels.  SMALL: the
// shape of small meshes
template <int N, typename T, bool VISC, int FX, bool SVA, bool CART, bool SMALL>
__global__ void __launch_bounds__(SMALL ? small_lanes(N) : wg_lanes(N))
    __attribute__((amdgpu_waves_per_eu(SMALL ? 2 : stage_waves_per_eu(N, sizeof(T) == 4, VISC, FX, SVA, CART))))
    stage_kernel(View v, int cur, double dt, double rkA, double rkB, int mode) {
  constexpr int EW = SMALL ? 1 : wg_elems(N);
  __shared__ __align__(16) char lds[StageLds<N, T, VISC, CART, EW>::bytes];
  stage_body<N, T, VISC, FX, SVA, CART, EW, SMALL ? small_lanes(N) : wg_lanes(N)>(
      lds, v, block_element((v.E + EW - 1) / EW), cur, dt, rkA, rkB, mode);
}

// FORM: the members' boxes.  Deformed members have kernels of their own since the registers of both forms
// in one kernel spilled: 16 solves of 10^3, N = 4 Navier-Stokes FP64, deformed, 3791 us for four RK3 steps
// (3166 so, 3534 with one general form before there was a plain one).
// SMALL: the shape of small meshes (kBatchSmallWaves)
template <int N, typename T, bool VISC, int FX, BoxForm FORM, bool SMALL>
__global__ void __launch_bounds__(SMALL ? small_lanes(N) : wg_lanes(N))
    __attribute__((amdgpu_waves_per_eu(SMALL ? 2 : batch_waves_per_eu(N, sizeof(T) == 4, VISC, FX, FORM))))
    stage_batch_kernel(BatchArgs B, double rkA, double rkB, int mode) {
  constexpr int EW = SMALL ? 1 : wg_elems(N), NT = SMALL ? small_lanes(N) : wg_lanes(N);
  __shared__ __align__(16) char lds[StageLds<N, T, VISC, FORM == BoxForm::plain, EW>::bytes];
  static_assert(StageLds<N, T, VISC, true, EW>::bytes <= StageLds<N, T, VISC, false, EW>::bytes, "one LDS buffer for both");
  int m, w;
  batch_member(B, m, w);
  ConstView& v = const_view(B.view[m]);
  if constexpr (FORM != BoxForm::both) {
    stage_body<N, T, VISC, FX, false, FORM == BoxForm::plain, EW, NT>(lds, v, w, B.cur[m], B.dt[m], rkA, rkB, mode);
  } else {
    if (v.deform)
      stage_body<N, T, VISC, FX, false, false, EW, NT>(lds, v, w, B.cur[m], B.dt[m], rkA, rkB, mode);
    else
      stage_body<N, T, VISC, FX, false, true, EW, NT>(lds, v, w, B.cur[m], B.dt[m], rkA, rkB, mode);
  }
}

// ------------------------------------------------------------------ launch helpers
template <int N, typename T, int FX, bool CART>
inline hipError_t stage_ntxc(const View& v, int cur, double dt, double a, double b, int mode,
                             hipStream_t st) {
  const dim3 grid(wg_count(N, v.E)), block(wg_lanes(N));
  if constexpr (FX == 0) {
    if (v.viscous && v.Fa) {
      hipLaunchKernelGGL((stage_kernel<N, T, true, 0, true, CART, false>), grid, block, 0, st, v, cur, dt, a, b, mode);
      return hipGetLastError();
    }
  }
  if (v.Fa) return hipErrorInvalidValue;  // the folded SVV term: Navier-Stokes, standard fluxes
  if constexpr (N <= kSmallMaxOrder) {
    if (small_mesh(N, v.E)) {
      const dim3 g1(v.E), b1(small_lanes(N));
      if (v.viscous)
        hipLaunchKernelGGL((stage_kernel<N, T, true, FX, false, CART, true>), g1, b1, 0, st, v, cur, dt, a, b, mode);
      else
        hipLaunchKernelGGL((stage_kernel<N, T, false, FX, false, CART, true>), g1, b1, 0, st, v, cur, dt, a, b, mode);
      return hipGetLastError();
    }
  }
  if (v.viscous)
    hipLaunchKernelGGL((stage_kernel<N, T, true, FX, false, CART, false>), grid, block, 0, st, v, cur, dt, a, b, mode);
  else
    hipLaunchKernelGGL((stage_kernel<N, T, false, FX, false, CART, false>), grid, block, 0, st, v, cur, dt, a, b, mode);
  return hipGetLastError();
}

template <int N, typename T, int FX>
inline hipError_t stage_ntx(const View& v, int cur, double dt, double a, double b, int mode, hipStream_t st) {
  return v.deform ? stage_ntxc<N, T, FX, false>(v, cur, dt, a, b, mode, st)
                  : stage_ntxc<N, T, FX, true>(v, cur, dt, a, b, mode, st);
}

template <int N, typename T, int FX, BoxForm FORM, bool SMALL>
inline hipError_t stage_batch_nts(const BatchArgs& B, bool visc, double a, double b, int mode, hipStream_t st) {
  const dim3 grid(B.start[B.n]), block(SMALL ? small_lanes(N) : wg_lanes(N));
  if (visc)
    hipLaunchKernelGGL((stage_batch_kernel<N, T, true, FX, FORM, SMALL>), grid, block, 0, st, B, a, b, mode);
  else
    hipLaunchKernelGGL((stage_batch_kernel<N, T, false, FX, FORM, SMALL>), grid, block, 0, st, B, a, b, mode);
  return hipGetLastError();
}

template <int N, typename T, int FX, BoxForm FORM>
inline hipError_t stage_batch_ntf(const BatchArgs& B, bool visc, double a, double b, int mode, hipStream_t st) {
  if constexpr (N <= kBatchSmallMaxOrder) {
    if (B.small) return stage_batch_nts<N, T, FX, FORM, true>(B, visc, a, b, mode, st);
  }
  return stage_batch_nts<N, T, FX, FORM, false>(B, visc, a, b, mode, st);
}

template <int N, typename T, int FX>
inline hipError_t stage_batch_nt(const BatchArgs& B, bool visc, BoxForm form, double a, double b, int mode,
                                 hipStream_t st) {
  switch (form) {
    case BoxForm::plain: return stage_batch_ntf<N, T, FX, BoxForm::plain>(B, visc, a, b, mode, st);
    case BoxForm::deformed: return stage_batch_ntf<N, T, FX, BoxForm::deformed>(B, visc, a, b, mode, st);
    default: return stage_batch_ntf<N, T, FX, BoxForm::both>(B, visc, a, b, mode, st);
  }
}

}  // namespace dg
