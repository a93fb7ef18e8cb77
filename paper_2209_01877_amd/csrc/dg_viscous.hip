// Viscous (Navier-Stokes) terms of eq. 11 in BR1 form for gfx950, FP64 and FP32.
//
// The paper rewrites the viscous equations with the auxiliary variable Z = grad U and
// takes the viscous interface flux in the form of Bassi and Rebay (BR1): both the
// lifting of Z and the viscous flux use central interface values.  Per element K,
// variable v, mode i, direction k:
//   |K| Z_k,i = -sum_q w_q |det J| dphi_i/dx_k U(q) + sum_f sum_q w^f_q (U- + U+)/2 N_k phi_i
//   Rv_i      = -(Vv_i - Sv_i) / |K|,   Vv_i = int_K F_v(U, Z) . grad phi_i,
//               Sv_i = sum_f int_f (F_v(U-, Z-) + F_v(U+, Z+))/2 . n phi_i
// with the inviscid ghost state as U+ on boundary faces and Z+ = Z- there.  Two kernels, with the
// stage kernel's MFMA operand tables:
//   ns_kernel        : everything of the residual that an element's own Z gives: the lifting of Z,
//                      the inviscid and viscous volume terms, the inviscid face fluxes and the
//                      element's own half of every viscous face term; the own half
//                      F_v(U-, Z-) . N / 2 at the face points is also stored
//   ns_update_kernel : adds the neighbours' halves, read from that store, then the RK update
// Since the BR1 interface flux is an average, the face term splits into two halves; the
// neighbour's half at our face points is minus its own half at its face points (opposite normal,
// and two elements sharing a face parametrise it identically), so it is computed once, by its
// owner.  Each kernel writes only its own elements' outputs: no atomics.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dg_kernels.hpp"
#include "dg_launch.hpp"
#include "dg_tile.hpp"

namespace tetdg {

namespace {

// Viscous flux F_v,j (j = 0..2, rows of Fv) at one point from U and Z[k][w] = d_k U_w,
// constant mu, Fourier heat flux with kappa = mu gamma / ((gamma - 1) Pr), T = p / rho.
template <class T>
__device__ __forceinline__ void visc_flux(const T U[5], const T Z[3][5], T gm1, T mu, T kappa, T Fv[3][5]) {
  const T ir = T(1) / U[0];
  const T u[3] = {U[1] * ir, U[2] * ir, U[3] * ir};
  const T q2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
  const T p = gm1 * (U[4] - T(0.5) * U[0] * q2);
  const T tt = p * ir;
  T gu[3][3], gT[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    T ug = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      gu[k][i] = (Z[k][1 + i] - u[i] * Z[k][0]) * ir;
      ug += u[i] * gu[k][i];
    }
    const T gp = gm1 * (Z[k][4] - T(0.5) * q2 * Z[k][0] - U[0] * ug);
    gT[k] = (gp - tt * Z[k][0]) * ir;
  }
  const T div = gu[0][0] + gu[1][1] + gu[2][2];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    T e = kappa * gT[j];
    Fv[j][0] = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      T tij = mu * (gu[j][i] + gu[i][j]);
      if (i == j) tij -= T(2.0 / 3.0) * mu * div;
      Fv[j][1 + i] = tij;
      e += u[i] * tij;
    }
    Fv[j][4] = e;
  }
}

// One direction dd of one point j of the projection: acc[mt][v] += P(mt, qt, 4 dd + j) y[v].
template <class Pr, int MT, bool kTail4, class L>
__device__ __forceinline__ void project_dir(const typename Pr::Op* __restrict__ tab, int qt, int j, int dd, int lane,
                                            typename Pr::T (&y)[5], typename Pr::Acc (&acc)[MT][5]) {
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const typename Pr::Op av = tab[L::proj(mt, qt, 4 * dd + j) * 64 + lane];
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[mt][v] = mfma_tile<Pr, kTail4>(mt == MT - 1, av, y[v], acc[mt][v]);
  }
}

// One point lk of the lift of a face tile: acc[mt][v] += L(mt, f, ft, lk) h[v].
template <class Pr, int MT, bool kTail4, class L>
__device__ __forceinline__ void lift_point(const typename Pr::Op* __restrict__ tab, int f, int ft, int lk, int lane,
                                           typename Pr::T (&h)[5], typename Pr::Acc (&acc)[MT][5]) {
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const typename Pr::Op av = tab[L::lift(mt, f, ft, lk) * 64 + lane];
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[mt][v] = mfma_tile<Pr, kTail4>(mt == MT - 1, av, h[v], acc[mt][v]);
  }
}

// Sum the lane groups' shares of the short last tile (FP32, as in the stage kernel).
template <class Pr, class V>
__device__ __forceinline__ V finish_tail(V t) {
  if constexpr (!Pr::f64) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      auto x = t[j];
      x += __shfl_xor(x, 16);
      x += __shfl_xor(x, 32);
      t[j] = x;
    }
  }
  return t;
}

// One 16-element group per workgroup of four wavefronts, as in the split stage kernel: wavefront
// w takes face w and the volume point tiles w, w + 4, ... in both passes.
//   1. Lifting.  Both parts of Z are linear in the rows of M = |det J| J^-1: the volume
//      integrand's contravariant components are M[d][k] U, and the face normal is N_f,k =
//      sum_d M[d][k] n_f,d with the reference normals n_0 = (1, 1, 1), n_f = -e_(f-1).  So one
//      interpolation, one set of traces and three reference-direction sums
//        D_d = sum_q w_q dphi/dxi_d U(q) - sum_f n_f,d int_f Uhat phi
//      serve all three directions: Z_k = -(sum_d M[d][k] D_d) / |K|.  The same traces give the
//      inviscid face fluxes.  The wavefronts' shares of D_d meet in LDS, one direction at a time;
//      the (mode tile, variable) pairs of Z are dealt out over the wavefronts, which leave them in
//      LDS as MFMA operands: Z never reaches memory.
//   2. Fluxes at the volume points and the element's own face points from U and Z (both in LDS).
// Bound by latency at one or two waves per SIMD (P3 FP64: MFMA 0.38, VALU 0.22 of the time, waves waiting
// 0.23 of theirs).  Before, Z was written by one kernel (2.4 KB per element at P3 FP64) and read back for
// every point tile by a second one, a third added the neighbours' halves and the stage kernel the
// inviscid part.  Whole stage at 32^3 x 6 elements, before and now, us, Rusanov: FP64 P1 634 -> 543, P2
// 1172 -> 1134, P3 2475 -> 1840, P4 12554 -> 10498; FP32 413 -> 381, 764 -> 642, 1381 -> 890, 5163 -> 3603;
// at 384 elements FP64 P1 59 -> 21, P3 188 -> 49, FP32 P3 145 -> 35.  Tables staged in LDS and workgroups
// that sweep several groups were slower (P3 FP64 2308: the loop costs registers, 284 bytes per lane
// spilled).  FP64 P4 spills 1452 (Roe 1468) bytes per lane, the kernels before it 1252 and 212.
//
// Waves per SIMD: FP64 P2 at two spills 344 bytes per lane and is still the faster one (1139
// against 1279 us); FP32 P1 at three spills 12 (a step at 32^3 x 6 elements 14 % faster than at two).
template <int P, class Pr>
constexpr int ns_waves() {
  if (P == 1 && !Pr::f64) return 3;
  return P <= (Pr::f64 ? 2 : 3) ? 2 : 1;
}

template <int P, class Pr, bool kRoe>
__global__ __launch_bounds__(256, (ns_waves<P, Pr>())) void ns_kernel(ViscArgs a) {
  using O = Ord<P>;
  using L = Layout<P, 1>;
  using S = typename Pr::S;
  using T = typename Pr::T;
  using Op = typename Pr::Op;
  using Acc = typename Pr::Acc;
  constexpr int NP = O::NP, NQ = O::NQ, NF = O::NF, MT = O::MT, QT = O::QT, FT = O::FT, KS = L::KS;
  constexpr int NPQ = npq_of(NP), W = 4, NPAIR = MT * 5;
  constexpr bool kTail4 = NP - 16 * (MT - 1) <= 4;
  // FP32 P1: the viscous part in sums of its own, and Z's combination of the D_d (below) in fp64 FMAs.
  // With the differences of the fluxes in one sum the residual was up to 5 % further from 64 bits than
  // with the separate kernels' sums (mu = 1e-6 .. 100); now 4 % closer to 0.5 % further.  From P2 on the
  // four wavefronts' short sums outweigh the difference's rounding (16-33 % closer with one sum).
  constexpr bool kTwoSums = !Pr::f64 && P == 1;
  // the wavefronts' accumulators of one reduction; Z's operands between the two passes
  constexpr size_t kRed = sizeof(Acc) * W * NPAIR * 64, kZ = sizeof(Op) * 15 * KS * 64;
  __shared__ __align__(32) char lds_raw[kRed > kZ ? kRed : kZ];
  __shared__ Op lds_u[5 * KS * 64];
  Acc* const red = reinterpret_cast<Acc*>(lds_raw);
  Op* const lz = reinterpret_cast<Op*>(lds_raw);
  const Op* __restrict__ tab = reinterpret_cast<const Op*>(a.tab);
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const MeshView& mv = a.mesh;
  const int64_t epad = mv.epad;
  // each XCD owns a contiguous eighth of the groups (workgroups go round-robin over the XCDs)
  const int64_t ngroups = epad / 16, chunk = (ngroups + 7) / 8;
  const int64_t grp = (blockIdx.x % 8) * chunk + blockIdx.x / 8;
  if (grp >= ngroups) return;
  const uint32_t quad_bytes = (uint32_t)(epad * 4 * sizeof(S));
  const uint32_t var_bytes = quad_bytes * NPQ;
  // the fp64 output: in FP32 mode a variable of it may pass 4 GiB, in FP64 mode its offsets are the
  // state's (written as such: other expressions for them cost 80 bytes per lane of spills at P2)
  using RQ = typename std::conditional<Pr::f64, uint32_t, size_t>::type;
  const RQ r_quad = Pr::f64 ? (RQ)quad_bytes : (RQ)(epad * 4 * sizeof(double));
  const char* __restrict__ ubase = reinterpret_cast<const char*>(a.u);
  S* __restrict__ hb = reinterpret_cast<S*>(a.hbuf);
  const T gamma = T(a.gamma), gm1 = T(a.gamma - 1.0);
  const T mu = T(a.mu), kappa = T(a.mu * a.gamma / ((a.gamma - 1.0) * a.prandtl));
  T far[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) far[v] = T(a.far[v]);
  OperandMap<Pr, NP, KS> om;
  om.init(g, quad_bytes);
  // leave x (plus y where `on`) in red / the sum of what the wavefronts left there
  auto share = [&](const Acc (&x)[MT][5], const Acc (&y)[MT][5], bool on) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int v = 0; v < 5; ++v)
        red[(w * NPAIR + mt * 5 + v) * 64 + lane] = on ? x[mt][v] + y[mt][v] : x[mt][v];
    __syncthreads();
  };
  auto shared_sum = [&](int mt, int v) {
    d4_t t = __builtin_convertvector(red[(mt * 5 + v) * 64 + lane], d4_t);
#pragma unroll
    for (int x = 1; x < W; ++x) t += __builtin_convertvector(red[(x * NPAIR + mt * 5 + v) * 64 + lane], d4_t);
    return t;
  };


  const int e = (int)(grp * 16 + col);
  const bool live = e < mv.n_elem;
  const uint32_t eoff = (uint32_t)e * 4 * sizeof(S);
  double Md[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) Md[i] = mv.M[i * epad + e];
  T Mt[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) Mt[i] = T(Md[i]);
  const double ivol = mv.inv_vol[e];
  // always true, but a branch to the compiler: without it the face's loads and fluxes are
  // scheduled into the neighbouring phases (P3 FP64 then spills 176 bytes per lane)
  const bool face = w < 4;
  const int wf = face ? w : 0;
  const int nbf = mv.nbr[wf * epad + e];
  const int fpl = (mv.fcode[e] >> (2 * wf)) & 3;
  // the element's own operands, shared by the wavefronts
  for (int v = w; v < 5; v += W) {
    Op b[1][KS];
    load_operands<Pr, NP, KS, 1>(ubase + (size_t)v * var_bytes, var_bytes, eoff, om, b);
#pragma unroll
    for (int s = 0; s < KS; ++s) lds_u[(v * KS + s) * 64 + lane] = b[0][s];
  }
  Op bn[5][KS];
  if (face) load_operands<Pr, NP, KS>(ubase, var_bytes, (uint32_t)(nbf >= 0 ? nbf : e) * 4 * sizeof(S), om, bn);
  T N[3];
  face_normal<T>(wf, Md, N);
  __syncthreads();

  // U at the points of a tile by table t(s)
  auto own_u = [&](auto&& table, Acc (&d)[5]) {
#pragma unroll
    for (int v = 0; v < 5; ++v) d[v] = Acc{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const Op av = tab[table(s) * 64 + lane];
#pragma unroll
      for (int v = 0; v < 5; ++v) d[v] = Pr::mfma(av, lds_u[(v * KS + s) * 64 + lane], d[v]);
    }
  };

  Acc lift[MT][5];  // face w's share of D_(w-1) (face 0: of every D_d)
  Acc acc[MT][5];   // (V - S) - (Vv - Sv)
  Acc accv[MT][5];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int v = 0; v < 5; ++v) lift[mt][v] = acc[mt][v] = accv[mt][v] = Acc{0, 0, 0, 0};
  // up to P3 a wavefront has one tile of each kind and keeps the face's inviscid flux and the
  // volume points' U until pass 2; at P4 it lifts the flux at once and interpolates U again.  FP64 P2
  // with Roe's flux lifts it at once too: kept, the kernel spilled 476 bytes per lane instead of 220
  // and was slower than four separate kernels (a step at 32^3 x 6 elements: 4169 us kept, 3590 lifted
  // at once, 3650 in four kernels).
  constexpr bool kKeep = P <= 3;
  constexpr bool kLiftAtOnce = !kKeep || kTwoSums || (kRoe && Pr::f64 && P == 2);
  T fi[4][5];

  // ---------------- pass 1: face w, Uhat = (U- + U+)/2 and the inviscid flux
  if (face) {
    const T nn = sqrt(N[0] * N[0] + N[1] * N[1] + N[2] * N[2]);
#pragma unroll 1
    for (int ft = 0; ft < FT; ++ft) {
      Acc dm[5], dp[5];
      own_u([&](int s) { return L::trace(w, ft, s); }, dm);
#pragma unroll
      for (int v = 0; v < 5; ++v) dp[v] = Acc{0, 0, 0, 0};
#pragma unroll 1
      for (int c = 0; c < 4; ++c) {
        const bool mine = nbf >= 0 && fpl == c;
        if (__any(mine)) {
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            const Op av = tab[L::trace(c, ft, s) * 64 + lane];
#pragma unroll
            for (int v = 0; v < 5; ++v) dp[v] = Pr::mfma(av, mine ? bn[v][s] : Op(0), dp[v]);
          }
        }
      }
      // n_f,d Uhat: +Uhat for face 0 (all d), -Uhat for face f > 0 (d = f - 1)
      const T sgn = w == 0 ? T(0.5) : T(-0.5);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = 16 * ft + drow(Pr::f64, g, j);
        T um[5], up[5], uh[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          um[v] = T(dm[v][j]);
          up[v] = T(dp[v][j]);
        }
        if (nbf < 0) ghost_state<T>(-nbf, um, N, far, up);
        num_flux<kRoe, T>(um, up, N, nn, gamma, fi[j]);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          uh[v] = q < NF ? sgn * (um[v] + up[v]) : T(0);
          fi[j][v] = q < NF ? fi[j][v] : T(0);
        }
        lift_point<Pr, MT, kTail4, L>(tab, w, ft, j, lane, uh, lift);
        if constexpr (kLiftAtOnce) lift_point<Pr, MT, kTail4, L>(tab, w, ft, j, lane, fi[j], acc);
      }
    }
  }
  // ---------------- pass 1: U at the volume points of this wavefront's tiles
  constexpr int NT = (QT + W - 1) / W;
  Acc du1[NT][5];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int qt = w + W * t;
    if (qt >= QT) continue;
    own_u([&](int s) { return L::interp(qt, s); }, du1[t]);
    // points past the rule count as zero
#pragma unroll
    for (int v = 0; v < 5; ++v)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (16 * qt + drow(Pr::f64, g, j) >= NQ) du1[t][v][j] = 0;
  }

  // ---------------- Z_k = -(sum_d M[d][k] D_d) / |K|, pairs 5 mt + v = w (mod 4) per wavefront
  constexpr int NVW = (5 + W - 1) / W;
  auto pair_v = [&](int mt, int i) {
    const int v = w - 5 * mt % W;
    return (v < 0 ? v + W : v) + W * i;
  };
  {
    Acc z[MT][NVW][3];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < NVW; ++i) z[mt][i][0] = z[mt][i][1] = z[mt][i][2] = Acc{0, 0, 0, 0};
#pragma unroll
    for (int dd = 0; dd < 3; ++dd) {
      // this wavefront's share of D_dd: its volume tiles, and its face where n_f,dd is not zero
      const bool on = w == 0 || w == dd + 1;
      Acc D[MT][5];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int v = 0; v < 5; ++v) D[mt][v] = kTwoSums && on ? lift[mt][v] : Acc{0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (w + W * t >= QT) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          T y[5];
#pragma unroll
          for (int v = 0; v < 5; ++v) y[v] = T(du1[t][v][j]);
          project_dir<Pr, MT, kTail4, L>(tab, w + W * t, j, dd, lane, y, D);
        }
      }
      if (dd > 0) __syncthreads();  // the previous direction's shares are read
      share(D, lift, !kTwoSums && on);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < NVW; ++i) {
          const int v = pair_v(mt, i);
          if (v >= 5) continue;
          const d4_t t = shared_sum(mt, v);
#pragma unroll
          for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if constexpr (kTwoSums)
                z[mt][i][k][j] = T(fma(Md[3 * dd + k], t[j], double(z[mt][i][k][j])));
              else
                z[mt][i][k][j] = fmaT(Mt[3 * dd + k], T(t[j]), T(z[mt][i][k][j]));
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < NVW; ++i) {
        const int v = pair_v(mt, i);
        if (v >= 5) continue;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          T x[4];
          if constexpr (kTail4)
            if (mt == MT - 1) z[mt][i][k] = finish_tail<Pr>(z[mt][i][k]);
          // |K| is fp64 in every mode: one product, rounded once (an fp32 1/|K| would scale all of Z
          // by the same wrong factor)
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] = T(-ivol * double(z[mt][i][k][j]));
          Op* const zk = lz + (5 * k + v) * KS * 64;
          if constexpr (Pr::f64) {
            // register j of lane group g: mode 16 mt + g + 4 j, operand step 4 mt + j of this lane
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (4 * mt + j < KS) zk[(4 * mt + j) * 64 + lane] = x[j];
          } else if (kTail4 && mt == MT - 1) {
            // modes 16 mt .. + 3 in every lane group's registers: operand step 4 mt, mode 16 mt + g
            zk[4 * mt * 64 + lane] = g == 0 ? x[0] : g == 1 ? x[1] : g == 2 ? x[2] : x[3];
          } else if (4 * mt + g < KS) {
            // register j of lane group g: mode 16 mt + 4 g + j, step 4 mt + g of lane group j
#pragma unroll
            for (int j = 0; j < 4; ++j) zk[(4 * mt + g) * 64 + 16 * j + col] = x[j];
          }
        }
      }
    __syncthreads();
  }

  // ---------------- pass 2: U and Z at the points of a tile by table t(s)
  auto z_values = [&](auto&& table, Acc (&dz)[3][5]) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int v = 0; v < 5; ++v) dz[k][v] = Acc{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const Op av = tab[table(s) * 64 + lane];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int v = 0; v < 5; ++v) dz[k][v] = Pr::mfma(av, lz[((5 * k + v) * KS + s) * 64 + lane], dz[k][v]);
    }
  };
  auto point = [&](const Acc (&du)[5], const Acc (&dz)[3][5], int j, T (&U)[5], T (&Z)[3][5]) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      U[v] = T(du[v][j]);
#pragma unroll
      for (int k = 0; k < 3; ++k) Z[k][v] = T(dz[k][v][j]);
    }
  };
#pragma unroll 1
  for (int qt = w; qt < QT; qt += W) {
    Acc du[5], dz[3][5];
    if constexpr (kKeep) {
#pragma unroll
      for (int v = 0; v < 5; ++v) du[v] = du1[0][v];
    } else {
      own_u([&](int s) { return L::interp(qt, s); }, du);
    }
    z_values([&](int s) { return L::interp(qt, s); }, dz);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = 16 * qt + drow(Pr::f64, g, j);
      T U[5], Z[3][5], Fv[3][5], yy[3][5];
      point(du, dz, j, U, Z);
      visc_flux<T>(U, Z, gm1, mu, kappa, Fv);
      contra_flux<T>(U, Mt, gm1, yy);
#pragma unroll
      for (int dd = 0; dd < 3; ++dd) {
        T y[5], yv[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          yv[v] = Mt[3 * dd] * Fv[0][v] + Mt[3 * dd + 1] * Fv[1][v] + Mt[3 * dd + 2] * Fv[2][v];
          y[v] = q < NQ ? (kTwoSums ? yy[dd][v] : yy[dd][v] - yv[v]) : T(0);
          yv[v] = q < NQ ? -yv[v] : T(0);
        }
        if constexpr (kTwoSums) project_dir<Pr, MT, kTail4, L>(tab, qt, j, dd, lane, yv, accv);
        project_dir<Pr, MT, kTail4, L>(tab, qt, j, dd, lane, y, acc);
      }
    }
  }
  // face w: the own half (and, on a boundary face, the ghost half with Z+ = Z-)
#pragma unroll 1
  for (int ft = face ? 0 : FT; ft < FT; ++ft) {
    Acc du[5], dz[3][5];
    own_u([&](int s) { return L::trace(w, ft, s); }, du);
    z_values([&](int s) { return L::trace(w, ft, s); }, dz);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = 16 * ft + drow(Pr::f64, g, j);
      T U[5], Z[3][5], Fv[3][5], h[5];
      point(du, dz, j, U, Z);
      visc_flux<T>(U, Z, gm1, mu, kappa, Fv);
#pragma unroll
      for (int v = 0; v < 5; ++v) h[v] = Fv[0][v] * N[0] + Fv[1][v] * N[1] + Fv[2][v] * N[2];
      if (nbf < 0) {
        T Ub[5];
        ghost_state<T>(-nbf, U, N, far, Ub);
        visc_flux<T>(Ub, Z, gm1, mu, kappa, Fv);
#pragma unroll
        for (int v = 0; v < 5; ++v) h[v] += Fv[0][v] * N[0] + Fv[1][v] * N[1] + Fv[2][v] * N[2];
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        h[v] = q < NF ? T(0.5) * h[v] : T(0);
        fi[j][v] = kLiftAtOnce ? -h[v] : fi[j][v] - h[v];
      }
      lift_point<Pr, MT, kTail4, L>(tab, w, ft, j, lane, fi[j], kTwoSums ? accv : acc);
      // the own half of an interior face, for the neighbour's side of this face: per
      // (element, face, variable) 16 FT values, the point held in register j of lane
      // group g at 16 ft + 4 g + j, so that a reader's lane gets its four points at once
      if (nbf >= 0 && live) {
#pragma unroll
        for (int v = 0; v < 5; ++v) hb[((((size_t)e * 4 + w) * 5 + v) * FT + ft) * 16 + 4 * g + j] = S(h[v]);
      }
    }
  }

  // ---------------- the residual without the neighbours' halves, in fp64 from here to the end of the
  // update: the wavefronts' sums, 1/|K| and the store
  __syncthreads();
  d4_t own[kTwoSums ? NVW : 1];  // P1 (one mode tile): the inviscid part
  if constexpr (kTwoSums) {
    share(acc, acc, false);
#pragma unroll
    for (int i = 0; i < NVW; ++i)
      if (pair_v(0, i) < 5) own[i] = shared_sum(0, pair_v(0, i));
    __syncthreads();
  }
  share(kTwoSums ? accv : acc, acc, false);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < NVW; ++i) {
      const int v = pair_v(mt, i);
      if (v >= 5) continue;
      d4_t t = shared_sum(mt, v);
      if constexpr (kTwoSums) t += own[i];
      if (kTail4 && mt == MT - 1) t = finish_tail<Pr>(t);
      if (!live) continue;
      char* const ob = reinterpret_cast<char*>(a.out) + (size_t)v * (Pr::f64 ? (RQ)var_bytes : r_quad * NPQ) +
                       (Pr::f64 ? (RQ)eoff : (RQ)e * 4 * sizeof(double));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int mode = 16 * mt + drow(Pr::f64, g, j);
        if ((mode >> 2) < NPQ)
          *reinterpret_cast<double*>(ob + (RQ)(mode >> 2) * r_quad + (mode & 3) * sizeof(double)) =
              mode < NP ? ivol * t[j] : 0.0;
      }
    }
}

// Neighbour halves of the viscous face term, then the stage's update: R = R_own - (sum_f int_f
// (F_v+ . N / 2) phi) / |K| (with the lift tables' sign), where F_v+ . N / 2 at our face point q is
// minus the neighbour's stored own half at point q of its face f+; R is stored or U_out =
// alpha U0 + (1 - alpha)(U_in + dt R).  Bound by its reads (6 KB per element at P3 FP64): a light
// kernel, the lift tables read through the caches, several workgroups per CU.
template <int P, class Pr>
__global__ __launch_bounds__(256) void ns_update_kernel(ViscArgs a) {
  using O = Ord<P>;
  using L = Layout<P, 1>;
  using S = typename Pr::S;
  using T = typename Pr::T;
  using Op = typename Pr::Op;
  using Acc = typename Pr::Acc;
  constexpr int NP = O::NP, MT = O::MT, FT = O::FT;
  constexpr int NPQ = npq_of(NP);
  constexpr bool kTail4 = NP - 16 * (MT - 1) <= 4;
  const Op* __restrict__ tab = reinterpret_cast<const Op*>(a.tab);
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  const MeshView& mv = a.mesh;
  const int64_t epad = mv.epad;
  const uint32_t quad_bytes = (uint32_t)(epad * 4 * sizeof(S));
  const uint32_t var_bytes = quad_bytes * NPQ;
  const int64_t ngroups = epad / 16, nblk8 = gridDim.x / 8;
  const int64_t chunk = (ngroups + 7) / 8;
  const int64_t first = (blockIdx.x % 8) * chunk;
  const int64_t last = first + chunk < ngroups ? first + chunk : ngroups;
  const S* __restrict__ hb = reinterpret_cast<const S*>(a.hbuf);
  const double dt = a.dt_dev ? *a.dt_dev : a.dt;
  for (int64_t grp = first + (int64_t)(blockIdx.x / 8) * 4 + (threadIdx.x >> 6); grp < last; grp += nblk8 * 4) {
    const int e = (int)(grp * 16 + col);
    const int fcode = mv.fcode[e];
    int nbr[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) nbr[f] = mv.nbr[f * epad + e];
    Acc acc[MT][5];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int v = 0; v < 5; ++v) acc[mt][v] = Acc{0, 0, 0, 0};
#pragma unroll 1
    for (int f = 0; f < 4; ++f) {
      const int nbf = f == 0 ? nbr[0] : f == 1 ? nbr[1] : f == 2 ? nbr[2] : nbr[3];
      if (!__any(nbf >= 0)) continue;
      const int fpl = (fcode >> (2 * f)) & 3;
      const size_t rec = nbf >= 0 ? ((size_t)nbf * 4 + fpl) * 5 * FT * 16 : 0;
      typedef S s4_t __attribute__((ext_vector_type(4)));
#pragma unroll 1
      for (int ft = 0; ft < FT; ++ft) {
        T h[4][5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          // the neighbour's values at points 16 ft + drow(g, j), j = 0..3 (zero past N_f)
          const s4_t x = *reinterpret_cast<const s4_t*>(hb + rec + ((size_t)v * FT + ft) * 16 + 4 * g);
#pragma unroll
          for (int j = 0; j < 4; ++j) h[j][v] = nbf >= 0 ? T(x[j]) : T(0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) lift_point<Pr, MT, kTail4, L>(tab, f, ft, j, lane, h[j], acc);
      }
    }
    if constexpr (kTail4) {
#pragma unroll
      for (int v = 0; v < 5; ++v) acc[MT - 1][v] = finish_tail<Pr>(acc[MT - 1][v]);
    }
    // the padding's elements get zeros (a caller may reduce over the padded array)
    const bool live = e < mv.n_elem;
    const double ivol = mv.inv_vol[e];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const char* const ro = reinterpret_cast<const char*>(a.r_own) + (size_t)v * NPQ * epad * 4 * sizeof(double);
        auto update = [&](double own, double x, double u, double u0) {
          double r = own + ivol * x;
          if (a.rk) r = a.alpha * u0 + (1.0 - a.alpha) * (u + dt * r);
          return r;
        };
        if constexpr (Pr::f64) {
          // register j of lane group g: position g of quad 4 mt + j
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int mode = 16 * mt + drow(true, g, j);
            if ((mode >> 2) < NPQ) {
              const size_t q = ((size_t)(mode >> 2) * epad + e) * 4 + (mode & 3);
              auto at = [&](const void* p) {
                return reinterpret_cast<const double*>(reinterpret_cast<const char*>(p) + (size_t)v * var_bytes)[q];
              };
              const double r = update(reinterpret_cast<const double*>(ro)[q], acc[mt][v][j], a.rk ? at(a.u) : 0.0,
                                      a.rk && a.alpha != 0.0 ? at(a.u0) : 0.0);
              reinterpret_cast<double*>(reinterpret_cast<char*>(a.out) + (size_t)v * var_bytes)[q] =
                  mode < NP && live ? r : 0.0;
            }
          }
        } else if (4 * mt + g < NPQ) {
          // lane group g holds quad 4 mt + g whole: one vector access each (value by value, the kernel
          // moved 2.7 TB/s)
          typedef S s4_t __attribute__((ext_vector_type(4)));
          const size_t q = (size_t)(4 * mt + g) * epad + e;
          auto at = [&](const void* p) {
            return reinterpret_cast<const s4_t*>(reinterpret_cast<const char*>(p) + (size_t)v * var_bytes)[q];
          };
          const d4_t own = reinterpret_cast<const d4_t*>(ro)[q];
          s4_t u = {0, 0, 0, 0}, u0 = {0, 0, 0, 0}, o;
          if (a.rk) u = at(a.u);
          if (a.rk && a.alpha != 0.0) u0 = at(a.u0);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const double r = update(own[j], double(acc[mt][v][j]), double(u[j]), double(u0[j]));
            o[j] = S(16 * mt + 4 * g + j < NP && live ? r : 0.0);
          }
          reinterpret_cast<s4_t*>(reinterpret_cast<char*>(a.out) + (size_t)v * var_bytes)[q] = o;
        }
      }
  }
}

template <int P, class Pr>
hipError_t launch_ns_impl(const ViscArgs& a, hipStream_t stream) {
  const int64_t ngroups = a.mesh.epad / 16;
  auto kern = a.flux == 1 ? ns_kernel<P, Pr, true> : ns_kernel<P, Pr, false>;
  // one group per workgroup, the same number of workgroups on every XCD
  hipLaunchKernelGGL(kern, dim3((unsigned)((ngroups + 7) / 8 * 8)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

template <int P, class Pr>
hipError_t launch_ns_update_impl(const ViscArgs& a, hipStream_t stream) {
  auto kern = ns_update_kernel<P, Pr>;
  int per_cu = 0;
  hipError_t err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, 0);
  if (err != hipSuccess) return err;
  if (per_cu < 1) per_cu = 1;
  int dev = 0, ncu = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  const int64_t want = (a.mesh.epad / 16 + 3) / 4, fill = (int64_t)ncu * per_cu;
  const int64_t nblk = want < fill ? want : fill;
  hipLaunchKernelGGL(kern, dim3((unsigned)((nblk + 7) / 8 * 8)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ns(int p, int prec, const ViscArgs& a, hipStream_t stream) {
#define TDG_CASE(PP) \
  if (p == PP) return prec == 1 ? launch_ns_impl<PP, PrecF32>(a, stream) : launch_ns_impl<PP, PrecF64>(a, stream);
  TDG_CASE(1) TDG_CASE(2) TDG_CASE(3) TDG_CASE(4)
#undef TDG_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_ns_update(int p, int prec, const ViscArgs& a, hipStream_t stream) {
#define TDG_CASE(PP)                                                                   \
  if (p == PP)                                                                         \
    return prec == 1 ? launch_ns_update_impl<PP, PrecF32>(a, stream) : launch_ns_update_impl<PP, PrecF64>(a, stream);
  TDG_CASE(1) TDG_CASE(2) TDG_CASE(3) TDG_CASE(4)
#undef TDG_CASE
  return hipErrorInvalidValue;
}

}  // namespace tetdg
