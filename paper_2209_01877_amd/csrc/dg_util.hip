// Layout conversion, quadrature-point coordinates and L2 projection kernels.
#include <hip/hip_runtime.h>

#include "dg_launch.hpp"

namespace tetdg {

namespace {

// Layout conversion between the caller's records ([E][5][N_p] doubles, caller's order) and the
// internal quads, 32 consecutive internal elements per workgroup through LDS, so that both sides
// move whole lines: a record is 40 N_p contiguous bytes, a (variable, quad) plane of the tile 32
// contiguous quads.  (One thread per element, striding over either side, moved 1.2 TB/s.)  An LDS
// record is 5 N_p + 1 doubles.
constexpr int kTileE = 32;

template <int P, class S>
__global__ __launch_bounds__(256) void set_state_kernel(MeshView m, const double* __restrict__ user,
                                                        S* __restrict__ out) {
  constexpr int NP = Ord<P>::NP, NPQ = npq_of(NP), REC = 5 * NP;
  __shared__ double tile[kTileE * (REC + 1)];
  const int64_t e0 = (int64_t)blockIdx.x * kTileE;
  __shared__ int perm[kTileE];
  if (threadIdx.x < kTileE) perm[threadIdx.x] = m.perm[e0 + threadIdx.x];
  __syncthreads();
  // all of a thread's reads are issued before the first LDS write
  constexpr int NIT = (kTileE * REC + 255) / 256;
  double x[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = (int)threadIdx.x + 256 * it;
    if (i < kTileE * REC) x[it] = user[(int64_t)perm[i / REC] * REC + i % REC];
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = (int)threadIdx.x + 256 * it;
    if (i < kTileE * REC) tile[i / REC * (REC + 1) + i % REC] = x[it];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 5 * NPQ * kTileE * 4; i += 256) {
    const int el = (i / 4) % kTileE, vk = i / (4 * kTileE), mode = 4 * (vk % NPQ) + i % 4;
    out[((int64_t)vk * m.epad + e0 + el) * 4 + i % 4] =
        mode < NP ? S(tile[el * (REC + 1) + vk / NPQ * NP + mode]) : S(0);
  }
}

template <int P, class S>
__global__ __launch_bounds__(256) void get_state_kernel(MeshView m, const S* __restrict__ in,
                                                        double* __restrict__ user) {
  constexpr int NP = Ord<P>::NP, NPQ = npq_of(NP), REC = 5 * NP;
  __shared__ double tile[kTileE * (REC + 1)];
  const int64_t e0 = (int64_t)blockIdx.x * kTileE;
  for (int i = threadIdx.x; i < 5 * NPQ * kTileE * 4; i += 256) {
    const int el = (i / 4) % kTileE, vk = i / (4 * kTileE), mode = 4 * (vk % NPQ) + i % 4;
    const S x = in[((int64_t)vk * m.epad + e0 + el) * 4 + i % 4];
    if (mode < NP) tile[el * (REC + 1) + vk / NPQ * NP + mode] = double(x);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kTileE * REC; i += 256) {
    const int el = i / REC, k = i % REC;
    if (e0 + el < m.n_elem) user[(int64_t)m.perm[e0 + el] * REC + k] = tile[el * (REC + 1) + k];
  }
}

// Points x = X0 + J xi_q, 32 elements per workgroup: their maps are staged in LDS, and every
// wavefront writes an element's 3 N_q coordinates as one run.
template <int P>
__global__ __launch_bounds__(256) void volume_points_kernel(MeshView m, RefView r, double* __restrict__ xyz) {
  constexpr int NQ = Ord<P>::NQ;
  __shared__ double map[12 * kTileE], xi[3 * NQ];
  const int64_t e0 = (int64_t)blockIdx.x * kTileE;
  for (int i = threadIdx.x; i < 12 * kTileE; i += 256) map[i] = m.x0j[(i / kTileE) * m.epad + e0 + i % kTileE];
  for (int i = threadIdx.x; i < 3 * NQ; i += 256) xi[i] = r.qx[i];
  __syncthreads();
  for (int el = threadIdx.x >> 6; el < kTileE; el += 4) {
    if (e0 + el >= m.n_elem) break;
    double* const dst = xyz + (int64_t)m.perm[e0 + el] * (3 * NQ);
    for (int i = threadIdx.x & 63; i < 3 * NQ; i += 64) {
      const int q = i / 3, d = i % 3;
      double x = map[d * kTileE + el];
      for (int c = 0; c < 3; ++c) x += map[(3 + 3 * d + c) * kTileE + el] * xi[3 * q + c];
      dst[i] = x;
    }
  }
}

// fp64 MFMA column tiles as in the stage kernel (16 elements per wavefront), for every state type.
typedef double util_d4 __attribute__((ext_vector_type(4)));

// c_i = (1/|K|) int_K U phi_i = 6 sum_q w_q U(x_q) phi_i(xi_q): rows = modes, k = points (lane group
// g holds point 4 s + g of step s and converts it once), the short last mode tile on the blocked
// 4x4x4 MFMA.  (One thread per (element, mode) converted every point N_p times.)
template <int P, class S>
__global__ __launch_bounds__(256) void project_kernel(MeshView m, RefView r, double gamma,
                                                      const double* __restrict__ prim, S* __restrict__ out) {
  constexpr int NP = Ord<P>::NP, NQ = Ord<P>::NQ, MT = Ord<P>::MT, NPQ = npq_of(NP), QS = (NQ + 3) / 4;
  constexpr bool kTail4 = NP - 16 * (MT - 1) <= 4;
  __shared__ double tab[MT * QS * 64];
  for (int i = threadIdx.x; i < MT * QS * 64; i += 256) {
    const int l = i % 64, st = i / 64 % QS, mt = i / 64 / QS;
    const int row = kTail4 && mt == MT - 1 ? l % 4 : l % 16, mode = 16 * mt + row, q = 4 * st + l / 16;
    tab[i] = mode < NP && q < NQ ? 6.0 * r.qw[q] * r.B[q * NP + mode] : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  const int64_t ngroups = m.epad / 16, stride = (int64_t)gridDim.x * 4;
  for (int64_t grp = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); grp < ngroups; grp += stride) {
    const int64_t e = grp * 16 + col;
    const double* const src = prim + (int64_t)m.perm[e] * (5 * NQ);
    util_d4 acc[MT][5];
    for (int mt = 0; mt < MT; ++mt)
      for (int v = 0; v < 5; ++v) acc[mt][v] = util_d4{0, 0, 0, 0};
#pragma unroll 4
    for (int st = 0; st < QS; ++st) {
      const bool in = 4 * st + g < NQ;
      const int q = in ? 4 * st + g : NQ - 1;
      const double rho = src[5 * q], u = src[5 * q + 1], v = src[5 * q + 2], w = src[5 * q + 3], p = src[5 * q + 4];
      const double U[5] = {rho, rho * u, rho * v, rho * w, p / (gamma - 1.0) + 0.5 * rho * (u * u + v * v + w * w)};
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const double a = tab[(mt * QS + st) * 64 + lane];
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          const double b = in ? U[c] : 0.0;  // past the rule: an infinity times a zero weight would be NaN
          if (kTail4 && mt == MT - 1)
            acc[mt][c][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, acc[mt][c][0], 0, 0, 0);
          else
            acc[mt][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[mt][c], 0, 0, 0);
        }
      }
    }
    // register j of lane group g: mode 16 mt + g + 4 j
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int c = 0; c < 5; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (4 * mt + j < NPQ)
            out[(((int64_t)c * NPQ + 4 * mt + j) * m.epad + e) * 4 + g] =
                16 * mt + 4 * j + g < NP ? S(acc[mt][c][j]) : S(0);
  }
}

// Integrated slip-wall pressure J = sum_{wall faces} sum_q 2 A_f w^f_q p(U-_q) and dJ/dU,
// one thread per element (fp64).  J accumulates atomically into *J (zeroed by the caller).
template <class S>
__global__ void wall_pressure_kernel(MeshView m, int np, int nf, RefView r, double gamma, const S* __restrict__ u,
                                     double* __restrict__ J, S* __restrict__ grad) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= m.epad) return;
  const double gm1 = gamma - 1.0;
  double Jloc = 0.0;
  const bool real = e < m.n_elem;
  if (grad)
    for (int v = 0; v < 5; ++v)
      for (int i = 0; i < 4 * npq_of(np); ++i) grad[sidx(v, i, e, m.epad, npq_of(np))] = S(0);
  for (int f = 0; f < 4 && real; ++f) {
    if (m.nbr[f * m.epad + e] != -2) continue;
    double Mr[9];
    for (int k = 0; k < 9; ++k) Mr[k] = m.M[k * m.epad + e];
    double N[3];
    for (int c = 0; c < 3; ++c)
      N[c] = f == 0 ? (Mr[c] + Mr[3 + c] + Mr[6 + c]) : f == 1 ? -Mr[c] : f == 2 ? -Mr[3 + c] : -Mr[6 + c];
    const double area2 = sqrt(N[0] * N[0] + N[1] * N[1] + N[2] * N[2]);  // 2 A_f
    for (int q = 0; q < nf; ++q) {
      const double* bq = r.Bf + ((int64_t)f * nf + q) * np;
      double U[5] = {0, 0, 0, 0, 0};
      for (int v = 0; v < 5; ++v)
        for (int i = 0; i < np; ++i) U[v] += bq[i] * double(u[sidx(v, i, e, m.epad, npq_of(np))]);
      const double ir = 1.0 / U[0];
      const double vel[3] = {U[1] * ir, U[2] * ir, U[3] * ir};
      const double q2 = vel[0] * vel[0] + vel[1] * vel[1] + vel[2] * vel[2];
      const double p = gm1 * (U[4] - 0.5 * U[0] * q2);
      const double wq = area2 * r.fw[q];
      Jloc += wq * p;
      if (grad) {
        const double dp[5] = {gm1 * 0.5 * q2, -gm1 * vel[0], -gm1 * vel[1], -gm1 * vel[2], gm1};
        for (int v = 0; v < 5; ++v)
          for (int i = 0; i < np; ++i) {
            S* gp = grad + sidx(v, i, e, m.epad, npq_of(np));
            *gp = S(double(*gp) + wq * dp[v] * bq[i]);
          }
      }
    }
  }
  if (Jloc != 0.0) atomicAdd(J, Jloc);
}

// Global minimum of the local explicit steps dt_K = cfl d_K / ((2p+1)(|u_K| + c_K)) over
// the cell means, d_K = 6|K| / sum_f A_f (the paper's minimum of local time steps, here a
// wavefront shuffle reduction per block and one atomic minimum on the bit pattern of a
// non-negative double; 0 when some cell mean is inadmissible).
__global__ void local_dt_kernel(MeshView m, int np, double gamma, double scale, const void* u, int f32,
                                unsigned long long* out) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  double dt = 1e300;
  if (e < m.n_elem) {
    double U[5];
    for (int v = 0; v < 5; ++v) {
      const int64_t idx = sidx(v, 0, e, m.epad, npq_of(np));
      U[v] = f32 ? double(((const float*)u)[idx]) : ((const double*)u)[idx];
    }
    const double ir = 1.0 / U[0];
    const double q2 = (U[1] * U[1] + U[2] * U[2] + U[3] * U[3]) * ir * ir;
    const double p = (gamma - 1.0) * (U[4] - 0.5 * U[0] * q2);
    const double lam = sqrt(q2) + sqrt(gamma * p * ir);
    double Mr[9], area2 = 0.0;
    for (int k = 0; k < 9; ++k) Mr[k] = m.M[k * m.epad + e];
    for (int f = 0; f < 4; ++f) {
      double N[3];
      for (int c = 0; c < 3; ++c)
        N[c] = f == 0 ? (Mr[c] + Mr[3 + c] + Mr[6 + c]) : f == 1 ? -Mr[c] : f == 2 ? -Mr[3 + c] : -Mr[6 + c];
      area2 += sqrt(N[0] * N[0] + N[1] * N[1] + N[2] * N[2]);  // 2 A_f
    }
    const double vol = 1.0 / m.inv_vol[e];
    const double d = 12.0 * vol / area2;  // 6 |K| / sum A_f
    dt = scale * d / lam;
    // an inadmissible cell mean (rho or p not positive, or not finite) gives a NaN, zero or
    // infinite local step: it becomes 0, so that the minimum reports it (a NaN would be
    // dropped by the comparisons below and by the atomic minimum on the bit pattern)
    if (!(dt > 0.0 && dt <= 1.79e308)) dt = 0.0;
  }
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_down(dt, off, 64);
    dt = o < dt ? o : dt;
  }
  __shared__ double wmin[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) wmin[w] = dt;
  __syncthreads();
  if (threadIdx.x == 0) {
    double b = wmin[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) b = wmin[i] < b ? wmin[i] : b;
    unsigned long long bits;
    __builtin_memcpy(&bits, &b, 8);
    atomicMin(out, bits);
  }
}

__global__ void fill_u64_kernel(unsigned long long* p, unsigned long long v) { *p = v; }

inline int np_of(int p) { return (p + 1) * (p + 2) * (p + 3) / 6; }
inline unsigned nblocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }


// Streaming probe: 16-byte accesses over caller buffers, grid-strided, non-temporal except
// kind 3.  kind 0 copies src to dst, kind 1 reads src (its XOR reduction reaches dst[0] only
// for one bit pattern, so the loads stay live), kind 2 zero-fills dst, kind 3 reads src with
// ordinary (cache-allocating) loads: repeated over a buffer that fits the last-level cache,
// it measures that cache's bandwidth.
typedef unsigned stream_u4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(512) void stream_kernel(int kind, const stream_u4* __restrict__ src,
                                                     stream_u4* __restrict__ dst, int64_t n16) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (kind == 0) {
    for (; i < n16; i += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
  } else if (kind == 1 || kind == 3) {
    stream_u4 x = {0u, 0u, 0u, 0u};
    if (kind == 1)
      for (; i < n16; i += stride) x ^= __builtin_nontemporal_load(src + i);
    else
      for (; i < n16; i += stride) x ^= src[i];
    if (x[0] == 0x9e3779b9u && x[1] == 0x7f4a7c15u && x[2] == 0xf39cc060u && x[3] == 0x5ced1e02u) dst[0] = x;
  } else {
    const stream_u4 z = {0u, 0u, 0u, 0u};
    for (; i < n16; i += stride) __builtin_nontemporal_store(z, dst + i);
  }
}

// Admissibility check: U at the volume quadrature points in fp64 (rows = points, k = modes, as the
// stage kernel's interpolation) and one count per element where any value is not finite or the
// density or pressure is not positive.  The count accumulates atomically into *n_bad, once per
// workgroup.  (One thread per element read its coefficients again for every point.)
template <int P, class S>
__global__ __launch_bounds__(256) void check_state_kernel(MeshView m, RefView r, double gamma,
                                                          const S* __restrict__ u,
                                                          unsigned long long* __restrict__ n_bad) {
  constexpr int NP = Ord<P>::NP, NQ = Ord<P>::NQ, QT = Ord<P>::QT, NPQ = npq_of(NP), KS = NPQ;
  __shared__ double tab[QT * KS * 64];
  __shared__ int count;
  if (threadIdx.x == 0) count = 0;
  for (int i = threadIdx.x; i < QT * KS * 64; i += 256) {
    const int l = i % 64, st = i / 64 % KS, q = 16 * (i / 64 / KS) + l % 16, mode = 4 * st + l / 16;
    tab[i] = q < NQ && mode < NP ? r.B[q * NP + mode] : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  const int64_t ngroups = m.epad / 16, stride = (int64_t)gridDim.x * 4;
  int found = 0;
  for (int64_t grp = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); grp < ngroups; grp += stride) {
    const int64_t e = grp * 16 + col;
    double b[5][KS];
#pragma unroll
    for (int c = 0; c < 5; ++c)
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        const S x = u[(((int64_t)c * NPQ + st) * m.epad + e) * 4 + g];
        b[c][st] = 4 * st + g < NP ? double(x) : 0.0;
      }
    bool bad = false;
#pragma unroll 1
    for (int qt = 0; qt < QT; ++qt) {
      util_d4 d[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) d[c] = util_d4{0, 0, 0, 0};
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        const double a = tab[(qt * KS + st) * 64 + lane];
#pragma unroll
        for (int c = 0; c < 5; ++c) d[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[c][st], d[c], 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double U[5] = {d[0][j], d[1][j], d[2][j], d[3][j], d[4][j]};
        const double p = (gamma - 1.0) * (U[4] - 0.5 * (U[1] * U[1] + U[2] * U[2] + U[3] * U[3]) / U[0]);
        bool finite = true;
#pragma unroll
        for (int c = 0; c < 5; ++c) finite = finite && isfinite(U[c]);
        if (16 * qt + g + 4 * j < NQ) bad = bad || !finite || !(U[0] > 0.0) || !(p > 0.0);
      }
    }
    unsigned long long any = __ballot(bad && e < m.n_elem);  // lane groups of an element: bits col + 16 g
    any |= any >> 32;
    any |= any >> 16;
    found += __popcll(any & 0xffffull);
  }
  if (lane == 0 && found) atomicAdd(&count, found);
  __syncthreads();
  if (threadIdx.x == 0 && count) atomicAdd(n_bad, (unsigned long long)count);
}

// Persistent column-tile launch: one wavefront per 16 elements, at most four workgroups per CU.
unsigned tile_blocks(const MeshView& m) {
  int dev = 0, ncu = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  const int64_t want = (m.epad / 16 + 3) / 4, fill = (int64_t)ncu * 4;
  return (unsigned)(want < fill ? want : fill);
}

}  // namespace

// Launch kernel<P, S> with S the mode's state type.
#define TDG_BY_ORDER(KERNEL, GRID, ...)                                                              \
  do {                                                                                               \
    switch (p) {                                                                                     \
      case 1: TDG_BY_STATE(KERNEL, 1, GRID, __VA_ARGS__); break;                                     \
      case 2: TDG_BY_STATE(KERNEL, 2, GRID, __VA_ARGS__); break;                                     \
      case 3: TDG_BY_STATE(KERNEL, 3, GRID, __VA_ARGS__); break;                                     \
      case 4: TDG_BY_STATE(KERNEL, 4, GRID, __VA_ARGS__); break;                                     \
      default: return hipErrorInvalidValue;                                                          \
    }                                                                                                \
    return hipGetLastError();                                                                        \
  } while (0)
#define TDG_BY_STATE(KERNEL, PP, GRID, ...)                                                          \
  do {                                                                                               \
    if (prec == 1) {                                                                                 \
      using S = float;                                                                               \
      hipLaunchKernelGGL((KERNEL<PP, S>), dim3(GRID), dim3(256), 0, s, __VA_ARGS__);                 \
    } else {                                                                                         \
      using S = double;                                                                              \
      hipLaunchKernelGGL((KERNEL<PP, S>), dim3(GRID), dim3(256), 0, s, __VA_ARGS__);                 \
    }                                                                                                \
  } while (0)

hipError_t launch_set_state(int p, int prec, const MeshView& m, const double* user, void* internal, hipStream_t s) {
  TDG_BY_ORDER(set_state_kernel, nblocks(m.epad, kTileE), m, user, (S*)internal);
}

hipError_t launch_get_state(int p, int prec, const MeshView& m, const void* internal, double* user, hipStream_t s) {
  TDG_BY_ORDER(get_state_kernel, nblocks(m.epad, kTileE), m, (const S*)internal, user);
}

hipError_t launch_volume_points(int p, const MeshView& m, const RefView& r, double* xyz, hipStream_t s) {
  const dim3 grid(nblocks(m.n_elem, kTileE)), block(256);
  switch (p) {
    case 1: hipLaunchKernelGGL(volume_points_kernel<1>, grid, block, 0, s, m, r, xyz); break;
    case 2: hipLaunchKernelGGL(volume_points_kernel<2>, grid, block, 0, s, m, r, xyz); break;
    case 3: hipLaunchKernelGGL(volume_points_kernel<3>, grid, block, 0, s, m, r, xyz); break;
    case 4: hipLaunchKernelGGL(volume_points_kernel<4>, grid, block, 0, s, m, r, xyz); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_wall_pressure(int p, int prec, const MeshView& m, const RefView& r, double gamma, const void* u,
                                double* J, void* grad, hipStream_t s) {
  const int np = np_of(p), nf = (p + 1) * (p + 1);
  hipLaunchKernelGGL(fill_u64_kernel, dim3(1), dim3(1), 0, s, (unsigned long long*)J, 0ULL);
  if (prec == 1)
    hipLaunchKernelGGL(wall_pressure_kernel<float>, dim3(nblocks(m.epad, 128)), dim3(128), 0, s, m, np, nf, r, gamma,
                       (const float*)u, J, (float*)grad);
  else
    hipLaunchKernelGGL(wall_pressure_kernel<double>, dim3(nblocks(m.epad, 128)), dim3(128), 0, s, m, np, nf, r,
                       gamma, (const double*)u, J, (double*)grad);
  return hipGetLastError();
}

hipError_t launch_check_state(int p, int prec, const MeshView& m, const RefView& r, double gamma, const void* u,
                              int64_t* n_bad, hipStream_t s) {
  hipLaunchKernelGGL(fill_u64_kernel, dim3(1), dim3(1), 0, s, (unsigned long long*)n_bad, 0ULL);
  TDG_BY_ORDER(check_state_kernel, tile_blocks(m), m, r, gamma, (const S*)u, (unsigned long long*)n_bad);
}

hipError_t launch_local_dt(int p, int prec, const MeshView& m, double gamma, double cfl, const void* u, double* dt,
                           hipStream_t s) {
  // start from +inf (bit pattern 0x7ff0...); the first atomic minimum replaces it
  hipLaunchKernelGGL(fill_u64_kernel, dim3(1), dim3(1), 0, s, (unsigned long long*)dt, 0x7ff0000000000000ULL);
  hipLaunchKernelGGL(local_dt_kernel, dim3(nblocks(m.n_elem, 256)), dim3(256), 0, s, m, np_of(p), gamma,
                     cfl / (2 * p + 1), u, prec == 1 ? 1 : 0, (unsigned long long*)dt);
  return hipGetLastError();
}

hipError_t launch_project(int p, int prec, const MeshView& m, const RefView& r, double gamma, const double* prim,
                          void* internal, hipStream_t s) {
  // padding elements map to caller element 0 (perm), so every row is a valid state
  TDG_BY_ORDER(project_kernel, tile_blocks(m), m, r, gamma, prim, (S*)internal);
}

hipError_t launch_stream_probe(int kind, const void* src, void* dst, size_t bytes, hipStream_t s) {
  const int64_t n16 = (int64_t)(bytes / 16);
  int64_t nb = (n16 + 511) / 512;
  if (nb > 65536) nb = 65536;  // grid-strided beyond 32 M threads
  hipLaunchKernelGGL(stream_kernel, dim3((unsigned)nb), dim3(512), 0, s, kind, (const stream_u4*)src, (stream_u4*)dst,
                     n16);
  return hipGetLastError();
}

}  // namespace tetdg
