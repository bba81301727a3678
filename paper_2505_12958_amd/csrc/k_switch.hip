// Dynamic switching parameter (paper: section "Adaptive-precision potential"
// and the appendix "Switching function" with the table of the adaptive-
// precision model's parameters), in the ACE-weight convention
// mu = 1 - lambda_paper:
//
//  1. CSP_i: the n/2 smallest |d_a + d_b|^2 over the pairs of the n nearest
//     neighbours (n = 14 for BCC), summed in ascending order; fewer than n
//     neighbours within the cutoff: (n/2) (2 r_c)^2;
//  2. time average c_i <- c_i + (CSP_i - c_i)/N_csp; detection mu0_i: 0 below
//     CSP_lo, 1 above CSP_hi, a cosine ramp between; 1 inside the precise
//     ball, 0 for surface atoms outside it;
//  3. spatial transition mu_i = max_j mu0_j g(r_ij), g = 1 up to r_lo, a
//     cosine down to 0 at r_hi;
//  4. time average m_i <- m_i + (mu_i - m_i)/N_lambda; lambda_i = m_i snapped
//     to 0 / 1 within dlambda_min; the ascending list of atoms with
//     lambda_i > 0.
//
// Every decision (which neighbours, which pair sums, inside or outside a
// zone or the transition range) is taken on FP64 values computed in a fixed
// operation order with nothing contracted, so it is bit-exact against any
// implementation of the same recipe; the max of step 3 does not depend on
// the order in which sources are combined.
#include "ap_internal.h"
#include "geom.h"
#include "scan.h"

#include <algorithm>

namespace ap {

constexpr int kCspWaves = 4;
constexpr int kMaxCsp = 16;

// (key, index) order: smaller key first, equal keys by index
__device__ __forceinline__ bool before(double a, int ia, double b, int ib) {
  return a < b || (a == b && ia < ib);
}

__device__ __forceinline__ double lane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Smallest value of the wavefront, by lane exchanges in registers.
__device__ __forceinline__ unsigned wave_min_u32(unsigned v) {
  v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xf, 0xf, true));   // lane ^ 1
  v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xf, 0xf, true));   // lane ^ 2
  v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xf, 0xf, true));  // half rows mirrored
  v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xf, 0xf, true));  // rows mirrored
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = min(r[0], r[1]);
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return min(h[0], h[1]);
}

// ---- 1. CSP, one wavefront per atom.
// Only the set of the n nearest matters, since the pair sums commute, and only
// the n/2 smallest sums in their order.  Both are found on FP32 keys (rounding
// keeps the order, up to ties): the n-th smallest distance by bisection of the
// key's bits with one ballot a step, the sums one after the other by a
// wavefront minimum.  A tie of keys that would decide is resolved on the FP64
// values.  Ranking all distances and all pair sums against each other in FP64
// took about 1200 of the kernel's 1600 vector instructions per atom (103,000
// atoms: 267 us, 77 us so).
// kR: candidates per lane; sel: the n nearest displacements
template <int kR>
__device__ __forceinline__ double csp_row(const SysView& sv, const double* __restrict__ pos,
                                          const int32_t* __restrict__ nbr, int i, int c, int n_csp,
                                          double* sel, int lane) {
#pragma clang fp contract(off)
  constexpr unsigned kNone = 0xffffffffu;
  const int n = sv.n_atoms;
  const int s = sv.sys_of[i];
  const bool ortho = sv.ortho[s] != 0;
  const double* H = sv.H + 9 * s;
  const double* Hi = sv.Hi + 9 * s;
  const double xi = pos[i], yi = pos[n + i], zi = pos[2 * n + i];
  double dx[kR], dy[kR], dz[kR], r2[kR] = {};
  unsigned key[kR];
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    key[r] = kNone;
    if (64 * r + lane < c) {
      const int j = nbr[(int64_t)(64 * r + lane) * n + i];
      displacement(ortho, H, Hi, sv.per, xi, yi, zi, pos[j], pos[n + j], pos[2 * n + j], dx[r], dy[r], dz[r]);
      r2[r] = norm2(dx[r], dy[r], dz[r]);
      key[r] = __float_as_uint((float)r2[r]);
    }
  }
  // the n-th smallest key: from the sorted keys of a row of one candidate per
  // lane, else the largest that fewer than n candidates lie below, bit by bit
  unsigned nth = 0;
  if constexpr (kR == 1) {
    // (non-negative floats order like signed integers too)
    nth = __builtin_amdgcn_readlane(wave_sort((int)min(key[0], 0x7fffffffu)), n_csp - 1);
  } else {
    for (int bit = 30; bit >= 0; --bit) {
      const unsigned t = nth | 1u << bit;
      int below = 0;
#pragma unroll
      for (int r = 0; r < kR; ++r) below += __popcll(__ballot(key[r] < t));
      if (below < n_csp) nth = t;
    }
  }
  int below = 0, upto = 0;
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    below += __popcll(__ballot(key[r] < nth));
    upto += __popcll(__ballot(key[r] <= nth));
  }
  int at = 0;
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    bool take = key[r] <= nth;
    if (upto > n_csp && key[r] == nth) {
      // more candidates share the n-th key than places are left: the first
      // of them in (r^2, slot) order; slots are in ascending neighbour index
      int rank = below;
#pragma unroll
      for (int q = 0; q < kR; ++q)
        for (int l = 0; l < 64; ++l) {
          const unsigned k = __builtin_amdgcn_readlane(key[q], l);
          const double v = lane_f64(r2[q], l);
          rank += k == nth && before(v, 64 * q + l, r2[r], 64 * r + lane) ? 1 : 0;
        }
      take = rank < n_csp;
    }
    const unsigned long long b = __ballot(take);
    const int p = at + __popcll(b & ((1ull << lane) - 1ull));
    if (take && p < n_csp) {
      double* o = sel + 3 * p;
      o[0] = dx[r];
      o[1] = dy[r];
      o[2] = dz[r];
    }
    at += __popcll(b);
  }
  __syncwarp_ap();
  // pair sums |d_a + d_b|^2, a < b: at most 120, two per lane
  const int np = n_csp * (n_csp - 1) / 2;
  double sum[2] = {};
  unsigned sk[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int q = 64 * r + lane;
    sk[r] = kNone;
    if (q < np) {
      const int m = 2 * n_csp - 1;
      int a = (int)((m - sqrtf((float)(m * m - 8 * q))) * 0.5f);
      if (a * (m - a) / 2 > q) --a;
      if ((a + 1) * (m - a - 1) / 2 <= q) ++a;
      const int b = a + 1 + q - a * (m - a) / 2;
      const double sx = sel[3 * a] + sel[3 * b];
      const double sy = sel[3 * a + 1] + sel[3 * b + 1];
      const double sz = sel[3 * a + 2] + sel[3 * b + 2];
      sum[r] = norm2(sx, sy, sz);
      sk[r] = __float_as_uint((float)sum[r]);
    }
  }
  // the n/2 smallest, in ascending order (equal values are interchangeable)
  double t = 0.0;
  for (int k = 0; k < n_csp / 2; ++k) {
    const unsigned mine = min(sk[0], sk[1]);
    const unsigned m = __builtin_amdgcn_readfirstlane(wave_min_u32(mine));
    unsigned long long b0 = __ballot(sk[0] == m), b1 = __ballot(sk[1] == m);
    int l = __ffsll(b0 | b1) - 1;
    bool second = !(b0 >> l & 1);
    double v = lane_f64(second ? sum[1] : sum[0], l);
    if (__popcll(b0) + __popcll(b1) > 1) {
      // of the sums with this key, the smallest
      for (unsigned long long x = b0 | b1; x; x &= x - 1) {
        const int y = __ffsll(x) - 1;
        const double u0 = lane_f64(sum[0], y), u1 = lane_f64(sum[1], y);
        if ((b0 >> y & 1) && u0 < v) { v = u0; l = y; second = false; }
        if ((b1 >> y & 1) && u1 < v) { v = u1; l = y; second = true; }
      }
    }
    t += v;
    if (lane == l) {
      if (second) sk[1] = kNone;
      else sk[0] = kNone;
    }
  }
  return t;
}

__global__ __launch_bounds__(64 * kCspWaves) void k_csp(SysView sv, const double* __restrict__ pos,
                                                        const int32_t* __restrict__ nbr,
                                                        const int32_t* __restrict__ count,
                                                        int n_csp, double csp_full,
                                                        double* __restrict__ csp) {
#pragma clang fp contract(off)
  __shared__ double lds[kCspWaves][3 * kMaxCsp];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = sv.n_atoms;
  const int i = xcd_chunk(blockIdx.x, gridDim.x) * kCspWaves + wave;
  if (i >= n) return;  // whole wavefront
  double* sel = lds[wave];  // [n][3]
  const int c = __builtin_amdgcn_readfirstlane(count[i]);
  if (c < n_csp) {
    if (lane == 0) csp[i] = csp_full;
    return;
  }
  // (rows beyond 64 entries keep up to four candidates per lane)
  const double t = c <= 64 ? csp_row<1>(sv, pos, nbr, i, c, n_csp, sel, lane)
                           : csp_row<kMaxCap / 64>(sv, pos, nbr, i, c, n_csp, sel, lane);
  if (lane == 0) csp[i] = t;
}

struct SwitchArgs {
  double csp_lo, csp_hi, r_lo, r_hi, n_csp_avg, n_lam_avg, dmin;
  double cx, cy, cz, r_precise, zsurf;
  int32_t init;
};

__device__ __forceinline__ double ramp_csp(double c, double lo, double hi) {
#pragma clang fp contract(off)
  if (c <= lo) return 0.0;
  if (c >= hi) return 1.0;
  return 0.5 * (1.0 - cos(M_PI * ((c - lo) / (hi - lo))));
}

// ---- 2. averaged CSP, detection value and fixed zones; flags of the sources
__global__ void k_switch_detect(int n, const double* __restrict__ pos, const double* __restrict__ csp,
                                double* __restrict__ c_avg, SwitchArgs a, double* __restrict__ mu0,
                                int32_t* __restrict__ flag) {
#pragma clang fp contract(off)
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double c = csp[i];
  const double ca = a.init ? c : c_avg[i] + (c - c_avg[i]) / a.n_csp_avg;
  c_avg[i] = ca;
  double m = ramp_csp(ca, a.csp_lo, a.csp_hi);
  const double x = pos[i], y = pos[n + i], z = pos[2 * n + i];
  bool inside = false;
  if (a.r_precise > 0.0) {
    const double dx = x - a.cx, dy = y - a.cy, dz = z - a.cz;
    inside = norm2(dx, dy, dz) <= a.r_precise * a.r_precise;
  }
  if (inside) m = 1.0;
  else if (z >= a.zsurf) m = 0.0;
  mu0[i] = m;
  flag[i] = m > 0.0 ? 1 : 0;
}

// ---- 3. spatial transition: one wavefront per source, the cells within
// r_hi of it (cell edge >= cutoff), max-combined into mu (FP64 bit patterns
// of non-negative values order like unsigned integers)
__global__ __launch_bounds__(256) void k_switch_spread(
    SysView sv, const double* __restrict__ pos, const int32_t* __restrict__ cell_of,
    const int32_t* __restrict__ cell_start, const int32_t* __restrict__ cell_count,
    const int32_t* __restrict__ cell_atoms, const double4* __restrict__ cell_pos,
    const int32_t* __restrict__ src, const int32_t* __restrict__ n_src_p,
    const double* __restrict__ mu0, SwitchArgs a, unsigned long long* __restrict__ mu_bits) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  const int n_src = *n_src_p;
  const int n = sv.n_atoms;
  const double rh2 = a.r_hi * a.r_hi;
  for (int w = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); w < n_src;
       w += gridDim.x * (blockDim.x >> 6)) {
    const int j = src[w];
    const double mj = mu0[j];
    const int s = sv.sys_of[j];
    const int* g = sv.grid + 3 * s;
    const double* H = sv.H + 9 * s;
    const int local = cell_of[j] - sv.cell_base[s];
    const int c0 = local / (g[1] * g[2]), c1 = (local / g[2]) % g[1], c2 = local % g[2];
    int R[3], lo[3], cnt[3];
    const int cc[3] = {c0, c1, c2};
    for (int k = 0; k < 3; ++k) {
      const double edge = H[4 * k] / g[k];
      R[k] = (int)ceil(a.r_hi / edge);
      if (sv.per[k] && 2 * R[k] + 1 >= g[k]) {
        lo[k] = 0;
        cnt[k] = g[k];
      } else {
        lo[k] = cc[k] - R[k];
        cnt[k] = 2 * R[k] + 1;
      }
    }
    const double xj = pos[j], yj = pos[n + j], zj = pos[2 * n + j];
    const int ncell = cnt[0] * cnt[1] * cnt[2];
    for (int q = lane; q < ncell; q += 64) {
      int o0 = lo[0] + q / (cnt[1] * cnt[2]);
      int o1 = lo[1] + (q / cnt[2]) % cnt[1];
      int o2 = lo[2] + q % cnt[2];
      const int o[3] = {o0, o1, o2};
      bool ok = true;
      int w3[3];
      for (int k = 0; k < 3; ++k) {
        int v = o[k];
        if (sv.per[k]) v = ((v % g[k]) + g[k]) % g[k];
        else if (v < 0 || v >= g[k]) ok = false;
        w3[k] = v;
      }
      if (!ok) continue;
      const int cell = sv.cell_base[s] + (w3[0] * g[1] + w3[1]) * g[2] + w3[2];
      const int b = cell_start[cell], e = b + cell_count[cell];
      for (int t = b; t < e; ++t) {
        const double4 p = cell_pos[t];
        double dx, dy, dz;
        displacement_ortho(sv.per, H[0], H[4], H[8], xj, yj, zj, p.x, p.y, p.z, dx, dy, dz);
        const double r2 = norm2(dx, dy, dz);
        if (r2 < rh2) {
          const double r = sqrt(r2);
          const double gr =
              r <= a.r_lo ? 1.0 : 0.5 * (1.0 + cos((M_PI * (r - a.r_lo)) / (a.r_hi - a.r_lo)));
          const double v = mj * gr;
          if (v > 0.0) atomicMax(&mu_bits[cell_atoms[t]], (unsigned long long)__double_as_longlong(v));
        }
      }
    }
  }
}

// ---- 4. averaged mu, snapping, flags of the ACE list
__global__ void k_switch_finish(int n, const unsigned long long* __restrict__ mu_bits,
                                double* __restrict__ m_avg, SwitchArgs a, double* __restrict__ lambda,
                                int32_t* __restrict__ flag) {
#pragma clang fp contract(off)
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double mu = __longlong_as_double((long long)mu_bits[i]);
  const double m = a.init ? mu : m_avg[i] + (mu - m_avg[i]) / a.n_lam_avg;
  m_avg[i] = m;
  const double l = m < a.dmin ? 0.0 : (m > 1.0 - a.dmin ? 1.0 : m);
  lambda[i] = l;
  flag[i] = l > 0.0 ? 1 : 0;
}

hipError_t launch_switching(const SysView& sv, const double* pos, const int32_t* nbr,
                            const int32_t* count, const int32_t* cell_of,
                            const int32_t* cell_start, const int32_t* cell_count,
                            const int32_t* cell_atoms, const double4* cell_pos,
                            const ap_switching& sw, double csp_full, double* csp, double* mu0,
                            unsigned long long* mu_bits, int32_t* flag, int32_t* src, int32_t* n_src,
                            int32_t* scan_tmp, double* lambda, int32_t* ace_list, int32_t* n_ace,
                            hipStream_t s) {
  const int n = sv.n_atoms;
  SwitchArgs a;
  a.csp_lo = sw.csp_lo;
  a.csp_hi = sw.csp_hi;
  a.r_lo = sw.r_lo;
  a.r_hi = sw.r_hi;
  a.n_csp_avg = (double)sw.n_csp_avg;
  a.n_lam_avg = (double)sw.n_lambda_avg;
  a.dmin = sw.dlambda_min;
  a.cx = sw.centre[0];
  a.cy = sw.centre[1];
  a.cz = sw.centre[2];
  a.r_precise = sw.r_precise;
  a.zsurf = sw.z_surface_min;
  a.init = sw.initialised ? 0 : 1;
  if (n > 0) {
    hipLaunchKernelGGL(k_csp, dim3((n + kCspWaves - 1) / kCspWaves), dim3(64 * kCspWaves), 0, s, sv,
                       pos, nbr, count, sw.n_csp, csp_full, csp);
    hipLaunchKernelGGL(k_switch_detect, dim3((n + 255) / 256), dim3(256), 0, s, n, pos, csp, sw.csp_avg,
                       a, mu0, flag);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = launch_compact(n, flag, src, n_src, scan_tmp, s)) != hipSuccess) return e;
  if ((e = launch_fill_i32(reinterpret_cast<int32_t*>(mu_bits), 0, 2 * (int64_t)n, s)) != hipSuccess) return e;
  if (n > 0) {
    const int blocks = std::min((n + 3) / 4, 65536);
    hipLaunchKernelGGL(k_switch_spread, dim3(blocks), dim3(256), 0, s, sv, pos, cell_of, cell_start,
                       cell_count, cell_atoms, cell_pos, src, n_src, mu0, a, mu_bits);
    hipLaunchKernelGGL(k_switch_finish, dim3((n + 255) / 256), dim3(256), 0, s, n, mu_bits,
                       sw.lambda_avg, a, lambda, flag);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_compact(n, flag, ace_list, n_ace, scan_tmp, s);
}

}  // namespace ap
