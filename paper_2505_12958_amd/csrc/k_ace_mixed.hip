// ACE part of the AP force: bond basis (kernel 1), embedding and bond
// gradients (kernel 3) of both precisions and the launchers of the three
// phases; the rank kernels (phase 1) are in k_ace_rank32.hip (mixed) and
// k_ace_rank64.hip (FP64).
#include "ace_basis.h"
#include "ap_internal.h"
#include "geom.h"
#include "scan.h"

#include <algorithm>
#include <type_traits>

namespace ap {

// ---- kernel 1: bond basis and atomic basis A, one wavefront per ACE atom
constexpr int kBasisWaves = 4;
// The number of listed atoms is on the device.  Up to kBondAtoms atoms every four
// have a workgroup, which leaves at once beyond the list; beyond, kBondGrid
// workgroups take the items in turn (kLoop).  An empty workgroup costs 0.2 ns:
// 2.66 million atoms, 37,000 listed, kernel 1 and 3 240 + 259 -> 107 + 131 us;
// the loop costs registers: 370,000 atoms, all listed, 506 + 824 -> 551 + 898 us.
constexpr int kBondAtoms = 524288;
constexpr int kBondGrid = 8192;

// T: the arithmetic of the precision (float: mixed, double: FP64).  NM, LM,
// KK > 0: model shape fixed at compile time (n_max, l_max, K), so
// every loop over radial and angular indices unrolls with constant trip
// counts and the radial weights are read as scalar loads at constant
// offsets; NM = 0: the shape is read from the model at run time.  Items
// item0 .. item0 + n_buf - 1 of the list; A_out and bn_out (mixed only) hold
// these n_buf items.
template <typename T, int NM, int LM, int KK, bool kLoop>
__global__ __launch_bounds__(64 * kBasisWaves) void k_ace_basis(
    SysView sv, BondDev<T> m, const double* __restrict__ pos, const double4* __restrict__ pos4,
    const int32_t* __restrict__ nbr, const int32_t* __restrict__ count, int cap,
    const int32_t* __restrict__ ace_list,
    const int32_t* __restrict__ n_ace_p, int n_all, int item0, int n_buf, T* __restrict__ A_out,
    float* __restrict__ bn_out, int32_t* __restrict__ nbr_ace, int32_t* __restrict__ halo,
    int32_t stamp) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_max = NM ? NM : m.n_max, l_max = NM ? LM : m.l_max, K = NM ? KK : m.K;
  const int lp1 = l_max + 1, nlm = lp1 * lp1, nnl = n_max * lp1, nA = n_max * nlm;
  // per bond the Chebyshev values g_k and the harmonics Y_lm go to LDS; the
  // wavefront sums B[k][lm] = sum_j g_k(r_j) Y_lm(u_j) and contracts with the
  // radial weights once per atom: A_nlm = sum_k W_nlk B[k][lm]
  const int nB = K * nlm;
  const int stride = K + nlm;
  T* RY = reinterpret_cast<T*>(lds) + wave * 64 * stride;
  const int n = sv.n_atoms;
  const int n_items = ace_list ? *n_ace_p : n_all;
  const int n_local = min(n_buf, n_items - item0);
  for (int local = blockIdx.x * kBasisWaves + wave; local < n_local; local += gridDim.x * kBasisWaves) {
  const int item = item0 + local;
  const int a = ace_list ? ace_list[item] : item;
  const int c = count[a];
  const int sy = sv.sys_of[a];
  const T rc = (T)m.rc;
  T acc[(kMaxN * kMaxLM + 63) / 64];
#pragma unroll
  for (int q = 0; q < (kMaxN * kMaxLM + 63) / 64; ++q) acc[q] = 0;
  // the atom and its neighbours carry an ACE force term: stamped for the gather
  if (lane == 0) halo[a] = stamp;
  for (int base = 0; base < c; base += 64) {
    const int s = base + lane;
    T* o = RY + lane * stride;
    if (s < c) {
      const int j = nbr[(int64_t)s * n + a];
      nbr_ace[(int64_t)item * cap + s] = j;  // the row again, atom-major, for the force gather
      halo[j] = stamp;
      double dx, dy, dz;
      displacement(sv.ortho[sy] != 0, sv.H + 9 * sy, sv.Hi + 9 * sy, sv.per, pos[a], pos[n + a],
                   pos[2 * n + a], pos4[j].x, pos4[j].y, pos4[j].z, dx, dy, dz);
      const T fx = (T)dx, fy = (T)dy, fz = (T)dz;
      const T r = t_sqrt<T>(fx * fx + fy * fy + fz * fz);
      T g[kMaxK], dg[kMaxK];
      cheb_basis<T>(K, rc, r, g, dg);
#pragma unroll
      for (int k = 0; k < kMaxK; ++k)
        if (k < K) o[k] = g[k];
      T Y[kMaxLM];
      const T ir = (T)1 / r;
      real_ylm<T>(l_max, m.ynorm, fx * ir, fy * ir, fz * ir, r, Y, nullptr);
#pragma unroll
      for (int q = 0; q < kMaxLM; ++q)
        if (q < nlm) o[K + q] = Y[q];
    } else {
      for (int q = 0; q < stride; ++q) o[q] = 0;
    }
    __syncwarp_ap();
    const int nb = min(64, c - base);
#pragma unroll
    for (int r = 0; r < (kMaxN * kMaxLM + 63) / 64; ++r) {
      const int e = lane + 64 * r;
      if (e >= nB) break;
      const int k = e / nlm, lm = e - k * nlm;
      T v = 0;
      const T* ga = RY + k;
      const T* ya = RY + K + lm;
#pragma unroll 4
      for (int s2 = 0; s2 < nb; ++s2) v += ga[s2 * stride] * ya[s2 * stride];
      acc[r] += v;
    }
    __syncwarp_ap();
  }
  // B through LDS (the staging area is free now), then A = W B
  T* B = RY;
  T Asq[(kMaxN * kMaxLM + 63) / 64];
#pragma unroll
  for (int r = 0; r < (kMaxN * kMaxLM + 63) / 64; ++r) Asq[r] = 0;
#pragma unroll
  for (int r = 0; r < (kMaxN * kMaxLM + 63) / 64; ++r) {
    const int e = lane + 64 * r;
    if (e < nB) B[e] = acc[r];
  }
  __syncwarp_ap();
#pragma unroll
  for (int r = 0; r < (kMaxN * kMaxLM + 63) / 64; ++r) {
    const int e = lane + 64 * r;
    if (e >= nA) continue;
    const int nn = e / nlm, lm = e - nn * nlm;
    int l = 0;
    while ((l + 1) * (l + 1) <= lm) ++l;
    const T* w = m.W + (nn * lp1 + l) * K;
    T v = 0;
#pragma unroll
    for (int k = 0; k < kMaxK; ++k)
      if (k < K) v += w[k] * B[k * nlm + lm];
    A_out[(int64_t)local * nA + e] = v;
    Asq[r] = v * v;
  }
  if constexpr (sizeof(T) == 8) {
    if constexpr (!kLoop) return;
    __syncwarp_ap();
    continue;
  }  // (the FP64 rank kernels scale nothing)
  // largest |A_(n,l)|^2 over the atom's single indices: it bounds every entry
  // of the coupled operand and fixes the atom's power-of-two scale there
  T* Q = RY + nB;
  __syncwarp_ap();
#pragma unroll
  for (int r = 0; r < (kMaxN * kMaxLM + 63) / 64; ++r) {
    const int e = lane + 64 * r;
    if (e < nA) Q[e] = Asq[r];
  }
  __syncwarp_ap();
  T bq = 0;
  if (lane < nnl) {
    const int nn = lane / lp1, l = lane - nn * lp1;
    for (int q = 0; q <= 2 * l; ++q) bq += Q[nn * nlm + l * l + q];
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) bq = max(bq, __shfl_xor(bq, d, 64));
  if (lane == 0) bn_out[local] = (float)bq;
  if constexpr (!kLoop) return;
  __syncwarp_ap();  // the staging area is written again
  }
}

// ---- kernel 3: embedding (FP64), bond gradients and virial, one wavefront per atom.
// The neighbours come from the atom-major rows that kernel 1 wrote, and the nine
// virial sums share their exchanges (250,000 atoms 104 -> 82 us; 370,000, all
// listed, 910 -> 812).
// om_in: the two sets are n_buf * nA apart
template <typename T, int NM, int LM, int KK, bool kLoop>
__global__ __launch_bounds__(64 * kBasisWaves) void k_ace_grad(
    SysView sv, BondDev<T> m, const double* __restrict__ pos, const double4* __restrict__ pos4,
    const int32_t* __restrict__ count, int cap, const double* __restrict__ lambda,
    const int32_t* __restrict__ ace_list, const int32_t* __restrict__ n_ace_p, int n_all,
    int item0, int n_buf, const int32_t* __restrict__ nbr_ace, const T* __restrict__ A_in,
    const T* __restrict__ om_in, const T* __restrict__ phi_in, T* __restrict__ pair_g, double* __restrict__ e_atom,
    double* __restrict__ vir, double* __restrict__ e_raw, int vir_acc) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  T* om = reinterpret_cast<T*>(lds) + wave * (m.apad + kMaxLM * kMaxK);
  T* Om = om + m.apad;  // [nlm][K]
  const int n = sv.n_atoms;
  const int n_items = ace_list ? *n_ace_p : n_all;
  const int n_local = min(n_buf, n_items - item0);
  const int64_t plane = (int64_t)n_buf * m.nA;
  auto om_at = [&](int64_t o, int p) {
    return (double)om_in[o + p * plane];
  };
  for (int local = blockIdx.x * kBasisWaves + wave; local < n_local; local += gridDim.x * kBasisWaves) {
  const int item = item0 + local;
  const int a = ace_list ? ace_list[item] : item;
  const double lam = lambda ? lambda[a] : 1.0;
  // phi_p = X.Z/2 summed over L.  X rows are homogeneous in A of degree 2
  // (coupled channels), 1 (A rows) and 0 (constant row); by Euler's theorem
  // phi_p = (A . dphi_p/dA + S_A + 2 Z_1)/4 with S_A = A.Z over the A rows and
  // Z_1 the constant row, accumulated in phi_in.
  double d1 = 0.0, d2 = 0.0;
  for (int e = lane; e < m.nA; e += 64) {
    const int64_t o = (int64_t)local * m.nA + e;
    const double av = (double)A_in[o];
    d1 += av * om_at(o, 0);
    d2 += av * om_at(o, 1);
  }
  d1 = wave_sum_f64(d1);
  d2 = wave_sum_f64(d2);
  const double p1 = 0.25 * (d1 + (double)phi_in[2 * (int64_t)local]);
  const double p2 = 0.25 * (d2 + (double)phi_in[2 * (int64_t)local + 1]);
  const double root = sqrt(fabs(p2) + 1e-6);
  const double E = p1 + root;
  const double sp = (p2 >= 0.0 ? 1.0 : -1.0) / (2.0 * root);
  for (int e = lane; e < m.nA; e += 64) {
    const int64_t o = (int64_t)local * m.nA + e;
    om[e] = (T)(lam * (om_at(o, 0) + sp * om_at(o, 1)));
  }
  __syncwarp_ap();
  const int c = count[a];
  const int sy = sv.sys_of[a];
  const int n_max = NM ? NM : m.n_max, l_max = NM ? LM : m.l_max, K = NM ? KK : m.K;
  const int lp1 = l_max + 1, nlm = lp1 * lp1;
  const T rc = (T)m.rc;
  // omega contracted with the radial weights once per atom:
  // Om[lm][k] = sum_n omega_nlm W_nlk, so that for every bond
  // sum_n omega_nlm R_nl = sum_k Om[lm][k] g_k (and likewise with g_k')
  for (int e = lane; e < nlm * K; e += 64) {
    const int q = e / K, k = e - q * K;
    int l = 0;
    while ((l + 1) * (l + 1) <= q) ++l;
    T acc = 0;
    for (int nn = 0; nn < n_max; ++nn) acc += om[nn * nlm + q] * m.W[(nn * lp1 + l) * K + k];
    Om[e] = acc;
  }
  __syncwarp_ap();
  double w9[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int s = lane; s < c; s += 64) {
    const int j = nbr_ace[(int64_t)item * cap + s];
    double dx, dy, dz;
    displacement(sv.ortho[sy] != 0, sv.H + 9 * sy, sv.Hi + 9 * sy, sv.per, pos[a], pos[n + a],
                 pos[2 * n + a], pos4[j].x, pos4[j].y, pos4[j].z, dx, dy, dz);
    const T fx = (T)dx, fy = (T)dy, fz = (T)dz;
    const T r = t_sqrt<T>(fx * fx + fy * fy + fz * fz);
    const T ir = (T)1 / r;
    T g[kMaxK], dg[kMaxK];
    cheb_basis<T>(K, rc, r, g, dg);
    T ca[kMaxLM], cb[kMaxLM];
#pragma unroll
    for (int q = 0; q < kMaxLM; ++q) {
      ca[q] = 0;
      cb[q] = 0;
      if (q < nlm) {
#pragma unroll
        for (int k = 0; k < kMaxK; ++k)
          if (k < K) {
            const T w = Om[q * K + k];
            ca[q] += w * g[k];
            cb[q] += w * dg[k];
          }
      }
      // compiler barrier: the loads of one row stay with it, so the row's
      // weights are the only ones live at a time
      asm volatile("" ::: "memory");
    }
    T rad, gx, gy, gz;
    ylm_contract<T>(l_max, m.ynorm, fx * ir, fy * ir, fz * ir, r, ca, cb, rad, gx, gy, gz);
    gx += rad * fx * ir;
    gy += rad * fy * ir;
    gz += rad * fz * ir;
    T* o = pair_g + ((int64_t)item * cap + s) * 3;
    o[0] = gx; o[1] = gy; o[2] = gz;
    w9[0] -= dx * gx; w9[1] -= dx * gy; w9[2] -= dx * gz;
    w9[3] -= dy * gx; w9[4] -= dy * gy; w9[5] -= dy * gz;
    w9[6] -= dz * gx; w9[7] -= dz * gy; w9[8] -= dz * gz;
  }
  if (vir) {
    const double w = wave_sums_f64(w9, lane);
    const int k = (lane >> 5 & 1) + (lane >> 4 & 1) * 2 + (lane >> 3 & 1) * 4 + (lane >> 2 & 1) * 8;
    if ((lane & 3) == 0 && k < 9) {
      double* v = vir + (int64_t)k * n + a;
      *v = vir_acc ? *v + w : w;
    }
  }
  if (lane == 0) {
    e_atom[a] += lam * E;
    if (e_raw) e_raw[a] = E;
  }
  if constexpr (!kLoop) return;
  __syncwarp_ap();  // om and Om are written again
  }
}

// kernels 1 and 3 of one precision over the items item0 .. item0 + n_buf - 1
// (wavefronts past *n_ace leave at once, or take every so many items up to it)
template <typename T>
static hipError_t launch_bonds(const BondDev<T>& m, const SysView& sv, const BondArgs& b, int phase,
                               int item0, int n_buf, T* pair_g, T* A_buf, T* om_buf, T* phi_buf,
                               float* bn_buf, hipStream_t s) {
  const int items = std::min(n_buf, b.n_atoms - item0);
  if (items <= 0) return hipSuccess;
  const int nlm = (m.l_max + 1) * (m.l_max + 1);
  const bool loop = b.n_atoms > kBondAtoms;
  const int groups = (items + kBasisWaves - 1) / kBasisWaves;
  const dim3 grid(loop ? std::min(groups, kBondGrid) : groups), block(64 * kBasisWaves);
  const size_t lds = kBasisWaves * sizeof(T) *
                     (phase == 0 ? (size_t)64 * (m.K + nlm) : (size_t)(m.apad + kMaxLM * kMaxK));
  auto attr = [&](auto kern) {
    return lds <= 65536 ? hipSuccess
                        : hipFuncSetAttribute((const void*)kern,
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  };
  auto basis = [&](auto kern) {
    const hipError_t e = attr(kern);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, lds, s, sv, m, b.pos, b.pos4, b.nbr, b.count, b.cap,
                       b.ace_list, b.n_ace, b.n_atoms, item0, n_buf, A_buf, bn_buf, b.nbr_ace, b.halo,
                       b.stamp);
    return hipGetLastError();
  };
  auto grad = [&](auto kern) {
    const hipError_t e = attr(kern);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, lds, s, sv, m, b.pos, b.pos4, b.count, b.cap,
                       b.lambda, b.ace_list, b.n_ace, b.n_atoms, item0, n_buf, b.nbr_ace, A_buf, om_buf, phi_buf,
                       pair_g, b.e_atom, b.vir_atom, b.e_raw, b.vir_acc ? 1 : 0);
    return hipGetLastError();
  };
  const bool w844 = m.n_max == 8 && m.l_max == 4 && m.K == 8;
  const bool s633 = m.n_max == 6 && m.l_max == 3 && m.K == 6;
  auto run = [&](auto lp) {
    constexpr bool kLoop = decltype(lp)::value;
    if (phase == 0)
      return w844 ? basis(k_ace_basis<T, 8, 4, 8, kLoop>)
                  : s633 ? basis(k_ace_basis<T, 6, 3, 6, kLoop>) : basis(k_ace_basis<T, 0, 0, 0, kLoop>);
    return w844 ? grad(k_ace_grad<T, 8, 4, 8, kLoop>)
                : s633 ? grad(k_ace_grad<T, 6, 3, 6, kLoop>) : grad(k_ace_grad<T, 0, 0, 0, kLoop>);
  };
  return loop ? run(std::true_type{}) : run(std::false_type{});
}

hipError_t launch_ace_bonds64(const Ctx& c, const SysView& sv, const BondArgs& b, int phase, int item0,
                              int n_buf, double* pair_g, double* A_buf, double* om_buf,
                              double* phi_buf, hipStream_t s) {
  const AceDev& a = c.ace;
  return launch_bonds<double>({a.n_max, a.l_max, a.K, a.nA, a.nA | 1, a.rc, a.W, a.ynorm}, sv, b, phase,
                              item0, n_buf, pair_g, A_buf, om_buf, phi_buf, nullptr, s);
}

hipError_t launch_ace_rank64(const Ctx& c, const int32_t* n_ace, int n_atoms, int item0, int n_buf,
                             double* A_buf, double* om_buf, double* phi_buf, hipStream_t s) {
  int dev = 0, n_cu = 256;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int tiles = (std::min(n_buf, n_atoms - item0) + kT64 - 1) / kT64;
  if (tiles <= 0) return hipSuccess;
  for (int L = 0; L <= c.ace.L_max; ++L) {
    const Rank64L& P = c.r64_lv[L];
    if (P.nrow == 0) continue;
    const void* fn = nullptr;
    const bool sm = P.small != 0;
    switch (L) {
      case 0: fn = rank64_kernel<0>(sm); break;
      case 1: fn = rank64_kernel<1>(sm); break;
      case 2: fn = rank64_kernel<2>(sm); break;
      case 3: fn = rank64_kernel<3>(sm); break;
      case 4: fn = rank64_kernel<4>(sm); break;
      case 5: fn = rank64_kernel<5>(sm); break;
      case 6: fn = rank64_kernel<6>(sm); break;
      case 7: fn = rank64_kernel<7>(sm); break;
      default: fn = rank64_kernel<8>(sm); break;
    }
    const size_t lds = c.r64_lds[L];
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int per_cu = sm ? 2 : 1;
    void* args[] = {(void*)&c.r64, (void*)&P, (void*)&n_ace, (void*)&n_atoms, (void*)&item0,
                    (void*)&n_buf, (void*)&A_buf, (void*)&om_buf, (void*)&phi_buf};
    e = hipLaunchKernel(fn, dim3(std::min(tiles, n_cu * per_cu)), dim3(64 * kRank64Waves), args, lds, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t launch_ace_mixed(const Ctx& c, const SysView& sv, const BondArgs& b, float* pair_g, float* A_buf, float* om_buf, float* phi_buf,
                            float* bn_buf, hipStream_t s, int phase, int rank_mode) {
  const MixDev& m = c.mix;
  const int n_atoms = b.n_atoms;
  if (phase != 1)
    return launch_bonds<float>({m.n_max, m.l_max, m.K, m.nA, m.apad, m.rc, m.Wf, m.ynorm}, sv, b, phase,
                               0, n_atoms, pair_g, A_buf, om_buf, phi_buf, bn_buf, s);
  int dev = 0, n_cu = 256;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int32_t* na = b.ace_list ? b.n_ace : nullptr;
  const int tiles = (n_atoms + kMT32 - 1) / kMT32;
  if (tiles == 0) return hipSuccess;
  const int v = rank_mode == AP_RANK_NARROW ? 0 : 1;
  for (int L = 0; L <= m.L_max; ++L) {
    const Rank32L& P = c.r32_lv[v][L];
    if (P.nrow == 0) continue;
    const void* fn = nullptr;
    const bool sm = P.small != 0;
    switch (L) {
      case 0: fn = rank32_kernel<0>(sm); break;
      case 1: fn = rank32_kernel<1>(sm); break;
      case 2: fn = rank32_kernel<2>(sm); break;
      case 3: fn = rank32_kernel<3>(sm); break;
      case 4: fn = rank32_kernel<4>(sm); break;
      case 5: fn = rank32_kernel<5>(sm); break;
      case 6: fn = rank32_kernel<6>(sm); break;
      case 7: fn = rank32_kernel<7>(sm); break;
      default: fn = rank32_kernel<8>(sm); break;
    }
    const int nw = sm ? kRank32WavesSmall : rank32_waves(L);
    const size_t lds = c.r32_lds[v][L];
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int per_cu = std::min<int>(rank32_groups(L, nw), 160 * 1024 / lds);
    void* args[] = {(void*)&c.r32, (void*)&P, (void*)&na, (void*)&n_atoms, (void*)&A_buf,
                    (void*)&om_buf, (void*)&phi_buf, (void*)&bn_buf};
    e = hipLaunchKernel(fn, dim3(std::min(tiles, n_cu * per_cu)), dim3(64 * nw), args, lds, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace ap
