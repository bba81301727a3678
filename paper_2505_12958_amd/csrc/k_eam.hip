// EAM part of the AP force: two gather passes over the full ELL lists, no
// atomics.  Paper, section "EAM potential": E_i = xi(sum_j zeta(r_ij)) +
// 1/2 sum_j Phi(r_ij); with weights w_i = 1 - lambda_i the force on atom k is
// F_k = sum_j [(w_k xi'_k + w_j xi'_j) zeta'(r) + (w_k + w_j) Phi'(r)/2] d_kj/r.
#include "ap_internal.h"
#include "geom.h"

#include <algorithm>
#include <type_traits>

namespace ap {

// coef: the table's (n-1) double4 coefficients, in global memory or staged in LDS
__device__ __forceinline__ void tab_eval(const TableDev& t, const double4* coef, double x,
                                         bool linear_beyond, double& v, double& dv) {
  int k = (int)floor((x - t.x0) * t.inv_dx);
  k = k < 0 ? 0 : (k > t.n - 2 ? t.n - 2 : k);
  const double u = x - (t.x0 + k * t.dx);
  const double4 c = coef[k];
  v = c.x + u * (c.y + u * (c.z + u * c.w));
  dv = c.y + u * (2.0 * c.z + u * 3.0 * c.w);
  const double x_end = t.x0 + (t.n - 1) * t.dx;
  if (x > x_end) {
    if (linear_beyond) {
      const double4 e = coef[t.n - 2];
      const double h = t.dx;
      const double ve = e.x + h * (e.y + h * (e.z + h * e.w));
      const double de = e.y + h * (2.0 * e.z + h * 3.0 * e.w);
      v = ve + de * (x - x_end);
      dv = de;
    } else {
      v = 0.0;
      dv = 0.0;
    }
  }
}

// ---- the paper's W EAM in closed form (appendix "AP potential for tungsten":
// equations eam_F_Marinica, eam_Phi_Marinica, eam_rho_Marinica,
// tungsten_rho_up, tungsten_F_up, tungsten_Phi_up), FP64.
// A knot sum sum_i a_i (d_i - r)^3 Theta(d_i - r) as the cubic of r's interval
// between the sorted distinct knots D_0 < D_1 < ...: for D_{k-1} < r <= D_k it is
// c0 + t (c1 + t (c2 + t c3)) with t = D_k - r, the coefficients expanded on the
// host in extended precision (KnotDev).  Adding up the knots one by one kept
// the vector units busy (511 instructions per bond of the force pass); the
// interval search is one compare and one add per knot.  Against extended
// precision the W pair function's error falls from 1.2e-14 (its knots cancel)
// to 6e-17, the density's from 9e-17 to 7e-17.  An r that is infinite or not a
// number lies beyond every knot and gives zero, as in the sum.
__device__ __forceinline__ void an_knots(const KnotDev& d, const double4* coef, double r, double& v,
                                         double& dv) {
  int k = 0;
  for (int i = 0; i < d.n4; i += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) k += !(d.knot[i + q] >= r) ? 1 : 0;  // padded with +inf
  }
  k = min(k, d.n);
  const double4 c = coef[k];
  // (beyond the last knot the coefficients are zero, and so is t)
  const double t = fmax(reinterpret_cast<const double*>(coef + d.n + 1)[k] - r, 0.0);
  v = c.x + t * (c.y + t * (c.z + t * c.w));
  dv = -(c.y + t * (2.0 * c.z + t * 3.0 * c.w));
}

// zeta(r) = zeta_0(max(r, r_cut))
__device__ __forceinline__ void an_density(const EamAnalyticDev& p, const double4* coef, double r,
                                           double& v, double& dv) {
  an_knots(p.rho, coef, r, v, dv);
  if (r <= p.r_cut_rho) {
    v = p.zeta_cut;
    dv = 0.0;
  }
}

// Phi^Fit(r): screened Coulomb below r_lo, quintic bridge up to r_hi, knot sum above
__device__ __forceinline__ void an_pair(const EamAnalyticDev& p, const double4* coef, double r, double& v,
                                        double& dv) {
  if (!(r <= p.r_hi)) {
    an_knots(p.phi, coef, r, v, dv);
  } else if (r < p.r_lo) {
    const double x = r / p.a_zbl;
    double s = 0.0, ds = 0.0;
    for (int k = 0; k < 4; ++k) {
      const double e = exp(-p.zbl_q[k] * x);
      s += p.zbl_c[k] * e;
      ds -= p.zbl_c[k] * p.zbl_q[k] / p.a_zbl * e;
    }
    v = p.zbl_pref * s / r;
    dv = p.zbl_pref * (ds / r - s / (r * r));
  } else {
    const double* b = p.b_phi;
    v = b[0] + r * (b[1] + r * (b[2] + r * (b[3] + r * (b[4] + r * b[5]))));
    dv = b[1] + r * (2.0 * b[2] + r * (3.0 * b[3] + r * (4.0 * b[4] + r * 5.0 * b[5])));
  }
}

// xi^Fit(x) = a1 sqrt(x) + a2 x^2 + Delta xi (the square root dropped for x <= 0)
__device__ __forceinline__ void an_embed(const EamAnalyticDev& p, double x, double& v, double& dv) {
  const double s = x > 0.0 ? sqrt(x) : 0.0;
  v = p.a_xi1 * s + p.a_xi2 * x * x + p.d_xi;
  dv = (x > 0.0 ? 0.5 * p.a_xi1 / s : 0.0) + 2.0 * p.a_xi2 * x;
}

// The interval cubics of a knot sum, then its knots (0 behind the last), to LDS.
__device__ __forceinline__ const double4* stage_knots(const KnotDev& d, double4* lds) {
  for (int q = threadIdx.x; q <= d.n; q += blockDim.x) {
    lds[q] = make_double4(d.c[q][0], d.c[q][1], d.c[q][2], d.c[q][3]);
    reinterpret_cast<double*>(lds + d.n + 1)[q] = q < d.n ? d.knot[q] : 0.0;
  }
  return lds;
}
// double4 records the staged knot sum takes
__host__ __device__ inline int knot_records(const KnotDev& d) { return d.n + 1 + (d.n + 4) / 4; }

// Copies n records of a table into LDS (whole workgroup, before any thread
// leaves); returns where the bond loop reads them from.
__device__ __forceinline__ const double4* stage_table(const double* c, int n, double4* lds, bool use) {
  const double4* g = reinterpret_cast<const double4*>(c);
  if (!use) return g;
  for (int q = threadIdx.x; q < n; q += blockDim.x) lds[q] = g[q];
  return lds;
}

// Sum over the LN parts of an atom's bonds: part p of the block's atom a sits
// in thread p * (256 / LN) + a, so that neighbouring lanes read neighbouring
// atoms of the slot-major list; the parts are added in order through LDS, and
// the result is valid in part 0.
template <int LN, int NV>
__device__ __forceinline__ void sum_parts(double (&v)[NV], double* lds) {
  if constexpr (LN > 1) {
    constexpr int kAtoms = 256 / LN;
    __syncthreads();  // the table staging shares this region
#pragma unroll
    for (int q = 0; q < NV; ++q) lds[q * 256 + threadIdx.x] = v[q];
    __syncthreads();
    if (threadIdx.x < kAtoms) {
#pragma unroll
      for (int q = 0; q < NV; ++q)
        for (int p = 1; p < LN; ++p) v[q] += lds[q * 256 + p * kAtoms + threadIdx.x];
    }
  }
}

// kOrtho: every system is orthorhombic, so the box edges are hoisted out of
// the bond loop (same arithmetic as the general displacement).  kLds: the
// pair tables are staged in LDS (dynamic shared memory sized by the host).
// LN threads share an atom's bonds (thread part, part + LN, ...).  pos4: the
// position and, in w, the atom's EAM weight 1 - lambda.  The closed form loads the
// list entries of four bonds together (1.27 million atoms 336 -> 303 us); with
// tables two bonds in flight are the better (2.66 million 630 us, batches of
// two 669, of four 655).
template <bool kOrtho, bool kLds, bool kAn, int LN>
__global__ __launch_bounds__(256) void k_eam_density(SysView sv, TableDev rho_t, TableDev F_t,
                                                     EamAnalyticDev an,
                                                     const double4* __restrict__ pos4,
                                                     const int32_t* __restrict__ nbr,
                                                     const int32_t* __restrict__ count,
                                                     double* __restrict__ wfp,
                                                     double* __restrict__ eF) {
  extern __shared__ double4 tab_lds[];
  const double4* rho_c = kAn ? stage_knots(an.rho, tab_lds)
                             : stage_table(rho_t.c, rho_t.n - 1, tab_lds, kLds);
  if (kLds || kAn) __syncthreads();
  const int n = sv.n_atoms;
  constexpr int kAtoms = 256 / LN, kBatch = kAn ? 4 : 1;
  const int i = xcd_chunk(blockIdx.x, gridDim.x) * kAtoms + threadIdx.x % kAtoms, part = threadIdx.x / kAtoms;
  const bool live = i < n;
  const double4 pi = live ? pos4[i] : make_double4(0.0, 0.0, 0.0, 0.0);
  const double w = pi.w;
  double rho[1] = {0.0};
  if (w > 0.0) {
    const int s = sv.sys_of[i];
    const bool ortho = sv.ortho[s] != 0;
    const double* H = sv.H + 9 * s;
    const double* Hi = sv.Hi + 9 * s;
    const double Lx = H[0], Ly = H[4], Lz = H[8];
    const int c = count[i];
#pragma unroll (kAn ? 1 : 2)
    for (int q = part; q < c; q += kBatch * LN) {
      int js[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) js[u] = q + u * LN < c ? nbr[(int64_t)(q + u * LN) * n + i] : -1;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = js[u];
        if (kBatch > 1 && j < 0) continue;
        const double4 pj = pos4[j];
        double dx, dy, dz;
        if (kOrtho)
          displacement_ortho(sv.per, Lx, Ly, Lz, pi.x, pi.y, pi.z, pj.x, pj.y, pj.z, dx, dy, dz);
        else
          displacement(ortho, H, Hi, sv.per, pi.x, pi.y, pi.z, pj.x, pj.y, pj.z, dx, dy, dz);
        const double r = sqrt(dx * dx + dy * dy + dz * dz);
        double v, dv;
        if constexpr (kAn) an_density(an, rho_c, r, v, dv);
        else tab_eval(rho_t, rho_c, r, false, v, dv);
        rho[0] += v;
      }
    }
  }
  sum_parts<LN>(rho, reinterpret_cast<double*>(tab_lds));
  if (!live || part != 0) return;
  if (!(w > 0.0)) {
    wfp[i] = 0.0;
    eF[i] = 0.0;
    return;
  }
  double Fv, Fp;
  if constexpr (kAn) an_embed(an, rho[0], Fv, Fp);
  else tab_eval(F_t, reinterpret_cast<const double4*>(F_t.c), rho[0], true, Fv, Fp);
  wfp[i] = w * Fp;
  eF[i] = Fv;
}

// Waits on the list entries and the gathered records, four wavefronts a SIMD; with
// tables also on LDS (a lookup's 16-byte reads start in half of the banks: 250,000
// atoms, 74 % of the LDS cycles are conflicts, 68 % in the density pass).  The
// entries of four bonds are loaded together, so their way from HBM is paid once
// for the four (us, against a bond at a time with five wavefronts a SIMD: 1.27
// million atoms closed form 620 -> 589, 2.66 million 1265 -> 1157, 250,000
// 102 -> 98; five wavefronts spill here: 600, 1265, 103; batches of eight 606,
// 2120, 179).
template <bool kOrtho, bool kLds, bool kAn, int LN>
__global__ __launch_bounds__(256, 4) void k_eam_force(SysView sv, TableDev rho_t, TableDev phi_t,
                                                   EamAnalyticDev an,
                                                   const double4* __restrict__ pos4,
                                                   const int32_t* __restrict__ nbr,
                                                   const int32_t* __restrict__ count,
                                                   const double* __restrict__ wfp,
                                                   const double* __restrict__ eF,
                                                   double* __restrict__ e_atom,
                                                   double* __restrict__ force,
                                                   double* __restrict__ vir, int accumulate,
                                                   double* __restrict__ e_raw) {
  extern __shared__ double4 tab_lds[];
  const double4* rho_c = kAn ? stage_knots(an.rho, tab_lds)
                             : stage_table(rho_t.c, rho_t.n - 1, tab_lds, kLds);
  const double4* phi_c = kAn ? stage_knots(an.phi, tab_lds + knot_records(an.rho))
                             : stage_table(phi_t.c, phi_t.n - 1, tab_lds + (rho_t.n - 1), kLds);
  if (kLds || kAn) __syncthreads();
  const int n = sv.n_atoms;
  constexpr int kAtoms = 256 / LN, kBatch = 4;
  const int k = xcd_chunk(blockIdx.x, gridDim.x) * kAtoms + threadIdx.x % kAtoms, part = threadIdx.x / kAtoms;
  const bool live = k < n;
  // force, pair energy and virial sums; atom k's bond gradients are parallel to
  // the bonds, so its virial -sum_j d (x) G_kj is symmetric: six sums
  double a10[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  double wk = 0.0;
  if (live) {
    const int s = sv.sys_of[k];
    const bool ortho = sv.ortho[s] != 0;
    const double* H = sv.H + 9 * s;
    const double* Hi = sv.Hi + 9 * s;
    const double Lx = H[0], Ly = H[4], Lz = H[8];
    const double4 pk = pos4[k];
    wk = pk.w;
    const double fk = wfp[k];
    const int c = count[k];
    for (int q = part; q < c; q += kBatch * LN) {
      int js[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) js[u] = q + u * LN < c ? nbr[(int64_t)(q + u * LN) * n + k] : -1;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = js[u];
        if (kBatch > 1 && j < 0) continue;
        const double4 pj = pos4[j];
        const double wj = pj.w, fj = wfp[j];
        if (wk == 0.0 && wj == 0.0) continue;
        double dx, dy, dz;
        if (kOrtho)
          displacement_ortho(sv.per, Lx, Ly, Lz, pk.x, pk.y, pk.z, pj.x, pj.y, pj.z, dx, dy, dz);
        else
          displacement(ortho, H, Hi, sv.per, pk.x, pk.y, pk.z, pj.x, pj.y, pj.z, dx, dy, dz);
        const double r = sqrt(dx * dx + dy * dy + dz * dz);
        const double ir = 1.0 / r;
        double z, dzr, p, dp;
        if constexpr (kAn) {
          an_density(an, rho_c, r, z, dzr);
          an_pair(an, phi_c, r, p, dp);
        } else {
          tab_eval(rho_t, rho_c, r, false, z, dzr);
          tab_eval(phi_t, phi_c, r, false, p, dp);
        }
        const double a = ((fk + fj) * dzr + 0.5 * (wk + wj) * dp) * ir;
        a10[0] += a * dx;
        a10[1] += a * dy;
        a10[2] += a * dz;
        a10[3] += p;
        // virial of atom k's own bond gradient G_kj = (w_k xi'_k zeta' + w_k Phi'/2) d/r
        if (vir) {
          const double g = (fk * dzr + 0.5 * wk * dp) * ir;
          const double gx = g * dx, gy = g * dy, gz = g * dz;
          a10[4] -= dx * gx; a10[5] -= dx * gy; a10[6] -= dx * gz;
          a10[7] -= dy * gy; a10[8] -= dy * gz;
          a10[9] -= dz * gz;
        }
      }
    }
  }
  sum_parts<LN>(a10, reinterpret_cast<double*>(tab_lds));
  if (!live || part != 0) return;
  const double fx = a10[0], fy = a10[1], fz = a10[2], ephi = a10[3];
  const double v00 = a10[4], v01 = a10[5], v02 = a10[6], v11 = a10[7], v12 = a10[8], v22 = a10[9];
  const double e_un = wk > 0.0 ? eF[k] + 0.5 * ephi : 0.0;  // E_k^EAM, unweighted
  const double e = wk > 0.0 ? wk * e_un : 0.0;
  if (e_raw) e_raw[k] = e_un;
  if (accumulate) {
    e_atom[k] += e;
    force[k] += fx;
    force[n + k] += fy;
    force[2 * n + k] += fz;
  } else {
    e_atom[k] = e;
    force[k] = fx;
    force[n + k] = fy;
    force[2 * n + k] = fz;
  }
  if (vir) {
    vir[0 * (int64_t)n + k] = v00; vir[1 * (int64_t)n + k] = v01; vir[2 * (int64_t)n + k] = v02;
    vir[3 * (int64_t)n + k] = v01; vir[4 * (int64_t)n + k] = v11; vir[5 * (int64_t)n + k] = v12;
    vir[6 * (int64_t)n + k] = v02; vir[7 * (int64_t)n + k] = v12; vir[8 * (int64_t)n + k] = v22;
  }
}

// Threads per atom.  An atom's 58 or so bonds are one chain of gathers, square
// roots and divisions: while the chip is not full, splitting it sets the time.
// On a full chip the split only shortens each block's chain.  us, density +
// force pass with 1, 2, 4 and 16 threads, tables:
//      2,000 atoms   23 +   44,  15 +   23,   9 +   15,   5 +    8
//     31,250 atoms   24 +   45,  16 +   25,  12 +   18,  13 +   21
//    108,000 atoms   35 +   62,  28 +   50,  25 +   47,  31 +   65
//    250,000 atoms   55 +  106,  54 +  102,  54 +  103,  68 +  144
//  2,660,283 atoms  568 + 1219, 610 + 1123, 647 + 1108, 746 + 1714
// closed form (418 + 958 with one thread when the knots were added up one by one):
//  1,272,112 atoms  297 +  577, 278 +  559, 260 +  577, 322 +  858
constexpr int kEamSplit16 = 8192, kEamSplit4 = 131072;

hipError_t launch_eam(const Ctx& c, const SysView& sv, const double4* pos4, const int32_t* nbr,
                      const int32_t* count, int32_t n_atoms, double* wfp, double* eF, double* e_atom,
                      double* force, double* vir_atom, bool accumulate, double* e_raw, hipStream_t s) {
  if (n_atoms == 0) return hipSuccess;
  // pair tables in LDS when both fit in a quarter of a CU's LDS (four
  // resident workgroups); otherwise they are read through the caches
  // (the closed form's interval cubics, at most 42 records each, always are)
  const size_t rho_b = 32 * (size_t)(c.eam_analytic ? knot_records(c.ean.rho) : c.rho.n - 1);
  const size_t phi_b = 32 * (size_t)(c.eam_analytic ? knot_records(c.ean.phi) : c.phi.n - 1);
  const bool lds = c.eam_analytic || rho_b + phi_b <= 40 * 1024;
  auto go = [&](auto dens, auto frc, int ln) {
    const dim3 g((unsigned)(((int64_t)n_atoms * ln + 255) / 256)), b(256);
    // the parts' sums reuse the region: 1 and 10 doubles per thread
    const size_t pd = ln > 1 ? 8 * 256 : 0, pf = ln > 1 ? 80 * 256 : 0;
    hipLaunchKernelGGL(dens, g, b, std::max(lds ? rho_b : 0, pd), s, sv, c.rho, c.F, c.ean, pos4, nbr,
                       count, wfp, eF);
    hipLaunchKernelGGL(frc, g, b, std::max(lds ? rho_b + phi_b : 0, pf), s, sv, c.rho, c.phi, c.ean, pos4,
                       nbr, count, wfp, eF, e_atom, force, vir_atom, accumulate ? 1 : 0, e_raw);
  };
  auto pick = [&](auto ln) {
    constexpr int LN = decltype(ln)::value;
    if (c.eam_analytic) {
      if (sv.all_ortho) go(k_eam_density<true, false, true, LN>, k_eam_force<true, false, true, LN>, LN);
      else go(k_eam_density<false, false, true, LN>, k_eam_force<false, false, true, LN>, LN);
    } else if (sv.all_ortho) {
      if (lds) go(k_eam_density<true, true, false, LN>, k_eam_force<true, true, false, LN>, LN);
      else go(k_eam_density<true, false, false, LN>, k_eam_force<true, false, false, LN>, LN);
    } else {
      if (lds) go(k_eam_density<false, true, false, LN>, k_eam_force<false, true, false, LN>, LN);
      else go(k_eam_density<false, false, false, LN>, k_eam_force<false, false, false, LN>, LN);
    }
  };
  if (n_atoms <= kEamSplit16) pick(std::integral_constant<int, 16>{});
  else if (n_atoms <= kEamSplit4) pick(std::integral_constant<int, 4>{});
  else pick(std::integral_constant<int, 2>{});
  return hipGetLastError();
}

}  // namespace ap
