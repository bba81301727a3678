// FP64 rank kernels of the ACE path (coupling, folded contraction and adjoint
// of one coupled rank L), one translation unit per L (-DAP_RANK_L=<L>).
//
// One workgroup (512 threads, 8 wavefronts) evaluates tiles of kT64 = 4 ACE
// atoms (persistent loop, tiles round-robin):
//  1. coupling: X_L = [AA_{c,M} | A_{n,L,M} | 1] for the 4 atoms in LDS,
//     X[row][t (2L+1) + M]; one lane per (channel, atom), channels grouped by
//     (l_a, l_b), so the coupling coefficients are compile-time constants;
//  2. contraction Z = C_L X of both coefficient sets with
//     v_mfma_f64_16x16x4_f64.  C_L is stored as 16 x 4 tiles and only the
//     tiles that hold a nonzero are visited: a product function couples
//     (a, b) with (c, d) only for b <= c, so with the channels ordered by
//     (n_b, n_a) 36 % of the tiles of the (8, 4, nu <= 4) model are empty, and
//     nearly all of a nu <= 3 model's.  The accumulators of both sets stay in
//     registers, so X is built once and Z overwrites it, one set at a time;
//  3. adjoint: lane = (target n, atom, half of the partners); job (l_t, l_p,
//     part of the M) forms W[m2][M] = sum_n' A_(n',l_p,m2) Z_({a,p},M) and
//     applies the coupling coefficients once.  Jobs of one target l that sit
//     on different wavefronts write to different slots, added in a fixed
//     order, so results are reproducible.
// What bounds it: 2,499 atoms of the (8, 4, nu <= 4) model take 1.11 ms over the
// nine ranks (one workgroup per atom and sparse FP64 sums: 4.46 ms for the
// whole ACE part); at L = 2..4 the contraction is 60 % of the time, at 55-65 %
// of the matrix rate; 20,518 atoms of the (6, 3, nu <= 3) model take 0.80 ms
// (4.27 ms before), bound by LDS latency and barriers in short phases.
// Why MFMA: FP64 matrix and vector rates are equal (78.6 TFLOP/s), but a
// sparse vector contraction needs one LDS read per two multiply-adds and LDS
// delivers one b64 read per 4 cycles and CU, half of what the vector units
// consume; the matrix instruction reads each operand once per 1024
// multiply-adds.  4 atoms per tile: 4 (2L+1) columns fill 62-94 % of the
// 16-column tiles for L >= 1, and X_L of the widest rank (308 rows x 36
// columns, 118 KB with the padding) still fits in LDS beside A and the slots.
#include "ace_cg.h"
#include "ap_internal.h"
#include "scan.h"

#include <utility>

#ifndef AP_RANK_L
#error "k_ace_rank64.hip is compiled once per coupled rank with -DAP_RANK_L=<L>"
#endif

namespace ap {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads64 = 64 * kRank64Waves;

// Read-only tables through the constant address space: wavefront-uniform
// indices become scalar loads (the kernel never writes them).
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p) { return (cptr<T>)p; }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <int LA, int LB, int L, int E>
__device__ __forceinline__ void x_entry(const double* Aa, const double* Ab, double* X) {
  constexpr int q = E % (2 * L + 1), i2 = (E / (2 * L + 1)) % (2 * LB + 1),
                i1 = E / ((2 * L + 1) * (2 * LB + 1));
  if constexpr (cg_rule(i1 - LA, i2 - LB, q - L)) {
    constexpr double c = ce_real_cg(LA, LB, L, i1 - LA, i2 - LB, q - L);
    if constexpr (c > 1e-15 || c < -1e-15) X[q] = fma(c, Aa[i1] * Ab[i2], X[q]);
  }
}
template <int LA, int LB, int L, int... E>
__device__ __forceinline__ void x_all(std::integer_sequence<int, E...>, const double* Aa,
                                      const double* Ab, double* X) {
  (x_entry<LA, LB, L, E>(Aa, Ab, X), ...);
}

// One channel (n, LA) x (n', LB) -> L of one atom.
template <int LA, int LB, int L>
__device__ __forceinline__ void x_channel(const double* At, int oa, int ob, double* out) {
  double Aa[2 * LA + 1], Ab[2 * LB + 1], X[2 * L + 1];
#pragma unroll
  for (int q = 0; q <= 2 * LA; ++q) Aa[q] = At[oa + q];
#pragma unroll
  for (int q = 0; q <= 2 * LB; ++q) Ab[q] = At[ob + q];
#pragma unroll
  for (int q = 0; q <= 2 * L; ++q) X[q] = 0.0;
  x_all<LA, LB, L>(std::make_integer_sequence<int, (2 * LA + 1) * (2 * LB + 1) * (2 * L + 1)>{}, Aa,
                   Ab, X);
#pragma unroll
  for (int q = 0; q <= 2 * L; ++q) out[q] = X[q];
}

// Adjoint of the pattern (LT, LP, L) for the M of [Q0, Q1): partner sum, then
// the coupling coefficients.
template <int LT, int LP, int L, int Q0, int Q1, int E>
__device__ __forceinline__ void ad_entry(const double* W, double* ga) {
  constexpr int mc = Q1 - Q0;
  constexpr int q = E % mc + Q0, i2 = (E / mc) % (2 * LP + 1), i1 = E / (mc * (2 * LP + 1));
  if constexpr (cg_rule(i1 - LT, i2 - LP, q - L)) {
    constexpr double c = ce_real_cg(LT, LP, L, i1 - LT, i2 - LP, q - L);
    if constexpr (c > 1e-15 || c < -1e-15) ga[i1] = fma(c, W[i2 * mc + q - Q0], ga[i1]);
  }
}
template <int LT, int LP, int L, int Q0, int Q1, int... E>
__device__ __forceinline__ void ad_all(std::integer_sequence<int, E...>, const double* W, double* ga) {
  (ad_entry<LT, LP, L, Q0, Q1, E>(W, ga), ...);
}

// At: the atom's A; Z: at the atom's first column; rows: channel rows of
// target (n, LT) for the partners (n', LP), stride lp1; h: this lane takes
// the partners n' = h, h + 2, ...  A missing channel's row is a row of zeros,
// and the diagonal channels' rows of C_L are doubled on the host.
template <int LT, int LP, int L, int NC, int K>
__device__ __forceinline__ void ad_job(const double* At, const double* Z, int cstr,
                                       const int16_t* rows, int lp1, int nlm, int n_max, int zrow,
                                       bool act, int h, double* out, bool first) {
  constexpr int w = 2 * L + 1, w2 = 2 * LP + 1, w1 = 2 * LT + 1;
  constexpr int Q0 = K * w / NC, Q1 = (K + 1) * w / NC, mc = Q1 - Q0;
  double W[w2 * mc];
#pragma unroll
  for (int e = 0; e < w2 * mc; ++e) W[e] = 0.0;
#pragma unroll 1
  for (int np = h; np < n_max + (n_max & 1); np += 2) {
    const bool ok = act && np < n_max;
    const int npc = np < n_max ? np : 0;
    const int row = ok ? (int)rows[npc * lp1 + LP] : zrow;
    const double* zr = Z + row * cstr + Q0;
    const double* ar = At + npc * nlm + LP * LP;
    double a[w2], z[mc];
#pragma unroll
    for (int q = 0; q < w2; ++q) a[q] = ar[q];
#pragma unroll
    for (int q = 0; q < mc; ++q) z[q] = zr[q];
#pragma unroll
    for (int i = 0; i < w2; ++i)
#pragma unroll
      for (int q = 0; q < mc; ++q) W[i * mc + q] = fma(a[i], z[q], W[i * mc + q]);
  }
  double ga[w1];
#pragma unroll
  for (int q = 0; q < w1; ++q) ga[q] = 0.0;
  ad_all<LT, LP, L, Q0, Q1>(std::make_integer_sequence<int, w1 * w2 * mc>{}, W, ga);
  // the two partner halves sit in neighbouring lanes
#pragma unroll
  for (int q = 0; q < w1; ++q) ga[q] += __shfl_xor(ga[q], 1);
  if (act && h == 0) {
#pragma unroll
    for (int q = 0; q < w1; ++q) out[q] = first ? ga[q] : out[q] + ga[q];
  }
}

// U: units (16 rows of one set) per wavefront; SMALL: the register budget of
// two workgroups per CU.
template <int L, int U, bool SMALL>
__global__ __launch_bounds__(kThreads64, SMALL ? 4 : 2) void k_ace_rank64(
    Rank64Dev m, Rank64L P, const int32_t* __restrict__ n_ace_p, int n_all, int item0, int n_buf,
    const double* __restrict__ A_in, double* __restrict__ om_buf, double* __restrict__ phi_buf) {
  constexpr int w = 2 * L + 1;
  constexpr int ncols = kT64 * w;
  constexpr int CT = (ncols + 15) / 16;
  extern __shared__ double lds64[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uni(tid >> 6);
  const int lp1 = m.l_max + 1, nlm = lp1 * lp1, nA = m.nA, nidx = m.n_max * lp1;
  double* A = lds64;                                         // [kT64][apad]
  double* part = A + kT64 * m.apad;                          // [slots][kT64][apad]
  double* X = part + m.slots * kT64 * m.apad;                // [zrow + 1][cstr], X then Z
  int4* mem_lds = reinterpret_cast<int4*>(X + (size_t)(P.zrow + 1) * P.cstr);
  int16_t* rows_lds = reinterpret_cast<int16_t*>(mem_lds + P.ngrp * (64 / kT64));
  const int n_items = min((n_ace_p ? *n_ace_p : n_all) - item0, n_buf);
  const int n_tiles = (n_items + kT64 - 1) / kT64;
  if ((int)blockIdx.x >= n_tiles) return;
  for (int q = tid; q < nidx * nidx; q += kThreads64) {
    const int r = m.rowtab[(size_t)L * nidx * nidx + q];
    rows_lds[q] = (int16_t)(r < 0 ? P.zrow : r);
  }
  for (int q = tid; q < P.ngrp * (64 / kT64); q += kThreads64)
    mem_lds[q] = m.grp_mem[(size_t)P.grp0 * (64 / kT64) + q];
  // the padding rows up to the last 4-row step (as X) and the row of zeros (as Z)
  for (int q = tid; q < ncols; q += kThreads64) X[(size_t)P.zrow * P.cstr + q] = 0.0;
  // the tile's A is fetched into registers one tile ahead (kT64 nA <= 1024)
  double pa[2];
  auto fetch = [&](int tile) {
    const int nt = min(kT64, n_items - tile * kT64);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int q = tid + r * kThreads64;
      pa[r] = q < nt * nA ? A_in[(int64_t)tile * kT64 * nA + q] : 0.0;
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int q = tid + r * kThreads64;
      if (q < kT64 * nA) A[(q / nA) * m.apad + q % nA] = pa[r];
    }
  };
  fetch(blockIdx.x);
  // the gradient entries this thread adds up: slot offset, slots, A-row entry of Z
  int gpart[2], gslots[2], gz[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int q = tid + r * kThreads64;
    const int t = q / nA, e = q - t * nA, nn = e / nlm, lm = e - nn * nlm;
    int l = 0;
    while ((l + 1) * (l + 1) <= lm) ++l;
    gpart[r] = t * m.apad + e;
    gslots[r] = P.nslots[l];
    gz[r] = P.arow && l == L ? (P.nch + nn) * P.cstr + t * w + lm - L * L : -1;
  }
  cptr<int32_t> units = as_const(reinterpret_cast<const int32_t*>(m.units)) + 4 * (P.unit0 + wave * P.nu);
  cptr<int32_t> jptr = as_const(m.job_ptr) + L * (kRank64Waves + 1);
  cptr<int32_t> jobs = as_const(reinterpret_cast<const int32_t*>(m.jobs));
  cptr<int32_t> kidx = as_const(m.kidx);
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int nt = min(kT64, n_items - tile * kT64);
    stage();
    __syncthreads();
    if (tile + (int)gridDim.x < n_tiles) fetch(tile + gridDim.x);
    // ---- coupling
    {
      const int t = lane & (kT64 - 1);
      const double* At = A + t * m.apad;
      for (int g = wave; g < P.ngrp; g += kRank64Waves) {
        const int4 mem = mem_lds[g * (64 / kT64) + lane / kT64];
        const int key = uni(mem.w);
        if (mem.x < 0) continue;
        double* out = X + mem.x * P.cstr + t * w;
        switch (key) {
#define AP_X(la, lb)                                                                        \
  case (la) * 5 + (lb):                                                                     \
    if constexpr (iabs_c((la) - (lb)) <= L && L <= (la) + (lb) && (((la) + (lb) + L) & 1) == 0) \
      x_channel<la, lb, L>(At, mem.y, mem.z, out);                                          \
    break;
#define AP_X5(la) AP_X(la, 0) AP_X(la, 1) AP_X(la, 2) AP_X(la, 3) AP_X(la, 4)
          AP_X5(0) AP_X5(1) AP_X5(2) AP_X5(3) AP_X5(4)
#undef AP_X5
#undef AP_X
          default: break;
        }
      }
      if (P.arow)
        for (int q = tid; q < m.n_max * ncols; q += kThreads64) {
          const int n = q / ncols, col = q % ncols;
          X[(P.nch + n) * P.cstr + col] = A[(col / w) * m.apad + n * nlm + L * L + col % w];
        }
      if (L == 0 && tid < kT64) X[(P.nch + m.n_max) * P.cstr + tid] = 1.0;
      for (int q = tid; q < (P.nrow4 - P.nrow) * ncols; q += kThreads64)
        X[(P.nrow + q / ncols) * P.cstr + q % ncols] = 0.0;
    }
    __syncthreads();
    // ---- contraction of both sets: this wavefront's units (16 rows of one set)
    f64x4 acc[U][CT];
    int urow[U], uset[U];
    const double* xb = X + (lane >> 4) * P.cstr + (lane & 15);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[u][c] = f64x4{0.0, 0.0, 0.0, 0.0};
      urow[u] = -1;
      uset[u] = 0;
      if (u < P.nu) {
        urow[u] = uni(units[4 * u]);
        uset[u] = uni(units[4 * u + 1]);
        const int s0 = uni(units[4 * u + 2]), ns = uni(units[4 * u + 3]);
        const double* cf = m.coef + (size_t)s0 * 64 + lane;
        // the coefficients of the next 4 steps load under this step's MFMAs
        double ca[4], cb[4];
        // (steps come in fours; the tail is padded with zero coefficients)
        int ka[4], kb[4];
        auto load = [&](double (&d)[4], int (&ki)[4], int s) {
          const int b = min(s, ns - 4);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            d[k] = cf[(size_t)(b + k) * 64];
            ki[k] = kidx[s0 + b + k];
          }
          asm volatile("" ::: "memory");
        };
        auto run = [&](const double (&d)[4], const int (&ki)[4]) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const double* xr = xb + ki[k];
#pragma unroll
            for (int c = 0; c < CT; ++c)
              acc[u][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[k], xr[16 * c], acc[u][c], 0, 0, 0);
          }
        };
        if (ns > 0) {
          load(ca, ka, 0);
          for (int s = 0; s < ns; s += 8) {
            load(cb, kb, s + 4);
            run(ca, ka);
            if (s + 4 < ns) {
              load(ca, ka, s + 8);
              run(cb, kb);
            }
          }
        }
      }
    }
    __syncthreads();  // X is dead from here on
    for (int p = 0; p < 2; ++p) {
      // the lower ranks' gradient, read ahead of its use
      double* om = om_buf + (int64_t)p * n_buf * nA + (int64_t)tile * kT64 * nA;
      double og[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int q = tid + r * kThreads64;
        og[r] = L > 0 && q < nt * nA ? om[q] : 0.0;
      }
      // ---- Z of set p over X: result rows (lane / 16) + 4 i
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (urow[u] >= 0 && uset[u] == p) {
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            const int col = c * 16 + (lane & 15);
            if (col < ncols) {
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int row = urow[u] + (lane >> 4) + 4 * i;
                if (row < P.nrow) X[row * P.cstr + col] = acc[u][c][i];
              }
            }
          }
        }
      __syncthreads();
      // ---- adjoint jobs of this wavefront
      {
        const int n = lane >> 3, t = (lane >> 1) & (kT64 - 1), h = lane & 1;
        const bool act = n < m.n_max;
        const double* At = A + t * m.apad;
        const int u0 = uni(jptr[wave]), u1 = uni(jptr[wave + 1]);
        for (int u = u0; u < u1; ++u) {
          const int key = uni(jobs[4 * u]), slot = uni(jobs[4 * u + 1]);
          const bool first = uni(jobs[4 * u + 2]) != 0;
          const int lt = uni(jobs[4 * u + 3]);
          const int16_t* rows = rows_lds + ((act ? n : 0) * lp1 + lt) * nidx;
          double* out = part + (slot * kT64 + t) * m.apad + (act ? n : 0) * nlm + lt * lt;
          switch (key) {
#define AP_J(lt, lp, k)                                                                         \
  case ((lt) * 5 + (lp)) * 4 + (k):                                                             \
    if constexpr (iabs_c((lt) - (lp)) <= L && L <= (lt) + (lp) && (((lt) + (lp) + L) & 1) == 0 && \
                  (k) < rank64_chunks(lp, L))                                             \
      ad_job<lt, lp, L, rank64_chunks(lp, L), k>(At, X + t * w, P.cstr, rows, lp1, nlm, m.n_max, \
                                                       P.zrow, act, h, out, first);             \
    break;
#define AP_J4(lt, lp) AP_J(lt, lp, 0) AP_J(lt, lp, 1) AP_J(lt, lp, 2) AP_J(lt, lp, 3)
#define AP_JT(lt) AP_J4(lt, 0) AP_J4(lt, 1) AP_J4(lt, 2) AP_J4(lt, 3) AP_J4(lt, 4)
            AP_JT(0) AP_JT(1) AP_JT(2) AP_JT(3) AP_JT(4)
#undef AP_JT
#undef AP_J4
#undef AP_J
            default: break;
          }
        }
      }
      __syncthreads();
      // ---- this rank's gradient: slots in order, then the A rows of X_L
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int q = tid + r * kThreads64;
        if (q < nt * nA) {
          double g = og[r];
          for (int s = 0; s < gslots[r]; ++s) g += part[s * kT64 * m.apad + gpart[r]];
          if (gz[r] >= 0) g += X[gz[r]];
          om[q] = g;
        }
      }
      // phi by Euler's theorem: A.Z over the A rows plus twice the constant row
      if (wave == kRank64Waves - 1) {
        const int t = lane >> 4;
        double sa = 0.0;
        if (P.arow)
          for (int q = lane & 15; q < m.n_max * w; q += 16) {
            const int nn = q / w, M = q % w;
            sa = fma(A[t * m.apad + nn * nlm + L * L + M], X[(P.nch + nn) * P.cstr + t * w + M], sa);
          }
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) sa += __shfl_xor(sa, d, 16);
        if ((lane & 15) == 0 && t < nt) {
          double* ph = phi_buf + 2 * ((int64_t)tile * kT64 + t) + p;
          if (L == 0) sa += 2.0 * X[(P.nch + m.n_max) * P.cstr + t];
          *ph = (L > 0 ? *ph : 0.0) + sa;
        }
      }
      __syncthreads();
    }
  }
}

}  // namespace

template <>
const void* rank64_kernel<AP_RANK_L>(bool small) {
  if constexpr (AP_RANK_L <= kRank64LSmall)
    if (small) return (const void*)k_ace_rank64<AP_RANK_L, kRank64USmall, true>;
  return (const void*)k_ace_rank64<AP_RANK_L, kRank64U[AP_RANK_L], false>;
}

}  // namespace ap
