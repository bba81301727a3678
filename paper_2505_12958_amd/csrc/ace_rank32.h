// Rank kernels of the mixed-precision ACE path: coupling, folded contraction
// and adjoint of one coupled rank L, one launch per rank.
//
// One workgroup evaluates tiles of kMT32 = 8 ACE atoms (persistent loop, tiles
// round-robin); per rank:
//  1. coupling: X_L = [AA_{c,M} | A_{n,L,M} | 1] for the 8 atoms (one lane per
//     (channel, atom), channels grouped by (l_a, l_b), so the coupling
//     coefficients are compile-time constants), scaled per atom by a power of
//     two and written to LDS as an fp16 hi/lo split (x = hi + lo to ~22 bits),
//     column-major (k contiguous);
//  2. contraction Z = C_L X of both coefficient sets with
//     v_mfma_f32_16x16x32_f16 as hi hi + hi lo + lo hi, FP32 accumulation.
//     C_L is stored as 16-row steps of four 8-column chunks, each row scaled
//     by a power of two; chunks without a nonzero are left out.  A product
//     function couples (a, b) with (c, d) only for b <= c, so with the channels
//     ordered by (n_b, n_a) 28 % of the chunks of the (8, 4, nu <= 4) model are
//     empty, and nearly all of a nu <= 3 model's.  A unit holds 16 rows of both
//     sets, so the operand reads of X serve both: with one set per unit these
//     LDS reads, not the matrix units, bound the contraction (L = 4 tile: 24.6k
//     cycles against 16.8k of MFMA).  The accumulators of both sets stay in
//     registers, so X is built once and Z overwrites it, one set at a time;
//  3. adjoint: lane = (target n, atom); job (l_t, l_p, part of the M) forms
//     W[m2][M] = sum_n' A_(n',l_p,m2) Z_({a,p},M) and applies the coupling
//     coefficients once.  Jobs of one target l on different wavefronts write to
//     different slots, added in a fixed order: results are reproducible.
// What bounds it: vector instruction issue (coupling and adjoint of L = 4 take
// 31k of 70k cycles per tile and keep the vector units busy), then the
// contraction, then barriers and LDS latency between the short phases.  More
// wavefronts hide those: 12 per workgroup (168 VGPRs; L = 4 spills 6) at
// L = 2..6, two workgroups of 8 (128 VGPRs; 26, 22 and 17 spill at L = 1, 7 and
// 8) at the others, and for models with few channels workgroups of 4, three to
// a CU (168 VGPRs; 5 and 30 spill at L = 2 and 3), four at L = 0 (128; 31).
// The previous layout (8 wavefronts of 256 VGPRs, dense
// coefficient tiles, X built per set, targets' components split over
// wavefronts) took 2.18 ms for 20,000 atoms of the (8, 4, nu <= 4) model, this
// one 1.51 ms; 389,694 atoms of (6, 3, nu <= 3): 7.23 ms, now 3.39 ms.  Also
// measured on these two: 16 wavefronts at L = 2..6 1.58 ms; one set per unit
// 1.83 ms; workgroups of 8 for the small model 4.02 ms, of 6 5.95 ms.
#pragma once

#include "ace_cg.h"
#include "ap_internal.h"
#include "scan.h"

#include <utility>

namespace ap {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p) { return (cptr<T>)p; }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ f16x8 as_f16x8(uint4 v) { return __builtin_bit_cast(f16x8, v); }

// Power-of-two scale of an atom's entries of X_L.  With B2 the largest
// squared norm |A_(n,l)|^2 over the atom's single indices, every coupled
// entry obeys |AA_{c,M}| <= |A_a| |A_b| <= B2 (the real coupling
// coefficients of one rank are orthonormal over (m1, m2)), every A row
// |A_{n,L,M}| <= sqrt(B2), and L = 0 holds the constant 1.  The scale puts
// the bound just below 2^13: fp16 keeps its full 11 bits in hi and in lo for
// all but negligibly small entries, and no product can overflow.
__device__ __forceinline__ int xscale_exp(float b2, int L) {
  float bound = fmaxf(b2, sqrtf(b2));
  if (L == 0) bound = fmaxf(bound, 1.f);
  int ex = 0;
  (void)frexpf(bound, &ex);
  return 13 - ex;
}

// x (scaled so that |x| < 2^13) as hi + lo in fp16: hi is x rounded to 11
// significant bits, lo the exact fp32 residual x - hi rounded again
__device__ __forceinline__ void put_split(_Float16* xh, int lo_off, float x) {
  const _Float16 hi = (_Float16)x;
  xh[0] = hi;
  xh[lo_off] = (_Float16)fmaf((float)hi, -1.0f, x);
}

template <int LA, int LB, int L, int E>
__device__ __forceinline__ void x_entry(const float* Aa, const float* Ab, float* X) {
  constexpr int q = E % (2 * L + 1), i2 = (E / (2 * L + 1)) % (2 * LB + 1),
                i1 = E / ((2 * L + 1) * (2 * LB + 1));
  if constexpr (cg_rule(i1 - LA, i2 - LB, q - L)) {
    constexpr float c = (float)ce_real_cg(LA, LB, L, i1 - LA, i2 - LB, q - L);
    if constexpr (c != 0.0f) X[q] = fmaf(c, Aa[i1] * Ab[i2], X[q]);
  }
}
template <int LA, int LB, int L, int... E>
__device__ __forceinline__ void x_all(std::integer_sequence<int, E...>, const float* Aa,
                                      const float* Ab, float* X) {
  (x_entry<LA, LB, L, E>(Aa, Ab, X), ...);
}

// One channel (n, LA) x (n', LB) -> L of one atom: the scale goes onto the
// first factor.  out: the channel's row in the atom's first column.
template <int LA, int LB, int L, int KSTR>
__device__ __forceinline__ void x_channel(const float* At, int oa, int ob, int sx, _Float16* out) {
  constexpr int w = 2 * L + 1;
  float Aa[2 * LA + 1], Ab[2 * LB + 1], X[w];
#pragma unroll
  for (int q = 0; q <= 2 * LA; ++q) Aa[q] = ldexpf(At[oa + q], sx);
#pragma unroll
  for (int q = 0; q <= 2 * LB; ++q) Ab[q] = At[ob + q];
#pragma unroll
  for (int q = 0; q < w; ++q) X[q] = 0.f;
  x_all<LA, LB, L>(std::make_integer_sequence<int, (2 * LA + 1) * (2 * LB + 1) * w>{}, Aa, Ab, X);
#pragma unroll
  for (int q = 0; q < w; ++q) put_split(out + q * KSTR, kMT32 * w * KSTR, X[q]);
}

template <int LT, int LP, int L, int Q0, int Q1, int E>
__device__ __forceinline__ void ad_entry(const float* W, float* ga) {
  constexpr int mc = Q1 - Q0;
  constexpr int q = E % mc + Q0, i2 = (E / mc) % (2 * LP + 1), i1 = E / (mc * (2 * LP + 1));
  if constexpr (cg_rule(i1 - LT, i2 - LP, q - L)) {
    constexpr float c = (float)ce_real_cg(LT, LP, L, i1 - LT, i2 - LP, q - L);
    if constexpr (c != 0.0f) ga[i1] = fmaf(c, W[i2 * mc + q - Q0], ga[i1]);
  }
}
template <int LT, int LP, int L, int Q0, int Q1, int... E>
__device__ __forceinline__ void ad_all(std::integer_sequence<int, E...>, const float* W, float* ga) {
  (ad_entry<LT, LP, L, Q0, Q1, E>(W, ga), ...);
}

// Adjoint of the pattern (LT, LP, L) for the M of part K of NC; lane = (target
// n, atom).  The partner sum W[m2][M] = sum_n' A_(n',LP,m2) Z_({a,p},M) comes
// first, so the coupling coefficients enter once per target.  rows: channel
// rows of target (n, LT) for the partners (n', LP), stride lp1, as offsets
// into Z; a missing channel's row is a row of zeros, and the diagonal
// channels' row scales are doubled on the host (both factors of A_a A_a).
template <int LT, int LP, int L, int NC, int K>
__device__ __forceinline__ void ad_job(const float* At, const float* Z, const int16_t* rows, int lp1,
                                       int nlm, int n_max, int zrow, int sx, bool act, float* out,
                                       bool first) {
  constexpr int w = 2 * L + 1, w2 = 2 * LP + 1, w1 = 2 * LT + 1, ZSTR = rank32_zstr(L);
  constexpr int Q0 = K * w / NC, Q1 = (K + 1) * w / NC, mc = Q1 - Q0;
  float W[w2 * mc];
#pragma unroll
  for (int e = 0; e < w2 * mc; ++e) W[e] = 0.f;
  const int16_t* rp = rows + LP;
  const float* ar = At + LP * LP;
  int row_next = act ? (int)rp[0] : zrow;
#pragma unroll 1
  for (int np = 0; np < n_max; ++np) {
    const float* zr = Z + row_next * ZSTR + Q0;
    rp += lp1;
    // the next partner's row, one partner ahead (the table has a row to spare)
    row_next = act ? (int)rp[0] : zrow;
    float a[w2], z[mc];
#pragma unroll
    for (int q = 0; q < w2; ++q) a[q] = ar[q];
#pragma unroll
    for (int q = 0; q < mc; ++q) z[q] = zr[q];
    ar += nlm;
#pragma unroll
    for (int i = 0; i < w2; ++i)
#pragma unroll
      for (int q = 0; q < mc; ++q) W[i * mc + q] = fmaf(a[i], z[q], W[i * mc + q]);
  }
  float ga[w1];
#pragma unroll
  for (int q = 0; q < w1; ++q) ga[q] = 0.f;
  ad_all<LT, LP, L, Q0, Q1>(std::make_integer_sequence<int, w1 * w2 * mc>{}, W, ga);
  if (act) {
    // the atom's column scale is undone here (a power of two)
#pragma unroll
    for (int q = 0; q < w1; ++q) {
      const float g = ldexpf(ga[q], -sx);
      out[q] = first ? g : out[q] + g;
    }
  }
}

// where the thread's gradient entries sit: LDS offset within A or a slot * 8 + l,
// and (atom << 16) | (n << 8) | lm
template <int PF>
struct Grad32 {
  int at[PF], id[PF];
};

template <int PF, int NT>
__device__ __forceinline__ void grad32_index(Grad32<PF>& G, int nA, int nlm, int apad, int tid) {
#pragma unroll
  for (int r = 0; r < PF; ++r) {
    const int q = tid + r * NT;
    const int t = q / nA, e = q - t * nA, nn = e / nlm, lm = e - nn * nlm;
    int l = 0;
    while ((l + 1) * (l + 1) <= lm) ++l;
    G.at[r] = (t * apad + e) * 8 + l;
    G.id[r] = (t << 16) | (nn << 8) | lm;
  }
}

// this rank's tables to LDS
template <int NT>
__device__ __forceinline__ void stage_tables(const Rank32Dev& m, const Rank32L& P, unsigned char* lds,
                                             int L, int tid) {
  const int nidx = m.n_max * (m.l_max + 1);
  float* rs = reinterpret_cast<float*>(lds + P.rs_off);
  int4* mem = reinterpret_cast<int4*>(lds + P.mem_off);
  int16_t* rows = reinterpret_cast<int16_t*>(lds + P.rows_off);
  for (int q = tid; q < nidx * nidx; q += NT) {
    const int r = m.rowtab[(size_t)L * nidx * nidx + q];
    rows[q] = (int16_t)(r < 0 ? P.zrow : r);
  }
  for (int q = tid; q < P.ngrp * kMT32; q += NT) mem[q] = m.grp_mem[(size_t)P.grp0 * kMT32 + q];
  for (int q = tid; q < 2 * P.nrow16; q += NT) rs[q] = m.rscale[P.rs0 + q];
}

// One rank of one tile; A, the column scales sx and the rank's tables are in
// LDS.  NW wavefronts; U: units (16 rows of NS sets) per wavefront; KSTR: k
// stride of X.  The gradient and phi are added to om_buf and phi_buf (the
// first rank writes).  Ends with a barrier.
template <int L, int NW, int U, int NS, int KSTR, int PF>
__device__ __forceinline__ void rank32_tile(const Rank32Dev& m, const Rank32L& P, unsigned char* lds,
                                            const float* A, float* part, const int* sx_lds,
                                            const Grad32<PF>& G, int n_all, int tile, int nt,
                                            float* __restrict__ om_buf, float* __restrict__ phi_buf,
                                            int tid, int wave) {
  constexpr int w = 2 * L + 1, kThreads = 64 * NW;
  constexpr int ncols = kMT32 * w, CT = (ncols + 15) / 16, ZSTR = rank32_zstr(L);
  const int lane = tid & 63;
  const int lp1 = m.l_max + 1, nlm = lp1 * lp1, nA = m.nA, nidx = m.n_max * lp1;
  const float* rs_lds = reinterpret_cast<const float*>(lds + P.rs_off);
  const int4* mem_lds = reinterpret_cast<const int4*>(lds + P.mem_off);
  const int16_t* rows_lds = reinterpret_cast<const int16_t*>(lds + P.rows_off);
  _Float16* X = reinterpret_cast<_Float16*>(lds + P.big_off);  // [ncols][KSTR] hi, then lo
  float* Z = reinterpret_cast<float*>(lds + P.big_off);        // [zrow + 1][ZSTR], over X
  cptr<int32_t> units = as_const(reinterpret_cast<const int32_t*>(m.units)) + 4 * (P.unit0 + wave * P.nu);
  cptr<int32_t> jptr = as_const(m.job_ptr) + P.job0;
  cptr<int32_t> jobs = as_const(reinterpret_cast<const int32_t*>(m.jobs));
  // ---- coupling: lane = (member of the group, atom)
  {
    const int t = lane & 7;
    const float* At = A + t * m.apad;
    const int sx = sx_lds[t];
    for (int g = wave; g < P.ngrp; g += NW) {
      const int4 mem = mem_lds[g * kMT32 + (lane >> 3)];
      const int key = uni(mem.w);
      if (mem.x < 0) continue;
      _Float16* out = X + t * w * KSTR + mem.x;
      switch (key) {
#define AP_X(la, lb)                                                                        \
  case (la) * 5 + (lb):                                                                     \
    if constexpr (iabs_c((la) - (lb)) <= L && L <= (la) + (lb) && (((la) + (lb) + L) & 1) == 0) \
      x_channel<la, lb, L, KSTR>(At, mem.y, mem.z, sx, out);                                \
    break;
#define AP_X5(la) AP_X(la, 0) AP_X(la, 1) AP_X(la, 2) AP_X(la, 3) AP_X(la, 4)
        AP_X5(0) AP_X5(1) AP_X5(2) AP_X5(3) AP_X5(4)
#undef AP_X5
#undef AP_X
        default: break;
      }
    }
    if (P.arow)
      for (int q = tid; q < m.n_max * ncols; q += kThreads) {
        const int n = q / ncols, col = q % ncols, tt = col / w;
        put_split(X + col * KSTR + P.nch + n, ncols * KSTR,
                  ldexpf(A[tt * m.apad + n * nlm + L * L + col % w], sx_lds[tt]));
      }
    if (L == 0 && tid < kMT32)
      put_split(X + tid * KSTR + P.nch + m.n_max, ncols * KSTR, ldexpf(1.f, sx_lds[tid]));
    // rows up to the last 8-row chunk
    const int padr = P.nrow8 - P.nrow;
    for (int q = tid; q < padr * ncols; q += kThreads) {
      X[(q / padr) * KSTR + P.nrow + q % padr] = (_Float16)0.f;
      X[(ncols + q / padr) * KSTR + P.nrow + q % padr] = (_Float16)0.f;
    }
  }
  __syncthreads();
  // ---- contraction of both sets: this wavefront's units
  f32x4 acc[U][NS][CT];
  int urow[U], uset[U];
  const int xcol = (lane & 15) * KSTR;
#pragma unroll
  for (int u = 0; u < U; ++u) {
#pragma unroll
    for (int p = 0; p < NS; ++p)
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[u][p][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    urow[u] = -1;
    uset[u] = 0;
    if (u < P.nu) {
      urow[u] = uni(units[4 * u]);
      uset[u] = uni(units[4 * u + 1]);
      const int s0 = uni(units[4 * u + 2]), ns = uni(units[4 * u + 3]);
      const uint4* cf = m.ctile + (size_t)s0 * 256 + uset[u] * 128 + lane;
      const int32_t* kx = m.kidx + (size_t)s0 * 4 + (lane >> 4);
      // two register buffers: the next PB steps' coefficients (and their
      // chunks of X) load under this step's MFMAs
      constexpr int PB = CT * NS >= 4 ? 1 : 2;
      uint4 ah[PB][NS], al[PB][NS], bh[PB][NS], bl[PB][NS];
      int ak[PB], bk[PB];
      auto load = [&](uint4 (&h)[PB][NS], uint4 (&l)[PB][NS], int (&k)[PB], int s) {
        const int b = min(s, ns - PB);
#pragma unroll
        for (int i = 0; i < PB; ++i) {
#pragma unroll
          for (int p = 0; p < NS; ++p) {
            h[i][p] = cf[(size_t)(b + i) * 256 + p * 128];
            l[i][p] = cf[(size_t)(b + i) * 256 + p * 128 + 64];
          }
          k[i] = kx[(size_t)(b + i) * 4];
        }
        asm volatile("" ::: "memory");
      };
      auto run = [&](const uint4 (&h)[PB][NS], const uint4 (&l)[PB][NS], const int (&k)[PB]) {
#pragma unroll
        for (int i = 0; i < PB; ++i) {
          const _Float16* xr = X + xcol + k[i];
          // the next column tile's operands are read under this one's MFMAs
          uint4 xh = *reinterpret_cast<const uint4*>(xr);
          uint4 xl = *reinterpret_cast<const uint4*>(xr + ncols * KSTR);
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            uint4 nh = xh, nl = xl;
            if (c + 1 < CT) {
              nh = *reinterpret_cast<const uint4*>(xr + (c + 1) * 16 * KSTR);
              nl = *reinterpret_cast<const uint4*>(xr + (c + 1) * 16 * KSTR + ncols * KSTR);
              asm volatile("" ::: "memory");
            }
            // the split products hi hi, hi lo, lo hi, the sets in turn
#pragma unroll
            for (int sp = 0; sp < 3; ++sp)
#pragma unroll
              for (int p = 0; p < NS; ++p)
                acc[u][p][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                    as_f16x8(sp == 2 ? l[i][p] : h[i][p]), as_f16x8(sp == 1 ? xl : xh), acc[u][p][c], 0, 0, 0);
            xh = nh;
            xl = nl;
          }
        }
      };
      if (ns > 0) {
        load(ah, al, ak, 0);
        for (int s = 0; s < ns; s += 2 * PB) {
          load(bh, bl, bk, s + PB);
          run(ah, al, ak);
          if (s + PB < ns) {
            load(ah, al, ak, s + 2 * PB);
            run(bh, bl, bk);
          }
        }
      }
    }
  }
  __syncthreads();  // X is dead from here on
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    float* om = om_buf + (int64_t)p * n_all * nA + (int64_t)tile * kMT32 * nA;
    // the lower ranks' gradient, read ahead of its use
    float og[PF];
#pragma unroll
    for (int r = 0; r < PF; ++r) {
      const int q = tid + r * kThreads;
      og[r] = L > 0 && q < nt * nA ? om[q] : 0.f;
    }
    // ---- Z of set p over X, the row scale undone: result rows 4 (lane / 16) + i
    if (tid < ZSTR) Z[P.zrow * ZSTR + tid] = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (urow[u] >= 0 && (NS == 2 || uset[u] == p)) {
        const int row0 = urow[u] + 4 * (lane >> 4);
        const float4 rs = *reinterpret_cast<const float4*>(rs_lds + p * P.nrow16 + row0);
        float* zp = Z + row0 * ZSTR + (lane & 15);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (row0 + i < P.nrow) {
            const float r = i == 0 ? rs.x : i == 1 ? rs.y : i == 2 ? rs.z : rs.w;
#pragma unroll
            for (int c = 0; c < CT; ++c)
              if (16 * c + 15 < ncols || (lane & 15) < ncols - 16 * c)
                zp[i * ZSTR + 16 * c] = (NS == 2 && p == 1 ? acc[u][NS - 1][c][i] : acc[u][0][c][i]) * r;
          }
        }
      }
    __syncthreads();
    // ---- adjoint jobs of this wavefront
    {
      const int n = lane >> 3, t = lane & 7;
      const bool act = n < m.n_max;
      const float* At = A + t * m.apad;
      const int sx = sx_lds[t];
      const int u0 = uni(jptr[wave]), u1 = uni(jptr[wave + 1]);
      for (int u = u0; u < u1; ++u) {
        const int key = uni(jobs[4 * u]), slot = uni(jobs[4 * u + 1]);
        const bool first = uni(jobs[4 * u + 2]) != 0;
        const int lt = uni(jobs[4 * u + 3]);
        const int16_t* rows = rows_lds + ((act ? n : 0) * lp1 + lt) * nidx;
        float* out = part + (slot * kMT32 + t) * m.apad + (act ? n : 0) * nlm + lt * lt;
        switch (key) {
#define AP_J(lt, lp, k)                                                                         \
  case ((lt) * 5 + (lp)) * 8 + (k):                                                             \
    if constexpr (iabs_c((lt) - (lp)) <= L && L <= (lt) + (lp) && (((lt) + (lp) + L) & 1) == 0 && \
                  (k) < rank32_chunks(lp, L))                                                   \
      ad_job<lt, lp, L, rank32_chunks(lp, L), k>(At, Z + t * w, rows, lp1, nlm, m.n_max, P.zrow, sx, \
                                                 act, out, first);                              \
    break;
#define AP_J6(lt, lp) AP_J(lt, lp, 0) AP_J(lt, lp, 1) AP_J(lt, lp, 2) AP_J(lt, lp, 3) AP_J(lt, lp, 4) AP_J(lt, lp, 5)
#define AP_JT(lt) AP_J6(lt, 0) AP_J6(lt, 1) AP_J6(lt, 2) AP_J6(lt, 3) AP_J6(lt, 4)
          AP_JT(0) AP_JT(1) AP_JT(2) AP_JT(3) AP_JT(4)
#undef AP_JT
#undef AP_J6
#undef AP_J
          default: break;
        }
      }
    }
    // phi by Euler's theorem: A.Z over the A rows plus twice the constant row,
    // by the wavefront with the least adjoint work; lane = (atom, n)
    if (wave == P.phi_wave) {
      const int t = lane >> 3, n = lane & 7;
      float sa = 0.f;
      if (P.arow && n < m.n_max) {
        const float* ar = A + t * m.apad + n * nlm + L * L;
        const float* zr = Z + (P.nch + n) * ZSTR + t * w;
#pragma unroll
        for (int q = 0; q < w; ++q) sa = fmaf(ar[q], zr[q], sa);
      }
#pragma unroll
      for (int d = 4; d >= 1; d >>= 1) sa += __shfl_xor(sa, d, 8);
      if (n == 0 && t < nt) {
        if (L == 0) sa += 2.f * Z[(P.nch + m.n_max) * ZSTR + t];
        sa = ldexpf(sa, -sx_lds[t]);
        float* ph = phi_buf + 2 * ((int64_t)tile * kMT32 + t) + p;
        *ph = L > 0 ? *ph + sa : sa;
      }
    }
    __syncthreads();
    // ---- this rank's gradient: slots in order, then the A rows of X_L
#pragma unroll
    for (int r = 0; r < PF; ++r) {
      const int q = tid + r * kThreads;
      if (q < nt * nA) {
        const int l = G.at[r] & 7, o = G.at[r] >> 3;
        int ns = P.nslots[0];
#pragma unroll
        for (int k = 1; k <= kMaxL; ++k) ns = l == k ? P.nslots[k] : ns;
        float g = 0.f;
        if (ns > 0) {
          float v[kSlots32];
#pragma unroll
          for (int s = 0; s < kSlots32; ++s) v[s] = part[min(s, ns - 1) * kMT32 * m.apad + o];
          g = v[0];
#pragma unroll
          for (int s = 1; s < kSlots32; ++s) g += s < ns ? v[s] : 0.f;
        }
        if (P.arow && l == L) {
          const int t = G.id[r] >> 16, nn = (G.id[r] >> 8) & 255, M = (G.id[r] & 255) - L * L;
          g += ldexpf(Z[(P.nch + nn) * ZSTR + t * w + M], -sx_lds[t]);
        }
        om[q] = og[r] + g;
      }
    }
    __syncthreads();
  }
}

}  // namespace ap
