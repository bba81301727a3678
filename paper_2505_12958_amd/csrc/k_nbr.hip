// Cell-list neighbour build: binning (counting sort), 27-cell stencil with
// the canonical FP64 test, ascending-order ELL lists and the reverse-slot
// index.  Also the generic fill and scan primitives.
#include <algorithm>
#include <type_traits>

#include "ap_internal.h"
#include "geom.h"
#include "scan.h"

namespace ap {

// --------------------------------------------------------------------------
template <typename T>
__global__ void k_fill(T* p, T v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

template <typename T>
static hipError_t fill(T* p, T v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) { return fill(p, v, n, s); }
hipError_t launch_fill_f64(double* p, double v, int64_t n, hipStream_t s) { return fill(p, v, n, s); }
hipError_t launch_fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t s) { return fill(p, v, n, s); }

// --------------------------------------------------------------------------
// cell of atom i: orthorhombic boxes bin Cartesian coordinates (clamped into
// the grid in free dimensions), triclinic boxes bin wrapped fractional ones.
// rel (where asked for): the position relative to the cell's centre, in FP32;
// infinite where that is not the nearest image of an atom near its cell (see
// k_fill_nbr_cell).
__device__ __forceinline__ int cell_coords(const SysView& sv, int s, double x, double y, double z,
                                           float3* rel) {
  const int* g = sv.grid + 3 * s;
  const double* H = sv.H + 9 * s;
  double f0, f1, f2;
  bool ok = true;
  if (sv.ortho[s]) {
    f0 = x / H[0];
    f1 = y / H[4];
    f2 = z / H[8];
    ok = (!sv.per[0] || (f0 >= 0.0 && f0 < 1.0)) && (!sv.per[1] || (f1 >= 0.0 && f1 < 1.0)) &&
         (!sv.per[2] || (f2 >= 0.0 && f2 < 1.0));
  } else {
    frac3(sv.Hi + 9 * s, x, y, z, f0, f1, f2);
    ok = f0 >= -0.25 && f0 < 1.25 && f1 >= -0.25 && f1 < 1.25 && f2 >= -0.25 && f2 < 1.25;
    f0 -= floor(f0);
    f1 -= floor(f1);
    f2 -= floor(f2);
  }
  // non-finite coordinates land in cell 0 (the force check reports them)
  int cx = isfinite(f0) ? (int)fmax(-1.0, fmin(floor(f0 * g[0]), (double)g[0])) : 0;
  int cy = isfinite(f1) ? (int)fmax(-1.0, fmin(floor(f1 * g[1]), (double)g[1])) : 0;
  int cz = isfinite(f2) ? (int)fmax(-1.0, fmin(floor(f2 * g[2]), (double)g[2])) : 0;
  cx = cx < 0 ? 0 : (cx >= g[0] ? g[0] - 1 : cx);
  cy = cy < 0 ? 0 : (cy >= g[1] ? g[1] - 1 : cy);
  cz = cz < 0 ? 0 : (cz >= g[2] ? g[2] - 1 : cz);
  if (rel) {
    const double a = f0 - (cx + 0.5) / g[0], b = f1 - (cy + 0.5) / g[1], c = f2 - (cz + 0.5) / g[2];
    double rx = a * H[0], ry = b * H[4], rz = c * H[8];
    if (!sv.ortho[s]) {
      rx += b * H[3] + c * H[6];
      ry += a * H[1] + c * H[7];
      rz += a * H[2] + b * H[5];
    }
    *rel = ok ? make_float3((float)rx, (float)ry, (float)rz) : make_float3(INFINITY, INFINITY, INFINITY);
  }
  return sv.cell_base[s] + (cx * g[1] + cy) * g[2] + cz;
}

// what a neighbour build counts in: cells, the fallback list, the overflow flag
__global__ void k_clear_nbr(int n_cells, int32_t* __restrict__ cell_count, int32_t* __restrict__ big_atoms,
                            int32_t* __restrict__ flag) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_cells) cell_count[i] = 0;
  if (i == 0) {
    big_atoms[0] = 0;
    if (flag) *flag = 0;
  }
}

hipError_t launch_clear_nbr(int32_t n_cells, int32_t* cell_count, int32_t* big_atoms, int32_t* flag,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_clear_nbr, dim3((n_cells + 255) / 256), dim3(256), 0, s, n_cells, cell_count,
                     big_atoms, flag);
  return hipGetLastError();
}

// cell_rank: the atom's place in its cell, in the order of arrival.  Taken here,
// where the count needs its atomic anyway, so that the scatter has none: both
// kernels at 1.27 million atoms 34 + 105 us with a second atomic in the
// scatter, 51 + 33 us so.
__global__ void k_bin(SysView sv, const double* __restrict__ pos, int32_t* __restrict__ cell_of,
                      int32_t* __restrict__ cell_rank, int32_t* __restrict__ cell_count) {
  const int n = sv.n_atoms;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int c = cell_coords(sv, sv.sys_of[i], pos[i], pos[n + i], pos[2 * n + i], nullptr);
  cell_of[i] = c;
  cell_rank[i] = atomicAdd(&cell_count[c], 1);
}

hipError_t launch_bin(const SysView& sv, const double* pos, int32_t* cell_of, int32_t* cell_rank,
                      int32_t* cell_count, hipStream_t s) {
  if (sv.n_atoms == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bin, dim3((sv.n_atoms + 255) / 256), dim3(256), 0, s, sv, pos, cell_of,
                     cell_rank, cell_count);
  return hipGetLastError();
}

__global__ void k_scatter(SysView sv, const double* __restrict__ pos, const int32_t* __restrict__ cell_of,
                          const int32_t* __restrict__ cell_rank,
                          const int32_t* __restrict__ cell_start, int32_t* __restrict__ cell_atoms, double4* __restrict__ cell_pos,
                          float4* __restrict__ cell_rel) {
  const int n = sv.n_atoms;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = pos[i], y = pos[n + i], z = pos[2 * n + i];
  float3 r;
  cell_coords(sv, sv.sys_of[i], x, y, z, &r);
  const int slot = cell_start[cell_of[i]] + cell_rank[i];
  cell_atoms[slot] = i;
  cell_pos[slot] = make_double4(x, y, z, (double)i);
  cell_rel[slot] = make_float4(r.x, r.y, r.z, __int_as_float(i));
}

hipError_t launch_scatter(const SysView& sv, const double* pos, const int32_t* cell_of,
                          const int32_t* cell_rank, const int32_t* cell_start, int32_t* cell_atoms,
                          double4* cell_pos, float4* cell_rel, hipStream_t s) {
  if (sv.n_atoms == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter, dim3((sv.n_atoms + 255) / 256), dim3(256), 0, s, sv, pos,
                     cell_of, cell_rank, cell_start, cell_atoms, cell_pos, cell_rel);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// One wavefront per atom.  The (at most 27, deduplicated) stencil cells are
// laid end to end; lanes walk the concatenated candidates 64 at a time,
// accepted indices are compacted into LDS with a ballot, then each lane
// ranks its entries (indices are unique) and stores them in ascending order.
constexpr int kWavesPerBlock = 4;
constexpr int kListLds = kMaxCap;

__device__ __forceinline__ void atom_list_direct(const SysView& sv, const double* __restrict__ pos,
                                                 const int32_t* __restrict__ cell_of,
                                                 const int32_t* __restrict__ cell_start,
                                                 const int32_t* __restrict__ cell_count,
                                                 const double4* __restrict__ cell_pos,
                                                 int32_t* __restrict__ nbr,
                                                 int32_t* __restrict__ count, int cap,
                                                 int32_t* __restrict__ overflow, int i,
                                                 int (&list)[kWavesPerBlock][kListLds],
                                                 int (&st_cell)[kWavesPerBlock][32],
                                                 int (&st_pre)[kWavesPerBlock][33]) {
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int n = sv.n_atoms;
  const int s = sv.sys_of[i];
  const double xi = pos[i], yi = pos[n + i], zi = pos[2 * n + i];
  const int* g = sv.grid + 3 * s;
  const int ci = cell_of[i] - sv.cell_base[s];
  const int c0 = ci / (g[1] * g[2]);
  const int c1 = (ci / g[2]) % g[1];
  const int c2 = ci % g[2];
  const int cc[3] = {c0, c1, c2};
  // stencil: lane k < 27 owns offset (k/9, k/3%3, k%3) of the per-axis lists
  int my_cell = -1, my_cnt = 0;
  if (lane < 27) {
    int idx[3] = {lane / 9, (lane / 3) % 3, lane % 3};
    int co[3];
    bool ok = true;
    for (int k = 0; k < 3; ++k) {
      const int gk = g[k];
      if (sv.per[k] && gk < 3) {
        if (idx[k] >= gk) ok = false;
        co[k] = idx[k];
      } else {
        int v = cc[k] + idx[k] - 1;
        if (sv.per[k]) {
          v = v < 0 ? v + gk : (v >= gk ? v - gk : v);
        } else if (v < 0 || v >= gk) {
          ok = false;
        }
        co[k] = v;
      }
    }
    if (ok) {
      my_cell = sv.cell_base[s] + (co[0] * g[1] + co[1]) * g[2] + co[2];
      my_cnt = cell_count[my_cell];
    }
  }
  const int incl = wave_incl_scan_i32(my_cnt, lane);
  const int total = __shfl(incl, 63);
  if (lane < 27) {
    st_cell[w][lane] = my_cell;
    st_pre[w][lane] = incl - my_cnt;
  }
  if (lane == 27) st_pre[w][27] = total;
  __syncwarp_ap();
  const bool ortho = sv.ortho[s] != 0;
  const double* H = sv.H + 9 * s;
  const double* Hi = sv.Hi + 9 * s;
  int cnt = 0;
  for (int base = 0; base < total; base += 64) {
    const int c = base + lane;
    bool acc = false;
    int j = -1;
    if (c < total) {
      int k = 0;
      while (k < 26 && st_pre[w][k + 1] <= c) ++k;
      const int slot = cell_start[st_cell[w][k]] + (c - st_pre[w][k]);
      const double4 q = cell_pos[slot];
      j = (int)q.w;
      if (j != i) {
        double dx, dy, dz;
        displacement(ortho, H, Hi, sv.per, xi, yi, zi, q.x, q.y, q.z, dx, dy, dz);
        acc = norm2(dx, dy, dz) < sv.rc2;
      }
    }
    const unsigned long long b = __ballot(acc);
    if (acc) {
      const int p = cnt + __popcll(b & ((1ull << lane) - 1ull));
      if (p < kListLds) list[w][p] = j;
    }
    cnt += __popcll(b);
  }
  __syncwarp_ap();
  if (cnt > cap && lane == 0) atomicMax(overflow, cnt);
  const int m = cnt < kListLds ? cnt : kListLds;
  for (int e = lane; e < m; e += 64) {
    const int v = list[w][e];
    int rank = 0;
    for (int q = 0; q < m; ++q) rank += list[w][q] < v;
    if (rank < cap) nbr[(int64_t)rank * n + i] = v;
  }
  if (lane == 0) count[i] = cnt < cap ? cnt : cap;
}

__global__ __launch_bounds__(256) void k_fill_nbr_big(SysView sv, const double* __restrict__ pos,
                                                      const int32_t* __restrict__ cell_of,
                                                      const int32_t* __restrict__ cell_start,
                                                      const int32_t* __restrict__ cell_count,
                                                      const double4* __restrict__ cell_pos,
                                                      int32_t* __restrict__ nbr,
                                                      int32_t* __restrict__ count, int cap,
                                                      int32_t* __restrict__ overflow,
                                                      const int32_t* __restrict__ big_atoms) {
  __shared__ int list[kWavesPerBlock][kListLds];
  __shared__ int st_cell[kWavesPerBlock][32];
  __shared__ int st_pre[kWavesPerBlock][33];
  // big_atoms = [m, atom_0, ..., atom_{m-1}]: one wavefront per listed atom,
  // grid-stride (the loop only holds wavefront-level synchronisation)
  const int m = big_atoms[0];
  const int waves = gridDim.x * kWavesPerBlock;
  for (int w = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6); w < m; w += waves)
    atom_list_direct(sv, pos, cell_of, cell_start, cell_count, cell_pos, nbr, count, cap, overflow,
                     big_atoms[1 + w], list, st_cell, st_pre);
}

// --------------------------------------------------------------------------
// One workgroup per cell.  The candidates of the cell's stencil (at most 27
// deduplicated cells) are gathered into LDS once, as FP32 positions relative
// to the cell's centre in the image next to it, and shared by the cell's
// atoms, one wavefront per atom: lanes test 64 candidates at a time, accepted
// indices are compacted into a per-wavefront LDS list, sorted across the lanes
// (at most 64 of them; more are ranked in LDS) and stored in ascending order.
//
// The result is the canonical FP64 rule's (geom.h), bit for bit, though nearly
// every pair is decided in FP32: a pair is accepted below r_c (1 - 2e-5) and
// rejected beyond r_c (1 + 2e-5); between, the wavefront evaluates the rule
// itself.  That is sound as long as
//  - coordinates stay below 8 r_c, those relative to an atom's own cell (FP32,
//    cell_rel) as well as the sums with the offset between the two cells: each
//    is rounded by at most 8 r_c 2^-24, a distance is off by less than 1e-5 r_c;
//  - every fractional coordinate lies in [-1/4, 5/4), so that the rule's single
//    wrap yields the nearest image, and the atom in the cell of its wrapped
//    position (orthorhombic boxes: in [0, 1), atoms outside are binned into the
//    box's outer cells unwrapped);
//  - the images agree, or both are out of reach.  With at least three cells
//    along an axis the staged image differs from the nearest only where the
//    two are a third of the box or more apart, at least one cell edge
//    (> r_c) in either; with fewer cells the pair is wrapped again, and a pair
//    within 1e-5 of half the box goes to the rule.
// A workgroup that holds any candidate outside these limits takes the rule for
// every pair.  A cell whose stencil holds more than kMaxCand candidates falls
// back to the kernel above for its atoms.
//
// The instruction issue bounds it (per atom about 230 vector and 175 scalar
// instructions; it was 412 vector with an FP32 screen that wrapped every pair,
// an FP64 test of each survivor and the rank loop).  Cells are dealt to the XCDs
// in contiguous runs, so that the 4-byte stores into the slot-major rows meet
// in one L2.  us, before -> after: 250,000 atoms 202 -> 134, 1.27 million
// 1032 -> 627, 2.66 million 2284 -> 1282, 96 sheared cells of 250 to 16,000 atoms
// (the FP64 test of every candidate fell away) 620 -> 201.  Seven workgroups a
// CU (2 VGPRs spill) rather than six: 1282 against 1336 us at 2.66 million; with
// eight more spill, 670 against 622 us at 1.27 million.
constexpr int kCellThreads = 256;
constexpr int kCellWaves = kCellThreads / 64;
constexpr int kMaxCand = 512;

__global__ __launch_bounds__(kCellThreads, 7) void k_fill_nbr_cell(
    SysView sv, const int32_t* __restrict__ cell_start, const int32_t* __restrict__ cell_count,
    const double4* __restrict__ cell_pos, const float4* __restrict__ cell_rel,
    int32_t* __restrict__ nbr, int32_t* __restrict__ count, int cap, int32_t* __restrict__ overflow,
    int32_t* __restrict__ big_atoms) {
  __shared__ float4 cposf[kMaxCand];  // x, y, z; w: the atom's index
  __shared__ int csrc[kMaxCand];      // its place in cell_pos
  __shared__ __align__(16) int list[kCellWaves][kMaxCand + 4];
  __shared__ float4 st_off[27];  // stencil cells: centre relative to this cell's; w: atoms
  __shared__ int2 st_src[27];    // first cell-ordered atom, exclusive prefix of the counts
  __shared__ int s_head[4];      // total, any candidate for the rule, system, home
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = xcd_chunk(blockIdx.x, gridDim.x);
  const int n_here = cell_count[c];
  if (n_here == 0) return;  // whole workgroup
  if (wave == 0) {
    // system of this cell
    int lo = 0, hi = sv.n_sys - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (sv.cell_base[mid] <= c) lo = mid; else hi = mid - 1;
    }
    const int s = lo;
    const int* g = sv.grid + 3 * s;
    const double* H = sv.H + 9 * s;
    const int ci = c - sv.cell_base[s];
    const int cc[3] = {ci / (g[1] * g[2]), (ci / g[2]) % g[1], ci % g[2]};
    int my_cnt = 0, home = 0;
    if (lane < 27) {
      const int idx[3] = {lane / 9, (lane / 3) % 3, lane % 3};
      int co[3], my_src = 0;
      double o[3];
      bool ok = true;
      for (int k = 0; k < 3; ++k) {
        const int gk = g[k];
        const bool few = sv.per[k] && gk < 3;  // the stencil is the whole axis
        home = 3 * home + (few ? cc[k] : 1);
        int v = few ? idx[k] : cc[k] + idx[k] - 1;
        o[k] = (double)(v - cc[k]) / gk;
        if (few) {
          if (v >= gk) ok = false;
        } else if (sv.per[k]) {
          v = v < 0 ? v + gk : (v >= gk ? v - gk : v);
        } else if (v < 0 || v >= gk) {
          ok = false;
        }
        co[k] = v;
      }
      if (ok) {
        const int my_cell = sv.cell_base[s] + (co[0] * g[1] + co[1]) * g[2] + co[2];
        my_cnt = cell_count[my_cell];
        my_src = cell_start[my_cell];
      }
      // (off-diagonal entries of an orthorhombic box are zero)
      st_off[lane] = make_float4((float)(o[0] * H[0] + o[1] * H[3] + o[2] * H[6]),
                                 (float)(o[0] * H[1] + o[1] * H[4] + o[2] * H[7]),
                                 (float)(o[0] * H[2] + o[1] * H[5] + o[2] * H[8]),
                                 __int_as_float(my_cnt));
      st_src[lane].x = my_src;
    }
    const int incl = wave_incl_scan_i32(my_cnt, lane);
    if (lane < 27) st_src[lane].y = incl - my_cnt;
    if (lane == 0) {
      s_head[1] = 0;
      s_head[2] = s;
      s_head[3] = home;
    }
    if (lane == 26) s_head[0] = incl;
  }
  __syncthreads();
  const int total = __builtin_amdgcn_readfirstlane(s_head[0]);
  const int n = sv.n_atoms;
  const int first = cell_start[c];
  if (total > kMaxCand) {
    // too many candidates for LDS: the cell's atoms go to the fallback
    // kernel's list (their order there does not matter, every row is
    // computed on its own)
    __shared__ int s_base;
    if (tid == 0) s_base = atomicAdd(big_atoms, n_here);
    __syncthreads();
    for (int a = tid; a < n_here; a += kCellThreads)
      big_atoms[1 + s_base + a] = (int)cell_pos[first + a].w;
    return;
  }
  // candidates, cell after cell, 16 threads to a stencil cell; the last batch
  // of 64 is padded with positions that pass no comparison
  {
    const float rc2 = (float)sv.rc2, reach2 = 64.f * rc2;
    bool exact = false;
    for (int k = tid >> 4; k < 27; k += kCellThreads / 16) {
      const float4 o = st_off[k];
      const int2 src = st_src[k];
      for (int q = tid & 15; q < __float_as_int(o.w); q += 16) {
        const float4 r = cell_rel[src.x + q];
        const float x = r.x + o.x, y = r.y + o.y, z = r.z + o.z;
        const float big = fmaxf(fmaxf(fmaxf(r.x * r.x, r.y * r.y), fmaxf(r.z * r.z, x * x)),
                                fmaxf(y * y, z * z));
        exact = exact || !(big < reach2) || isnan(x) || isnan(y) || isnan(z);
        cposf[src.y + q] = make_float4(x, y, z, r.w);
        csrc[src.y + q] = src.x + q;
      }
    }
    const int pad = ((total + 63) & ~63) - total;
    if (tid < pad) cposf[total + tid] = make_float4(NAN, NAN, NAN, __int_as_float(-1));
    if (exact) s_head[1] = 1;
  }
  __syncthreads();
  const bool exact = __builtin_amdgcn_readfirstlane(s_head[1]) != 0;
  const int s = __builtin_amdgcn_readfirstlane(s_head[2]);
  const int self0 = __builtin_amdgcn_readfirstlane(st_src[s_head[3]].y);
  const bool ortho = sv.ortho[s] != 0;
  const int* g = sv.grid + 3 * s;
  const double* H = sv.H + 9 * s;
  const double* Hi = sv.Hi + 9 * s;
  const bool few[3] = {sv.per[0] && g[0] < 3, sv.per[1] && g[1] < 3, sv.per[2] && g[2] < 3};
  const float near2 = (float)(sv.rc2 * ((1.0 - 2e-5) * (1.0 - 2e-5)));
  const float far2 = (float)(sv.rc2 * ((1.0 + 2e-5) * (1.0 + 2e-5)));
  // the pair's wrap along the few-cell axes: fractional rows and lattice vectors
  const bool wrap = few[0] || few[1] || few[2];
  __shared__ float s_wrap[3][6];
  if (wrap) {
    if (tid < 9) {
      const int k = tid / 3, x = tid % 3;
      s_wrap[k][x] = ortho ? (k == x ? 1.f / (float)H[4 * k] : 0.f) : (float)Hi[3 * x + k];
      s_wrap[k][3 + x] = (float)H[3 * k + x];
    }
    __syncthreads();
  }
  int* lw = list[wave];
  // the accepted candidates of the cell's atom a, in candidate order: their
  // number.  kMode 0: pairs in FP32; 1: after the wrap along the few-cell axes;
  // 2: every pair by the rule
  auto scan = [&](auto mode, int a) {
    constexpr int kMode = decltype(mode)::value;
    const float4 me = cposf[self0 + a];
    const int i = __float_as_int(me.w);
    int cnt = 0;
    for (int base = 0; base < total; base += 64) {
      const float4 pf = cposf[base + lane];
      const int j = __float_as_int(pf.w);
      unsigned long long in = 0, open = ~0ull;
      if constexpr (kMode < 2) {
        float dx = pf.x - me.x, dy = pf.y - me.y, dz = pf.z - me.z;
        bool edge = false;
        if constexpr (kMode == 1) {
#pragma unroll
          for (int k = 0; k < 3; ++k)
            if (few[k]) {
              const float* w = s_wrap[k];
              const float t = w[0] * dx + w[1] * dy + w[2] * dz, u = rintf(t);
              edge = edge || fabsf(t - u) > 0.49999f;
              dx -= u * w[3];
              dy -= u * w[4];
              dz -= u * w[5];
            }
        }
        const float r2 = dx * dx + dy * dy + dz * dz;
        in = __ballot(r2 < near2);
        open = __ballot(r2 < far2) & ~in;
        if constexpr (kMode == 1) open |= __ballot(edge);
      }
      if (open) {
        bool acc = false;
        if ((open >> lane & 1) && base + lane < total) {
          const double4 pi = cell_pos[first + a], pj = cell_pos[csrc[base + lane]];
          double ex, ey, ez;
          displacement(ortho, H, Hi, sv.per, pi.x, pi.y, pi.z, pj.x, pj.y, pj.z, ex, ey, ez);
          acc = norm2(ex, ey, ez) < sv.rc2;
        }
        in = (in & ~open) | __ballot(acc);
      }
      in &= __ballot(j != i);
      if (__builtin_amdgcn_inverse_ballot_w64(in))
        lw[__builtin_amdgcn_mbcnt_hi((unsigned)(in >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in, cnt))] = j;
      cnt += __popcll(in);
    }
    return cnt;
  };
  for (int a = wave; a < n_here; a += kCellWaves) {
    const int i = __builtin_amdgcn_readfirstlane(__float_as_int(cposf[self0 + a].w));
    const int cnt = exact  ? scan(std::integral_constant<int, 2>{}, a)
                    : wrap ? scan(std::integral_constant<int, 1>{}, a)
                           : scan(std::integral_constant<int, 0>{}, a);
    if (cnt <= 64) {
      __syncwarp_ap();
      const int v = wave_sort(lane < cnt ? lw[lane] : 0x7fffffff);
      if (lane < (cnt < cap ? cnt : cap)) nbr[(int64_t)lane * n + i] = v;
    } else {
      if (lane < 4) lw[cnt + lane] = 0x7fffffff;  // sentinels: the rank loop reads whole int4
      __syncwarp_ap();
      for (int e = lane; e < cnt; e += 64) {
        const int v = lw[e];
        int rank = 0;
        for (int q = 0; q < cnt; q += 4) {
          const int4 u = *reinterpret_cast<const int4*>(lw + q);
          rank += (u.x < v) + (u.y < v) + (u.z < v) + (u.w < v);
        }
        if (rank < cap) nbr[(int64_t)rank * n + i] = v;
      }
    }
    if (lane == 0) {
      count[i] = cnt < cap ? cnt : cap;
      if (cnt > cap) atomicMax(overflow, cnt);
    }
    __syncwarp_ap();
  }
}

hipError_t launch_fill_nbr_cells(const SysView& sv, int32_t n_cells, const double* pos,
                                 const int32_t* cell_of, const int32_t* cell_start,
                                 const int32_t* cell_count, const double4* cell_pos,
                                 const float4* cell_rel, int32_t* nbr, int32_t* count, int32_t cap,
                                 int32_t* overflow, int32_t* big_atoms, hipStream_t s) {
  if (sv.n_atoms == 0 || n_cells == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_nbr_cell, dim3(n_cells), dim3(kCellThreads), 0, s, sv, cell_start,
                     cell_count, cell_pos, cell_rel, nbr, count, cap, overflow, big_atoms);
  const int blocks = std::min((sv.n_atoms + kWavesPerBlock - 1) / kWavesPerBlock, 1024);
  hipLaunchKernelGGL(k_fill_nbr_big, dim3(blocks), dim3(64 * kWavesPerBlock), 0, s, sv, pos, cell_of,
                     cell_start, cell_count, cell_pos, nbr, count, cap, overflow, big_atoms);
  return hipGetLastError();
}

// rev[s][i] = slot of i in the (ascending) list of j = nbr[s][i]
__global__ void k_rev(int n, const int32_t* __restrict__ nbr, const int32_t* __restrict__ count,
                      int32_t* __restrict__ rev) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int ci = count[i];
  for (int s = 0; s < ci; ++s) {
    const int j = nbr[(int64_t)s * n + i];
    int lo = 0, hi = count[j] - 1, r = -1;
    while (lo <= hi) {
      const int mid = (lo + hi) >> 1;
      const int v = nbr[(int64_t)mid * n + j];
      if (v == i) { r = mid; break; }
      if (v < i) lo = mid + 1; else hi = mid - 1;
    }
    rev[(int64_t)s * n + i] = r;
  }
}

hipError_t launch_rev(int32_t n_atoms, const int32_t* nbr, const int32_t* count, int32_t* rev,
                      hipStream_t s) {
  if (n_atoms == 0) return hipSuccess;
  hipLaunchKernelGGL(k_rev, dim3((n_atoms + 255) / 256), dim3(256), 0, s, n_atoms, nbr, count, rev);
  return hipGetLastError();
}

}  // namespace ap
