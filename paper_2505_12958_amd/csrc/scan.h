// Wavefront (64-lane) and workgroup prefix-sum / reduction helpers.
#pragma once
#include <hip/hip_runtime.h>

namespace ap {

// Orders LDS traffic between the lanes of one wavefront.
__device__ __forceinline__ void __syncwarp_ap() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int wave_incl_scan_i32(int v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(v, d, 64);
    if (lane >= d) v += t;
  }
  return v;
}

// Fixed-order butterfly sum over the 64 lanes (same order every run).
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

__device__ __forceinline__ float wave_sum_f32(float v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// Sums over the wavefront of up to 16 values at once: the first four exchanges
// halve the number of values a lane holds (13 exchanges for nine values instead
// of 54).  Lane l returns the sum of value 8 (l>>2&1) + 4 (l>>3&1) + 2 (l>>4&1)
// + (l>>5&1).
template <int NV>
__device__ __forceinline__ double wave_sums_f64(const double (&v)[NV], int lane) {
  static_assert(NV > 8 && NV <= 16, "nine to sixteen values");
  double t[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) t[q] = q < NV ? v[q] : 0.0;
#pragma unroll
  for (int step = 0; step < 4; ++step) {
    const int d = 32 >> step;
#pragma unroll
    for (int q = 0; q < (8 >> step); ++q) {
      if (q * (2 << step) >= NV) continue;  // (zeros)
      const double lo = t[2 * q], hi = t[2 * q + 1];
      const bool up = lane & d;
      t[q] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, d, 64);
    }
#pragma unroll
    for (int q = 0; q < (8 >> step); ++q)
      if (q * (2 << step) >= NV) t[q] = 0.0;
  }
  double r = t[0];
  r += __shfl_xor(r, 2, 64);
  r += __shfl_xor(r, 1, 64);
  return r;
}

// Ascending sort of one value per lane over the wavefront: the bitonic network
// on lane exchanges (DPP up to distance 8, row and half swaps beyond).
template <int D>
__device__ __forceinline__ void lane_pair(int v, int& lo, int& hi) {
  int a = v, b;
  if constexpr (D == 1) b = __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, true);        // quad_perm 1,0,3,2
  else if constexpr (D == 2) b = __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, true);   // quad_perm 2,3,0,1
  else if constexpr (D == 4) {
    b = __builtin_amdgcn_update_dpp(v, v, 0x1B, 0xf, 0xf, true);                            // quad_perm 3,2,1,0
    b = __builtin_amdgcn_update_dpp(b, b, 0x141, 0xf, 0xf, true);                           // row_half_mirror
  } else if constexpr (D == 8) b = __builtin_amdgcn_update_dpp(v, v, 0x128, 0xf, 0xf, true);  // row_ror 8
  else {
    const auto p = D == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false)
                           : __builtin_amdgcn_permlane32_swap(v, v, false, false);
    a = (int)p[0];
    b = (int)p[1];
  }
  lo = a < b ? a : b;
  hi = a < b ? b : a;
}

// lanes that keep the smaller value of a pair at distance D in runs of S
__host__ __device__ constexpr unsigned long long keep_low(int D, int S) {
  unsigned long long m = 0;
  for (int l = 0; l < 64; ++l)
    if (((l & D) == 0) == ((l & S) == 0)) m |= 1ull << l;
  return m;
}

template <int D, int S>
__device__ __forceinline__ void sort_step(int& v) {
  int lo, hi;
  lane_pair<D>(v, lo, hi);
  constexpr unsigned long long m = keep_low(D, S);
  v = __builtin_amdgcn_inverse_ballot_w64(m) ? lo : hi;
  if constexpr (D > 1) sort_step<D / 2, S>(v);
}

__device__ __forceinline__ int wave_sort(int v) {
  sort_step<1, 2>(v);
  sort_step<2, 4>(v);
  sort_step<4, 8>(v);
  sort_step<8, 16>(v);
  sort_step<16, 32>(v);
  sort_step<32, 64>(v);
  return v;
}

// Sum over a workgroup of NW wavefronts; result valid in every thread.
template <int NW>
__device__ __forceinline__ double block_sum_f64(double v, double* lds /* NW doubles */) {
  v = wave_sum_f64(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[w] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int k = 0; k < NW; ++k) t += lds[k];
  return t;
}

}  // namespace ap
