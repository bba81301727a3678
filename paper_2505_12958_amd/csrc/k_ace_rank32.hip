// Mixed rank kernel, one launch and one translation unit per coupled rank L
// (-DAP_RANK_L=<L>).
#include "ace_rank32.h"

#ifndef AP_RANK_L
#error "k_ace_rank32.hip is compiled once per coupled rank with -DAP_RANK_L=<L>"
#endif

namespace ap {

namespace {

template <int L, int NW, int U, int NS, int KSTR>
__global__ __launch_bounds__(64 * NW, rank32_occ(L, NW)) void k_ace_rank32(
    Rank32Dev m, Rank32L P, const int32_t* __restrict__ n_ace_p, int n_all,
    const float* __restrict__ A_in, float* __restrict__ om_buf, float* __restrict__ phi_buf,
    const float* __restrict__ bn_in) {
  constexpr int kThreads = 64 * NW;
  constexpr bool kSmall = NW == kRank32WavesSmall;
  constexpr int PF = (kMT32 * (kSmall ? kRank32NaSmall : 8 * kMaxLM) + kThreads - 1) / kThreads;
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid0 = threadIdx.x;
  const int wave = uni(tid0 >> 6);
  const int nlm = (m.l_max + 1) * (m.l_max + 1), nA = m.nA;
  float* A = reinterpret_cast<float*>(lds);                  // [kMT32][apad]
  float* part = A + kMT32 * m.apad;                          // [slots][kMT32][apad]
  int* sx_lds = reinterpret_cast<int*>(lds + P.sx_off);      // [kMT32]
  const int n_items = n_ace_p ? *n_ace_p : n_all;
  const int n_tiles = (n_items + kMT32 - 1) / kMT32;
  if ((int)blockIdx.x >= n_tiles) return;
  stage_tables<kThreads>(m, P, lds, L, tid0);
  // the tile's A is fetched into registers one tile ahead
  float pa[PF];
  float pbn = 0.f;
  auto fetch = [&](int tile) {
    const int nt = min(kMT32, n_items - tile * kMT32);
#pragma unroll
    for (int r = 0; r < PF; ++r) {
      const int q = tid0 + r * kThreads;
      pa[r] = q < nt * nA ? A_in[(int64_t)tile * kMT32 * nA + q] : 0.f;
    }
    if (tid0 < kMT32) pbn = tid0 < nt ? bn_in[(int64_t)tile * kMT32 + tid0] : 0.f;
  };
  Grad32<PF> G;
  grad32_index<PF, kThreads>(G, nA, nlm, m.apad, tid0);
  fetch(blockIdx.x);
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int nt = min(kMT32, n_items - tile * kMT32);
    // index arithmetic is redone per tile rather than kept in registers across
    // the tile loop
    int tid = tid0;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int r = 0; r < PF; ++r)
      if (tid + r * kThreads < kMT32 * nA) A[G.at[r] >> 3] = pa[r];
    if (tid < kMT32) sx_lds[tid] = xscale_exp(pbn, L);
    __syncthreads();
    if (tile + (int)gridDim.x < n_tiles) fetch(tile + gridDim.x);
    rank32_tile<L, NW, U, NS, KSTR>(m, P, lds, A, part, sx_lds, G, n_all, tile, nt, om_buf, phi_buf, tid,
                                    wave);
  }
}

}  // namespace

template <>
const void* rank32_kernel<AP_RANK_L>(bool small) {
  constexpr int L = AP_RANK_L;
  if constexpr (L <= kRank32LSmall)
    if (small) return (const void*)k_ace_rank32<L, kRank32WavesSmall, kRank32USmall, 2, kRank32KstrSmall>;
  return (const void*)k_ace_rank32<L, rank32_waves(L), kRank32U[L], rank32_sets(L), kRank32Kstr[L]>;
}

}  // namespace ap
