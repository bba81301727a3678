// Internal declarations of the AP library: context, device-side model
// tables, kernel launchers.  Not part of the public ABI (include/ap.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <string>
#include <vector>

#include "../../include/ap.h"

namespace ap {

constexpr int kMaxSys = 1 << 20;
constexpr int kMaxL = 4;                   // l_max limit of the ACE model
constexpr int kMaxLM = (kMaxL + 1) * (kMaxL + 1);
constexpr int kMaxN = 16;
constexpr int kMaxK = 16;
constexpr int kMaxCap = 256;               // neighbour-list capacity limit
constexpr int kReduceChunk = 4096;         // atoms per deterministic partial sum

#define AP_HIP(call)                                                    \
  do {                                                                  \
    hipError_t e_ = (call);                                             \
    if (e_ != hipSuccess) return fail_hip(ctx, e_, #call, __FILE__, __LINE__); \
  } while (0)

// Workgroups go to the eight XCDs in turn; this numbers them so that each XCD
// gets one contiguous run of the work items, whose neighbours then share its L2.
constexpr unsigned kXcds = 8;
__host__ __device__ inline unsigned xcd_chunk(unsigned b, unsigned n) {
  const unsigned q = n / kXcds, r = n % kXcds, x = b % kXcds;
  return x * q + (x < r ? x : r) + b / kXcds;
}

// The same in runs of `run` workgroups: where the work sits in a part of the
// grid that the host doesn't know, every XCD still gets its share.
__host__ __device__ inline unsigned xcd_runs(unsigned b, unsigned n, unsigned run) {
  const unsigned group = kXcds * run, g0 = b / group * group;
  if (g0 + group > n) return b;
  const unsigned r = b - g0;
  return g0 + r % kXcds * run + r / kXcds;
}

// --------------------------------------------------------------------------
// device view of the systems of one call
struct SysView {
  int32_t n_sys;
  int32_t n_atoms;
  const int64_t* off;      // n_sys+1
  const double* H;         // 9 per system
  const double* Hi;        // 9 per system (triclinic inverse; unused for orthorhombic)
  const uint8_t* ortho;    // per system
  const int32_t* grid;     // 3 per system: cells along each axis
  const int32_t* cell_base;// n_sys+1: first global cell of each system
  const int32_t* sys_of;   // per atom
  int32_t per[3];
  int32_t all_ortho;        // every system orthorhombic (kernels may specialise)
  double rc2;
};

// piecewise-cubic table on device (4 coefficients per interval)
struct TableDev {
  double x0, dx, inv_dx;
  int32_t n;                // knots
  const double* c;          // (n-1)*4
  const float* cf;          // same, float
};

// the paper's W EAM in closed form (passed to the EAM kernels by value)
constexpr int kMaxEamKnots = 32;
// a knot sum as cubics between its sorted distinct knots
struct KnotDev {
  int32_t n, n4;                    // distinct knots; padded to a multiple of 4
  double knot[kMaxEamKnots];        // ascending, padded with +inf
  double c[kMaxEamKnots + 1][4];    // interval below knot[k] (k = n: zero): powers of knot[k] - r
};
struct EamAnalyticDev {
  KnotDev phi, rho;
  double r_cut_rho, zeta_cut;       // zeta = zeta_0(max(r, r_cut)); zeta_cut = zeta_0(r_cut)
  double a_xi1, a_xi2, d_xi;
  double zbl_pref, a_zbl;           // Z^2 / (4 pi eps0), screening length
  double zbl_c[4], zbl_q[4];
  double r_lo, r_hi, b_phi[6];
};

// ACE model folded for the device
// one term of the FP64 path's sparse sums, read as a single 16-byte load:
// coefficient c and the two operand indices i, j
struct alignas(16) PairTerm {
  double c;
  int32_t i, j;
};

struct AceDev {
  int32_t n_max, l_max, K, nlm, nA, nnl;
  int32_t L_max;            // largest coupled L
  double rc;
  const double* W;          // [n_max][l_max+1][K]
  const float* Wf;
  const double* ynorm;      // N_lm for m >= 0 at l*l + l + m (sqrt2 folded in for m > 0)
  // per L (0..L_max): X_L rows = [channels | A rows (n, l=L) | one-row (L=0)]
  int32_t nrow[2 * kMaxL + 1];
  int32_t nch[2 * kMaxL + 1];
  int32_t has_arow[2 * kMaxL + 1];
  // CSR building X: entry e of (channel row r, M) at dst = r*(2L+1)+M
  int32_t xb_off[2 * kMaxL + 2];    // offset of the L block in xb_ptr (size nch*(2L+1)+1 each)
  const int32_t* xb_ptr;
  const PairTerm* xb_t;             // c A[i] A[j]
  // Cext_L CSR over rows (symmetric, both coefficient sets)
  int32_t cx_off[2 * kMaxL + 2];    // offset of the L block in cx_ptr (nrow+1 each)
  const int32_t* cx_ptr;
  const int32_t* cx_col;
  const double2* cx_val;
  // adjoint CSR over A targets: terms (z index, partner A index, coef)
  int32_t ad_off[2 * kMaxL + 2];    // offset of the L block in ad_ptr (nA+1 each)
  const int32_t* ad_ptr;
  const PairTerm* ad_t;             // c A[i] Z[j]
  int32_t max_xsize;        // max_L nrow*(2L+1)
};

// wavefronts of a workgroup of the FP64 rank kernels
constexpr int kRank64Waves = 8;
// modes of the mixed rank phase: the narrow variant of the ranks that have one
// (few channels), or the wide variant of every rank (2 is accepted as 1)
enum { AP_RANK_NARROW = 0, AP_RANK_WIDE = 1, AP_RANK_WIDE_2 = 2, AP_RANK_N_MODES = 3 };

// the ACE model as the mixed path's bond kernels read it
struct MixDev {
  int32_t n_max, l_max, K, nA, apad, L_max;
  double rc;
  const float* Wf;
  const double* ynorm;
};

// ---- FP64 rank kernels (k_ace_rank64.hip): C_L as 16 x 4 tiles for the FP64
// MFMA, empty tiles left out
constexpr int kT64 = 4;              // atoms per tile
// ACE atoms whose A and adjoint are held at once.  The list's length is on the
// device, so the buffers are sized by the atoms (4.8 KB each at nA = 200, 1.3 GB
// at most) and batches beyond the list are launched empty, about 20 us each.
// Smaller batches trade the one for the other: 250,000 atoms, 20,000 listed,
// 1.78, 1.21 and 0.89 GB of scratch in all at 262,144, 131,072 and 65,536 items,
// 7.62, 7.64 and 7.68 ms; 2.66 million, 35,229 listed, 6.7, 6.0 and 5.7 GB, 16.1,
// 16.4 and 16.8 ms.
constexpr int kRank64Items = 262144;
constexpr int kRank64MaxN = 8;       // lanes per atom of the adjoint: n_max <= 8
// doubles of the adjoint's partner sum a lane holds at once (two VGPRs each)
constexpr int kRank64Lim = 27;
// units (16 rows of one set) per wavefront and rank: what the complete basis of
// n_max 8, l_max 4, nu 4 needs
constexpr int kRank64U[2 * kMaxL + 1] = {3, 5, 6, 6, 5, 3, 3, 1, 1};
// L <= 1 with at most 3 units per wavefront runs in 128 VGPRs (L = 1 spills 48),
// so two workgroups share a CU (20,518 atoms of the (6, 3, nu <= 3) model: L = 0
// 122 -> 85 us, L = 1 190 -> 124 us); at L >= 2 the spills cost more than that
// gives (L = 2 284 -> 290 us, L = 3 292 -> 308 us)
constexpr int kRank64USmall = 3, kRank64LSmall = 1;
// parts the M of rank L are cut into for a partner of rank lp (at most 4)
__host__ __device__ constexpr int rank64_chunks(int lp, int L) {
  const int n = ((2 * lp + 1) * (2 * L + 1) + kRank64Lim - 1) / kRank64Lim;
  return n > 4 ? 4 : n;
}
struct Rank64L {
  int32_t nrow, nrow4, nch, arow;   // rows of X_L, padded to the 4-row steps, channel rows, has A rows
  int32_t zrow, cstr;               // row of zeros (= nrow4), row stride in doubles
  int32_t grp0, ngrp;               // channel groups (64 / kT64 members each)
  int32_t unit0, nu;                // first unit, units per wavefront
  int32_t small;                    // two workgroups per CU
  int32_t nslots[kMaxL + 1];        // gradient slots per target l
};
struct Rank64Dev {
  int32_t n_max, l_max, nA, apad, slots;
  const int4* grp_mem;              // {row (-1: none), A offset of a, of b, la * 5 + lb}
  const int32_t* rowtab;            // [L][a][p]: row of the coupled channel {a, p}, or -1
  const int4* units;                // {first row (-1: none), set, first step, steps}
  const int32_t* kidx;              // per step: LDS offset of its 4 rows of X
  const double* coef;               // per step: 16 x 4 coefficients in lane order
  const int32_t* job_ptr;           // [L][kRank64Waves + 1]
  const int4* jobs;                 // {(lt * 5 + lp) * 4 + part, slot, first of its slot, lt}
};

// ---- mixed rank kernels (k_ace_rank32.hip): C_L as 16-row steps of four
// 8-column chunks in split fp16, empty chunks left out
constexpr int kMT32 = 8;             // atoms per tile
__host__ __device__ constexpr int rank32_zstr(int L) { return 8 * (2 * L + 1) + 4; }
// wavefronts per workgroup: 16 (128 VGPRs each) or 12 (168) fill a CU, two
// workgroups of 8 (128) share it where their LDS fits
__host__ __device__ constexpr int rank32_waves(int L) { return L < 2 || L > 6 ? 8 : 12; }
constexpr int kRank32WavesSmall = 4;
// wavefronts per SIMD (512 / this VGPRs each) and workgroups per CU
__host__ __device__ constexpr int rank32_occ(int L, int nw) { return nw == 8 || L == 0 ? 4 : 3; }
__host__ __device__ constexpr int rank32_groups(int L, int nw) { return 4 * rank32_occ(L, nw) / nw; }
// sets a unit (16 rows) holds: both, which then share the operand reads of X,
// but where a rank has fewer row tiles than wavefronts
__host__ __device__ constexpr int rank32_sets(int L) { return L == 0 || L >= 7 ? 1 : 2; }
// units per wavefront and k stride of X (fp16): what the complete basis of
// n_max 8, l_max 4, nu 4 needs; the stride is 8, 24, 40 or 56 mod 64, so the
// 16-byte operand reads of 8 consecutive columns hit distinct banks
constexpr int kRank32U[2 * kMaxL + 1] = {3, 3, 2, 2, 2, 1, 1, 1, 1};
constexpr int kRank32Kstr[2 * kMaxL + 1] = {200, 264, 344, 328, 312, 200, 136, 72, 40};
// the narrow variant of L = 0..3 for models with few channels: 4 wavefronts per
// workgroup, so that three or four workgroups share a CU
constexpr int kRank32USmall = 3, kRank32KstrSmall = 136, kRank32LSmall = 3, kRank32NaSmall = 128;
constexpr int kSlots32 = 4;          // gradient slots of a target l, at most
// parts the M of rank L are cut into for a partner of rank lp: floats of the
// adjoint's partner sum a lane holds beside the accumulators of the other set
__host__ __device__ constexpr int rank32_chunks(int lp, int L) {
  constexpr int lims[2 * kMaxL + 1] = {27, 27, 45, 42, 36, 54, 45, 27, 27};
  const int lim = lims[L];
  const int n = ((2 * lp + 1) * (2 * L + 1) + lim - 1) / lim;
  return n > 6 ? 6 : n;
}
struct Rank32L {
  int32_t nrow, nrow8, nrow16, nch, arow;  // rows of X_L, padded to chunks and row tiles
  int32_t zrow;                            // row of zeros of Z (= nrow)
  int32_t grp0, ngrp;                      // channel groups (8 members each)
  int32_t unit0, nu;                       // first unit, units per wavefront
  int32_t job0, rs0;                       // first entry of job_ptr, of rscale
  int32_t slots, nslots[kMaxL + 1];        // gradient slots: most, per target l
  // LDS offsets: column scales, row scales, channel groups, channel rows, X / Z
  int32_t sx_off, rs_off, mem_off, rows_off, big_off;
  int32_t phi_wave;                        // wavefront that sums phi
  int32_t small;                           // the narrow variant
};
struct Rank32Dev {
  int32_t n_max, l_max, nA, apad;
  const int4* grp_mem;                     // {row (-1: none), A offset of a, of b, la * 5 + lb}
  const int32_t* rowtab;                   // [L][a][p]: row of the coupled channel {a, p}, or -1
  const int4* units;                       // {first row (-1: none), set, first step, steps}
  const int32_t* kidx;                     // per step: first row of each of its four chunks
  const uint4* ctile;                      // per step and set: 64 lanes of hi, 64 of lo (8 fp16 each)
  const float* rscale;                     // per set and row: inverse of the row's scale
  const int32_t* job_ptr;
  const int4* jobs;                        // {(lt * 5 + lp) * 8 + part, slot, first of its slot, lt}
};

struct Buffer {
  void* p = nullptr;
  size_t bytes = 0;
};

struct SysCache {
  bool valid = false;
  std::vector<int64_t> off;
  std::vector<double> box;
  uint8_t periodic[3] = {0, 0, 0};
  double cutoff = 0;
  int32_t n_cells = 0;
  int32_t n_chunks = 0;
  bool one_chunk_each = false;
  bool all_ortho = false;
  // device
  Buffer off_d, H_d, Hi_d, ortho_d, grid_d, cell_base_d, sys_of_d;
  Buffer chunk_lo_d, chunk_hi_d, sys_chunk_d;  // reduction chunks
};

// the mixed rank phase's mode for a bucket of the atom count
struct RankChoice {
  int mode = -1;
  bool settled = false;         // measured on a list that stands for the bucket, or read from the file
  int64_t calls = 0, next = 0;  // until then: calls so far, the call that measures again
};

struct Ctx {
  int device = 0;
  int precision = AP_PREC_FP64;
  std::string err;
  bool has_eam = false, has_ace = false;
  TableDev phi{}, rho{}, F{};
  bool eam_analytic = false;            // EAM in closed form (ean) instead of the tables
  EamAnalyticDev ean{};
  AceDev ace{};
  MixDev mix{};
  Rank32Dev r32{};
  Rank32L r32_lv[2][2 * kMaxL + 1]{};   // [narrow, wide][L]
  size_t r32_lds[2][2 * kMaxL + 1] = {{0}};
  bool rank_narrow = false;             // some rank has a narrow variant
  // FP64 path: tables of the rank kernels; rank64 is false for models outside
  // their tiling, which run the one-workgroup-per-atom kernel
  bool rank64 = false;
  Rank64Dev r64{};
  Rank64L r64_lv[2 * kMaxL + 1]{};
  size_t r64_lds[2 * kMaxL + 1] = {0};
  std::vector<Buffer> owned;            // model tables
  SysCache sys;
  // scratch, grown on demand
  Buffer cell_big, pos4;               // cell_big: [m, atoms of the cells too big for LDS]
  Buffer cell_count, cell_start, cell_rank, cell_atoms, cell_pos, cell_rel, cell_of;
  Buffer scan_tmp;
  Buffer wfp, eF, vir_atom, e_tmp;
  Buffer ace_row, pair_g, ace_counter, ace_rows_list, ace_halo, nbr_ace;
  int32_t halo_stamp = 0;           // last stamp written into ace_halo (0: cleared)
  Buffer mix_A, mix_om, mix_phi;        // rank kernels of both paths: A, adjoint (2 sets), phi per ACE atom
  Buffer mix_bn;                        // mixed path: largest |A_(n,l)|^2 per ACE atom (X scale)
  Buffer partials, flags;               // flags: [0] nbr overflow max count, [1] nonfinite
  Buffer ind_atom;
  Buffer nvt_ke, nvt_sums, nvt_fac;      // Nose-Hoover layer: per-atom m v^2, per-system sums, scale
  Buffer sw_csp, sw_mu0, sw_mu, sw_flag, sw_src, sw_nsrc;   // dynamic switching scratch
  Buffer e_eam_raw, e_ace_raw;          // unweighted per-atom energies of the last force calls
  int64_t cells_n_atoms = -1;           // atoms of the last neighbour build (its cell list)
  int32_t* host_flag = nullptr;        // pinned: read-backs of the flags
  void* static_scratch = nullptr;      // this device's address of the static scratch array
  // launch mode of the mixed rank phase: forced (AP_RANK_MODE, >= 0) or tuned
  // per bucket of the atom count (timed on first use, optionally cached in
  // the JSON file named by AP_AUTOTUNE_CACHE)
  int rank_mode_forced = -1;
  std::map<int, RankChoice> rank_choice;
  std::string tune_key;                 // device and model shape, prefix of the cache keys
  std::string tune_cache;               // cache file path ("" = none)
  int last_rank_mode = -1;
  size_t ace_lds = 0;
  // set by ap_step's force evaluation, whose EAM and ACE calls see the same
  // positions: the ACE call reuses the positions the EAM call packed, and with
  // a virial the EAM call leaves its per-atom virial unreduced and the ACE call
  // adds to it and reduces both at once
  bool fused_eval = false;
  // algorithmic work counts (ap_info)
  double flops_atom = 0, flops_contract = 0, flops_bond = 0, nnz = 0, x_rows = 0;
  double mix_tiles = 0;        // stored 16x32 coefficient tiles (mixed path)
  double mix_mfma_flops = 0;   // executed MFMA FLOPs per ACE atom (3 split products)
  // per-phase event timing (ap_profile)
  bool prof = false;
  struct Ev { int phase; hipEvent_t a, b; };
  std::vector<Ev> evs;
  double prof_ms[AP_N_PHASES] = {0};
  int64_t prof_calls[AP_N_PHASES] = {0};
};

// Records a HIP event pair around a phase when profiling is on.
struct PhaseTimer {
  Ctx* c;
  int ph;
  hipStream_t s;
  hipEvent_t a = nullptr;
  PhaseTimer(Ctx* c_, int ph_, hipStream_t s_) : c(c_), ph(ph_), s(s_) {
    if (c->prof && hipEventCreate(&a) == hipSuccess) hipEventRecord(a, s);
  }
  ~PhaseTimer() {
    if (!a) return;
    hipEvent_t b;
    if (hipEventCreate(&b) == hipSuccess) {
      hipEventRecord(b, s);
      c->evs.push_back({ph, a, b});
    }
  }
};

// error helpers (ap_api.hip)
ap_status fail(Ctx* ctx, ap_status s, const std::string& msg);
ap_status fail_hip(Ctx* ctx, hipError_t e, const char* what, const char* file, int line);
ap_status ensure(Ctx* ctx, Buffer& b, size_t bytes);

// launchers ---------------------------------------------------------------
// neighbours (k_nbr.hip)
hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);
hipError_t launch_fill_f64(double* p, double v, int64_t n, hipStream_t s);
hipError_t launch_fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t s);
hipError_t launch_clear_nbr(int32_t n_cells, int32_t* cell_count, int32_t* big_atoms, int32_t* flag,
                            hipStream_t s);
hipError_t launch_bin(const SysView& sv, const double* pos, int32_t* cell_of, int32_t* cell_rank,
                      int32_t* cell_count, hipStream_t s);
hipError_t launch_scan_exclusive(const int32_t* in, int32_t* out, int32_t n, int32_t* tmp,
                                 hipStream_t s);
hipError_t launch_scatter(const SysView& sv, const double* pos, const int32_t* cell_of,
                          const int32_t* cell_rank, const int32_t* cell_start, int32_t* cell_atoms,
                          double4* cell_pos, float4* cell_rel, hipStream_t s);
hipError_t launch_fill_nbr_cells(const SysView& sv, int32_t n_cells, const double* pos,
                                 const int32_t* cell_of, const int32_t* cell_start,
                                 const int32_t* cell_count, const double4* cell_pos,
                                 const float4* cell_rel, int32_t* nbr, int32_t* count, int32_t cap,
                                 int32_t* overflow, int32_t* big_atoms, hipStream_t s);
hipError_t launch_rev(int32_t n_atoms, const int32_t* nbr, const int32_t* count, int32_t* rev,
                      hipStream_t s);
// switching and compaction (k_misc.hip)
hipError_t launch_blend(int32_t n, const double* pos, const ap_lambda_rule& rule, double* lambda,
                        int32_t* flag, hipStream_t s);
hipError_t launch_compact(int32_t n, const int32_t* flag, int32_t* out_list, int32_t* out_n,
                          int32_t* tmp, hipStream_t s);
hipError_t launch_seq(int32_t n, int32_t* out, hipStream_t s);
// reductions
hipError_t launch_reduce(const SysView& sv, int32_t n_chunks, bool one_chunk_each, const int64_t* chunk_lo,
                         const int64_t* chunk_hi, const int32_t* sys_chunk, const double* vals,
                         int32_t m, int64_t stride, double* partials, double* out, bool accumulate,
                         hipStream_t s, double* copy0 = nullptr, double* copy1 = nullptr);
// indenter / integration / checks
hipError_t launch_indenter(int32_t n, const double* pos, const uint8_t* fixed, const double* c,
                           double R, double K, const double* dir, double* force, double* e_atom2,
                           hipStream_t s);
hipError_t launch_kick_drift(int32_t n, const SysView& sv, double* pos, double* vel,
                             const double* force, const double* mass, const uint8_t* fixed,
                             const uint8_t* nvt, const double* nvt_fac, double dt, bool drift,
                             hipStream_t s);
hipError_t launch_nvt_ke(int32_t n, const double* vel, const double* mass, const uint8_t* nvt,
                         const uint8_t* fixed, double* out, hipStream_t s);
hipError_t launch_nvt_half(int32_t n_sys, double* sums, double* xi, double* fac, double T0,
                           double tau, double dt, hipStream_t s);
hipError_t launch_nvt_scale(int32_t n, const SysView& sv, double* vel, const uint8_t* nvt,
                            const uint8_t* fixed, const double* fac, hipStream_t s);
hipError_t launch_check_finite(int32_t n, const double* force, int32_t* flag, hipStream_t s);
hipError_t launch_lambda_grad(int32_t n, const double* pos, const ap_lambda_rule& rule,
                              const double* lambda, const double* e_ace, const double* e_eam,
                              double* force, double* vir_atom, hipStream_t s);
// dynamic switching (k_switch.hip)
hipError_t launch_switching(const SysView& sv, const double* pos, const int32_t* nbr,
                            const int32_t* count, const int32_t* cell_of,
                            const int32_t* cell_start, const int32_t* cell_count,
                            const int32_t* cell_atoms, const double4* cell_pos,
                            const ap_switching& sw, double csp_full, double* csp, double* mu0,
                            unsigned long long* mu_bits, int32_t* flag, int32_t* src, int32_t* n_src,
                            int32_t* scan_tmp, double* lambda, int32_t* ace_list, int32_t* n_ace,
                            hipStream_t s);
// EAM (k_eam.hip)
// p4 = position and, in w, the EAM weight 1 - lambda (1 when lambda is NULL)
hipError_t launch_pack_pos(int32_t n, const double* pos, const double* lambda, double4* p4,
                           hipStream_t s);
hipError_t launch_eam(const Ctx& c, const SysView& sv, const double4* pos4, const int32_t* nbr,
                      const int32_t* count, int32_t n_atoms, double* wfp, double* eF, double* e_atom,
                      double* force, double* vir_atom, bool accumulate, double* e_raw, hipStream_t s);
// ACE (k_ace.hip)
size_t ace_lds_bytes(const AceDev& a, int precision);
hipError_t launch_ace_reset(int32_t* counter, hipStream_t s);
hipError_t launch_ace(const Ctx& c, const SysView& sv, const double* pos, const double4* pos4,
                      const int32_t* nbr,
                      const int32_t* count, int32_t cap, int32_t n_atoms, const double* lambda,
                      const int32_t* ace_list, const int32_t* n_ace, int32_t* ace_row,
                      int32_t* counter, void* pair_g, double* e_atom, double* vir_atom,
                      double* e_raw, int32_t* nbr_ace, int32_t* halo, int32_t stamp,
                      bool vir_acc, hipStream_t s);
// arguments the bond kernels of both precisions share
struct BondArgs {
  const double* pos;
  const double4* pos4;
  const int32_t* nbr;
  const int32_t* count;
  int32_t cap, n_atoms;
  const double* lambda;
  const int32_t* ace_list;
  const int32_t* n_ace;
  double* e_atom;
  double* vir_atom;
  double* e_raw;
  int32_t* nbr_ace;
  int32_t* halo;
  int32_t stamp;
  bool vir_acc;
};
// the model as the bond kernels of one precision read it
template <typename T>
struct BondDev {
  int32_t n_max, l_max, K, nA, apad;
  double rc;
  const T* W;              // [n_max][l_max+1][K]
  const double* ynorm;
};
// phase 0: bond basis -> A (and the listed atoms' rows, atom-major, ->
// nbr_ace; the listed atoms and their neighbours stamped in halo); 1:
// coupling/contraction/adjoint -> om, phi; 2: embedding, bond gradients, virial
hipError_t launch_ace_mixed(const Ctx& c, const SysView& sv, const BondArgs& b, float* pair_g, float* A_buf, float* om_buf, float* phi_buf,
                            float* bn_buf, hipStream_t s, int phase, int rank_mode);
// FP64 path: phases 0 and 2, and phase 1, over the items item0 .. item0 + n_buf - 1
// (A, om, phi hold n_buf items)
hipError_t launch_ace_bonds64(const Ctx& c, const SysView& sv, const BondArgs& b, int phase, int item0,
                              int n_buf, double* pair_g, double* A_buf, double* om_buf,
                              double* phi_buf, hipStream_t s);
hipError_t launch_ace_rank64(const Ctx& c, const int32_t* n_ace, int n_atoms, int item0, int n_buf,
                             double* A_buf, double* om_buf, double* phi_buf, hipStream_t s);
// mixed rank kernel of coupled rank L (k_ace_rank32.hip); small: the narrow
// variant
template <int L>
const void* rank32_kernel(bool small);
// FP64 rank kernel of coupled rank L (k_ace_rank64.hip); small: the variant
// for two workgroups per CU (L <= kRank64LSmall)
template <int L>
const void* rank64_kernel(bool small);
hipError_t launch_ace_gather(const Ctx& c, int32_t n_atoms, const int32_t* nbr, const int32_t* count,
                             const int32_t* rev, const int32_t* nbr_ace, int32_t cap,
                             const int32_t* ace_row, const int32_t* halo, int32_t stamp,
                             const void* pair_g, double* force, bool accumulate, hipStream_t s);
hipError_t launch_ace_prep(int32_t n_atoms, const double* pos, const int32_t* ace_list,
                           const int32_t* n_ace, int32_t* ace_row, double* e_atom, double* vir,
                           double4* p4, hipStream_t s);

}  // namespace ap
