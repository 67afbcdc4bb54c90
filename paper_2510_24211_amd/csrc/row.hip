// Per-row part of the SCD step: top-k threshold, softmax normaliser, Modified
// Rejection Sampling (accept test + residual resample) and -- through a
// last-arriver ticket per sequence -- first rejection, emission and window
// slide.  (Alg. 1; Sec. 4.3 "Implementation Details": every window position is
// verified, none is skipped after a rejection, and only the offset of the first
// rejection is kept; appendix "Algorithms", Alg. SCD(pi_MC); top-k / temperature
// from the appendix "Experimental Details".)
//
//   thr  = K-th largest z (exact),  kept = { v : z_v >= thr }
//   lse  = m + log sum_kept exp(z_v - m),  p_v = [z_v >= thr] exp(z_v - lse)
//   accept iff fl(u * q(x)) <= p(x);  else y = argmin_{r_v > 0} -ln(U_v) / r_v
//
// gfx950 mapping.  A row of up to 65536 logits is far more than one CU should
// chew through alone, and with few sequences there are few rows, so the work is cut in two:
//   list_kernel   a wavefront per piece of 1024 or 2048 ids.  It emits the piece's largest logits as
//                 (id, logit) pairs, twice to three times its share of the row's top K, and a cut below
//                 which the others lie.  slice_kernel does the same for pieces of 8192 ids and an exact
//                 rank, where K is too large for lists that short (list_width).
//   row_kernel    one workgroup per row.  Loads the <= 6144 candidates into
//                 registers (6 per thread), selects the K-th largest key among
//                 them, and accepts the answer only if it is >= every list's
//                 cut (then no unseen logit can be >= it): exact, verified.
//                 Sum of exponentials, accept test, residual race and the
//                 commit follow from the same registers.
// Rows of <= 16384 logits need no candidates (the whole row fits the row
// kernel's registers); on longer ones the lists come from the LM head's
// epilogue, one per column tile, when that kernel emits them.  If the verification fails (massive ties, adversarial
// layouts) or no list is long enough, the row kernel falls back to a complete in-place
// path: one coalesced read of the row, 16-bit key prefixes parked in LDS,
// histogram select, candidate list or in-place scans; the scans alone where nothing filters.  Under a nucleus
// filter without top-k such rows stay in registers too (nucleus_path).
// Rows of more than 65536 logits (the LONG instance; top-k and the maximal coupling only) take the
// lists and the candidate path like the others.  32 rows of 131072 ids under top-k 2000: 9 us +
// 15 us, where one kernel per stage (radix select over the row, MRS, commit) took 124 + 64 + 5 us.
// Their complete path (long_path) makes whole passes over the row in memory.
// Logits supplied by the caller (a.src) are copied into the ring by whichever kernel reads them first; a
// copy kernel of its own took 66 us for 32 rows of 65536 ids (32 workgroups, 4-byte accesses), more than
// twice the rest of the iteration (9 + 19 us), and one of two launches of 6.8 us each for short rows.
// The K-th largest key is always found by integer counting (LDS histograms
// whose bins adapt to the key range, so lanes rarely collide); all
// floating-point sums use a fixed assignment of ids to threads and a fixed
// reduction tree, so results are run-to-run identical.
//
// This file is compiled three times: 1024 threads per row; 512 (row_batched.hip defines SCD_ROW_BATCHED) for rows of at
// most 8192 ids; 256 (row_short.hip defines SCD_ROW_SHORT) for rows of at most 1024.  What a row does once (range, sums,
// accept test, winners) every wavefront of it does, at 16 cycles an instruction when four share a SIMD: short rows spend
// most of their time on that, so they take few wavefronts.  Long rows want all the lanes.  Four steps on supplied logits
// (us, 1024 / 512 / 256 threads): 8 x 1024 ids 38.2 / 34.0 / 31.8; 32 x 2048 42.4 / 34.4 / 40.7, under top-k 500
// 45.2 / 35.3 / 39.7, with all options 68.9 / 53.4 / 61.9; 32 x 4096 40.8 / 42.7, under top-k 40.0 / 39.2, with all
// options 65.5 / 63.0; 32 x 8192 behind the LM head 107.4 / 111.4.
// The lines were drawn with 8 and 32 rows; with more rows than CUs the same way round (four steps, 512 rows, 1024 threads where
// options are on and else 512, against now): 1024 ids 53.3 / 48.1, with all options 135.1 / 71.5; 2048 ids 55.2 / 50.9,
// 136.1 / 73.9; 4096 ids (512 threads before, where no option is on) 68.7 / 64.0, 138.8 / 89.0.
//   More rows than CUs: a workgroup of 512 threads takes up to 118 registers per lane and 51 KB of LDS, so two of them
// share a CU and the barrier-separated phases of one row overlap with another's instead of the rows queueing in rounds.
#include "scd_device.h"
#include "scd_kernels.h"
#include "window_division.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

#ifdef SCD_ROW_BATCHED
#define SCD_ROW_THREADS 512
#define SCD_ROW_DIRECT_MAX 8192
#define row_kernel row_kernel_batched        // distinct names in traces
#define slice_kernel slice_kernel_batched
#define LAUNCH_ROW launch_row_batched
#define SCD_ROW_WAVES(EXTRA) ((EXTRA) ? 2 : 4)   // wavefronts per SIMD: two workgroups per CU
#elif defined(SCD_ROW_SHORT)
#define SCD_ROW_THREADS 256
#define SCD_ROW_DIRECT_MAX 4096              // (only the quarter of that is used)
#define row_kernel row_kernel_short
#define slice_kernel slice_kernel_short
#define LAUNCH_ROW launch_row_short
#define SCD_ROW_WAVES(EXTRA) ((EXTRA) ? 2 : 4)
#else
#define LAUNCH_ROW launch_row
#define SCD_ROW_WAVES(EXTRA) 4
#endif
#if defined(SCD_ROW_BATCHED) || defined(SCD_ROW_SHORT)
#define SCD_ROW_DIRECT_ONLY                  // whole rows in registers
#endif

namespace scd {
namespace {

#ifndef SCD_ROW_THREADS
#define SCD_ROW_THREADS 1024
#endif
// Few, fat threads: the per-wavefront bookkeeping (scans, reductions, the accept draw)
// costs issue slots per wavefront, the per-logit work does not care how it is cut.
constexpr int THREADS = SCD_ROW_THREADS;
constexpr int NW = THREADS / kWave;
constexpr int NBINS = 4096;
constexpr int kHistWords = NBINS + kWave;     // and a word per lane for what is not to be counted
constexpr int kListCap = kRowListCap;         // candidate ids per row (LDS list / slice or tile output)
constexpr int PER_LIST = kListCap / THREADS; // candidates per thread
#ifndef SCD_ROW_DIRECT_MAX
#define SCD_ROW_DIRECT_MAX kRowDirectMaxN
#endif
constexpr int kDirectMaxN = SCD_ROW_DIRECT_MAX;   // whole row in registers up to this many ids
constexpr int PER_DIRECT = kDirectMaxN / THREADS;   // (rows of half that size take half of them)
constexpr int kSliceMax = 8192;              // logits per slice workgroup
constexpr int PER_SLICE = kSliceMax / THREADS;
static_assert(THREADS >= 256 && kListCap % THREADS == 0 && PER_DIRECT % 8 == 0 && PER_SLICE % 4 == 0,
              "row kernels: unsupported workgroup size");
constexpr int kKeptCap = 4096;               // kept ids that long_path parks in LDS

struct Small {
  float fred[NW];
  uint32_t ured[NW];
  uint32_t umin[NW];      // complements
  uint32_t umax[NW];
  int ired[NW];
  int wtot[NW];
  uint4 sel;              // find_bin's bin, the population above it and its own
  uint32_t sel_bin;
  uint32_t cursor;        // append cursor of select_regs ...
  uint32_t members[64];   // ... and what it appends
  float u_accept;         // the accept test's uniform
  int ired2[NW];          // second slot of block_offsets
  unsigned long long win[2];   // winners of the two races: bits of the score, then the id
  int last;
  unsigned long long mtot[NW];   // nucleus: per-wavefront masses
  unsigned long long sel_mass;
  float dred[3][NW];             // statistics: per-wavefront sums
  int hamm[6];                   // (differing, compared) drafts 1, 2, 3 iterations apart
  int xnew[256];                 // the sequence's new drafts by ring slot
};

// hist[0..NBINS): find the bin holding the `need`-th largest element counting
// from the top bin; lowers `need` by the population of the bins above it.  members: its population.
// The trailing barrier keeps a later writer of sel / wtot away from slow
// readers; a caller whose next such write comes after another barrier anyway may drop it.
// T: threads of the workgroup (the row kernel's, or the slice kernel's smaller one).
template <int T = THREADS>
__device__ __forceinline__ uint32_t find_bin(const uint32_t* hist, uint32_t& need, uint32_t& members, Small& sm,
                                             bool trailing = true) {
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
  constexpr int PER = NBINS / T;         // consecutive bins per thread, top bins in thread 0
  static_assert(PER % 4 == 0, "find_bin: 16-byte reads");
  uint32_t c[PER], local = 0;
#pragma unroll
  for (int j = 0; j < PER; j += 4) {
    const uint4 t = *reinterpret_cast<const uint4*>(&hist[NBINS - 4 - (tid * PER + j)]);
    c[j] = t.w; c[j + 1] = t.z; c[j + 2] = t.y; c[j + 3] = t.x;
    local += (t.w + t.z) + (t.y + t.x);
  }
  const uint32_t incl_wave = static_cast<uint32_t>(wave_inclusive_sum_i32(static_cast<int>(local)));
  if (lane == 63) sm.wtot[wave] = static_cast<int>(incl_wave);
  __syncthreads();
  int total;
  const uint32_t incl = incl_wave + static_cast<uint32_t>(fold_before<T / kWave>(sm.wtot, wave, total));
  const uint32_t excl = incl - local;
  if (excl < need && need <= incl) {     // exactly one thread
    uint32_t above = excl, skipped = 0, mine = c[0];
#pragma unroll
    for (int j = 0; j + 1 < PER; ++j) {
      const bool further = skipped == static_cast<uint32_t>(j) && above + c[j] < need;
      above += further ? c[j] : 0u;
      mine = further ? c[j + 1] : mine;
      skipped += further ? 1u : 0u;
    }
    sm.sel = make_uint4(static_cast<uint32_t>(NBINS - 1 - tid * PER) - skipped, above, mine, 0u);
  }
  __syncthreads();
  const uint4 sel = sm.sel;
  need -= sel.y;
  members = sel.z;
  if (trailing) __syncthreads();
  return sel.x;
}
template <int T = THREADS>
__device__ __forceinline__ uint32_t find_bin(const uint32_t* hist, uint32_t& need, Small& sm,
                                             bool trailing = true) {
  uint32_t members;
  return find_bin<T>(hist, need, members, sm, trailing);
}

template <int T = THREADS>
__device__ __forceinline__ void zero_hist(uint32_t* hist) {
#pragma unroll
  for (int j = 0; j < NBINS / T; j += 4)
    *reinterpret_cast<uint4*>(&hist[threadIdx.x * 4 + j * T]) = make_uint4(0u, 0u, 0u, 0u);
}

__device__ __forceinline__ float prob(float z, float thr, float lse) {
  const float e = exp_of(z - lse);
  return z >= thr ? e : 0.f;
}

// Exclusive offset of this thread's `cnt` in a fixed thread order, and the total.
// `slot` picks one of two exchange arrays; without the trailing barrier the caller must
// have another barrier between this call and the next one on the same slot.
template <int T = THREADS>
__device__ __forceinline__ int block_offsets(int cnt, int& total, Small& sm, int slot = 0,
                                             bool trailing = true) {
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int incl = wave_inclusive_sum_i32(cnt);
  int* const ex = slot ? sm.ired2 : sm.ired;
  if (lane == 63) ex[wave] = incl;
  __syncthreads();
  const int base = fold_before<T / kWave>(ex, wave, total);
  if (trailing) __syncthreads();
  return base + incl - cnt;
}

// max / min of keys over the workgroup
template <int T = THREADS>
__device__ __forceinline__ void block_minmax(uint32_t& kmin, uint32_t& kmax, Small& sm,
                                             bool trailing = true) {
  const int lane = threadIdx.x & 63, wave = wave_index();
  kmax = wave_max_u32(kmax);
  kmin = ~wave_max_u32(~kmin);
  if (lane == 0) {
    sm.umax[wave] = kmax;
    sm.umin[wave] = ~kmin;
  }
  __syncthreads();
  kmax = fold_max<T / kWave>(sm.umax);
  kmin = ~fold_max<T / kWave>(sm.umin);
  if (trailing) __syncthreads();
}

constexpr float kRangeFloor = -1.0e30f;
// This thread's share of the row's range: keys of its largest logit (all ones if one is NaN) and of the
// smallest above kRangeFloor, of PER logits valid where ok[e].  One instruction per logit where all of the
// wavefront's are valid and above the floor; the rest (ragged rows, masked ids, NaN) is looked at one by one.
template <int PER>
__device__ __forceinline__ void thread_range(const float (&zv)[PER], const bool (&ok)[PER], uint32_t& kmin,
                                             uint32_t& kmax, bool& nan) {
  float hi = zv[0], lo = zv[0], sum = 0.f;
  bool plain = true, some = false;
#pragma unroll
  for (int e = 0; e < PER; ++e) some |= ok[e];
  kmax = 0u;
  kmin = 0xFFFFFFFFu;
  nan = false;
  if (__builtin_amdgcn_ballot_w64(some) == 0ull) return;      // a wavefront past the end of a short row
#pragma unroll
  for (int e = 0; e + 1 < PER; e += 2) {
    hi = max3(hi, zv[e], zv[e + 1]);
    lo = min3(lo, zv[e], zv[e + 1]);
  }
  if (PER & 1) {
    hi = max3(hi, zv[PER - 1], zv[PER - 1]);
    lo = min3(lo, zv[PER - 1], zv[PER - 1]);
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    sum += zv[e];
    plain &= ok[e];
  }
  if (__builtin_amdgcn_ballot_w64(!(plain && lo > kRangeFloor && sum == sum)) != 0ull) {
    hi = -INFINITY;
    lo = INFINITY;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      hi = ok[e] ? fmaxf(hi, zv[e]) : hi;
      lo = ok[e] && zv[e] > kRangeFloor ? fminf(lo, zv[e]) : lo;
      nan |= ok[e] && zv[e] != zv[e];
    }
    kmax = nan ? 0xFFFFFFFFu : zkey(hi);
    kmin = lo < INFINITY ? zkey(lo) : 0xFFFFFFFFu;
  } else {
    kmax = zkey(hi);
    kmin = zkey(lo);
  }
}

// To an unsigned integer: what is negative or NaN becomes 0, what is too large the largest.
__device__ __forceinline__ uint32_t saturating_u32(float f) {
  uint32_t r;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(f));
  return r;
}

// `need`-th largest key among the register-resident logits zv[e] (valid where ok[e]).  zlo is the
// smallest of the valid logits above -1e30, zhi the largest.
//   Level 1 bins the logits LINEARLY in value between those two (any monotone map
//   of the value preserves the order statistic; a linear one spreads a bell-shaped
//   row over all bins, where the float bit pattern would pile it into a few
//   exponent bins and serialise the LDS atomics).
//   Level 2 ranks the handful of members of the selected bin against each other, in every wavefront for
//   itself (lane to lane: an exchange through LDS costs a barrier and a round trip per member).
//   Should that bin hold more than kRankMax members (massive ties, or a few far logits that widen the
//   range and with it every bin), radix levels over the key bits finish the job: three histograms, 4 us
//   whatever their number.
constexpr uint32_t kRankMax = kWave;         // one per lane
static_assert(sizeof(Small::members) == kRankMax * 4, "a member per lane");
template <int PER, int T = THREADS>
__device__ __forceinline__ uint32_t select_regs(const float (&zv)[PER], const bool (&ok)[PER], float zlo,
                                                float zhi, uint32_t need, uint32_t* hist, Small& sm) {
  // hist (kHistWords) was zeroed by the caller before the barrier of block_minmax.  When a wavefront returns, no other
  // reads hist any more.
  const float scale = (zhi > zlo) ? fminf(__fdiv_rn(static_cast<float>(NBINS - 1), zhi - zlo), 3.0e38f) : 0.f;
  const int lane = threadIdx.x & 63;
  uint32_t bin[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    // Below the floor, or where the range is empty or infinite (NaN): bin 0, which the conversion gives for
    // what is negative or no number.  At most (zhi - zlo) * scale < NBINS (the scale is kept finite for ranges
    // of a few denormal numbers).  No logit: a word of the lane's own behind the bins, so that the counting
    // needs no branches.
    const uint32_t b = saturating_u32((zv[e] - zlo) * scale);
    bin[e] = ok[e] ? b : static_cast<uint32_t>(NBINS + lane);
  }
  if (threadIdx.x == 0) sm.cursor = 0u;          // append cursor, published by the next barrier
#pragma unroll
  for (int e = 0; e < PER; ++e) atomicAdd(&hist[bin[e]], 1u);
  __syncthreads();
  // no trailing barrier: sm.sel is next written after the barrier that follows the append
  uint32_t members;
  const uint32_t b1 = find_bin<T>(hist, need, members, sm, false);
  if (members <= kRankMax) {
    bool any = false;
#pragma unroll
    for (int e = 0; e < PER; ++e) any |= bin[e] == b1;
    if (__builtin_amdgcn_ballot_w64(any) != 0ull) {        // most wavefronts have none
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if (bin[e] == b1) sm.members[atomicAdd(&sm.cursor, 1u)] = zkey(zv[e]);
    }
    __syncthreads();
    // Every wavefront holds one member per lane and ranks them against each other: the smallest that has fewer
    // than `need` above it is the one.
    const int m = __builtin_amdgcn_readfirstlane(static_cast<int>(members));
    const uint32_t mine = lane < m ? sm.members[lane] : 0u;
    uint32_t above = 0;
    for (int i = 0; i < m; ++i)
      above += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mine), i)) > mine ? 1u : 0u;
    return ~wave_max_u32(lane < m && above < need ? ~mine : 0u);
  }
  __syncthreads();          // every thread has read its bins before the histogram is reused
  // radix levels over the key bits of the members, range [lo, lo + width)
  uint32_t lo = 0;
  uint64_t width = 1ull << 32;
  for (;;) {
    int s2 = 0;
    while (((width - 1) >> s2) >= static_cast<uint64_t>(NBINS)) ++s2;
    zero_hist<T>(hist);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const uint32_t k = zkey(zv[e]);
      if (bin[e] == b1 && k >= lo && static_cast<uint64_t>(k - lo) < width)
        atomicAdd(&hist[(k - lo) >> s2], 1u);
    }
    __syncthreads();
    const uint32_t dgt = find_bin<T>(hist, need, sm);
    lo += dgt << s2;
    width = 1ull << s2;
    if (s2 == 0) return lo;
  }
}

// ---------------------------------------------------------------------------------
// Nucleus (top-p) filter (appendix "Experimental Details", video setting p = 0.8), applied
// to the set K1 that top-k left:  keep v  iff  the mass of the ids with a LARGER logit is
// below top_p times the mass of K1 -- the shortest most-probable prefix reaching top_p, ids
// tied with its last member included.  Like top-k the result is a threshold on the logit.
//   Masses are 64-bit fixed point, w_v = trunc(expf(z_v - m) * 2^40): integer sums do not
//   depend on the order of the LDS atomics, so the decision is run-to-run identical, and it
//   is taken exactly:  above(v) * 2^24 < P24 * S  with P24 = round(top_p * 2^24).
//   Search: one histogram of masses over bins LINEAR in the logit (spreads a bell-shaped row
//   over the bins), then radix levels over the key bits of the selected bin's members.
// `each(f)` must call f(key, z) for every element of K1.  After the first level
// `prepare(klo, khi)` is called once and then `near(f)` must call f for at least the elements of
// K1 whose key lies in [klo, khi] (a path that can find them without reading the whole row again
// does so; extra elements are filtered here).
// mh: NBINS_P 64-bit bins (the space of the count histogram).  Uniform over the workgroup.
constexpr int NBINS_P = NBINS / 2;
static_assert(NBINS_P % THREADS == 0 || THREADS % NBINS_P == 0, "nucleus: bins per thread");

// Both words of trunc(e^(z - m) 2^40), at most 2^40: multiplications by powers of two and the subtraction are exact,
// so this is the conversion to 64 bits in 6 instructions (the general one takes twice as many).  NaN: 0.
__device__ __forceinline__ unsigned long long mass_of(float z, float m) {
  // As exp_of.  Far below, the product's rounding error alone would take the exponential unit to infinity: from e^-150 on
  // there is no mass, nor has a NaN any.
  const float y = fmaxf(z - m, -150.f);
  const float t = __fmul_rn(y, 1.44269502f);
  const float rest = __fmaf_rn(y, 1.92596303e-8f, __fmaf_rn(y, 1.44269502f, -t));
  const float k = __builtin_rintf(t);
  const float e = __builtin_ldexpf(__builtin_amdgcn_exp2f((t - k) + rest), static_cast<int>(k)) * 256.f;
  const uint32_t hi = saturating_u32(e);
  const uint32_t lo = saturating_u32((e - static_cast<float>(hi)) * 4294967296.f);
  return static_cast<unsigned long long>(hi) << 32 | lo;
}

__device__ __forceinline__ unsigned long long wave_inclusive_sum_u64(unsigned long long v) {
  // three 24-bit limbs: 64 lanes x 2^24 stays inside an int
  const int l0 = wave_inclusive_sum_i32(static_cast<int>(v & 0xFFFFFFull));
  const int l1 = wave_inclusive_sum_i32(static_cast<int>((v >> 24) & 0xFFFFFFull));
  const int l2 = wave_inclusive_sum_i32(static_cast<int>(v >> 48));
  return static_cast<unsigned long long>(static_cast<uint32_t>(l0)) +
         (static_cast<unsigned long long>(static_cast<uint32_t>(l1)) << 24) +
         (static_cast<unsigned long long>(static_cast<uint32_t>(l2)) << 48);
}

// ceil(P24 * S / 2^24) for S < 2^58
__device__ __forceinline__ unsigned long long nucleus_target(unsigned long long S, uint32_t p24) {
  const unsigned long long hi = (S >> 32) * p24, lo = (S & 0xFFFFFFFFull) * p24;
  return (hi << 8) + ((lo + 0xFFFFFFull) >> 24);
}

// The bin b with  above + mass(bins > b) < target <= above + mass(bins >= b);  `above` grows
// by mass(bins > b).  FIRST: target is derived here from the total mass of the histogram.
template <bool FIRST>
__device__ __forceinline__ uint32_t find_bin_mass(const unsigned long long* mh, unsigned long long& target,
                                                  unsigned long long& above, uint32_t p24, Small& sm) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int PER = NBINS_P >= THREADS ? NBINS_P / THREADS : 1;
  unsigned long long c[PER], local = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int idx = tid * PER + j;                 // top bins first
    c[j] = idx < NBINS_P ? mh[NBINS_P - 1 - idx] : 0ull;
    local += c[j];
  }
  unsigned long long incl = wave_inclusive_sum_u64(local);
  if (lane == 63) sm.mtot[wave] = incl;
  __syncthreads();
  unsigned long long base = above, total = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    base += w < wave ? sm.mtot[w] : 0ull;
    total += sm.mtot[w];
  }
  if (FIRST) target = nucleus_target(total, p24);
  incl += base;
  const unsigned long long excl = incl - local;
  if (excl < target && target <= incl) {           // exactly one thread
    unsigned long long ab = excl;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (ab + c[j] >= target) {
        sm.sel_bin = static_cast<uint32_t>(NBINS_P - 1 - (tid * PER + j));
        sm.sel_mass = ab;
        break;
      }
      ab += c[j];
    }
  }
  __syncthreads();
  const uint32_t bin = sm.sel_bin;
  above = sm.sel_mass;
  __syncthreads();
  return bin;
}

template <class Each, class Prepare, class Near>
__device__ __forceinline__ uint32_t nucleus_key(Each&& each, Prepare&& prepare, Near&& near, float m, float zmin, uint32_t p24,
                                                unsigned long long* mh, Small& sm) {
  const int tid = threadIdx.x;
  // logits more than 110 below the maximum weigh nothing: they all go to bin 0
  const float zlo = fmaxf(zmin, m - 110.f);
  const float scale = (m > zlo) ? __fdiv_rn(static_cast<float>(NBINS_P - 1), m - zlo) : 0.f;
  auto lin_bin = [&](float z) {
    return static_cast<int>(__builtin_amdgcn_fmed3f((z - zlo) * scale, 0.f, static_cast<float>(NBINS_P - 1)));
  };
  auto zero = [&]() {
    for (int i = tid; i < NBINS_P; i += THREADS) mh[i] = 0ull;
  };
  __syncthreads();                                  // earlier users of the histogram space are done
  zero();
  __syncthreads();
  each([&](uint32_t key, float z) { atomicAdd(&mh[lin_bin(z)], mass_of(z, m)); });
  __syncthreads();
  unsigned long long target = 0, above = 0;
  const int b1 = static_cast<int>(find_bin_mass<true>(mh, target, above, p24, sm));
  // keys that can fall into bin b1: its interval of logits widened by a bin on either side
  // (the rounding of lin_bin's arithmetic moves a logit by far less than a bin)
  uint32_t near_lo = 0u, near_hi = 0xFFFFFFFFu;
  if (scale > 0.f) {
    const float inv = __fdiv_rn(m - zlo, static_cast<float>(NBINS_P - 1));
    if (b1 > 1) near_lo = zkey(zlo + static_cast<float>(b1 - 1) * inv);
    if (b1 < NBINS_P - 2) near_hi = zkey(zlo + static_cast<float>(b1 + 2) * inv);
  }
  prepare(near_lo, near_hi);
  // A bin near the boundary holds a few dozen ids: they are parked in LDS, and for each the masses of those above it
  // are added up, every wavefront taking its share of the summands (all of them in one thread per member are as many
  // round trips to LDS: 11000 -> 5000 cycles on rows of 64000 ids); the smallest
  // key whose sum stays below the target is the threshold.
  constexpr uint32_t kFew = 512;
  unsigned long long* const mm = mh;
  unsigned long long* const over = mh + kFew;
  uint32_t* const mk = reinterpret_cast<uint32_t*>(over + kFew);
  static_assert(NBINS_P * 8 >= kFew * 20, "members' masses, sums and keys in the histogram's space");
  __syncthreads();                                  // the cursor may still be read by prepare()'s users
  for (uint32_t i = tid; i < kFew; i += THREADS) over[i] = 0ull;
  if (tid == 0) {
    sm.cursor = 0u;
    sm.sel_bin = 0xFFFFFFFFu;
  }
  __syncthreads();
  near([&](uint32_t key, float z) {
    if (lin_bin(z) == b1) {
      const uint32_t slot = atomicAdd(&sm.cursor, 1u);
      if (slot < kFew) {
        mk[slot] = key;
        mm[slot] = mass_of(z, m);
      }
    }
  });
  __syncthreads();
  const uint32_t members = sm.cursor;
  if (members <= kFew) {
    for (uint32_t a = tid & (kWave - 1); a < (members + kWave - 1) / kWave * kWave; a += kWave) {
      const uint32_t key = a < members ? mk[a] : 0xFFFFFFFFu;
      unsigned long long sum = 0ull;
      for (uint32_t i = wave_index(); i < members; i += NW) sum += mk[i] > key ? mm[i] : 0ull;
      if (sum != 0ull) atomicAdd(&over[a], sum);
    }
    __syncthreads();
    for (uint32_t i = tid; i < members; i += THREADS)
      if (above + over[i] < target) atomicMin(&sm.sel_bin, mk[i]);
    __syncthreads();
    const uint32_t key = sm.sel_bin;
    __syncthreads();                                // the next user of the space or of sel_bin
    return key;
  }
  __syncthreads();                                  // everybody has read the cursor
  // many (ties): radix levels over the key bits of the members of bin b1
  uint32_t lo = 0;
  int s2 = 32;
  while (s2 > 0) {
    const int width_bits = s2;                      // candidates: keys in [lo, lo + 2^width_bits)
    s2 = width_bits > 11 ? width_bits - 11 : 0;
    zero();
    __syncthreads();
    near([&](uint32_t key, float z) {
      if (lin_bin(z) == b1 && key >= lo &&
          (width_bits == 32 || (key - lo) >> width_bits == 0u))
        atomicAdd(&mh[(key - lo) >> s2], mass_of(z, m));
    });
    __syncthreads();
    lo += find_bin_mass<false>(mh, target, above, p24, sm) << s2;
  }
  return lo;
}

// Lanes below this one whose bit is set, plus `more`.
__device__ __forceinline__ int lanes_before(unsigned long long mask, int more) {
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                          __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), static_cast<uint32_t>(more))));
}
// LDS operations of a wavefront are performed in order: what its lanes wrote before, its lanes read behind.
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Where a kernel instance finds its row.
struct RowRef {
  const float* zc;
  const float* zp;
  float* zw;      // supplied logits: the ring row that takes a copy of zc, else null
  float thr_p, lse_p;
  bool active;
  int age;        // earlier evaluations of the position (kept as it is read: a comparison would wait for it on the spot)
  __device__ __forceinline__ bool fresh() const { return age == 0; }
  int x, b, s, p0, live, it;
  int first_slot; // ring slot of the window's first position
  size_t widx, oidx, sidx;
  size_t pidx;    // where the previous evaluation of the slot left its per-slot results (ring mode)
};

// pos, iter, mode, L, N repeat a.pos, a.iter, mode, L, N: the kernels receive them as plain
// leading arguments, which the hardware preloads into SGPRs at wavefront launch, so that the first
// dependent load (pos[b]) does not wait for a fetch of the kernel-argument segment.
__device__ __forceinline__ RowRef locate_row(const RowArgs& a, int r, const int32_t* pos,
                                             const int32_t* iter, int mode, int L, int N) {
  RowRef R{};
  R.widx = r;
  R.oidx = r;
  R.it = a.iter_scalar;
  R.x = -1;
  R.active = true;
  const int n = a.n;
  if (mode == kRowSelectOnly) {
    R.zc = a.z_cur + static_cast<size_t>(r) * n;
    return R;
  }
  R.b = div_window(r, L, a.recip_L);
  R.s = r - R.b * L;
  R.p0 = pos[R.b];
  R.live = max(0, min(L, N - R.p0));
  R.widx = static_cast<size_t>(R.b) * L + R.s;
  if (R.s >= R.live) {
    R.active = false;
    return R;
  }
  if (mode == kRowRing) {
    R.it = iter[R.b];
    R.first_slot = R.p0 - div_window(R.p0, L, a.recip_L) * L;
    int slot = R.first_slot + R.s;
    if (slot >= L) slot -= L;
    const int par = R.it & 1;
    const size_t sidx = static_cast<size_t>(R.b) * L + slot;
    const size_t half = static_cast<size_t>(a.B) * L;
    R.oidx = par * half + sidx;
    R.pidx = (par ^ 1) * half + sidx;
    float* const ring = const_cast<float*>(a.z_cur) + static_cast<size_t>(par) * a.parity_stride + sidx * n;
    R.zc = a.src ? a.src + R.widx * n : ring;
    R.zw = a.src ? ring : nullptr;
    R.zp = a.z_cur + static_cast<size_t>(par ^ 1) * a.parity_stride + sidx * n;
    R.sidx = sidx;
  } else {
    R.oidx = R.widx;
    R.zc = a.z_cur + R.widx * n;
    R.zp = a.z_prev + R.widx * n;
  }
  return R;
}
// One word of a uniform address through the scalar cache, which nothing of this launch has written before (a row's words are
// read before its sequence's commit, at the earliest behind all of them, rewrites them).  As vector loads the row's words
// would come back behind its logits, and the draft's logits, whose addresses they give, be asked for a round trip later
// (those four steps: 93.1 us for 94.4, 103.5 for 104.6).
template <class T>
__device__ __forceinline__ T scalar_word(const T* p) {
  static_assert(sizeof(T) == 4, "a word");
  return *reinterpret_cast<const __attribute__((address_space(4))) T*>(reinterpret_cast<uintptr_t>(p));
}
// The rest, for the caller to read once the row's logits are on their way: draft, whether its position is new,
// what the slot's previous evaluation left (memory that exists and holds nothing useful for a new one; read
// without waiting for the answer).  Before the loads of the logits this is a round trip of its own.
__device__ __forceinline__ void read_row_scalars(const RowArgs& a, RowRef& R) {
  if (a.mode == kRowSelectOnly) return;
  if (a.mode == kRowRing) {
    R.x = scalar_word(a.x + R.sidx);
    R.age = scalar_word(a.age + R.sidx);
    R.thr_p = scalar_word(a.thr + R.pidx);
    R.lse_p = scalar_word(a.lse + R.pidx);
  } else {
    R.age = a.fresh && a.fresh[R.widx] != 0 ? 0 : 1;
    R.x = scalar_word(a.x + R.widx);
    R.thr_p = scalar_word(a.thr_prev + R.widx);
    R.lse_p = scalar_word(a.lse_prev + R.widx);
  }
}

// Groups of four neighbouring logits of a row of `end` ids, those at group(0), group(1), ..., all requested before one is
// waited for.  A group that is not whole reads the row's last four and is shifted into place afterwards (load4 needs no
// alignment); what lies past the end holds any logit of the row.  No lane leaves the line meanwhile: with element-wise
// loads in a branch for the ragged group, the compiler waited for every group before it requested the next (their
// registers may be in flight from either side of the branch).  Without, four steps of 32 x 16384 ids over 1280 take 94.4 us
// for 96.5, of 32 x 8192 over 4096 104.6 for 107.1.
// TINY: rows of less than four ids.
template <int PER, bool TINY = false, class Group>
__device__ __forceinline__ void load_groups(const float* row, int end, Group&& group, float (&z)[PER]) {
#pragma unroll
  for (int u = 0; u < PER / 4; ++u) {
    if constexpr (TINY) {
#pragma unroll
      for (int e = 0; e < 4; ++e) z[u * 4 + e] = row[min(group(u) + e, end - 1)];
    } else {
      const float4 t = load4(row + min(group(u), end - 4));
      z[u * 4 + 0] = t.x; z[u * 4 + 1] = t.y; z[u * 4 + 2] = t.z; z[u * 4 + 3] = t.w;
    }
  }
}
// The shift, once the logits are wanted: rows of a multiple of four ids have no such group, others one in one lane, and the
// other wavefronts step over it.
template <int PER, class Group>
__device__ __forceinline__ void align_groups(int end, Group&& group, float (&z)[PER]) {
  if ((end & 3) == 0) return;                  // uniform
#pragma unroll
  for (int u = 0; u < PER / 4; ++u) {
    const int by = group(u) - (end - 4);       // 1 .. 3: that many of the four are the group's predecessors
    if (__builtin_amdgcn_ballot_w64(static_cast<uint32_t>(by - 1) < 3u) == 0ull) continue;
    const float t1 = z[u * 4 + 1], t2 = z[u * 4 + 2], t3 = z[u * 4 + 3];
    z[u * 4] = by == 1 ? t1 : by == 2 ? t2 : by == 3 ? t3 : z[u * 4];
    z[u * 4 + 1] = by == 1 ? t2 : by == 2 ? t3 : t1;
    z[u * 4 + 2] = by == 1 ? t3 : t2;
  }
}

#ifndef SCD_ROW_DIRECT_ONLY
// ---------------------------------------------------------------------------------
// slice kernel: lists from slices of 8192 ids by an exact rank (see list_kernel and list_width)
// ---------------------------------------------------------------------------------
// ST threads: 1024, or 512 when there are more slices than two per CU (four such workgroups
// fit a CU by LDS and wavefronts, so that all of them run at once: C4 192 -> 186 us per step)
template <int ST>
__global__ __launch_bounds__(ST) void slice_kernel(const int32_t* const pos_, const int32_t* const iter_,
                                                        const int mode_, const int L_, const int N_,
                                                        const int P, const int capE, const int rank,
                                                        const RowArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t hist[kHistWords];
  __shared__ Small sm;
  constexpr int PS = kSliceMax / ST;   // logits per thread
  const int tid = threadIdx.x;
  const int r = blockIdx.x / P, p = blockIdx.x % P;
  const RowRef R = locate_row(a, r, pos_, iter_, mode_, L_, N_);
  if (!R.active) return;
  const int n = a.n;
  const int slice_len = (((n + P - 1) / P) + 3) & ~3;
  const int lo_id = p * slice_len;
  const int hi_id = min(n, lo_id + slice_len);
  uint32_t* const cnt_out = a.cand_cnt + static_cast<size_t>(r) * P;
  uint32_t* const cut_out = a.cand_cut + static_cast<size_t>(r) * P;
  if (lo_id >= hi_id) {
    for (int i = tid; i < capE; i += ST)
      a.cand[static_cast<size_t>(r) * kListCap + static_cast<size_t>(p) * capE + i] = make_uint2(kNoId, 0u);
    if (tid == 0) {
      cnt_out[p] = 0;
      cut_out[p] = 0;
    }
    return;
  }
  float zv[PS];
  int vid[PS];
  bool ok[PS];
  auto group = [&](int u) { return lo_id + ((tid + u * ST) << 2); };
  load_groups<PS>(R.zc, hi_id, group, zv);     // (rows that have slices are long: hi_id > 4)
  align_groups<PS>(hi_id, group, zv);
#pragma unroll
  for (int u = 0; u < PS / 4; ++u) {
    const int v0 = group(u);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      vid[u * 4 + e] = v0 + e;
      ok[u * 4 + e] = v0 + e < hi_id;
    }
    if (R.zw) {
      if (v0 + 3 < hi_id) {
        store4(R.zw + v0, zv[u * 4], zv[u * 4 + 1], zv[u * 4 + 2], zv[u * 4 + 3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v0 + e < hi_id) R.zw[v0 + e] = zv[u * 4 + e];
      }
    }
  }
  uint32_t kmax, kmin;
  bool nan;
  thread_range<PS>(zv, ok, kmin, kmax, nan);
  if (nan && a.flags) atomicOr(a.flags, 1);                    // NaN of either sign
  zero_hist<ST>(hist);                        // published by the barrier inside block_minmax
  block_minmax<ST>(kmin, kmax, sm, false);
  const int nvalid = hi_id - lo_id;
  uint32_t cut = 0;                       // 0: the whole slice is emitted
  if (nvalid > rank)
    cut = select_regs<PS, ST>(zv, ok, key_to_float(kmin), key_to_float(kmax), static_cast<uint32_t>(rank), hist, sm);
  bool take[PS];
  int mine = 0;
#pragma unroll
  for (int e = 0; e < PS; ++e) {
    take[e] = ok[e] && zkey(zv[e]) >= cut;
    mine += take[e] ? 1 : 0;
  }
  int total;
  int off = block_offsets<ST>(mine, total, sm, 0, false);
  uint2* const dst = a.cand + (static_cast<size_t>(r) * kListCap + static_cast<size_t>(p) * capE);
  for (int i = total + tid; i < capE; i += ST) dst[i] = make_uint2(kNoId, 0u);
#pragma unroll
  for (int e = 0; e < PS; ++e) {
    if (take[e]) {
      if (off < capE) dst[off] = make_uint2(static_cast<uint32_t>(vid[e]), __float_as_uint(zv[e]));
      ++off;
    }
  }
  if (tid == 0) {
    cnt_out[p] = static_cast<uint32_t>(total);   // > capE signals overflow
    cut_out[p] = cut;
  }
}

// ---------------------------------------------------------------------------------
// list kernel: the same lists from pieces that a wavefront holds in registers
// ---------------------------------------------------------------------------------
// A wavefront takes 64 E ids of a row, one line of 64 out of every P, and emits the `cap` largest of them or somewhat
// fewer as (id, logit) pairs in a fixed order, with their number and a cut: every logit of the piece that is not emitted
// lies below it.
//   Lines are dealt over the pieces because likely ids tend to be neighbours: of neighbouring ids alone, a piece holds a
// whole such neighbourhood, more than a list takes, and the row is read whole.  Four steps on supplied logits of 32 x 65536
// ids, top-k 2000, in pieces of neighbours : of lines (us): independent logits 79.3 : 79.4, runs of 1024 ids that differ by
// half of a logit's own deviation 183 : 78, logits falling with log(id) 209 : 76, one half masked 282 : 96, sorted 352 : 86;
// of 32 x 131072, top-k 1000, 80.9 : 81.2, 285 : 82, 272 : 270, 855 : 114, 479 : 488.  Lines of 32 take falling logits there
// too (81) but cost independent ones more: 65536 ids 80.4, 81146 84.9 for 82.7 in lines of 64 (rows whose lines are not the
// memory's pay for those of 64 already, 288 x 24577 138.5 : 141.5).  Lines of 128 fail runs of 128 to 512 ids.
//   A line's place moves by two from stripe to stripe: at one place in all, a load's lines lie 8 KB apart at 65536 ids, on
// few channels (82.4).
// As in the LM head's epilogue the emitted set is found on a monotone image of the logits, linear between their mean and
// their largest: one LDS histogram per wavefront, the lowest bin whose upper set holds at most `cap`.  A list needs no exact
// length, only to hold what the row's K-th largest leaves to this piece, so that bins of a few logits will do; where they
// are too wide (a far logit, masks of -1e10) the bin below the cut is counted again on its own range (refine_list).
// Masked ids (kListFloor and below) are never emitted.  What is not finite, or ties by the hundred, reports more pairs than
// fit: the row kernel reads the row whole.
//   Bound by latency: a wavefront works for itself, 400 instructions and no barrier, where the slice kernel's
// workgroups select an exact rank in eight barrier-separated phases.  Four steps on supplied logits of 32 x 65536 ids take
// 79.1 us for 91.2, of 32 x 81146 83.2 for 100.3, four steps of 32 x 131072 behind the LM head 737.8 for 745.7, three stage
// calls on 60 x 30001 42.4 for 48.5.
constexpr int kListBins = 256;
constexpr int kListHist = kWave + kListBins;       // words: one per lane for what lies far below the bins
constexpr int kListWaves = 4;                      // per workgroup
constexpr int kListLine = 64, kListSkew = 2;
constexpr float kListFloor = kRangeFloor;
__device__ __forceinline__ float list_scale(float range) {
  return range > 0.f ? fminf(__builtin_amdgcn_rcpf(range) * (kListBins - 1.01f), 3.0e38f) : 0.f;
}
__device__ __forceinline__ void zero_list_bins(uint32_t* bins, int lane) {
  *reinterpret_cast<uint4*>(&bins[4 * lane]) = make_uint4(0u, 0u, 0u, 0u);
}
// The lowest bin whose upper set holds at most `room` of the counted logits (kListBins: not even the last one's), and
// how many that are.
__device__ __forceinline__ int list_cut(const uint32_t* bins, int lane, int room, int& taken) {
  static_assert(kListBins == 4 * kWave, "four bins per lane");
  const uint4 t = *reinterpret_cast<const uint4*>(&bins[kListBins - 4 - 4 * lane]);      // top bins in lane 0
  const int c[4] = {static_cast<int>(t.w), static_cast<int>(t.z), static_cast<int>(t.y), static_cast<int>(t.x)};
  const int local = (c[0] + c[1]) + (c[2] + c[3]);
  int sum = wave_inclusive_sum_i32(local) - local;
  int fits = 0;
  taken = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    sum += c[j];
    fits += __builtin_popcountll(__builtin_amdgcn_ballot_w64(sum <= room));
    taken = max(taken, sum <= room ? sum : 0);
  }
  taken = static_cast<int>(wave_max_u32(static_cast<uint32_t>(taken)));
  return kListBins - fits;
}
// bin[e] >= cut: the logit is emitted.  Where the list stays short, the logits of the bin below the cut (more than there are
// free slots) are counted on an image of their own range, and those of its upper bins are lifted above every cut; again
// on the next bin while the list is short and the members differ.
constexpr int kListLifted = 1 << 20;
template <int E>
__device__ __forceinline__ void refine_list(const float (&v)[E], int (&bin)[E], int cut, int cap, int enough, int total,
                                            uint32_t* bins, int lane) {
  uint64_t in = 0;                                       // a bit per logit (E <= 64)
#pragma unroll
  for (int e = 0; e < E; ++e)
    in |= (cut > 0 ? bin[e] == cut - 1 : bin[e] < 0 && bin[e] >= -kWave) ? 1ull << e : 0ull;
#pragma unroll 1
  for (int round = 0; round < 6 && total < enough; ++round) {
    float mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool is = (in >> e & 1u) != 0u;
      mx = is ? fmaxf(mx, v[e]) : mx;
      mn = is ? fminf(mn, v[e]) : mn;
    }
    const float hi = wave_max_f32(mx), lo = wave_min_f32(mn);
    if (!(hi > lo)) return;                              // they tie (or there are none)
    const float scale = list_scale(hi - lo);
    zero_list_bins(bins, lane);
    wave_lds_fence();
    int image[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      image[e] = static_cast<int>(__builtin_amdgcn_fmed3f((v[e] - lo) * scale, 0.f, kListBins - 1.f));
      if ((in >> e & 1u) != 0u) atomicAdd(&bins[image[e]], 1u);
    }
    wave_lds_fence();
    int taken;
    const int part = list_cut(bins, lane, cap - total, taken);
    total += taken;
    uint64_t next = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool is = (in >> e & 1u) != 0u;
      bin[e] = is && image[e] >= part ? kListLifted : bin[e];
      next |= is && image[e] == part - 1 ? 1ull << e : 0ull;
    }
    in = next;
  }
}

template <int E>
__global__ __launch_bounds__(kListWaves * kWave) void list_kernel(const int32_t* const pos_, const int32_t* const iter_,
                                                                  const float* const rows_, const int mode_, const int L_,
                                                                  const int N_, const int n_, const int P, const int cap,
                                                                  const RowArgs a) {
  // rows_: the rows' logits in the order of the launch, or null: in the ring, where pos and iter say
  __shared__ __attribute__((aligned(16))) uint32_t hist[kListWaves * kListHist];
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int r = blockIdx.x, p = static_cast<int>(blockIdx.y) * kListWaves + wave;
  if (p >= P) return;
  uint32_t* const bins = hist + wave * kListHist + kWave;
  // The piece's line of stripe j, P lines each, is its (p + 2 j mod P)-th; four stripes in a load, and only the last load's
  // may end before their P lines (list_width).
  constexpr int kLanes = kListLine / 4, kStripes = kWave / kLanes, kLast = E - 4;
  int ids[E / 4];                                        // the lane's four of each load begin here
  {
    int j = lane / kLanes, at = p + kListSkew * j;
    at = at >= P ? at - P : at;
#pragma unroll
    for (int u = 0; u < E / 4; ++u) {
      ids[u] = (j * P + at) * kListLine + ((lane & (kLanes - 1)) << 2);
      j += kStripes;
      at += kListSkew * kStripes;
      at = at >= P ? at - P : at;
    }
  }
  auto group = [&](int u) { return ids[u]; };
  const bool whole = __builtin_amdgcn_ballot_w64(group(E / 4 - 1) + 3 >= n_) == 0ull;
  float v[E];
  RowRef R;
  const float* row = rows_ + static_cast<size_t>(r) * n_;
  if (!rows_) {
    R = locate_row(a, r, pos_, iter_, mode_, L_, N_);
    if (!R.active) return;
    row = R.zc;
  }
  load_groups<E>(row, n_, group, v);
  zero_list_bins(bins, lane);
  if (rows_) {                                           // (while they are on their way)
    R = locate_row(a, r, pos_, iter_, mode_, L_, N_);
    if (!R.active) return;
  }
  int have = kWave * E;                                  // ids of the piece
  float least[4], addend[4];                             // of the last load
  {
    float last[4] = {v[kLast], v[kLast + 1], v[kLast + 2], v[kLast + 3]};
    align_groups<4>(n_, [&](int) { return group(E / 4 - 1); }, last);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[kLast + e] = least[e] = addend[e] = last[e];
  }
  if (!whole) {                                          // what lies past the end takes a value below every other's
    have = kWave * kLast;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool is = group(E / 4 - 1) + e < n_;
      have += __builtin_popcountll(__builtin_amdgcn_ballot_w64(is));
      v[kLast + e] = is ? v[kLast + e] : -INFINITY;
      least[e] = is ? least[e] : INFINITY;
      addend[e] = is ? addend[e] : 0.f;
    }
  }
  float given[E];                                        // (the copy's: the logits may change below)
#pragma unroll
  for (int e = 0; e < E; ++e) given[e] = v[e];
  float mx = -INFINITY, mn = INFINITY, sum = 0.f;
  int there = have;                                      // logits above the floor
#pragma unroll
  for (int e = 0; e < E; e += 2) {
    mx = max3(mx, v[e], v[e + 1]);
    mn = e < kLast ? min3(mn, v[e], v[e + 1]) : min3(mn, least[e & 3], least[(e & 3) + 1]);
    sum += e < kLast ? v[e] : addend[e & 3];
    sum += e < kLast ? v[e + 1] : addend[(e & 3) + 1];
  }
  bool nan = false;
  if (__builtin_amdgcn_ballot_w64(!(mn > kListFloor && sum == sum)) != 0ull) {
    // masked, or not finite: those do not count either
    int mine = 0;
    sum = 0.f;
    mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      nan |= v[e] != v[e];
      const bool counts = v[e] > kListFloor;
      v[e] = counts ? v[e] : -INFINITY;
      sum += counts ? v[e] : 0.f;
      mx = fmaxf(mx, v[e]);
      mine += counts ? 1 : 0;
    }
    there = wave_sum_i32(mine);
  }
  nan = __builtin_amdgcn_ballot_w64(nan) != 0ull;
  if (nan && a.flags && lane == 0) atomicOr(a.flags, 1);         // NaN of either sign
  mx = wave_max_f32(mx);
  const float mean = there > 0 ? wave_sum(sum) * __builtin_amdgcn_rcpf(static_cast<float>(there)) : 0.f;
  const float range = mx - mean;
  const size_t list = static_cast<size_t>(r) * P + p;
  uint2* const dst = a.cand + (static_cast<size_t>(r) * kListCap + static_cast<size_t>(p) * cap);
  int bin[E], cut = 0, total = 0;
  const bool all = there <= cap;                         // every logit above the floor is emitted
  const bool finite = !nan && mx < INFINITY && mean > -INFINITY;
  if (all) {
#pragma unroll
    for (int e = 0; e < E; ++e) bin[e] = v[e] > -INFINITY ? 0 : -1;
  } else if (finite) {
    const float scale = list_scale(range), below = -1.f - static_cast<float>(lane);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      bin[e] = static_cast<int>(__builtin_amdgcn_fmed3f((v[e] - mean) * scale, below, kListBins - 1.f));
      atomicAdd(&bins[bin[e]], 1u);
      if (v[e] == -INFINITY) bin[e] = -1 - kWave;        // never a member of anything
    }
    wave_lds_fence();
    cut = list_cut(bins, lane, cap, total);
    const int enough = min(cap - cap / 4, there * 3 / 8);    // (a piece that is masked for the most part has a smaller share)
    if (__builtin_expect(total < enough, 0)) refine_list<E>(v, bin, cut, cap, enough, total, bins, lane);
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) bin[e] = -1;
  }
  int at = 0;
  float vmin = INFINITY;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const bool take = bin[e] >= cut;
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(take);
    if (take) {
      dst[lanes_before(mask, at)] = make_uint2(static_cast<uint32_t>(group(e >> 2) + (e & 3)), __float_as_uint(v[e]));
      vmin = fminf(vmin, v[e]);
    }
    at += __builtin_popcountll(mask);
  }
  for (int i = at + lane; i < cap; i += kWave) dst[i] = make_uint2(kNoId, 0u);
  // Supplied logits: keep them for the next iteration.  Last, so that nothing waits behind the stores, and through the L2:
  // 32 x 65536 ids 83.2 -> 79.1 us in four steps (81.2 with plain stores here), x 81146 88.4 -> 83.2.
  if (R.zw) {
    const auto ring = row_buffer(R.zw, n_);
#pragma unroll
    for (int u = 0; u < E / 4; ++u) {
      const int v0 = group(u);
      if (u < E / 4 - 1 || whole || v0 + 3 < n_) {
        store4_through(ring, v0, given[u * 4], given[u * 4 + 1], given[u * 4 + 2], given[u * 4 + 3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v0 + e < n_) R.zw[v0 + e] = given[u * 4 + e];
      }
    }
  }
  vmin = wave_min_f32(vmin);
  if (lane == 0) {
    const bool good = all || (finite && at > 0);
    a.cand_cnt[list] = good && !nan ? static_cast<uint32_t>(at) : static_cast<uint32_t>(cap) + 1u;   // > cap: overflow
    // what is not emitted lies below this key: nothing (0), masked ids, everything below the smallest emitted
    a.cand_cut[list] = !all ? zkey(vmin) : at == have ? 0u : zkey(kListFloor) + 1u;
  }
}

// Ids per lane of the list kernel for these rows (a list per 64 times as many), or 0: the slice kernel.  The lists of a row
// share kRowListCap slots; a list has to hold what the row's top_k leaves to its piece: its mean, five of its standard
// deviations and some more have to fit into the three quarters of the slots that are filled.  Longer pieces vary less.
// (top-k 1000: any row that has lists but for a few lengths near the 524288th id; 2000: up to 196608 ids; 3072: up to 53248.)
// Where both would do the lists are faster than the slices: four steps of 32 rows behind an LM head over 1280 that leaves none,
// slices : lists (us), 20000 ids under top-k 2500 128 : 119, 40000 under 2434 158 : 149, 65536 under 2600 193 : 188; of 128
// rows 188 : 162, 248 : 223, 294 : 280.
int list_width(int n, int top_k) {
  for (int per : {16, 32}) {
    const int P = (n + kWave * per - 1) / (kWave * per);
    // list_kernel looks for the row's end in the last load only: a piece has `per` lines, its last four may be missing
    if (P > kRowMaxTiles || (P - 1) * per < (per - 4) * P) continue;
    const double cap = kRowListCap / P, mean = static_cast<double>(top_k) / P;
    if (mean + 5.0 * std::sqrt(mean) + 4.0 <= 0.75 * cap) return per;
  }
  return 0;
}
#endif  // !SCD_ROW_DIRECT_ONLY

// Per-position statistics of the iteration (Sec. 3: acceptance rate beta = 1 - D_TV(p, q) =
// sum_v min(p_v, q_v); Prop. "SJD Collision Probability": C = sum_v p_v q_v and its bound
// sqrt(sum p^2 * sum q^2) = exp(-(H_2(p) + H_2(q)) / 2)).  d0..d2: this thread's share of
// sum min(p, q), sum p q, sum p^2 over the kept ids.  sum q^2 is what the slot's previous
// evaluation stored (1/n for a never-evaluated position).  Uniform over the workgroup.
__device__ __forceinline__ void row_statistics_out(const RowArgs& a, const RowRef& R, float d0, float d1,
                                                   float d2, float q_uniform, Small& sm) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  d0 = wave_sum(d0);
  d1 = wave_sum(d1);
  d2 = wave_sum(d2);
  if (lane == 0) {
    sm.dred[0][wave] = d0;
    sm.dred[1][wave] = d1;
    sm.dred[2][wave] = d2;
  }
  __syncthreads();
  if (tid == 0) {
    float s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      s0 += sm.dred[0][w];
      s1 += sm.dred[1][w];
      s2 += sm.dred[2][w];
    }
    const float s2q = R.fresh() ? q_uniform : a.s2[R.pidx];
    *reinterpret_cast<float4*>(a.diag + R.widx * 4) = make_float4(s0, s1, s2, s2q);
    a.s2[R.oidx] = s2;
  }
}

// ---------------------------------------------------------------------------------
// row kernel
// ---------------------------------------------------------------------------------
struct RowOut {      // what a path hands to the common tail
  bool accept;
  bool prace;         // the row makes a Gumbel-max draw from p (GS kernels only)
  float px, qx;
  float best;         // residual race (on rejection)
  int best_id;
  float gbest;        // Gumbel-sharing draft (GS kernels only)
  int gbest_id;
};

// Entry of id v, probability pv > 0, in the shared-noise Gumbel-max draw of position j
// (Alg. GS / Alg. SCD(pi_GS)): argmax_v(log p_v + G_v) with G_v = -ln(-ln U_v) is the
// argmin of -ln(U_v) / p_v (appendix proof of the Gumbel-coupling theorem).  U_v is keyed by
// (seed, sequence, position, id) only -- not by the iteration -- so that every iteration
// redraws the position with the same noise (w3s = stream 3, it = 0).  The independent redraft
// of the alpha-coupling is the same draw with fresh noise (stream 5, it = the iteration).
// Ties go to the lowest id.
__device__ __forceinline__ void gumbel_entry(RowOut& out, uint2 key, uint32_t w3s, int j, int it,
                                             int v, float pv) {
  const uint4 rr = philox4x32_10(make_uint4(static_cast<uint32_t>(v >> 2), static_cast<uint32_t>(j),
                                            static_cast<uint32_t>(it), w3s), key);
  const uint32_t lanes[4] = {rr.x, rr.y, rr.z, rr.w};
  const float sc = __fdiv_rn(neg_log(u01(lanes[v & 3])), pv);
  if (sc < out.gbest || (sc == out.gbest && v < out.gbest_id)) {
    out.gbest = sc;
    out.gbest_id = v;
  }
}

// Which Gumbel-max draw from p the row makes for its next draft, if any (uniform over the
// workgroup).  alpha-coupling (Sec. 5.3): with probability 1 - alpha the redraft is independent:
// fresh noise.  Otherwise the shared-noise draw under pi_GS, and none under pi_MC (the MRS output
// is the redraft).
struct PRace {
  bool on;
  uint32_t w3s;
  int it;
};
__device__ __forceinline__ PRace p_race_of_row(const RowArgs& a, uint2 key, uint32_t w3, int j, int it) {
  if (a.alpha < 1.0f) {
    const uint4 rs = philox4x32_10(make_uint4(0u, static_cast<uint32_t>(j), static_cast<uint32_t>(it),
                                              w3 | kStreamAlpha), key);
    if (!(u01(rs.x) <= a.alpha)) return {true, w3 | kStreamIndep, it};
  }
  return {a.gumbel != 0, w3 | kStreamGumbel, 0};
}

// The draw of a row that concerns all of its ids, the accept test's uniform: ten Philox rounds by one wavefront
// while the row's logits are on their way, not by all of them behind the normaliser.  Published by the next
// barrier.
__device__ __forceinline__ void draw_accept_uniform(const RowArgs& a, const RowRef& R, Small& sm) {
  if (a.mode == kRowSelectOnly || wave_index() != NW - 1) return;
  const uint4 ra = philox4x32_10(make_uint4(0u, static_cast<uint32_t>(R.p0 + R.s), static_cast<uint32_t>(R.it),
                                            (static_cast<uint32_t>(R.b) << 8) | kStreamAccept), seed_key(a.seed));
  if ((threadIdx.x & 63) == 0) sm.u_accept = u01(ra.x);
}

// Kept ids that a wavefront parks in LDS; with more (only where a thread holds more than 8 logits) it works from
// its registers, where then every second lane or more has work anyway.
constexpr int kWaveCap = 512;
template <int PER>
constexpr int wave_cap() { return PER * kWave < kWaveCap ? PER * kWave : kWaveCap; }

// Normaliser, accept test, residual race (and the optional parts) over a row's kept ids, behind the threshold.  Every
// wavefront works on its own: `cnt` of them parked at kid / kz / kq (compact), or those that each_reg(f) calls f with.
template <bool PREQ, bool GS, bool EXTRA, class EachReg>
__device__ __forceinline__ void finish_kept(const RowArgs& a, const RowRef& R, uint32_t* kid, float* kz, float* kq, int cnt,
                                            bool compact, EachReg&& each_reg, float m, float thr, float zcx, float zpx,
                                            Small& sm, RowOut& out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
  const int n = a.n;
  wave_lds_fence();
  // the previous logits of the first kAhead lanes' worth of kept ids are requested now, of any more when needed
  constexpr int kAhead = 3;
  float qa[kAhead];
  const bool gather = !PREQ && a.mode != kRowSelectOnly && !R.fresh();
  if (gather) {
#pragma unroll
    for (int s = 0; s < kAhead; ++s) qa[s] = R.zp[s * kWave + lane < cnt ? kid[s * kWave + lane] : 0u];
  }
  // f(valid, id, z, q) for this wavefront's kept ids, every lane taking part in every call
  auto from_lds = [&](auto&& f) {
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {
      const int i = s * kWave + lane;
      if (s * kWave < cnt) f(i < cnt, static_cast<int>(kid[i]), kz[i], PREQ ? kq[i] : qa[s]);
    }
    if constexpr (PREQ) {
#pragma unroll 1
      for (int s = kAhead * kWave; s < cnt; s += kWave) {
        const int i = s + lane, id = i < cnt ? static_cast<int>(kid[i]) : 0;
        f(i < cnt, id, kz[i], kq[i]);
      }
    } else if (cnt > kAhead * kWave) {
      // the loads of the next round are under way while f works on this one
      auto id_at = [&](int i) { return i < cnt ? static_cast<int>(kid[i]) : 0; };
      int next = id_at(kAhead * kWave + lane);
      float qnext = gather ? R.zp[next] : 0.f;
#pragma unroll 1
      for (int s = kAhead * kWave; s < cnt; s += kWave) {
        const int i = s + lane, id = next;
        const float q = qnext;
        next = id_at(i + kWave);
        if (gather && s + kWave < cnt) qnext = R.zp[next];
        f(i < cnt, id, kz[i], q);
      }
    }
  };
  auto each_kept = [&](auto&& f) {
    if (compact) from_lds(f);
    else each_reg(f);
  };
  float sum = 0.f;
  each_kept([&](bool valid, int, float z, float) {
    const float w = exp_of(z - m);
    sum += valid ? w : 0.f;
  });
  sum = wave_sum(sum);
  if (lane == 0) {
    sm.fred[wave] = sum;
    sm.ired[wave] = cnt;
  }
  __syncthreads();
  int Cn;
  fold_before<NW>(sm.ired, 0, Cn);
  const float S = fold_sum<NW>(sm.fred);
  const float lse_c = m + logf(S);
  if (tid == 0) {
    a.thr[R.oidx] = thr;
    a.lse[R.oidx] = lse_c;
    a.nkept[R.oidx] = Cn;
    if (a.flags && !(lse_c == lse_c && fabsf(lse_c) < INFINITY)) atomicOr(a.flags, 1);
  }
  if (a.mode == kRowSelectOnly) return;

  // Modified Rejection Sampling
  const int j = R.p0 + R.s;
  const float q_uniform = a.q_uniform;
  const uint2 key = seed_key(a.seed);
  const uint32_t w3 = static_cast<uint32_t>(R.b) << 8;
  const bool x_ok = R.x >= 0 && R.x < n;
  out.px = x_ok ? prob(zcx, thr, lse_c) : 0.f;
  out.qx = R.fresh() ? q_uniform : (x_ok ? prob(zpx, R.thr_p, R.lse_p) : 0.f);
  out.accept = __fmul_rn(sm.u_accept, out.qx) <= out.px;
  out.best = INFINITY;
  out.best_id = 0x7FFFFFFF;
  out.gbest = INFINITY;
  out.gbest_id = 0x7FFFFFFF;
  auto q_of = [&](float z) { return R.fresh() ? q_uniform : prob(z, R.thr_p, R.lse_p); };
  if (EXTRA && a.diag != nullptr && a.mode == kRowRing) {
    float d0 = 0.f, d1 = 0.f, d2 = 0.f;
    each_kept([&](bool valid, int, float zc_v, float zq_v) {
      const float pv = valid ? exp_of(zc_v - lse_c) : 0.f;
      const float qv = valid ? q_of(zq_v) : 0.f;
      d0 += fminf(pv, qv);
      d1 += pv * qv;
      d2 += pv * pv;
    });
    row_statistics_out(a, R, d0, d1, d2, q_uniform, sm);
  }
  if (GS) {                        // next draft should the row survive
    const PRace pr = p_race_of_row(a, key, w3, j, R.it);
    out.prace = pr.on;
    if (pr.on)
      each_kept([&](bool valid, int v, float z, float) {
        const float pv = valid ? exp_of(z - lse_c) : 0.f;
        if (pv > 0.f) gumbel_entry(out, key, pr.w3s, j, pr.it, v, pv);
      });
  }
  if (out.accept) return;          // uniform over the workgroup

  auto race_one = [&](int v, float rv) {   // exponential-race entry of id v, residual rv > 0
    const uint4 rr = philox4x32_10(make_uint4(static_cast<uint32_t>(v >> 2), static_cast<uint32_t>(j),
                                              static_cast<uint32_t>(R.it), w3 | kStreamResid), key);
    const uint32_t lanes[4] = {rr.x, rr.y, rr.z, rr.w};
    const float sc = __fdiv_rn(neg_log(u01(lanes[v & 3])), rv);
    if (sc < out.best || (sc == out.best && v < out.best_id)) {
      out.best = sc;
      out.best_id = v;
    }
  };
  auto residual = [&](float z, float q) { return __fsub_rn(exp_of(z - lse_c), q_of(q)); };
  if (compact) {
    int positive = 0;              // written over the entries, at or before the place just read
    from_lds([&](bool valid, int v, float z, float q) {
      const float rv = residual(z, q);
      const bool pos = valid && rv > 0.f;
      const unsigned long long mask = __builtin_amdgcn_ballot_w64(pos);
      const int at = lanes_before(mask, positive);
      positive += __builtin_popcountll(mask);
      if (pos) {
        kid[at] = static_cast<uint32_t>(v);
        kz[at] = rv;
      }
    });
    wave_lds_fence();
    for (int i = lane; i < positive; i += kWave) race_one(static_cast<int>(kid[i]), kz[i]);
  } else {
    each_kept([&](bool valid, int v, float z, float q) {
      const float rv = residual(z, q);
      if (valid && rv > 0.f) race_one(v, rv);
    });
  }
}

// Everything after the candidates sit in registers: threshold (if top-k filters),
// normaliser, accept test, residual race.  Returns false if the threshold could not
// be certified against `cut_max` (the caller then takes the complete path).
// PREQ: zq[e] is the previous iteration's logit of id vid[e], read by the caller together
// with zv (coalesced; unused for a fresh position).  Otherwise the previous
// logits of the KEPT ids are gathered here, right after the compaction, so that the round trip hides behind the
// normaliser.  LDS: hist (kHistWords), and lds (NW * wave_cap * 12 or 8 bytes), which may lie over it.
//
// The kept ids are a random ~K/n of each thread's logits.  Every wavefront compacts its own into its part of LDS
// (a fixed order), so that the expensive per-id work that follows runs on full wavefronts instead of at the pace
// of the unluckiest lane; the positive residuals, about half of them, are compacted again before the race.  No
// barrier stands between the threshold and the normaliser, nor between the normaliser and the race: with the
// row compacted as a whole, three barriers and a prefix sum over the workgroup did (16 x 32 rows of 8192 ids 24 ->
// 19 us, 32 rows of 16384 15 -> 13.5).  The callers deal ids out in small pieces, so the wavefronts' shares differ
// by chance only.
template <int PER, bool PREQ, bool GS, bool EXTRA>
__device__ __forceinline__ bool finish_regs(const RowArgs& a, const RowRef& R, const int (&vid)[PER],
                                            const float (&zv)[PER], const float (&zq)[PER],
                                            const bool (&ok)[PER], bool filter, uint32_t cut_max,
                                            float zcx, float zpx, uint32_t* hist, unsigned char* lds,
                                            Small& sm, RowOut& out, bool have_thr = false, float thr_given = 0.f) {
  const int wave = wave_index();
  uint32_t kmin, kmax;
  bool nan;
  thread_range<PER>(zv, ok, kmin, kmax, nan);
  if (nan && a.flags) atomicOr(a.flags, 1);                    // NaN of either sign
  if (filter) zero_hist(hist);            // published by the barrier inside block_minmax
  block_minmax(kmin, kmax, sm, false);
  const float m = key_to_float(kmax);
  float thr = have_thr ? thr_given : -INFINITY;   // given: the caller has applied the filters
  if (filter) {
    const uint32_t tkey = select_regs<PER>(zv, ok, key_to_float(kmin), m, static_cast<uint32_t>(a.top_k), hist, sm);
    if (tkey < cut_max) return false;     // an unseen logit could be >= the K-th candidate
    thr = key_to_float(tkey);
  }
  if (EXTRA && a.top_p24 != 0u && !have_thr) {   // nucleus filter on what top-k left
    const float thr_k = thr;
    const float zmin = filter ? thr_k : (kmin <= kmax ? key_to_float(kmin) : m);
    auto each = [&](auto&& f) {
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if (ok[e] && zv[e] >= thr_k) f(zkey(zv[e]), zv[e]);
    };
    const uint32_t pkey = nucleus_key(each, [](uint32_t, uint32_t) {}, each, m, zmin, a.top_p24,
                                      reinterpret_cast<unsigned long long*>(hist), sm);
    thr = key_to_float(pkey);
  }
  constexpr int CAP = wave_cap<PER>();
  constexpr bool ALL_FIT = CAP == PER * kWave;
  uint32_t* const kid = reinterpret_cast<uint32_t*>(lds) + wave * (PREQ ? 3 : 2) * CAP;
  float* const kz = reinterpret_cast<float*>(kid + CAP);
  float* const kq = kz + CAP;
  int cnt = 0;                            // this wavefront's kept ids, a scalar
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const bool keep = ok[e] && zv[e] >= thr;
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(keep);
    const int at = lanes_before(mask, cnt);
    cnt += __builtin_popcountll(mask);
    if (keep && (ALL_FIT || at < CAP)) {
      kid[at] = static_cast<uint32_t>(vid[e]);
      kz[at] = zv[e];
      if (PREQ) kq[at] = zq[e];
    }
  }
  const bool compact = ALL_FIT || cnt <= CAP;
  finish_kept<PREQ, GS, EXTRA>(a, R, kid, kz, kq, cnt, compact, [&](auto&& f) {
    if constexpr (!ALL_FIT) {
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        float q = 0.f;
        if constexpr (PREQ) q = zq[e];
        else if (a.mode != kRowSelectOnly && !R.fresh() && ok[e] && zv[e] >= thr) q = R.zp[vid[e]];
        f(ok[e] && zv[e] >= thr, vid[e], zv[e], q);
      }
    }
  }, m, thr, zcx, zpx, sm, out);
  return true;
}

// The draft token's logits in this and the previous iteration: their latency hides behind the selection.
__device__ __forceinline__ void draft_logits(const RowArgs& a, const RowRef& R, float& zcx, float& zpx) {
  const bool x_ok = a.mode != kRowSelectOnly && R.x >= 0 && R.x < a.n;
  zcx = x_ok ? R.zc[R.x] : 0.f;
  zpx = x_ok ? R.zp[R.x] : 0.f;              // (of a new position: never used)
}

// f(v0, z) for every four neighbouring ids v0 .. v0 + 3 of a row, -inf past its end, read in coalesced 32-byte pieces,
// two per thread in flight.
template <class F>
__device__ __forceinline__ void each_four(const float* zc, int n, F&& f) {
  const int nchunks = (n + 7) >> 3;
  for (int c0 = threadIdx.x; c0 < nchunks; c0 += 2 * THREADS) {
    float zz[2][2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int c = c0 + u * THREADS;
      if (c < nchunks && (c << 3) + 7 < n) {
        const float4 lo4 = load4(zc + (c << 3));
        const float4 hi4 = load4(zc + (c << 3) + 4);
        zz[u][0][0] = lo4.x; zz[u][0][1] = lo4.y; zz[u][0][2] = lo4.z; zz[u][0][3] = lo4.w;
        zz[u][1][0] = hi4.x; zz[u][1][1] = hi4.y; zz[u][1][2] = hi4.z; zz[u][1][3] = hi4.w;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          zz[u][e >> 2][e & 3] = (c < nchunks && (c << 3) + e < n) ? zc[(c << 3) + e] : -INFINITY;
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int c = c0 + u * THREADS;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (c < nchunks && (c << 3) + 4 * h < n) f((c << 3) + 4 * h, zz[u][h]);
    }
  }
}
// f(v, z) for every id
template <class F>
__device__ __forceinline__ void each_logit(const float* zc, int n, F&& f) {
  each_four(zc, n, [&](int v0, const float (&z)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (v0 + e < n) f(v0 + e, z[e]);
  });
}

// Normaliser, accept test and races over all ids that `for_each_logit` brings, where the kept ones are too many to park.
// WHOLE: that is the whole row, and the residual race takes it four ids at a time, which share a draw of random bits (four
// steps of 32 x 64000 ids of which 27000 are kept: 445 -> 396 us).
template <bool GS, bool EXTRA, bool WHOLE, class Each>
__device__ __forceinline__ void finish_in_place(const RowArgs& a, const RowRef& R, Each&& for_each_logit, float m, float thr,
                                                float zcx, float zpx, Small& sm, RowOut& out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.n;
  const float* const zp = R.zp;
  float sum = 0.f;
  int cnt = 0;
  for_each_logit([&](int, float z) {
    if (z >= thr) {
      sum += exp_of(z - m);
      ++cnt;
    }
  });
  sum = wave_sum(sum);
  cnt = wave_sum_i32(cnt);
  if (lane == 0) {
    sm.fred[wave] = sum;
    sm.ired[wave] = cnt;
  }
  __syncthreads();
  const float S = fold_sum<NW>(sm.fred);
  int Cn;
  fold_before<NW>(sm.ired, 0, Cn);
  const float lse_c = m + logf(S);
  if (tid == 0) {
    a.thr[R.oidx] = thr;
    a.lse[R.oidx] = lse_c;
    a.nkept[R.oidx] = Cn;
    if (a.flags && !(lse_c == lse_c && fabsf(lse_c) < INFINITY)) atomicOr(a.flags, 1);
  }
  if (a.mode == kRowSelectOnly) return;
  const int j = R.p0 + R.s;
  const float q_uniform = a.q_uniform;
  const uint2 key = seed_key(a.seed);
  const uint32_t w3 = static_cast<uint32_t>(R.b) << 8;
  const bool x_ok = R.x >= 0 && R.x < n;
  out.px = x_ok ? prob(zcx, thr, lse_c) : 0.f;
  out.qx = R.fresh() ? q_uniform : (x_ok ? prob(zpx, R.thr_p, R.lse_p) : 0.f);
  const uint4 ra = philox4x32_10(make_uint4(0u, static_cast<uint32_t>(j), static_cast<uint32_t>(R.it),
                                            w3 | kStreamAccept), key);
  out.accept = __fmul_rn(u01(ra.x), out.qx) <= out.px;
  out.best = INFINITY;
  out.best_id = 0x7FFFFFFF;
  out.gbest = INFINITY;
  out.gbest_id = 0x7FFFFFFF;
  if (EXTRA && a.diag != nullptr && a.mode == kRowRing) {
    float d0 = 0.f, d1 = 0.f, d2 = 0.f;
    for_each_logit([&](int v, float z) {
      const float pv = prob(z, thr, lse_c);
      if (pv > 0.f) {
        const float qv = R.fresh() ? q_uniform : prob(zp[v], R.thr_p, R.lse_p);
        d0 += fminf(pv, qv);
        d1 += pv * qv;
        d2 += pv * pv;
      }
    });
    row_statistics_out(a, R, d0, d1, d2, q_uniform, sm);
  }
  if (GS) {
    const PRace pr = p_race_of_row(a, key, w3, j, R.it);
    out.prace = pr.on;
    if (pr.on) {
      for_each_logit([&](int v, float z) {
        const float pv = prob(z, thr, lse_c);
        if (pv > 0.f) gumbel_entry(out, key, pr.w3s, j, pr.it, v, pv);
      });
    }
  }
  if (out.accept) return;
  if constexpr (WHOLE) {
    each_four(R.zc, n, [&](int v0, const float (&z)[4]) {
      float q[4] = {0.f, 0.f, 0.f, 0.f}, rv[4];
      bool any = false;
      if (!R.fresh()) {
        if (v0 + 3 < n) {
          const float4 t = load4(zp + v0);
          q[0] = t.x; q[1] = t.y; q[2] = t.z; q[3] = t.w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) q[e] = v0 + e < n ? zp[v0 + e] : 0.f;
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float pv = v0 + e < n ? prob(z[e], thr, lse_c) : 0.f;
        rv[e] = pv > 0.f ? __fsub_rn(pv, R.fresh() ? q_uniform : prob(q[e], R.thr_p, R.lse_p)) : 0.f;
        any |= rv[e] > 0.f;
      }
      if (!any) return;
      const uint4 rr = philox4x32_10(make_uint4(static_cast<uint32_t>(v0 >> 2), static_cast<uint32_t>(j),
                                                static_cast<uint32_t>(R.it), w3 | kStreamResid), key);
      const uint32_t lanes[4] = {rr.x, rr.y, rr.z, rr.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float sc = rv[e] > 0.f ? __fdiv_rn(neg_log(u01(lanes[e])), rv[e]) : INFINITY;
        if (rv[e] > 0.f && (sc < out.best || (sc == out.best && v0 + e < out.best_id))) {
          out.best = sc;
          out.best_id = v0 + e;
        }
      }
    });
  } else {
    for_each_logit([&](int v, float z) {
      const float pv = prob(z, thr, lse_c);
      if (pv > 0.f) {
        const float qv = R.fresh() ? q_uniform : prob(zp[v], R.thr_p, R.lse_p);
        const float rv = __fsub_rn(pv, qv);
        if (rv > 0.f) {
          const uint4 rr = philox4x32_10(make_uint4(static_cast<uint32_t>(v >> 2), static_cast<uint32_t>(j),
                                                    static_cast<uint32_t>(R.it), w3 | kStreamResid), key);
          const uint32_t lanes[4] = {rr.x, rr.y, rr.z, rr.w};
          const float sc = __fdiv_rn(neg_log(u01(lanes[v & 3])), rv);
          if (sc < out.best || (sc == out.best && v < out.best_id)) {
            out.best = sc;
            out.best_id = v;
          }
        }
      }
    });
  }
}

// Rows of more than kDirectMaxN ids under a nucleus filter alone: the whole row in registers, 32 or 64 logits per
// thread, until the threshold is known and the kept ids are parked in LDS.
//   Bound by the vector instructions of one CU per row, about 30 per id for the masses (an exponential, a conversion to
// fixed point and a 64-bit LDS addition each): 28000 of 88000 cycles.  Against a row read from memory three times and
// scanned three more through 16-bit prefixes in LDS, four steps on supplied logits of 32 x 65536 take 198 us for 228,
// of 2 x 64 x 64000 ids behind the LM head 678 for 705, of 8 x 32 x 65536 over 2048 without guidance 680 for 776.
// Up to 18432 kept ids are parked (what LDS holds); rows that keep more are read again, which is the better way for them.
constexpr int kNucleusCap = 1152;            // kept ids that a wavefront parks ...
constexpr int kNucleusPark = kNucleusCap + kWave;   // ... and a place per lane for what is not kept
template <int PER, bool GS>
__device__ __forceinline__ void nucleus_path(const RowArgs& a, RowRef& R, unsigned char* smem, Small& sm, RowOut& out) {
  const int lane = threadIdx.x & 63, wave = wave_index();
  int n = a.n;
  // the sizes' comparisons are made anew in every phase: kept, they fill the scalar registers
  auto new_phase = [&]() { asm volatile("" : "+s"(n)); __builtin_amdgcn_sched_barrier(0); };
  constexpr int STEP = 8 * NW * 32;          // ids per group of four registers, dealt out as in direct_path
  const int first = wave * 32 + (lane >> 3) * (NW * 32) + ((lane & 7) << 2);
  // Past the end of the row: -inf, which has no mass and is below every threshold (a mask per logit would be kept from
  // phase to phase); whole groups past it are skipped.
  // a scalar base and 32 bits per lane: no registers for addresses
  auto at_byte = [](auto* base, uint32_t bytes) {
    using T = decltype(base);
    if constexpr (std::is_const_v<std::remove_pointer_t<T>>) return reinterpret_cast<T>(reinterpret_cast<const char*>(base) + bytes);
    else return reinterpret_cast<T>(reinterpret_cast<char*>(base) + bytes);
  };
  float zv[PER];
#pragma unroll
  for (int u = 0; u < PER / 4; ++u) {
    const int v0 = first + u * STEP;
    if ((u + 1) * STEP <= n) {               // uniform
      const float4 t = load4(at_byte(R.zc + u * STEP, 4u * first));
      zv[4 * u] = t.x; zv[4 * u + 1] = t.y; zv[4 * u + 2] = t.z; zv[4 * u + 3] = t.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) zv[4 * u + e] = -INFINITY;
      if (u * STEP < n) {
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = *at_byte(R.zc, 4u * min(v0 + e, n - 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) zv[4 * u + e] = v0 + e < n ? t[e] : -INFINITY;
      }
    }
  }
  read_row_scalars(a, R);
  float zcx, zpx;
  draft_logits(a, R, zcx, zpx);
  draw_accept_uniform(a, R, sm);
  new_phase();
  float hi = -INFINITY, lo = INFINITY;
  bool nan = false;
#pragma unroll
  for (int u = 0; u < PER / 4; ++u) {
    if (u * STEP >= n) continue;             // uniform
    float* const z = &zv[4 * u];
    const int v0 = first + u * STEP;
    if (R.zw) {                              // supplied logits: keep them for the next iteration
      if (v0 + 3 < n) {
        store4(at_byte(R.zw + u * STEP, 4u * first), z[0], z[1], z[2], z[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v0 + e < n) *at_byte(R.zw, 4u * (v0 + e)) = z[e];
      }
    }
    hi = max3(max3(hi, z[0], z[1]), z[2], z[3]);
    if ((u + 1) * STEP <= n) {
      lo = min3(min3(lo, z[0], z[1]), z[2], z[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) lo = z[e] > -INFINITY ? min3(lo, z[e], z[e]) : lo;
    }
    const float sum = (z[0] + z[1]) + (z[2] + z[3]);
    if (sum != sum) {                        // a NaN, or infinities of both signs
#pragma unroll
      for (int e = 0; e < 4; ++e) nan |= z[e] != z[e];
    }
  }
  if (nan && a.flags) atomicOr(a.flags, 1);
  uint32_t kmax = nan ? 0xFFFFFFFFu : zkey(hi), kmin = zkey(lo);
  block_minmax(kmin, kmax, sm, false);
  const float m = key_to_float(kmax);
  // Members of the boundary's bin: gathered in LDS behind the histogram, then taken up by all threads evenly.
  float* const list = reinterpret_cast<float*>(smem + NBINS_P * 8);
  int near_cnt = 0;
  bool near_dense = false;
  float nz[PER_LIST];
  const uint32_t pkey = nucleus_key(
      [&](auto&& f) {
        new_phase();
#pragma unroll
        for (int u = 0; u < PER / 4; ++u) {
          if (u * STEP >= n) continue;
#pragma unroll
          for (int e = 0; e < 4; ++e) f(0u, zv[4 * u + e]);
          __builtin_amdgcn_sched_barrier(0);               // (64 logits leave no registers for more at a time)
        }
      },
      [&](uint32_t klo, uint32_t khi) {
        const float flo = klo != 0u ? key_to_float(klo) : -INFINITY, fhi = khi != 0xFFFFFFFFu ? key_to_float(khi) : INFINITY;
        // four ids at a time, most of them far away: a distance to a place in the interval that none of its logits exceeds.
        // Both are rounded, and the interval may be a single float wide (its middle is then one of its ends): the larger
        // distance of the two ends is computed like a logit's, and rounding keeps their order.
        const bool bounded = flo > -INFINITY && fhi < INFINITY;
        const float middle = bounded ? 0.5f * flo + 0.5f * fhi : 0.f;
        const float reach = bounded ? fmaxf(fhi - middle, middle - flo) : INFINITY;
        if (threadIdx.x == 0) sm.cursor = 0u;
        __syncthreads();
        new_phase();
#pragma unroll
        for (int u = 0; u < PER / 4; ++u) {
          if (u * STEP >= n) continue;
          float d[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) d[e] = fabsf(zv[4 * u + e] - middle);
          if (__builtin_amdgcn_ballot_w64(fminf(fminf(d[0], d[1]), fminf(d[2], d[3])) <= reach) == 0ull) continue;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float z = zv[4 * u + e];
            if (z >= flo && z <= fhi) {
              const uint32_t slot = atomicAdd(&sm.cursor, 1u);
              if (slot < static_cast<uint32_t>(kListCap)) list[slot] = z;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        const uint32_t found = sm.cursor;
        near_dense = found > static_cast<uint32_t>(kListCap);
        near_cnt = near_dense ? 0 : static_cast<int>(found);
#pragma unroll
        for (int e = 0; e < PER_LIST; ++e) {
          const int i = threadIdx.x + e * THREADS;
          nz[e] = i < near_cnt ? list[i] : 0.f;
        }
      },
      [&](auto&& f) {
        if (near_dense) {
          each_logit(R.zc, n, [&](int, float z) { f(zkey(z), z); });
        } else {
#pragma unroll
          for (int e = 0; e < PER_LIST; ++e)
            if (static_cast<int>(threadIdx.x) + e * THREADS < near_cnt) f(zkey(nz[e]), nz[e]);
        }
      },
      m, key_to_float(kmin), a.top_p24, reinterpret_cast<unsigned long long*>(smem), sm);
  const float thr = key_to_float(pkey);
  new_phase();
  int mine = 0;
#pragma unroll
  for (int u = 0; u < PER / 4; ++u) {
    if (u * STEP >= n) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) mine += zv[4 * u + e] >= thr ? 1 : 0;
  }
  const int incl = wave_inclusive_sum_i32(mine);
  const int cnt = __builtin_amdgcn_readlane(incl, kWave - 1);
  if (lane == 0) sm.ured[wave] = static_cast<uint32_t>(cnt);
  __syncthreads();
  if (fold_max<NW>(sm.ured) > static_cast<uint32_t>(kNucleusCap)) {        // uniform: a flat row
    finish_in_place<GS, true, true>(a, R, [&](auto&& f) { each_logit(R.zc, n, f); }, m, thr, zcx, zpx, sm, out);
    return;
  }
  uint32_t* const kid = reinterpret_cast<uint32_t*>(smem) + wave * 2 * kNucleusPark;
  float* const kz = reinterpret_cast<float*>(kid + kNucleusPark);
  int at = incl - mine;
  new_phase();
#pragma unroll
  for (int u = 0; u < PER / 4; ++u) {
    if (u * STEP >= n) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool keep = zv[4 * u + e] >= thr;
      const int to = keep ? at : kNucleusCap + lane;
      kid[to] = static_cast<uint32_t>(min(first + u * STEP + e, n - 1));
      kz[to] = zv[4 * u + e];
      at += keep ? 1 : 0;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  wave_lds_fence();
  finish_kept<false, GS, true>(a, R, kid, kz, nullptr, cnt, true, [](auto&&) {}, m, thr, zcx, zpx, sm, out);
}

// The complete in-place path: one coalesced read of the row, 16-bit key prefixes in
// LDS, histogram select; then a candidate list in registers, or in-place scans when
// top-k is off or the candidates do not fit.
template <bool GS, bool EXTRA>
__device__ __forceinline__ void full_path(const RowArgs& a, const RowRef& R, unsigned char* smem,
                                          float zcx, float zpx, Small& sm, RowOut& out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.n;
  const int n8 = (n + 7) & ~7;
  uint16_t* k16 = reinterpret_cast<uint16_t*>(smem);
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem + static_cast<size_t>(n8) * 2);
  uint16_t* list = reinterpret_cast<uint16_t*>(smem + static_cast<size_t>(n8) * 2 + NBINS * 4);
  const float* zc = R.zc;
  float* const zw = a.cand ? nullptr : R.zw;     // whoever made the lists has made the copy already

  // pass 1: batches of 8 independent 16-byte loads per thread
  const int ngroups8 = n8 >> 2;
  // (the range is taken on the floats, two instructions a logit, and turned into keys at the end; rows of odd
  // length are read with 16-byte loads as well)
  float hi = -INFINITY, lo = INFINITY;
  bool nan = false;
  constexpr int UNR = 8;
  for (int g0 = tid; g0 < ngroups8; g0 += THREADS * UNR) {
    float f[UNR][4];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int v0 = (g0 + u * THREADS) << 2;
      if (v0 + 3 < n) {
        const float4 t = load4(zc + v0);
        f[u][0] = t.x; f[u][1] = t.y; f[u][2] = t.z; f[u][3] = t.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[u][e] = (v0 + e < n) ? zc[v0 + e] : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int g = g0 + u * THREADS;
      if (g < ngroups8) {
        const int v0 = g << 2;
        uint32_t h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = zkey(f[u][e]) >> 16;
        if (v0 + 3 < n) {
          hi = max3(max3(hi, f[u][0], f[u][1]), f[u][2], f[u][3]);
          lo = min3(min3(lo, f[u][0], f[u][1]), f[u][2], f[u][3]);
          const float sum = (f[u][0] + f[u][1]) + (f[u][2] + f[u][3]);
          if (sum != sum) {                  // a NaN, or infinities of both signs
#pragma unroll
            for (int e = 0; e < 4; ++e) nan |= f[u][e] != f[u][e];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (v0 + e < n) {
              hi = fmaxf(hi, f[u][e]);
              lo = fminf(lo, f[u][e]);
              nan |= f[u][e] != f[u][e];
            }
        }
        *reinterpret_cast<uint2*>(&k16[v0]) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
        if (zw) {
          if (v0 + 3 < n) {
            store4(zw + v0, f[u][0], f[u][1], f[u][2], f[u][3]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (v0 + e < n) zw[v0 + e] = f[u][e];
          }
        }
      }
    }
  }
  if (nan && a.flags) atomicOr(a.flags, 1);  // NaN of either sign; its prefix may be any
  uint32_t kmax = nan ? 0xFFFFFFFFu : zkey(hi);
  uint32_t p16min = nan ? 0u : zkey(lo) >> 16, p16max = kmax >> 16;
  kmax = wave_max_u32(kmax);
  if (lane == 0) sm.ured[wave] = kmax;
  block_minmax(p16min, p16max, sm);      // its barriers also publish ured and the LDS prefixes
  kmax = fold_max<NW>(sm.ured);
  const float m = key_to_float(kmax);

  const int nchunks = n8 >> 3;           // thread owns the 8-id chunks tid, tid + THREADS, ...
  const bool filter = a.top_k > 0 && a.top_k < n;
  const uint32_t K = static_cast<uint32_t>(a.top_k);
  const uint32_t range = p16max - p16min;
  int sh = 0;
  while ((range >> sh) >= static_cast<uint32_t>(NBINS)) ++sh;
  auto prefix_hist = [&](bool low_bits, uint32_t only) {
    zero_hist(hist);
    __syncthreads();
    const uint32_t mask = (1u << sh) - 1u;
    for (int c = tid; c < nchunks; c += THREADS) {
      const uint4 raw = *reinterpret_cast<const uint4*>(&k16[c << 3]);
      const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if ((c << 3) + e < n) {
          const uint32_t p = ((w4[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu) - p16min;
          if (!low_bits) atomicAdd(&hist[p >> sh], 1u);
          else if ((p >> sh) == only) atomicAdd(&hist[p & mask], 1u);
        }
      }
    }
    __syncthreads();
  };
  uint32_t t16 = 0, need_ab = K;
  int ncand = 0, my_off = 0;
  // ids whose 16-bit key prefix is >= t16: this thread's offset in a fixed order, and the total
  auto count_candidates = [&]() {
    int my_cnt = 0;
    for (int c = tid; c < nchunks; c += THREADS) {
      const uint4 raw = *reinterpret_cast<const uint4*>(&k16[c << 3]);
      const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t p = (w4[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu;
        my_cnt += ((c << 3) + e < n && p >= t16) ? 1 : 0;
      }
    }
    my_off = block_offsets(my_cnt, ncand, sm);
  };
  // those ids (at most kListCap) as a list, their logits in registers, and the common tail;
  // have_thr: the filters have been applied already and thr_given is their threshold
  auto run_list = [&](bool have_thr, float thr_given) {
    int o = my_off;
    for (int c = tid; c < nchunks; c += THREADS) {
      const uint4 raw = *reinterpret_cast<const uint4*>(&k16[c << 3]);
      const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t p = (w4[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu;
        if ((c << 3) + e < n && p >= t16) list[o++] = static_cast<uint16_t>((c << 3) + e);
      }
    }
    __syncthreads();
    int vid[PER_LIST];
    float zv[PER_LIST];
    bool ok[PER_LIST];
#pragma unroll
    for (int e = 0; e < PER_LIST; ++e) {
      const int i = tid + e * THREADS;
      ok[e] = i < ncand;
      vid[e] = ok[e] ? static_cast<int>(list[i]) : 0;
    }
#pragma unroll
    for (int e = 0; e < PER_LIST; ++e) zv[e] = ok[e] ? zc[vid[e]] : 0.f;
    // the prefixes and the list in LDS are spent: their space takes what finish_regs parks
    finish_regs<PER_LIST, false, GS, EXTRA>(a, R, vid, zv, zv, ok, !have_thr, 0u, zcx, zpx, hist, smem, sm, out,
                                            have_thr, thr_given);
  };
  if (filter) {
    prefix_hist(false, 0u);
    const uint32_t binA = find_bin(hist, need_ab, sm);
    uint32_t low = 0;
    if (sh > 0) {
      prefix_hist(true, binA);
      low = find_bin(hist, need_ab, sm);
    }
    t16 = p16min + (binA << sh) + low;
    count_candidates();
    if (ncand <= kListCap) {
      run_list(false, 0.f);
      return;
    }
  }

  // in place: no filter, or the candidates do not fit (massive ties).  Candidates: ids whose 16-bit key prefix is >= t16
  auto for_each_candidate = [&](auto&& f) {
    for (int c = tid; c < nchunks; c += THREADS) {
      const uint4 raw = *reinterpret_cast<const uint4*>(&k16[c << 3]);
      const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int v = (c << 3) + e;
        const uint32_t p = (w4[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu;
        if (v < n && p >= t16) f(v, p);
      }
    }
  };
  // with their logits, gathered: f(v, z)
  auto for_each_logit = [&](auto&& f) {
    for_each_candidate([&](int v, uint32_t) { f(v, zc[v]); });
  };
  float thr = -INFINITY;
  if (filter) {
    uint32_t lowkey = 0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      zero_hist(hist);
      __syncthreads();
      const int shift = pass == 0 ? 8 : 0;
      for_each_candidate([&](int v, uint32_t p) {
        if (p == t16) {
          const uint32_t kk = zkey(zc[v]) & 0xFFFFu;
          if (pass == 0 || (kk >> 8) == (lowkey >> 8)) atomicAdd(&hist[(kk >> shift) & 0xFFu], 1u);
        }
      });
      __syncthreads();
      lowkey |= find_bin(hist, need_ab, sm) << shift;
    }
    thr = key_to_float((t16 << 16) | lowkey);
  }
  if (EXTRA && a.top_p24 != 0u) {          // nucleus filter on what top-k left (alone: nucleus_path)
    const float thr_k = thr;
    // members of the selected bin: ids found by the prefixes in LDS (appended in any order:
    // the masses are integers), their logits gathered once and kept for the three radix levels
    int near_cnt = 0;
    bool near_dense = false;
    float nz[PER_LIST];
    const uint32_t pkey = nucleus_key(
        [&](auto&& f) {
          for_each_logit([&](int, float z) {
            if (z >= thr_k) f(zkey(z), z);
          });
        },
        [&](uint32_t klo, uint32_t khi) {
          const uint32_t pa = klo >> 16, pb = khi >> 16;
          if (tid == 0) sm.cursor = 0u;
          __syncthreads();
          for_each_candidate([&](int v, uint32_t p) {
            if (p >= pa && p <= pb) {
              const uint32_t slot = atomicAdd(&sm.cursor, 1u);
              if (slot < static_cast<uint32_t>(kListCap)) list[slot] = static_cast<uint16_t>(v);
            }
          });
          __syncthreads();
          const uint32_t found = sm.cursor;
          near_dense = found > static_cast<uint32_t>(kListCap);
          near_cnt = near_dense ? 0 : static_cast<int>(found);
#pragma unroll
          for (int e = 0; e < PER_LIST; ++e) {
            const int i = tid + e * THREADS;
            nz[e] = i < near_cnt ? zc[list[i]] : 0.f;
          }
        },
        [&](auto&& f) {
          if (near_dense) {
            for_each_logit([&](int, float z) {
              if (z >= thr_k) f(zkey(z), z);
            });
          } else {
#pragma unroll
            for (int e = 0; e < PER_LIST; ++e)
              if (tid + e * THREADS < near_cnt && nz[e] >= thr_k) f(zkey(nz[e]), nz[e]);
          }
        },
        m, thr_k, a.top_p24, reinterpret_cast<unsigned long long*>(hist), sm);
    thr = key_to_float(pkey);
    // the kept ids sit at or above the threshold's prefix: a short list takes the common tail
    t16 = max(t16, pkey >> 16);
    count_candidates();
    if (ncand <= kListCap) {
      run_list(true, thr);
      return;
    }
  }
  if (filter) finish_in_place<GS, EXTRA, false>(a, R, for_each_logit, m, thr, zcx, zpx, sm, out);
  else finish_in_place<GS, EXTRA, true>(a, R, [&](auto&& f) { each_logit(zc, n, f); }, m, thr, zcx, zpx, sm, out);
}

// Rows of more than kRowKernelMaxN ids whose candidates were not certified, or that have none
// (no top-k, or one too large for the lists): whole passes over the row in memory -- the key prefixes
// of full_path would not fit LDS.  Bound by the vector instructions of one CU, 30 to 40 us per pass
// over 131072 ids: three passes without a filter (111 us; 137 us as three kernels of one stage each),
// four with a top-k of 5000 or more (an iteration on supplied logits 32 x 131072 ids: 144 us; 154 us with every
// kept id appended to a full list, 338 us as one kernel per stage).  Odd rows are read with 16-byte loads too (100003 ids
// without a filter: 87 us against 121 us with 4-byte loads).
__device__ __forceinline__ void long_path(const RowArgs& a, const RowRef& R, unsigned char* smem, float zcx,
                                          float zpx, Small& sm, RowOut& out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.n;
  uint32_t* const hist = reinterpret_cast<uint32_t*>(smem);
  uint32_t* const kid = hist + NBINS;                       // kept ids (or members of a bin) ...
  float* const kz = reinterpret_cast<float*>(kid + kKeptCap);   // ... and their logits
  const int ngroups = n >> 2;                                // whole groups of four ids
  constexpr int UNR = 4;
  // f(v0, z) for every group of four ids v0 .. v0 + 3, z[e] = pad where there is no such id; the same
  // groups in the same order in every pass of a thread
  auto groups = [&](float pad, auto&& f) {
    for (int g0 = tid; g0 < ngroups; g0 += THREADS * UNR) {
      float4 t[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int g = g0 + u * THREADS;
        t[u] = load4(R.zc + (g < ngroups ? g << 2 : 0));
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const float z[4] = {t[u].x, t[u].y, t[u].z, t[u].w};
        if (g0 + u * THREADS < ngroups) f((g0 + u * THREADS) << 2, z);
      }
    }
    if ((n & 3) != 0 && tid == 0) {                          // the last ids of a ragged row
      float z[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = (ngroups << 2) + e < n ? R.zc[(ngroups << 2) + e] : pad;
      f(ngroups << 2, z);
    }
  };
  // f(v, z) for every id
  auto each = [&](auto&& f) {
    groups(0.f, [&](int v0, const float (&z)[4]) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v0 + e < n) f(v0 + e, z[e]);
    });
  };
  uint32_t kmax = 0, kmin = 0xFFFFFFFFu;
  {
    float hi = -INFINITY, lo = INFINITY, nan = 0.f;
    float* const zw = a.cand ? nullptr : R.zw;               // whoever made the lists has made the copy already
    groups(-INFINITY, [&](int v0, const float (&z)[4]) {
      if (zw) {
        if (v0 + 3 < n) {
          store4(zw + v0, z[0], z[1], z[2], z[3]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (v0 + e < n) zw[v0 + e] = z[e];
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hi = fmaxf(hi, z[e]);
        lo = z[e] > kRangeFloor ? fminf(lo, z[e]) : lo;
        nan = z[e] != z[e] ? z[e] : nan;                     // NaN of either sign
      }
    });
    kmax = zkey(hi);
    kmin = zkey(lo);
    if (nan != 0.f) {
      kmax = 0xFFFFFFFFu;                                    // sorts above every logit: the normaliser shows it too
      if (a.flags) atomicOr(a.flags, 1);
    }
  }
  __syncthreads();                                           // earlier users of LDS are done
  zero_hist(hist);
  if (tid == 0) sm.cursor = 0u;
  block_minmax(kmin, kmax, sm);                              // its barriers publish the zeroed bins
  const float m = key_to_float(kmax);
  const bool filter = a.top_k > 0 && a.top_k < n;
  float thr = -INFINITY;
  if (filter) {
    // first level linear in the logit (see select_regs), then radix levels over the key bits of the
    // selected bin's members, which are kept in LDS when they fit
    const float zlo = key_to_float(kmin);
    const float scale = (m > zlo) ? __fdiv_rn(static_cast<float>(NBINS - 1), m - zlo) : 0.f;
    auto lin_bin = [&](float z) {
      const float t = z > kRangeFloor ? (z - zlo) * scale : 0.f;
      return t >= 0.f ? (t >= static_cast<float>(NBINS - 1) ? NBINS - 1 : static_cast<int>(t)) : 0;
    };
    each([&](int, float z) { atomicAdd(&hist[lin_bin(z)], 1u); });
    __syncthreads();
    uint32_t need = static_cast<uint32_t>(a.top_k);
    uint32_t members;
    const int b1 = static_cast<int>(find_bin(hist, need, members, sm));
    const bool parked = members <= static_cast<uint32_t>(kKeptCap);
    if (parked)                                              // in any order: they are only counted
      each([&](int, float z) {
        if (lin_bin(z) == b1) kid[atomicAdd(&sm.cursor, 1u)] = zkey(z);
      });
    uint32_t lo = 0;
    for (int width = 32; width > 0;) {
      const int s2 = width > 12 ? width - 12 : 0;
      __syncthreads();
      zero_hist(hist);
      __syncthreads();
      auto count = [&](uint32_t key) {
        if (key >= lo && (width == 32 || (key - lo) >> width == 0u)) atomicAdd(&hist[(key - lo) >> s2], 1u);
      };
      if (parked) {
        for (uint32_t i = tid; i < members; i += THREADS) count(kid[i]);
      } else {
        each([&](int, float z) {
          if (lin_bin(z) == b1) count(zkey(z));
        });
      }
      __syncthreads();
      lo += find_bin(hist, need, sm) << s2;
      width = s2;
    }
    thr = key_to_float(lo);
    if (tid == 0) sm.cursor = 0u;
    __syncthreads();
  }
  // sum in a fixed order; the kept ids are parked for the race where a top-k says that they are few (in any
  // order: the race's winner does not depend on it)
  const bool park = filter && a.top_k <= kKeptCap;
  float sum = 0.f;
  int cnt = 0;
  each([&](int v, float z) {
    if (z >= thr) {
      sum += exp_of(z - m);
      ++cnt;
      if (park) {                         // ties at the threshold may be more than fit
        const uint32_t slot = atomicAdd(&sm.cursor, 1u);
        if (slot < static_cast<uint32_t>(kKeptCap)) {
          kid[slot] = static_cast<uint32_t>(v);
          kz[slot] = z;
        }
      }
    }
  });
  sum = wave_sum(sum);
  cnt = wave_sum_i32(cnt);
  if (lane == 0) {
    sm.fred[wave] = sum;
    sm.ired[wave] = cnt;
  }
  __syncthreads();
  const float S = fold_sum<NW>(sm.fred);
  int Cn;
  fold_before<NW>(sm.ired, 0, Cn);
  const float lse_c = m + logf(S);
  if (tid == 0) {
    a.thr[R.oidx] = thr;
    a.lse[R.oidx] = lse_c;
    a.nkept[R.oidx] = Cn;
    if (a.flags && !(lse_c == lse_c && fabsf(lse_c) < INFINITY)) atomicOr(a.flags, 1);
  }
  if (a.mode == kRowSelectOnly) return;
  const int j = R.p0 + R.s;
  const float q_uniform = a.q_uniform;
  const uint2 key = seed_key(a.seed);
  const uint32_t w3 = static_cast<uint32_t>(R.b) << 8;
  const bool x_ok = R.x >= 0 && R.x < n;
  out.px = x_ok ? prob(zcx, thr, lse_c) : 0.f;
  out.qx = R.fresh() ? q_uniform : (x_ok ? prob(zpx, R.thr_p, R.lse_p) : 0.f);
  const uint4 ra = philox4x32_10(make_uint4(0u, static_cast<uint32_t>(j), static_cast<uint32_t>(R.it),
                                            w3 | kStreamAccept), key);
  out.accept = __fmul_rn(u01(ra.x), out.qx) <= out.px;
  out.best = INFINITY;
  out.best_id = 0x7FFFFFFF;
  if (out.accept) return;
  auto enter = [&](uint32_t bits, int v, float rv) {          // exponential-race entry of id v
    const float sc = __fdiv_rn(neg_log(u01(bits)), rv);
    if (sc < out.best || (sc == out.best && v < out.best_id)) {
      out.best = sc;
      out.best_id = v;
    }
  };
  auto noise = [&](int v) {                                   // random bits of ids v & ~3 .. v | 3
    return philox4x32_10(make_uint4(static_cast<uint32_t>(v >> 2), static_cast<uint32_t>(j),
                                    static_cast<uint32_t>(R.it), w3 | kStreamResid), key);
  };
  if (park && Cn <= kKeptCap) {
    for (int i = tid; i < Cn; i += THREADS) {
      const int v = static_cast<int>(kid[i]);
      const float rv = __fsub_rn(exp_of(kz[i] - lse_c), R.fresh() ? q_uniform : prob(R.zp[v], R.thr_p, R.lse_p));
      if (!(rv > 0.f)) continue;
      const uint4 rr = noise(v);
      const uint32_t lanes[4] = {rr.x, rr.y, rr.z, rr.w};
      enter(lanes[v & 3], v, rv);
    }
    return;
  }
  groups(-INFINITY, [&](int v0, const float (&z)[4]) {
    float q[4] = {0.f, 0.f, 0.f, 0.f};
    if (!R.fresh()) {
      if (v0 + 3 < n) {
        const float4 t = load4(R.zp + v0);
        q[0] = t.x; q[1] = t.y; q[2] = t.z; q[3] = t.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = v0 + e < n ? R.zp[v0 + e] : 0.f;
      }
    }
    float rv[4];
    bool any = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float pv = v0 + e < n ? prob(z[e], thr, lse_c) : 0.f;
      rv[e] = __fsub_rn(pv, R.fresh() ? q_uniform : prob(q[e], R.thr_p, R.lse_p));
      any |= pv > 0.f && rv[e] > 0.f;
    }
    if (!any) return;
    const uint4 rr = noise(v0);
    const uint32_t lanes[4] = {rr.x, rr.y, rr.z, rr.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (rv[e] > 0.f) enter(lanes[e], v0 + e, rv[e]);
  });
}

// The whole row in registers, PER logits per thread (n <= PER * THREADS).  A wavefront takes every NW-th piece of
// 32 ids (a 128-byte line): ids that are likelier than others tend to be neighbours, and every wavefront works
// on the kept ones among its own.
//   PARTS: this iteration's logits come as the LM head's sums over parts of k.
template <int PER, bool TINY, bool PARTS, bool GS, bool EXTRA>
__device__ __forceinline__ void direct_path(const RowArgs& a, RowRef& R, unsigned char* smem, bool filter, Small& sm,
                                            RowOut& out) {
  const int lane = threadIdx.x & 63, n = a.n;
  const int first = wave_index() * 32 + (lane >> 3) * (NW * 32) + ((lane & 7) << 2);
  auto group = [&](int u) { return first + u * (8 * NW * 32); };   // four ids each
  // The kept ids' previous logits are gathered behind the threshold, except 16 to a thread without options: there the whole
  // row's are read up front (four steps of 464 rows x 4688 ids 233 : 236 us, of 32 x 16384 92.9 : 93.9).  With the options the 16
  // more registers spilled (128 rows x 10457 ids 149.8 -> 135.0, 128 x 9137 140.5 -> 132.0); shorter rows save the bytes
  // (104 x 2546 75.7 -> 74.5; 512 x 8192 behind the LM head the same).
  constexpr bool PREQ = PER >= 16 && !EXTRA;
  int vid[PER];
  float zv[PER], zq[PER];
  bool ok[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    vid[e] = group(e >> 2) + (e & 3);
    ok[e] = vid[e] < n;
    zq[e] = 0.f;
  }
  float zcx, zpx;
  if constexpr (PARTS) {
    const size_t arr = static_cast<size_t>(a.rows) * n;                         // floats between the arrays [part][cond, uncond]
    const float* const mine = a.part + R.widx * n;
    static_assert(!PREQ, "the previous logits are not read here");
    zcx = 0.f;
    auto add_up = [&](auto c_, auto ks_) {
      constexpr int C = decltype(c_)::value, KS = decltype(ks_)::value;
      float t[C * KS][PER];
#pragma unroll
      for (int q = 0; q < C * KS; ++q) load_groups<PER>(mine + q * arr, n, group, t[q]);   // q = part * C + {cond, uncond}
      read_row_scalars(a, R);
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        float c = t[0][e], u = t[C - 1][e];
#pragma unroll
        for (int p = 1; p < KS; ++p) {
          c += t[p * C][e];
          u += t[p * C + C - 1][e];
        }
        zv[e] = processed_logit<C>(a.lam, a.one_plus_lam, a.tau, c, u);
      }
      if (R.x >= 0 && R.x < n) {                                                // the draft's, by itself
        float d[C * KS];
#pragma unroll
        for (int q = 0; q < C * KS; ++q) d[q] = scalar_word(mine + q * arr + R.x);
        float c = d[0], u = d[C - 1];
#pragma unroll
        for (int p = 1; p < KS; ++p) {
          c += d[p * C];
          u += d[p * C + C - 1];
        }
        zcx = processed_logit<C>(a.lam, a.one_plus_lam, a.tau, c, u);
      }
    };
    using std::integral_constant;
    auto by_parts = [&](auto c_) {                                              // (as many as launch_row lets through)
      if constexpr (PER <= 4) {
        if (a.ksplit == 8) return add_up(c_, integral_constant<int, 8>{});
      }
      if (a.ksplit == 4) return add_up(c_, integral_constant<int, 4>{});
      add_up(c_, integral_constant<int, 2>{});
    };
    if (a.C == 2) by_parts(integral_constant<int, 2>{});
    else by_parts(integral_constant<int, 1>{});
    zpx = R.x >= 0 && R.x < n ? R.zp[R.x] : 0.f;
    R.zw = const_cast<float*>(R.zc);
  } else {
    load_groups<PER, TINY>(R.zc, n, group, zv);
    if (PREQ && a.mode != kRowSelectOnly) load_groups<PER, TINY>(R.zp, n, group, zq);   // previous logits, for a rejection
    read_row_scalars(a, R);
    draft_logits(a, R, zcx, zpx);
  }
  draw_accept_uniform(a, R, sm);
  if constexpr (!TINY) {
    align_groups<PER>(n, group, zv);
    if (PREQ) align_groups<PER>(n, group, zq);
  }
  if (R.zw) {                                  // supplied logits: keep them for the next iteration
#pragma unroll
    for (int u = 0; u < PER / 4; ++u) {
      const int v0 = group(u);
      if (v0 + 3 < n) {
        store4(R.zw + v0, zv[u * 4], zv[u * 4 + 1], zv[u * 4 + 2], zv[u * 4 + 3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v0 + e < n) R.zw[v0 + e] = zv[u * 4 + e];
      }
    }
  }
  finish_regs<PER, PREQ, GS, EXTRA>(a, R, vid, zv, zq, ok, filter, 0u, zcx, zpx, reinterpret_cast<uint32_t*>(smem), smem,
                                    sm, out);
}

// What a position that is not live any more leaves.
template <bool GS, bool EXTRA>
__device__ __forceinline__ void inactive_row(const RowArgs& a, const RowRef& R) {
  if (threadIdx.x != 0) return;
  a.y[R.widx] = -1;
  a.k[R.widx] = 1;
  if (GS) a.g[R.widx] = -1;
  if (a.px) a.px[R.widx] = 0.f;
  if (a.qx) a.qx[R.widx] = 0.f;
  if (a.mode == kRowRing && R.s == 0) a.accept_len[R.b] = 0;   // finished sequence
  if (EXTRA && a.diag != nullptr && a.mode == kRowRing) {
    *reinterpret_cast<float4*>(a.diag + R.widx * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
    if (R.s == 0)
      for (int i = 0; i < 6; ++i) a.hamm[6 * R.b + i] = 0;
  }
}

// GS: the row also makes a Gumbel-max draw from p; EXTRA: the optional parts are compiled in
// (nucleus filter, per-position statistics; kept out of the other instances: their live ranges
// cost the hot kernels registers).  PATH: which way rows of this length go.  One instance per way, because
// with all of them in one kernel the compiler keeps every way's arguments in scalar registers and spills them
// (184 spills; 46 vector registers spilled in the optional instances).  Four-step decodes over 8192 ids: 132 ->
// 129 us, with every option 206 -> 193 us.
enum Path { kDirectTiny, kDirectQuarter, kDirectHalf, kDirectWhole, kPartsQuarter, kPartsHalf, kLists, kLong, kNucleusHalf, kNucleusWhole };
template <bool GS, bool EXTRA, int PATH>
__global__ __launch_bounds__(THREADS, SCD_ROW_WAVES(EXTRA)) void row_kernel(
    const int32_t* const pos_, const int32_t* const iter_, const uint2* const cand_, const uint32_t* const cand_cnt_,
    const int mode_, const int L_, const int N_, const int P, const int capE, const RowArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ Small sm;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.n;
  const int r = blockIdx.x;
  RowRef R;
  RowOut out{};
  out.accept = true;
  if (tid < 2) sm.win[tid] = ~0ull;          // (barriers stand between this and the races)
  if constexpr (PATH <= kPartsHalf) {
    R = locate_row(a, r, pos_, iter_, mode_, L_, N_);
    if (!R.active) {
      inactive_row<GS, EXTRA>(a, R);
      return;
    }
    // ---- the whole row in registers ------------------------------------------------
    constexpr bool PARTS = PATH >= kPartsQuarter;
    constexpr int PER = PATH == kDirectWhole ? PER_DIRECT : PATH == kDirectHalf || PATH == kPartsHalf ? PER_DIRECT / 2 : PER_DIRECT / 4;
    direct_path<PER, PATH == kDirectTiny, PARTS, GS, EXTRA>(a, R, smem, a.top_k > 0 && a.top_k < n, sm, out);
  } else if constexpr (PATH == kNucleusHalf || PATH == kNucleusWhole) {
    R = locate_row(a, r, pos_, iter_, mode_, L_, N_);
    if (!R.active) {
      inactive_row<GS, EXTRA>(a, R);
      return;
    }
    nucleus_path<PATH == kNucleusHalf ? 32 : 64, GS>(a, R, smem, sm, out);
  } else {
    // ---- candidate lists (P > 0: a top-k filters and somebody has made them) ---------
    // The P counts and cuts of the row's lists (P pieces of the list or slice kernel, or P column tiles
    // of the LM head's epilogue; thread t holds those of list t) and the slots themselves are fetched in ONE round trip,
    // that of the row's place in the window.  Slots that a list does not fill hold an id past the end (kNoId); behind the
    // P lists' slots there may be room that nobody writes.
    uint32_t tc = 0, tq = 0;
    uint2 raw[PER_LIST];
    if (P > 0) {
      const uint2* const src = cand_ + static_cast<size_t>(r) * kListCap;
#pragma unroll
      for (int e = 0; e < PER_LIST; ++e) raw[e] = src[tid + e * THREADS];
      if (tid < P) {
        tc = (cand_cnt_ + static_cast<size_t>(r) * P)[tid];
        tq = (a.cand_cut + static_cast<size_t>(r) * P)[tid];
      }
    }
    R = locate_row(a, r, pos_, iter_, mode_, L_, N_);
    if (!R.active) {
      inactive_row<GS, EXTRA>(a, R);
      return;
    }
    bool done = false;
    float zcx = 0.f, zpx = 0.f;
    read_row_scalars(a, R);
    draft_logits(a, R, zcx, zpx);
    draw_accept_uniform(a, R, sm);
    if (P > 0) {
      // every list fits its capacity, how many candidates there are, the largest cut
      {
        const int tot = wave_sum_i32(static_cast<int>(tc <= static_cast<uint32_t>(capE) ? tc : 0u));
        const uint32_t cm = wave_max_u32(tq);
        const bool anybad = __builtin_amdgcn_ballot_w64(tc > static_cast<uint32_t>(capE)) != 0ull;
        if (lane == 0) {
          sm.ired2[wave] = tot;
          sm.ured[wave] = cm;
          sm.ired[wave] = anybad ? 1 : 0;
        }
      }
      __syncthreads();                // their next writers sit behind the barrier of block_minmax
      int bad, total;
      fold_before<NW>(sm.ired, 0, bad);
      fold_before<NW>(sm.ired2, 0, total);
      const uint32_t cut_max = fold_max<NW>(sm.ured);
      if (bad == 0 && total >= a.top_k) {
        int vid[PER_LIST];
        float zv[PER_LIST];
        bool ok[PER_LIST];
#pragma unroll
        for (int e = 0; e < PER_LIST; ++e) {
          ok[e] = raw[e].x < static_cast<uint32_t>(n) && tid + e * THREADS < P * capE;
          vid[e] = ok[e] ? static_cast<int>(raw[e].x) : 0;
          zv[e] = ok[e] ? __uint_as_float(raw[e].y) : 0.f;
        }
        done = finish_regs<PER_LIST, false, GS, EXTRA>(a, R, vid, zv, zv, ok, true, cut_max, zcx, zpx,
                                                       reinterpret_cast<uint32_t*>(smem), smem, sm, out);
      }
    }
    if constexpr (PATH == kLong) {
      if (!done) long_path(a, R, smem, zcx, zpx, sm, out);
    } else {
      if (!done) full_path<GS, EXTRA>(a, R, smem, zcx, zpx, sm, out);
    }
  }
  if (a.mode == kRowSelectOnly) return;

  // ---- winners of the races (lexicographic (score, id) minima) ------------------
  // Score and id as one integer, the smallest of the wavefronts' by one LDS atomic each, one barrier for both races; the
  // last wavefront alone does everything up to the hand-off, because the first ones prepare the commit meanwhile: what every
  // wavefront of a row repeats is paid four times over per SIMD.  Requesting the commit's words before the ticket comes back
  // takes its 5500 cycles to 3000.  Four-step decodes: 8 x 1024 ids 50.0 -> 45.6 us, 32 x 8192 behind the LM head 128.0 -> 122.0.
  auto enter_winner = [&](int which, float score, int id) {
    wave_min_score_id(score, id);
    if (lane == 0)
      atomicMin(&sm.win[which], static_cast<unsigned long long>(__float_as_uint(score)) << 32 | static_cast<uint32_t>(id));
  };
  if (!out.accept) enter_winner(0, out.best, out.best_id);
  if (GS) enter_winner(1, out.gbest, out.gbest_id);
  if (GS || !out.accept) __syncthreads();
  const bool speaker = wave == NW - 1;
  int y_out = R.x, k_out = 1, g_out = -1;
  if (speaker) {
    auto winner = [&](int which) { return __builtin_amdgcn_readfirstlane(static_cast<int>(sm.win[which])); };
    if (!out.accept) {
      const int id = winner(0);
      if (id != 0x7FFFFFFF) {      // else: empty residual (rounding only) counts as accept
        y_out = id;
        k_out = 0;
      }
    }
    // Gumbel-sharing draft of the row.  Empty support cannot happen (the maximum is kept); -1: the row made
    // no such draw
    if (GS && out.prace) {
      const int id = winner(1);
      g_out = id != 0x7FFFFFFF ? id : R.x;
    }
  }
  if (a.mode != kRowRing) {
    if (speaker && lane == 0) {
      a.y[R.widx] = y_out;
      a.k[R.widx] = static_cast<uint8_t>(k_out);
      if (a.px) a.px[R.widx] = out.px;
      if (a.qx) a.qx[R.widx] = out.qx;
      if (GS) a.g[R.widx] = g_out;
    }
    return;
  }

  // ---- last workgroup of the sequence: first rejection, emit, slide -----------
  // Hand-off between workgroups WITHOUT an agent-scope fence (on this chip such a fence
  // writes back the whole L2 and costs tens of microseconds per launch).  The few bytes that
  // travel (y, k, g) are stored with agent-scope atomic stores, which are written through
  // to the device-coherent level.  The storing wavefront then WAITS until those stores have
  // been acknowledged (s_waitcnt vmcnt(0): the vector-memory counter of a wavefront covers
  // its stores on gfx950) and only then bumps the sequence's ticket with an agent-scope
  // atomic; a workgroup-scope fence alone does not make the compiler emit that wait.  The
  // last arriver (the one that reads live - 1 from the ticket) reads y, k, g back with
  // agent-scope atomic loads, which bypass the non-coherent cache levels.
  // Assumption about gfx950 stated here on purpose: an agent-scope atomic store is complete
  // at the device-coherent level when the issuing wavefront's vmcnt reaches zero, and
  // agent-scope atomic RMWs on one address are totally ordered, so every store of a row that
  // took an earlier ticket is visible to the workgroup that takes the last one.
  const int b = R.b, p0 = R.p0, live = R.live;
  const size_t base = static_cast<size_t>(b) * a.L;
  int slot = tid < a.L ? R.first_slot + tid : 0;
  if (slot >= a.L) slot -= a.L;
  int age_old = 0, verified_old = 0, entering = -1;
  if (speaker) {
    if (lane == 0) {
      __hip_atomic_store(&a.y[R.widx], y_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&a.k[R.widx], static_cast<uint8_t>(k_out), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (GS) __hip_atomic_store(&a.g[R.widx], g_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the stores above have completed
      sm.last = __hip_atomic_fetch_add(&a.ticket[b], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == live - 1;
    }
  } else if (tid < a.L) {
    // While the ticket travels: what the commit will need, should this workgroup be the last.  Nothing but
    // the commit writes these words.
    age_old = a.age_w[base + slot];
    if (tid == 0) {
      verified_old = a.verified[b];
      if (a.px) a.px[R.widx] = out.px;
      if (a.qx) a.qx[R.widx] = out.qx;
    }
    const int np = p0 + a.L + tid;
    if (np < a.N) entering = init_token(a.seed, b, np, n);
  }
  __syncthreads();
  if (!sm.last) return;
  // nothing below may be moved above the ticket read (the barrier orders the other threads)
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  if (!EXTRA && wave * kWave >= live) return;              // (the statistics below need every wavefront)
  int yy = -1, gg = -1;
  if (tid < live) {
    yy = __hip_atomic_load(&a.y[base + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (GS) gg = __hip_atomic_load(&a.g[base + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // every wavefront reads all accept bits (a window has at most 256 positions): no exchange, no barrier
  uint8_t kk[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int s = c * kWave + lane;
    kk[c] = 1;
    if (c * kWave < live)                                  // uniform
      kk[c] = __hip_atomic_load(&a.k[base + min(s, live - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  int first_rej = live;                                    // (a lane past the end repeats the last bit)
#pragma unroll
  for (int c = 3; c >= 0; --c) {
    const unsigned long long m = __builtin_amdgcn_ballot_w64(kk[c] == 0);
    if (m != 0ull) first_rej = min(c * kWave + __builtin_ctzll(m), live - 1);
  }
  const int acc = min(first_rej + 1, live);
  if (tid < acc) a.out[static_cast<size_t>(b) * a.N + p0 + tid] = a.v_lo + yy;
  const bool stats = EXTRA && a.diag != nullptr;
  const int ring = R.it % 3;
  if (stats) {
    // the drafts this iteration started with, by ring slot, and where its window started
    if (tid < a.L) a.xhist[(static_cast<size_t>(ring) * a.B + b) * a.L + tid] = a.X[base + tid];
    if (tid == 0) a.phist[ring * a.B + b] = p0;
    if (tid < 6) sm.hamm[tid] = 0;
    __syncthreads();                 // slot tid is rewritten by another thread below
  }
  if (tid < live) {
    // survivors: the MRS output is the coupled redraft (pi_MC); under pi_GS, or when the
    // alpha-coupling switch chose the independent redraft, it is the row's Gumbel-max draw
    const bool survives = tid >= acc;
    const int next = survives ? ((GS && gg >= 0) ? gg : yy) : entering;
    a.age_w[base + slot] = survives ? age_old + 1 : 0;
    a.X[base + slot] = next;
    if (stats) sm.xnew[slot] = next;
  }
  if (tid == 0) {
    a.accept_len[b] = acc;
    a.pos[b] = p0 + acc;
    a.iter[b] = R.it + 1;
    a.verified[b] = verified_old + live;
    a.ticket[b] = 0;
  }
  if (stats) {
    // Hamm(t + 1 - n, t + 1), n = 1..3 (Sec. 5.3 "Multi-Step Behavior"): the new drafts against
    // those of n iterations earlier over the positions that sit in both windows.  The thread of
    // ring slot tid owns the position j of the new window with j % L == tid.
    __syncthreads();
    const int pnew = p0 + acc;
    if (tid < a.L) {
      const int j = pnew + (tid - pnew % a.L + a.L) % a.L;
      if (j < a.N && j < p0 + a.L) {               // a position the step left in the window
        const int xn = sm.xnew[tid];
#pragma unroll
        for (int back = 0; back < 3; ++back) {
          const int ri = (ring + 3 - back) % 3;
          const int ph = back == 0 ? p0 : a.phist[ri * a.B + b];
          if (j >= ph && j < ph + a.L) {
            const int xo = a.xhist[(static_cast<size_t>(ri) * a.B + b) * a.L + tid];
            atomicAdd(&sm.hamm[2 * back + 1], 1);
            if (xo != xn) atomicAdd(&sm.hamm[2 * back], 1);
          }
        }
      }
    }
    __syncthreads();
    if (tid < 6) a.hamm[6 * b + tid] = sm.hamm[tid];
  }
}

// LDS of a workgroup: the histogram and, over it, what the wavefronts park (finish_regs); long_path's three
// arrays; full_path's key prefixes, histogram and list.
size_t lds_bytes_for(int n) {
  const size_t hist = kHistWords * sizeof(uint32_t);
  if (n <= kDirectMaxN / 2) return std::max(hist, static_cast<size_t>(NW) * wave_cap<PER_DIRECT / 2>() * 12);
  if (n <= kDirectMaxN) return std::max(hist, static_cast<size_t>(NW) * wave_cap<PER_DIRECT>() * 12);
  const size_t lists = std::max(hist, static_cast<size_t>(NW) * wave_cap<PER_LIST>() * 8);
  if (n > kRowKernelMaxN) return std::max(lists, hist + static_cast<size_t>(kKeptCap) * 8);
  return std::max(lists, static_cast<size_t>((n + 7) & ~7) * 2 + NBINS * sizeof(uint32_t) + kListCap * sizeof(uint16_t));
}

#ifndef SCD_ROW_DIRECT_ONLY
constexpr size_t kNucleusLds = static_cast<size_t>(NW) * kNucleusPark * 8;      // the histogram of masses lies under it
static_assert(kNucleusLds >= NBINS_P * 8 + kListCap * 4 && kNucleusLds + sizeof(Small) <= 160 * 1024, "nucleus_path: LDS");
static_assert(64 * 1024 >= kRowKernelMaxN, "nucleus_path: a row in registers");
#endif

inline size_t small_block(int rows) {
  return (static_cast<size_t>(rows) * kRowMaxTiles * 4 + 255) / 256 * 256;
}

}  // namespace

#ifndef SCD_ROW_DIRECT_ONLY
size_t row_candidate_bytes(int rows) {
  // per row: kListCap (id, logit) pairs, kRowMaxTiles list counts, kRowMaxTiles list cuts
  return static_cast<size_t>(rows) * kListCap * sizeof(uint2) + 2 * small_block(rows);
}

void row_candidate_layout(void* base_, int rows, uint2** cand, uint32_t** cnt, uint32_t** cut) {
  char* base = static_cast<char*>(base_);
  const size_t pairs = static_cast<size_t>(rows) * kListCap * sizeof(uint2);
  *cand = reinterpret_cast<uint2*>(base);
  *cnt = reinterpret_cast<uint32_t*>(base + pairs);
  *cut = reinterpret_cast<uint32_t*>(base + pairs + small_block(rows));
}

bool row_uses_candidates(int n, int top_k) {
  const bool filter = top_k > 0 && top_k < n;
  // at most kRowMaxTiles lists per row (longer rows are read whole).  top-k: a slice
  // emits about twice its share of the row's top_k logits, which has to fit its part of the lists.
  return n > kRowDirectMaxN && n <= kRowMaxTiles * kSliceMax && filter && top_k <= kListCap / 2;
}

#endif  // !SCD_ROW_DIRECT_ONLY

hipError_t LAUNCH_ROW(const RowArgs& a_in, hipStream_t s, size_t* lds_configured) {
  if (a_in.rows <= 0) return hipSuccess;
#ifdef SCD_ROW_DIRECT_ONLY
  if (a_in.n > kDirectMaxN) return hipErrorInvalidValue;     // these builds hold whole rows in registers only
#else
  // short rows: few wavefronts (figures at the head of this file)
  if (a_in.n <= kRowShortMaxN && a_in.L <= kRowShortMaxL)
    return launch_row_short(a_in, s, lds_configured ? lds_configured + 2 : nullptr);
  // more rows than compute units (256 on this chip), longer ones, the hot instances: the build
  // of this file whose workgroups pair up on a CU
  if (a_in.n <= kRowBatchedMaxN / 2 ||
      (a_in.rows > 256 && a_in.n <= kRowBatchedMaxN && a_in.top_p24 == 0u && a_in.diag == nullptr))
    return launch_row_batched(a_in, s, lds_configured ? lds_configured + 1 : nullptr);
#endif
  RowArgs a = a_in;
  a.q_uniform = 1.0f / static_cast<float>(a.n);
  a.recip_L = window_reciprocal(a.rows, a.N, a.L);
  // (mentioned first, these kernels lie first in the library: behind the list kernels, which shrank, all options on 32 x 8192 ids
  // took 136.7 us for 135.2 with the same instructions)
  using Kernel = void (*)(const int32_t*, const int32_t*, const uint2*, const uint32_t*, int, int, int, int, int, RowArgs);
#define SCD_ROW_INSTANCES(PATH) \
  {row_kernel<false, false, PATH>, row_kernel<true, false, PATH>, row_kernel<false, true, PATH>, row_kernel<true, true, PATH>}
  static const Kernel kernels[][4] = {
#if defined(SCD_ROW_SHORT)
      SCD_ROW_INSTANCES(kDirectTiny), SCD_ROW_INSTANCES(kDirectQuarter), {}, {}, SCD_ROW_INSTANCES(kPartsQuarter)
#elif defined(SCD_ROW_BATCHED)
      SCD_ROW_INSTANCES(kDirectTiny), SCD_ROW_INSTANCES(kDirectQuarter), SCD_ROW_INSTANCES(kDirectHalf),
      {row_kernel<false, false, kDirectWhole>, row_kernel<true, false, kDirectWhole>, nullptr, nullptr},
      SCD_ROW_INSTANCES(kPartsQuarter), SCD_ROW_INSTANCES(kPartsHalf)
#else
      {}, {}, SCD_ROW_INSTANCES(kDirectHalf), SCD_ROW_INSTANCES(kDirectWhole),
      {}, {}, SCD_ROW_INSTANCES(kLists),
      {row_kernel<false, false, kLong>, nullptr, nullptr, nullptr},
      {nullptr, nullptr, row_kernel<false, true, kNucleusHalf>, row_kernel<true, true, kNucleusHalf>},
      {nullptr, nullptr, row_kernel<false, true, kNucleusWhole>, row_kernel<true, true, kNucleusWhole>}
#endif
  };
#undef SCD_ROW_INSTANCES
  int P = 0, capE = 0;
  a.cand = nullptr;
#ifndef SCD_ROW_DIRECT_ONLY
  if (a.cand_base && row_uses_candidates(a.n, a.top_k)) {
    row_candidate_layout(a.cand_base, a.rows, &a.cand, &a.cand_cnt, &a.cand_cut);
    if (a.tiles > 0) {
      // the LM head's epilogue has filled the lists: one per column tile
      P = a.tiles;
      capE = kListCap / P;
    } else {
      const int per = list_width(a.n, a.top_k);
      if (per > 0) {
        P = (a.n + kWave * per - 1) / (kWave * per);
        capE = kListCap / P;
        hipLaunchKernelGGL(per == 16 ? list_kernel<16> : list_kernel<32>, dim3(a.rows, (P + kListWaves - 1) / kListWaves),
                           dim3(kListWaves * kWave), 0, s, a.pos, a.iter,
                           a.src ? a.src : a.mode == kRowRing ? nullptr : a.z_cur, a.mode, a.L, a.N, a.n, P, capE, a);
      } else {
        P = (a.n + kSliceMax - 1) / kSliceMax;                   // 3 .. kRowMaxTiles
        capE = kListCap / P;
        int rank = (2 * a.top_k + P - 1) / P;
        rank = rank < 64 ? 64 : rank;
        if (rank > capE * 4 / 5) rank = capE * 4 / 5;
        if (a.rows * P > 512)
          hipLaunchKernelGGL(slice_kernel<512>, dim3(a.rows * P), dim3(512), 0, s, a.pos, a.iter, a.mode, a.L, a.N, P,
                             capE, rank, a);
        else
          hipLaunchKernelGGL(slice_kernel<THREADS>, dim3(a.rows * P), dim3(THREADS), 0, s, a.pos, a.iter, a.mode, a.L,
                             a.N, P, capE, rank, a);
      }
      if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
  }
#endif
#ifdef SCD_ROW_DIRECT_ONLY
  const size_t lds = lds_bytes_for(a.n), most = lds_bytes_for(kDirectMaxN);
#else
  const bool nucleus = a.n > kDirectMaxN && a.n <= kRowKernelMaxN && a.top_p24 != 0u && !(a.top_k > 0 && a.top_k < a.n);
  const size_t lds = nucleus ? kNucleusLds : lds_bytes_for(a.n);
  const size_t most = std::max({lds_bytes_for(kRowKernelMaxN), lds_bytes_for(kDirectMaxN), kNucleusLds});
#endif
  const bool gs = (a.gumbel || a.alpha < 1.0f) && a.g && a.mode != kRowSelectOnly;
  const bool extra = a.top_p24 != 0u || a.diag != nullptr;   // the instances with the optional parts
  // The dynamic-LDS limit is an attribute of the function on a device.  Every context asks
  // for the same value, the largest any row needs, once (a context has one stream, hence one
  // device), so contexts of different row lengths cannot lower each other's limit.
  size_t none = 0;
  size_t& configured = lds_configured ? *lds_configured : none;
  if (configured == 0) {
    for (const auto& row : kernels)
      for (Kernel f : row)
        if (f)
          if (hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 static_cast<int>(most));
              e != hipSuccess)
            return e;
    configured = most;
  }
#ifdef SCD_ROW_DIRECT_ONLY
  int path = a.n < 4 ? kDirectTiny : a.n <= kDirectMaxN / 4 ? kDirectQuarter : a.n <= kDirectMaxN / 2 ? kDirectHalf : kDirectWhole;
#else
  int path = a.n <= kDirectMaxN / 2 ? kDirectHalf : a.n <= kDirectMaxN ? kDirectWhole
                   : nucleus ? (a.n <= 32 * THREADS ? kNucleusHalf : kNucleusWhole) : a.n <= kRowKernelMaxN ? kLists : kLong;
#endif
  if (a.part) {
    const bool quarter = path == kDirectQuarter;
    if (!(quarter || path == kDirectHalf) || !(a.ksplit == 2 || a.ksplit == 4 || (quarter && a.ksplit == 8)))
      return hipErrorInvalidValue;                   // sums that no instance adds up
    path += kPartsQuarter - kDirectQuarter;
  }
  const Kernel kernel = kernels[path][(gs ? 1 : 0) + (extra ? 2 : 0)];
  if (!kernel) return hipErrorInvalidValue;          // long rows with options: refused when the context is created
  hipLaunchKernelGGL(kernel, dim3(a.rows), dim3(THREADS), lds, s, a.pos, a.iter, a.cand, a.cand_cnt, a.mode, a.L, a.N, P, capE,
                     a);
  return hipGetLastError();
}

}  // namespace scd
