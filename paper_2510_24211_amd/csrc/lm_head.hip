// LM head of the window ("Evaluate" step of the SCD / SJD algorithms):
//   logit[m, v] = sum_k h[m, k] * W[v, k]      bf16 x bf16 -> fp32 (MFMA)
// with the first logit processors fused into the epilogue (Sec. 4.3 defines
// p^(t) after post-processing; Sec. 5.1 gives the guidance mix):
//   z = fl(fl((1+lambda) * c) - fl(lambda * u)),   z <- z / tau
// Only the allowed vocabulary rows of W are streamed (the mask to -inf of the
// other ids is realised by never forming their columns).
//
// gfx950 mapping.  The contraction is skinny: M = B*C*L rows (1..1024) against n = |allowed| columns
// (1k..128k) over d = 1k..4k: a stream over W for few rows, a GEMM for many.  choose() picks among
//   * lm_head_tile_kernel: LDS-staged tiles fed by LDS-direct loads (see there); most shapes.
//   * lm_head_splitk_kernel (few rows, few columns): a workgroup owns only 32 columns, so that enough of
//     them exist; its KS wavefronts take a 1/KS part of k each and stage their own W and h tiles
//     PRIVATELY: coalesced 16-byte loads (8 lanes cover one 128-byte row segment), D k-tiles ahead in
//     registers, parked in LDS (pitch 144 bytes against bank conflicts) and read back in the operand layout
//     of v_mfma_f32_32x32x16_bf16 (lane l: row l%32, k-group l/32, 8 consecutive k); no barrier in the loop.
//     The partial sums are added in wavefront order through LDS at the end (a fixed order: deterministic).
//   * lm_head_kernel (32 rows without guidance on long streams; tiny d): NW wavefronts take 32 neighbouring
//     columns each with private W staging as above and SHARE the h tile through LDS (double buffered, one
//     barrier per h tile).
// Common to all: window rows are packed into blocks of 32 (p = b * L + s), a block's cond and uncond tiles
// live in the same lanes, so the guidance mix needs no data movement; every workgroup walks k cyclically
// from its own starting tile: rows of W are d*2 bytes apart, and without the rotation all of the chip asks for
// the same address bits at the same time and camps on a few channels.
#include "scd_device.h"
#include "scd_kernels.h"

#include <hip/hip_ext.h>

#include <stdio.h>

#include <utility>

namespace scd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
// 16-byte register value; a native vector (the HIP struct type is copied with memcpy,
// which keeps arrays of it in scratch memory)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One 16-byte piece of W.  NT: non-temporal load -- the line is not kept in the caches it
// passes.  A slice of W that cannot stay in the 256 MB memory-side cache until the next step
// only evicts what could (the hidden rows in L2, the logits): streaming it past the caches
// took the full-vocabulary LM head from 96 to 87 us.  A slice that fits (C2: 67 MB) is served
// from that cache step after step and loses 3 us when loaded this way.
template <bool NT>
__device__ __forceinline__ u32x4 load_w(const u32x4* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

constexpr int BK = 64;          // k elements per W tile (128 bytes per row)
constexpr int PITCH = BK + 8;   // LDS row pitch in bf16 elements (144 bytes)

struct TrueT { static constexpr bool value = true; };
struct FalseT { static constexpr bool value = false; };
template <int N>
struct IntT { static constexpr int value = N; };

__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }
// Also a boundary for the machine scheduler, which otherwise treats loads of never-written
// global memory as freely movable and may sink a prefetch down to its use.
__device__ __forceinline__ void hard_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Which rows of W (= columns of z) a workgroup works on.  Workgroup ids go round robin over
// the 8 XCDs.  Read bandwidth on this chip is markedly higher when every XCD keeps to its own
// residue class of 128 KB address blocks (block number mod 8 == XCD; measured: 5.8 against
// 4.5 TB/s for the same bytes otherwise).  So when a row of W divides 128 KB, rows are dealt
// out in groups of G = 128 KB / row bytes consecutive rows: group g (rows g*G .. g*G+G-1)
// belongs to XCD (g + rot) mod 8, where rot places group 0 in the class of the block that
// holds most of it, and the workgroups of an XCD take its rows in order.  Otherwise
// (gshift < 0) workgroup tile t simply owns rows t * BN .. t * BN + BN - 1.
struct RowMap {
  int gshift;   // log2 G, or -1
  int rot;      // residue class of group 0
};
// Row of W for position `local` of workgroup tile jt of XCD xcd; >= n: no such row.  Rows grow
// with `local`.
__device__ __forceinline__ int mapped_row(const RowMap& m, int xcd, int jt, int BN, int local) {
  if (m.gshift < 0) return (jt * 8 + xcd) * BN + local;
  const int idx = jt * BN + local;                        // idx-th row owned by this XCD
  const int g = ((idx >> m.gshift) << 3) + ((xcd - m.rot) & 7);
  return (g << m.gshift) + (idx & ((1 << m.gshift) - 1));
}

template <int RBW, int C, int NWV>
struct Cfg {
  static constexpr int NW = NWV;                  // wavefronts per workgroup
  static constexpr int THREADS = NW * 64;
  static constexpr int NBLK = RBW * C;            // accumulator tiles per wavefront
  static constexpr int HROWS = NBLK * 32;         // h rows per tile
  static constexpr int D = 4;                     // W tiles in flight per wavefront (registers)
  static constexpr int DH = 2;                    // h tiles in flight (registers)
  static constexpr int HT = NBLK <= 2 ? 2 : 1;    // W tiles per shared h tile
  static constexpr int BKH = BK * HT;
  static constexpr int PITCH_H = BKH + 8;
  static constexpr int BN = NW * 32;              // columns per workgroup
  static constexpr int W_LDS = NW * 32 * PITCH;   // elements
  static constexpr int H_LDS = 2 * HROWS * PITCH_H;
  static constexpr int LDS_BYTES = (W_LDS + H_LDS) * 2;
};

// Window rows are packed: row p = b * L + s of the B * L rows, blocks of 32 whatever the window length.
// row_dest: where window row p is stored, as a row of z [2, B, L] (ring slot (pos[b] + s) % L of half
// iter[b] & 1 when the decode state is given, else row p), or -1 if it is not live.  The kernels leave it
// in a table in LDS.  The two words of the state are fetched ahead of everything else and without a branch
// (from h where there is no state), so that nothing waits for them before they are used.
struct RowState {
  int p, b, p0, it;
};
__device__ __forceinline__ RowState row_state(const LmHeadArgs& a, int p) {
  const int q = min(p, a.B * a.L - 1);
  RowState r{p, q / a.L, 0, 0};
  const int32_t* const any = reinterpret_cast<const int32_t*>(a.h);
  r.p0 = (a.pos ? a.pos : any)[a.pos ? r.b : 0];
  r.it = (a.iter ? a.iter : any)[a.iter ? r.b : 0];
  return r;
}
__device__ __forceinline__ int row_dest(const LmHeadArgs& a, const RowState& r) {
  if (r.p >= a.B * a.L) return -1;
  if (!a.pos) return r.p;
  const int s = r.p - r.b * a.L, par = a.iter ? (r.it & 1) : 0;
  return s < a.N - r.p0 ? (par * a.B + r.b) * a.L + (r.p0 + s) % a.L : -1;
}
// First h row (of [B, C, L]) of the sequence that holds window row p.  A workgroup addresses its h rows from
// there: the whole of h may exceed the 4 GiB that a 32-bit offset reaches.
__device__ __forceinline__ int first_h_row(int p, int C, int L) { return p / L * C * L; }
// h row (of [B, C, L]) of row r < 32 of the block that starts at window row p0 (uniform; the last row where
// there is none: its results are not stored).  Windows of 32 or more positions end at most once in a block.
__device__ __forceinline__ int h_row(int p0, int r, int c, int C, int L, int rows) {
  int b = p0 / L, s = p0 - b * L + min(r, rows - 1 - p0);
  if (L >= 32) {
    const bool next = s >= L;
    b += next ? 1 : 0;
    s -= next ? L : 0;
  } else {
    const int w = s / L;
    b += w;
    s -= w * L;
  }
  return (b * C + c) * L + s;
}

template <int C>
__device__ __forceinline__ float processed_logit(const LmHeadArgs& a, float c, float u) {
  return scd::processed_logit<C>(a.lam, a.one_plus_lam, a.tau, c, u);
}
// A logit on its way to the ring.  THROUGH: written through the L2.  Every kernel stores its logits at its end; left in the
// L2 they are written back when others need the room, or all together behind the last workgroup.  Where W is streamed past
// the caches in several rounds of workgroups that costs most: four steps of one sequence x 32 x 131072 ids over 4096
// 777 -> 743 us, 32 x 101632 over 2048 alone 81 -> 74.5; of 32 x 16384 over 1280 (split kernel) 97.7 -> 96.9; no gain in the
// other kernels (sixteen x 32 x 8192 from 316 -> 311 to 328 -> 329).  Only where the 32 columns that a half wavefront
// stores are whole 128-byte lines (through_lines): lines written in two parts cost more than they save (60 rows x 51285
// ids over 2048 42.1 -> 43.5).  Nor where tile_candidates stores 16 bytes per lane (65536 ids 397 -> 399).
template <bool THROUGH>
__device__ __forceinline__ void store_logit(float* p, float z) {
  if constexpr (THROUGH) __hip_atomic_store(p, z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = z;
}
__device__ __forceinline__ bool through_lines(const LmHeadArgs& a) { return (a.n & 31) == 0; }
template <class F>
__device__ __forceinline__ void with_bool(bool b, F&& f) {
  if (b) f(TrueT{});
  else f(FalseT{});
}
// Epilogue of a wavefront that holds whole sums.  Element j of lane (ln, lg) is row
// (j/4)*8 + lg*4 + j%4, column ln of the 32x32 tile.  zout takes the processed logits.
// table: row_dest of the workgroup's RBW * 32 window rows.  v: this lane's column, `there` if it exists.
template <int RBW, int C>
__device__ __forceinline__ void epilogue(const LmHeadArgs& a, const f32x16 (&acc)[RBW * C], const int* table, int64_t v,
                                         bool there, int lg, float (&zout)[RBW][16]) {
#pragma unroll
  for (int rbw = 0; rbw < RBW; ++rbw) {
    int4 to[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) to[g] = *reinterpret_cast<const int4*>(&table[rbw * 32 + g * 8 + lg * 4]);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int4 t = to[j >> 2];
      const int row = (j & 3) == 0 ? t.x : (j & 3) == 1 ? t.y : (j & 3) == 2 ? t.z : t.w;
      zout[rbw][j] = processed_logit<C>(a, acc[rbw * C][j], acc[rbw * C + C - 1][j]);
      if (row >= 0 && there) a.z[static_cast<int64_t>(row) * a.n + v] = zout[rbw][j];
    }
  }
}

// ---- per-tile top-k candidates (first half of the top-k selection, fused into the epilogue) ----
// A workgroup that owns COLS = 256 or 128 neighbouring columns parks its processed logits in LDS as a tile
// zt[row][COLS + 8] and every wavefront then reduces some rows of it: of the row's COLS
// logits it emits the `cap` largest or a few less as (id, logit) pairs in a FIXED order (lane, then column within
// the lane), their number, and the cut = the smallest emitted logit (as a key): every logit of
// the tile row that was not emitted lies strictly below it.  The row kernel selects the K-th largest
// among the emitted logits of all tiles and accepts it only if it is not below any tile's cut (then no
// logit that was not emitted can reach it): exact, and certified per row.
//   The emitted set is found on a monotone 7-bit image of the logits, linear between the tile row's mean (only
// what lies above it can be among the largest, unless the row is lopsided) and its largest (equal images: both
// emitted or neither), by counting it: one LDS histogram of 128 bins per row, and the lowest bin whose upper set
// holds at most `cap` logits (a bin near the cut holds about one logit, so 23 of 24 slots are used).  Where the
// bins are wide against the spread of the logits (one far logit is enough) the list would come
// out short or empty: if more than kTileSlack slots stay free, the bin below the cut is counted again on an image
// of its own range (refine_cut).  If more than `cap` logits tie at the top (or a logit is not finite, which
// collapses the image) the tile reports an overflowing count and the row kernel reads the row whole.
//   Bound by the instructions of a CU: with one or two wavefronts per SIMD nothing else runs meanwhile.  Four tile
// rows lie side by side in a wavefront, a row of 16 lanes each: reductions are four lane exchanges for four rows at once,
// and what is once per row (range, cut, offsets) is once per four: about 130 instructions per tile row.  z is stored from here,
// 16 bytes per lane.  Against a whole wavefront per tile row and 4-byte stores of z, four steps of two sequences
// x 64 positions x 64000 ids over 4096 take 590 us for 626, of one sequence x 32 x 65536 398 for 409, of eight x 32 x
// 65536 over 2048 without guidance 507 for 526 (tiles of 256 x 256 in two passes: the second one's logits spill).
constexpr int kTilePad = 8;                 // floats: rows 4 apart fall into disjoint banks
constexpr int kTileBins = 128;
constexpr int kTileRows = 4;                // rows that a wavefront reduces side by side
constexpr int kTileLanes = kWave / kTileRows;
constexpr int kTileBelow = kTileLanes;      // words in front of a row's bins, for logits below the first one
constexpr int kTileHistRow = kTileBelow + kTileBins;
constexpr int kTileHist = kTileRows * kTileHistRow * 4;   // LDS bytes per wavefront
static_assert(kTileLanes == 16 && kTileBins % (4 * kTileLanes) == 0 && kTileHistRow % 4 == 0, "a DPP row per tile row");

// Reductions over the 16 lanes of a tile row, in every lane.
template <class T, class F>
__device__ __forceinline__ T tile_row_fold(T v, F&& f) {
  static_assert(sizeof(T) == 4, "one register");
  auto other = [&](auto ctrl) { return __builtin_bit_cast(T, dpp_u32<decltype(ctrl)::value>(__builtin_bit_cast(uint32_t, v))); };
  v = f(v, other(IntT<kDppXor1>{}));
  v = f(v, other(IntT<kDppXor2>{}));
  v = f(v, other(IntT<kDppHalfMirror>{}));
  return f(v, other(IntT<kDppMirror>{}));
}
__device__ __forceinline__ float tile_row_max(float v) {
  return tile_row_fold(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float tile_row_min(float v) {
  return tile_row_fold(v, [](float a, float b) { return fminf(a, b); });
}
__device__ __forceinline__ float tile_row_sum(float v) {
  return tile_row_fold(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ int tile_row_sum(int v) {
  return tile_row_fold(v, [](int a, int b) { return a + b; });
}

// The largest image is below kTileBins: scale times the range, rounding included.  0 for an empty range; kept finite
// for ranges of a few denormal numbers.
__device__ __forceinline__ float tile_scale(float range) {
  return range > 0.f ? fminf(__builtin_amdgcn_rcpf(range) * (kTileBins - 1.01f), 3.0e38f) : 0.f;
}
// Per tile row: the lowest bin whose upper set holds at most `room` of the counted logits (kTileBins: not even
// the last one's does).  A lane reads kTileBins / 16 bins.
__device__ __forceinline__ void zero_tile_bins(uint32_t* bins, int l) {
#pragma unroll
  for (int j = 0; j < kTileBins / kTileLanes; j += 4)
    *reinterpret_cast<uint4*>(&bins[l * (kTileBins / kTileLanes) + j]) = make_uint4(0u, 0u, 0u, 0u);
}
__device__ __forceinline__ int find_cut(const uint32_t* bins, int l, int room) {
  constexpr int PER = kTileBins / kTileLanes;
  int c[PER], above = 0;
#pragma unroll
  for (int j = 0; j < PER; j += 4) {
    const uint4 t = *reinterpret_cast<const uint4*>(&bins[l * PER + j]);
    c[j] = static_cast<int>(t.x); c[j + 1] = static_cast<int>(t.y);
    c[j + 2] = static_cast<int>(t.z); c[j + 3] = static_cast<int>(t.w);
    above += (c[j] + c[j + 1]) + (c[j + 2] + c[j + 3]);
  }
  above += dpp_i32<kDppRowShl + 1>(above);          // logits in this lane's bins and those of the lanes behind
  above += dpp_i32<kDppRowShl + 2>(above);
  above += dpp_i32<kDppRowShl + 4>(above);
  above += dpp_i32<kDppRowShl + 8>(above);
  int cut = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    cut += above > room ? 1 : 0;
    above -= c[j];
  }
  return tile_row_sum(cut);
}
// bin[e] >= cut: the logit is emitted.  Where more than kTileSlack slots of a tile row stay free, the logits of the
// bin below the cut (more than there are free slots) are counted on an image of
// their own range, and those of its upper bins are lifted above every cut; again on the next bin while
// more than kTileSlack slots are free and the members differ (each round resolves the range 127 times finer).
// `may`: this lane's row is live and finite.
constexpr int kTileLifted = 2 * kTileBins;
template <int E>
__device__ __forceinline__ void refine_cut(const float (&v)[E], int (&bin)[E], int cut, int cap, bool may, uint32_t* bins, int l) {
  uint32_t in = 0u;                                      // a bit per logit
  int taken = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    in |= (cut > 0 ? bin[e] == cut - 1 : bin[e] < 0 && bin[e] >= -kTileBelow) ? 1u << e : 0u;
    taken += bin[e] >= cut ? 1 : 0;
  }
  int total = tile_row_sum(taken);
#pragma unroll 1
  for (int round = 0; round < 4; ++round) {
    float mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool is = (in >> e & 1u) != 0u;
      mx = is ? fmaxf(mx, v[e]) : mx;
      mn = is ? fminf(mn, v[e]) : mn;
    }
    const float hi = tile_row_max(mx), lo = tile_row_min(mn);
    const bool go = may && total < cap - kTileSlack && hi > lo;      // else: full enough, or they tie
    if (__builtin_amdgcn_ballot_w64(go) == 0ull) return;
    const float scale = tile_scale(hi - lo);
    zero_tile_bins(bins, l);
    compiler_fence();
    int image[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      image[e] = static_cast<int>(__builtin_amdgcn_fmed3f((v[e] - lo) * scale, 0.f, kTileBins - 1.f));
      if (go && (in >> e & 1u) != 0u) atomicAdd(&bins[image[e]], 1u);
    }
    compiler_fence();
    const int part = find_cut(bins, l, cap - total);     // at least 1: all members are more than fit
    taken = 0;
    uint32_t next = 0u;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool is = go && (in >> e & 1u) != 0u;
      bin[e] = is && image[e] >= part ? kTileLifted : bin[e];
      taken += is && image[e] >= part ? 1 : 0;
      next |= is && image[e] == part - 1 ? 1u << e : 0u;
    }
    total += tile_row_sum(taken);
    in = next;
  }
}

// Rows q0 .. q0 + 3 of the tile, a row per 16 lanes; dest: where the lane's row is stored (row_dest) or -1, wrow: its
// window row (b * L + s); v0 = id of the tile's first column; tile / T = its index and the
// number of tiles per row.  hist: kTileHist bytes of this wavefront's own.  STORE: the logits are not in z yet.
// The rows of zt are spent behind this: they take the emitted pairs on their way to memory.
template <int COLS, bool STORE>
__device__ __forceinline__ void tile_candidates(const LmHeadArgs& a, float* zt, uint32_t* hist, int lane,
                                                int q0, int dest, int wrow, int v0, int tile, int T) {
  const int cap = a.cand_cap;
  constexpr int E = COLS / kTileLanes;                   // logits per lane: columns 64 k + 4 l .. + 3
  const int l = lane & (kTileLanes - 1), sub = lane / kTileLanes;
  const int nvalid = min(COLS, a.n - v0);                // columns of this tile that exist
  const bool live = dest >= 0;
  uint32_t* const bins = hist + sub * kTileHistRow + kTileBelow;
  float* const ztrow = zt + (q0 + sub) * (COLS + kTilePad);
  auto column = [&](int e) { return (e >> 2) * 64 + 4 * l + (e & 3); };
  float v[E];
  int bin[E];
#pragma unroll
  for (int k = 0; k < E / 4; ++k) {
    const float4 t = *reinterpret_cast<const float4*>(ztrow + 4 * l + 64 * k);
    v[4 * k] = t.x; v[4 * k + 1] = t.y; v[4 * k + 2] = t.z; v[4 * k + 3] = t.w;
  }
  zero_tile_bins(bins, l);
  float* const to = a.z + (static_cast<int64_t>(dest) * a.n + v0 + 4 * l);
  float range;
  // RAGGED: columns that do not exist (in the last tile of a row only)
  auto images = [&](auto is_ragged) {
    constexpr bool RAGGED = decltype(is_ragged)::value;
    auto there = [&](int e) { return !RAGGED || column(e) < nvalid; };
    if (STORE && live) {
#pragma unroll
      for (int k = 0; k < E / 4; ++k) {
        if (!RAGGED) {
          store4(to + 64 * k, v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (there(4 * k + j)) to[64 * k + j] = v[4 * k + j];
        }
      }
    }
    float mx = -INFINITY, sum = 0.f;
#pragma unroll
    for (int e = 0; e < E; e += 2) {
      mx = max3(mx, there(e) ? v[e] : -INFINITY, there(e + 1) ? v[e + 1] : -INFINITY);
      v[e] = there(e) ? v[e] : 0.f;
      v[e + 1] = there(e + 1) ? v[e + 1] : 0.f;
      sum += v[e];
      sum += v[e + 1];
    }
    // a NaN (or +inf next to -inf) among the lane's logits poisons their sum
    if (sum != sum && a.flags && live) atomicOr(a.flags, 1);
    const float mean = tile_row_sum(sum) * (RAGGED ? __fdiv_rn(1.f, static_cast<float>(nvalid)) : 1.f / COLS);
    range = tile_row_max(mx) - mean;
    const float scale = tile_scale(range), below = -1.f - static_cast<float>(l);
    // What lies below the bins is counted in the words in front of them, far below in the lane's own (half of the
    // lanes would add to one word otherwise).
#pragma unroll
    for (int e = 0; e < E; ++e) {
      bin[e] = static_cast<int>(__builtin_amdgcn_fmed3f((v[e] - mean) * scale, below, kTileBins - 1.f));
      if (RAGGED) bin[e] = there(e) ? bin[e] : -1 - l;
      atomicAdd(&bins[bin[e]], 1u);
    }
    if (RAGGED) {                                        // counted; from here on never emitted, or all of the others
#pragma unroll
      for (int e = 0; e < E; ++e) bin[e] = !there(e) ? -kTileLifted : nvalid <= cap ? kTileLifted : bin[e];
    }
  };
  // LDS operations of a wavefront are performed in order: the zeroing above, the counting, the reading
  compiler_fence();
  if (nvalid == COLS) images(FalseT{});
  else images(TrueT{});
  compiler_fence();
  const int cut = find_cut(bins, l, cap);
  int mine, incl, total;
  auto offsets = [&]() {                                 // emitted logits of this lane, up to it, of the tile row
    mine = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) mine += bin[e] >= cut ? 1 : 0;
    incl = mine + dpp_i32<kDppRowShr + 1>(mine);
    incl += dpp_i32<kDppRowShr + 2>(incl);
    incl += dpp_i32<kDppRowShr + 4>(incl);
    incl += dpp_i32<kDppRowShr + 8>(incl);
    total = tile_row_sum(mine);
  };
  offsets();
  const bool may = live && range < INFINITY;             // (no NaN)
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(may && total < min(nvalid, cap - kTileSlack)) != 0ull, 0)) {
    refine_cut<E>(v, bin, cut, cap, may, bins, l);
    offsets();
  }
  // The pairs are put in order in the row's part of zt (what is not emitted goes to a place of the lane's own behind
  // them: a branch per logit takes longer) and leave it 16 at a time.
  constexpr int PAIRS = (COLS + kTilePad) / 2;
  static_assert(kRowListCap / (kRowDirectMaxN / COLS + 1) <= PAIRS - kTileLanes, "the longest list of the shortest row");
  uint2* const pairs = reinterpret_cast<uint2*>(ztrow);
  compiler_fence();
  int at = incl - mine;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const bool take = bin[e] >= cut;
    pairs[take ? at : PAIRS - kTileLanes + l] = make_uint2(static_cast<uint32_t>(v0 + column(e)), __float_as_uint(v[e]));
    at += take ? 1 : 0;
  }
  compiler_fence();
  uint2* const dst = a.cand + (static_cast<size_t>(wrow) * kRowListCap + static_cast<size_t>(tile) * cap);
  float vmin = INFINITY;
  for (int i = l; i < cap; i += kTileLanes) {
    const uint2 t = i < total ? pairs[i] : make_uint2(kNoId, __float_as_uint(INFINITY));
    if (live) dst[i] = t;
    vmin = fminf(vmin, __uint_as_float(t.y));
  }
  vmin = tile_row_min(vmin);                             // smallest emitted logit
  if (live && l == 0) {
    const size_t slot = static_cast<size_t>(wrow) * T + tile;
    a.cand_cnt[slot] = total > 0 ? static_cast<uint32_t>(total) : static_cast<uint32_t>(cap) + 1u;   // > cap: overflow
    a.cand_cut[slot] = total == nvalid ? 0u : zkey(vmin);    // 0: the whole tile row is emitted
  }
}

template <int RBW, int C, int NWV, bool NT>
__global__ __launch_bounds__((Cfg<RBW, C, NWV>::THREADS)) void lm_head_kernel(
    const LmHeadArgs a, const int VT, const int MT) {
  using K = Cfg<RBW, C, NWV>;
  constexpr int NBLK = K::NBLK, HROWS = K::HROWS, D = K::D, DH = K::DH, HT = K::HT;
  constexpr int THREADS = K::THREADS;
  __shared__ __attribute__((aligned(16))) unsigned char lds_raw[K::LDS_BYTES];
  uint16_t* const Ws_all = reinterpret_cast<uint16_t*>(lds_raw);
  uint16_t* const Hs_all = Ws_all + K::W_LDS;

  // Workgroups with consecutive ids land on different XCDs (round robin over 8).  The
  // MT row-block tiles that share one slab of W get ids 8 apart, i.e. the same XCD and
  // the same L2.
  const int id = blockIdx.x;
  const int xcd = id % 8, jt = id / (8 * MT);
  const int vt = jt * 8 + xcd;
  const int mt = (id / 8) % MT;
  if (vt >= VT) return;
  const int v_base = vt * K::BN, v_left = a.n - v_base;   // first column; columns that exist from there
  const int p_base = mt * RBW * 32, rows = a.B * a.L;     // first window row; all of them
  __shared__ __attribute__((aligned(16))) int table[RBW * 32];

  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int ln = lane & 31;     // row (A) / column (B) inside a 32x32 tile
  const int lg = lane >> 5;     // k-group
  const int chunk = lane & 7;   // 16-byte chunk inside a 128-byte row segment
  const int lrow = lane >> 3;   // 0..7

  const int d = a.d;
  const int KT = (d + BK - 1) / BK;
  const int ntiles = KT;
  const int ntiles_pad = (ntiles + D - 1) / D * D;
  // Row tiles that share a slab of W, and column tiles that share the same h rows, read the same
  // bytes; with several row tiles (MT > 1: the h rows no longer fit one L2 beside the W stream)
  // all workgroups of an XCD therefore start at the same k, so that they meet in L2 (C3: 86 -> 82 us).
  const int rot = (MT > 1 ? xcd * 5 : vt * 5) % ntiles_pad;
  // logical tile t -> k-tile index; `valid` is false for the padding tiles of the rotation
  // and for prefetches past the end.  Loads are NEVER predicated (a predicated load is a
  // branch, and branches keep the scheduler from batching the loads): an invalid tile reads
  // tile 0 of W (finite weights) against an h tile that is forced to zero.
  auto ktile = [&](int t, bool& valid) {
    int r = t + rot;
    if (r >= ntiles_pad) r -= ntiles_pad;
    valid = t < ntiles_pad && r < ntiles;
    return valid ? r : 0;
  };

  uint16_t* const Ws = Ws_all + wave * 32 * PITCH;          // private W staging

  // ---- W: coalesced private loads, D tiles ahead -----------------------------------
  // 32-bit byte offsets from the workgroup's first row; rows past the end are clamped to the last
  // row (their columns are never stored), k past the end to the last 16-byte chunk.
  const char* const Wb = reinterpret_cast<const char*>(a.W) + static_cast<size_t>(v_base) * d * 2;
  uint32_t woff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    woff[i] = static_cast<uint32_t>(min(wave * 32 + lrow + 8 * i, v_left - 1)) * static_cast<uint32_t>(d) * 2u;
  const uint32_t kclamp = static_cast<uint32_t>(d - 8) * 2u;
  u32x4 wreg[D][4];
  auto wload = [&](int slot, int t) {       // logical tile index t
    bool valid;
    const int kt = ktile(t, valid);
    const uint32_t kb = min(static_cast<uint32_t>(kt * BK + chunk * 8) * 2u, kclamp);
#pragma unroll
    for (int i = 0; i < 4; ++i) wreg[slot][i] = load_w<NT>(reinterpret_cast<const u32x4*>(Wb + (woff[i] + kb)));
  };
  auto wstore = [&](int slot) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<u32x4*>(&Ws[(lrow + 8 * i) * PITCH + chunk * 8]) = wreg[slot][i];
  };

  // ---- h: shared tile, BKH = HT * 64 wide --------------------------------------------
  constexpr int CH = K::BKH / 8;                 // 16-byte chunks per h row
  constexpr int CHW = BK / 8;                    // 16-byte chunks per W tile width
  constexpr int RPP = THREADS / CH;              // rows covered per pass of the workgroup
  constexpr int HL = HROWS / RPP;                // loads per thread per h tile
  static_assert(HROWS % RPP == 0, "h tile must divide over the workgroup");
  const int hchunk = tid % CH, hr0 = tid / CH;
  const int h0 = first_h_row(p_base, C, a.L);
  const char* const Hb = reinterpret_cast<const char*>(a.h) + static_cast<size_t>(h0) * d * 2;
  uint32_t hoff[HL];
#pragma unroll
  for (int i = 0; i < HL; ++i) {
    const int rr = hr0 + RPP * i, blk = rr >> 5;  // tile row 0..HROWS-1
    hoff[i] = static_cast<uint32_t>(h_row(min(p_base + (blk / C) * 32, rows - 1), rr & 31, blk % C, C, a.L, rows) - h0) *
              static_cast<uint32_t>(d) * 2u;
  }
  u32x4 hreg[DH][HL];
  bool hkok[DH];
  // logical h tile st = logical W tiles st*HT .. st*HT+HT-1; after the rotation these
  // need not be neighbours in k (wrap-around), so every 64-wide part is placed on its own.
  // Loaded unconditionally from a clamped address, then zeroed where k is not real.
  auto hload = [&](int slot, int st) {
    bool valid;
    const int kt = ktile(st * HT + hchunk / CHW, valid);
    const int k = kt * BK + (hchunk % CHW) * 8;
    const bool kok = valid && k < d;
    const uint32_t kb = min(static_cast<uint32_t>(k) * 2u, kclamp);
#pragma unroll
    for (int i = 0; i < HL; ++i) hreg[slot][i] = *reinterpret_cast<const u32x4*>(Hb + (hoff[i] + kb));
    hkok[slot] = kok;
  };
  // the zeroing waits for the load, so it happens here, when the tile moves to LDS
  auto hstore = [&](int slot, int buf) {
    uint16_t* dst = Hs_all + buf * HROWS * K::PITCH_H;
#pragma unroll
    for (int i = 0; i < HL; ++i) {
      const u32x4 t4 = hreg[slot][i];
      *reinterpret_cast<u32x4*>(&dst[(hr0 + RPP * i) * K::PITCH_H + hchunk * 8]) =
          (hkok[slot] ? t4 : u32x4{0u, 0u, 0u, 0u});
    }
  };

  f32x16 acc[NBLK];
#pragma unroll
  for (int i = 0; i < NBLK; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;

  // MFMAs of one W tile against h tile `Hs_tile` at column offset koff.  The operands of
  // k-step kk + 1 are read from LDS before the MFMAs of k-step kk are issued, so that the
  // matrix pipe does not wait for an LDS round trip per instruction.
  auto compute = [&](const uint16_t* Hs_tile, int koff) {
    constexpr int KK = BK / 16;
    u32x4 bq[2], aq[2][NBLK];
    auto fetch = [&](int buf, int kk) {
      bq[buf] = *reinterpret_cast<const u32x4*>(&Ws[ln * PITCH + kk * 16 + lg * 8]);
#pragma unroll
      for (int i = 0; i < NBLK; ++i)
        aq[buf][i] = *reinterpret_cast<const u32x4*>(
            &Hs_tile[(i * 32 + ln) * K::PITCH_H + koff + kk * 16 + lg * 8]);
    };
    fetch(0, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk + 1 < KK) fetch((kk + 1) & 1, kk + 1);
      const bf16x8 bfrag = __builtin_bit_cast(bf16x8, bq[kk & 1]);
#pragma unroll
      for (int i = 0; i < NBLK; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, aq[kk & 1][i]),
                                                         bfrag, acc[i], 0, 0, 0);
      if (kk + 1 < KK) {                       // keep that order: reads of kk + 1, MFMAs of kk
        __builtin_amdgcn_sched_group_barrier(0x100, NBLK + 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, NBLK, 0);
      }
    }
  };

  // h tile st travels: registers (stage st % 2, loaded at the end of h tile st - 3), LDS
  // buffer st % 2 (moved at the end of h tile st - 1), consumed during h tile st.  One
  // barrier per h tile: it publishes the moved tile and ends the reads of the buffer that
  // the next move overwrites.
  static_assert(D % (2 * HT) == 0, "register stages of h must be static in the unrolled body");
#pragma unroll
  for (int j = 0; j < D; ++j) wload(j, j);
  hload(0, 0);
  hstore(0, 0);
  hload(1, 1);
  hload(0, 2);
  const RowState mine = row_state(a, p_base + tid);
  __syncthreads();
  // One pass over D tiles.  The last pass (PF false) issues no load that would fall past
  // the end: such a load would fetch real bytes a second time.
  auto body = [&](int t0, auto pf) {
    constexpr bool PF = decltype(pf)::value;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int t = t0 + j;
      const int st = t / HT;
      const int stage = (j / HT) & 1;            // == st & 1 because t0 / HT is even
      compiler_fence();
      wstore(j);
      if (PF) wload(j, t + D);
      compiler_fence();
      compute(Hs_all + stage * HROWS * K::PITCH_H, (j % HT) * BK);
      compiler_fence();
      if (j % HT == HT - 1 && (PF || j / HT + 1 < D / HT)) {
        hstore(stage ^ 1, stage ^ 1);            // h tile st + 1 -> the other LDS buffer
        if (PF || j / HT + 3 < D / HT) hload(stage ^ 1, st + 3);
        __syncthreads();
      }
    }
  };
  for (int t0 = 0; t0 < ntiles_pad - D; t0 += D) body(t0, TrueT{});
  if (tid < RBW * 32) table[tid] = row_dest(a, mine);     // published by the last pass's barriers
  body(ntiles_pad - D, FalseT{});

  float zv[RBW][16];
  epilogue<RBW, C>(a, acc, table, static_cast<int64_t>(v_base) + wave * 32 + ln, wave * 32 + ln < v_left, lg, zv);

  if constexpr (RBW == 1 && NWV == 8) {
    // ---- per-tile candidates for the row kernel (a.cand is uniform) --------------------------
    constexpr int PITCH_Z = K::BN + kTilePad, ZT = 32 * PITCH_Z;   // floats of the logit tile; the histograms follow
    static_assert(K::BN == 256 && K::LDS_BYTES >= ZT * 4 + NWV * kTileHist, "logit tile must fit");
    if (a.cand == nullptr) return;
    __syncthreads();                       // every wavefront is done with the staging buffers
    float* const zt = reinterpret_cast<float*>(lds_raw);
#pragma unroll
    for (int j = 0; j < 16; ++j) zt[((j >> 2) * 8 + lg * 4 + (j & 3)) * PITCH_Z + wave * 32 + ln] = zv[0][j];
    __syncthreads();
    uint32_t* const hist = reinterpret_cast<uint32_t*>(zt + ZT) + wave * (kTileHist / 4);
#pragma unroll 1
    for (int q0 = wave * 4; q0 < wave * 4 + 4; q0 += kTileRows) {
      const int row = q0 + lane / kTileLanes;
      tile_candidates<K::BN, false>(a, zt, hist, lane, q0, table[row], p_base + row, v_base, vt, VT);
    }
  }
}

// ---- many rows: LDS-staged tiles of HR h rows x BN columns, fed by LDS-direct loads -------------------
// With more than about 64 h rows per byte of W the matrix pipe carries real load and the work is a GEMM.
// A workgroup of 8 wavefronts owns HR h rows (HR / C window rows, cond and uncond) x BN columns and walks
// k in tiles of 64.  What is done against each of the limits that were met:
//   * Rows are packed: h rows of a tile are HR / C consecutive window rows p = b * L + s whatever the
//     window length (blocks of 32 per sequence would multiply 37 % padding at L = 20, 75 % at L = 8).
//   * W and h tiles go from memory straight into LDS (global_load_lds, 16 bytes per lane), SW / SH stages
//     deep, one to two tiles ahead, so no registers are spent on loads in flight.  A load instruction moves
//     8 rows of 128 bytes; lane l writes slot l % 8 of row l / 8 (the hardware's fixed layout) and
//     therefore READS chunk (l % 8) ^ ((row >> 1) & 7): operand reads are then free of bank conflicts
//     without padding.
//   * The loads are inline assembly that names no output register: the compiler, which cannot see which
//     LDS bytes such a load fills, otherwise waits for ALL loads in flight before the next LDS read.  The
//     waits are written out: s_waitcnt vmcnt counts a wavefront's own loads, the barrier that follows
//     publishes them to the others.
//   * One barrier per k-tile, in the middle of the last k-step: when it is passed the next tile is in
//     LDS, its first operands are read under the last MFMAs of this tile, and the stage just read is free.
//   * The loads of a tile are issued one by one between MFMAs: eight wavefronts issuing all of theirs after
//     the barrier queue at the CU's one address unit (16 clocks per instruction) with their MFMAs behind them
//     (256 x 128 tiles, 64 workgroups: 52 -> 43 us).
//   * A wavefront multiplies 64 x 128 or 64 x 64 (NC x NB accumulator tiles of 32 x 32): the LDS reads of a
//     k-tile take less than its MFMAs (by the counters 33 of 66 thousand cycles on 256 x 128 tiles, no bank conflicts).
//   * Small calls add k up in 4 or 8 partial sums (k_parts): every `per` k-tiles the accumulators are added to
//     whole sums and start again from zero.  In the register form of the MFMAs (launch bounds of 512: with one
//     wavefront per SIMD the compiler takes accumulation registers, and each fold copies them out and back)
//     this takes 0 to 6 % (64 rows with guidance x 2000 ids over 4096: 17.7 -> 18.8 us).
// What is left: on 1024 h rows x 8192 ids the matrix pipes are busy for 66 thousand cycles of the 96 that a CU has
// wavefronts, a third of the wavefronts' cycles pass at waits and barriers, and a quarter of the kernel lies before a
// CU's first and after its last wavefront.  Above it stands power: with real operands all 256 CUs sustain about 1.45 PFLOP/s
// (MFMAs alone, operands fixed in registers; 1.9 on zeros).  Against register-staged kernels:
// 1024 h rows x 8192 ids over 4096 84 -> 62 us (1.10 PFLOP/s; the vendor GEMM 66), 256 x 64000 148 -> 124
// without candidates (4.2 TB/s and 1.08 PFLOP/s at once), 128 x 65536 107 -> 88, 64 x 30000 71 -> 44,
// 120 packed rows x 51285 over 2048 63 -> 42.
template <int C_, int HR_, int BN_, int S_>
struct TileCfg {
  static constexpr int C = C_, HR = HR_, BN = BN_;
  static constexpr int NW = HR == 64 && BN == 128 ? 4 : 8;                  // wavefronts
  static constexpr int THREADS = NW * 64;
  static constexpr int CW = HR * BN <= 128 * 128 ? 32 : 64;                 // columns per wavefront
  static constexpr int NC = CW / 32;
  static constexpr int WCOL = BN / CW, WROW = NW / WCOL;
  static constexpr int RW = HR / WROW;               // h rows per wavefront
  static constexpr int NB = RW / 32;
  static constexpr int RB = NB / C;                  // blocks of 32 window rows per wavefront
  static constexpr int WR = HR / C;                  // window rows per workgroup
  static constexpr int WL = BN / 8 / NW, HL = HR / 8 / NW;   // loads per wavefront and k-tile
  static constexpr int WB = BN * 128, HB = HR * 128; // bytes per stage
  static constexpr int SW = S_, SH = HR == 256 && BN == 256 ? S_ - 1 : S_;   // stages
  static_assert(SW >= 3 && SH >= 2, "stages");
  static constexpr bool SPLITS = HR == 64 && BN == 128;      // may have k dealt over workgroups
  static constexpr bool PARTS = HR * BN < 256 * 256; // registers left for whole sums beside the partial ones
  static constexpr int STAGES = SW * WB + SH * HB;
  // epilogue: row table, then the logit tile of up to 128 window rows and the histograms
  static constexpr int ZROWS = WR < 128 ? WR : 128;
  static constexpr int TABLE = 1024;
  static constexpr int PITCH_Z = BN + kTilePad;
  static constexpr int EPI = TABLE + ZROWS * PITCH_Z * 4 + NW * kTileHist;
  static constexpr int LDS_BYTES = STAGES > EPI ? STAGES : EPI;
  static_assert(WCOL * WROW == NW && NB % C == 0 && WR * 4 <= TABLE && LDS_BYTES <= 160 * 1024, "tile shape");
};

// 16 bytes per lane from base + off (per lane) to LDS byte address lds + ADD + 16 * lane (lds uniform).  The
// LDS address travels in m0, a reserved register: the compiler warns that it does not save what a statement
// clobbers there.  It has nothing to save, but has to see that whatever it sets m0 for itself is set again behind.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool NT, int ADD>
__device__ __forceinline__ void load_lds16(uint64_t base, uint32_t off, uint32_t lds) {
  if constexpr (NT)
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 ::"s"(lds), "v"(off), "s"(base), "n"(ADD) : "memory", "m0", "scc");
  else
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 ::"s"(lds), "v"(off), "s"(base), "n"(ADD) : "memory", "m0", "scc");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_loads() {       // until at most N of this wavefront's loads are in flight
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(IntT<I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

template <int C, int HR, int BN, int S, bool NT>
__global__ __launch_bounds__(512) void lm_head_tile_kernel(const LmHeadArgs a, const int VT, const int MT, const int KS,
                                                            const int per) {
  using K = TileCfg<C, HR, BN, S>;
  constexpr int NC = K::NC, NB = K::NB, WL = K::WL, HL = K::HL, SW = K::SW, SH = K::SH;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[K::LDS_BYTES];
  // Workgroups with consecutive ids land on different XCDs; the MT row tiles that share a slab of W get
  // ids 8 apart: the same XCD, the same L2; so do the KS parts of k (1 unless the sums go to a.part).
  const int id = blockIdx.x, xcd = id % 8;
  int mt = (id / 8) % MT, kp = 0, vt = (id / (8 * MT)) * 8 + xcd;
  if constexpr (K::SPLITS) {
    if (KS > 1) {
      kp = (id / (8 * MT)) % KS;
      vt = id / (8 * MT * KS) * 8 + xcd;
    }
  }
  if (vt >= VT) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % K::WCOL, wr = wave / K::WCOL;
  const int ln = lane & 31, lg = lane >> 5;
  const int d = a.d, rows = a.B * a.L, p_base = mt * K::WR;
  const int v_left = a.n - vt * BN;                  // columns that exist from this tile's first
  // whole k-tiles of this part of k, its first, elements of the ragged one (the last part's)
  int kt0 = 0, KT = d / 64, dtail = d % 64;
  if constexpr (K::SPLITS) {
    if (KS > 1) {                                    // (a division is about thirty instructions ahead of the first load)
      const int all = KT;
      kt0 = all * kp / KS;
      KT = all * (kp + 1) / KS - kt0;
      if (kp < KS - 1) dtail = 0;
    }
  }
  const int rot = (MT > 1 ? xcd * 5 : vt * 5) % KT;  // where this workgroup's cyclic walk over k starts

  const RowState mine = row_state(a, p_base + tid);  // for the epilogue's row table

  // byte offsets of this lane's pieces; rows past the end read the last one (their results are not stored)
  auto piece_row = [&](int per_wave, int i) { return (wave * per_wave + i) * 8 + (lane >> 3); };
  auto piece_chunk = [&](int r) { return (lane & 7) ^ ((r >> 1) & 7); };
  const int h0 = first_h_row(p_base, C, a.L);
  uint32_t wo[WL], ho[HL];
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    const int r = piece_row(WL, i);
    wo[i] = static_cast<uint32_t>(min(r, v_left - 1)) * static_cast<uint32_t>(d) * 2u + piece_chunk(r) * 16;
  }
#pragma unroll
  for (int i = 0; i < HL; ++i) {
    // tile row r: block r / 32 holds the (cond, uncond) pair in turn, row r % 32 of its 32 window rows
    const int r = piece_row(HL, i), blk = r >> 5;
    ho[i] = static_cast<uint32_t>(h_row(min(p_base + (blk / C) * 32, rows - 1), r & 31, blk % C, C, a.L, rows) - h0) *
                static_cast<uint32_t>(d) * 2u + piece_chunk(r) * 16;
  }
  const uint64_t wbase = reinterpret_cast<uint64_t>(a.W) + static_cast<uint64_t>(vt) * BN * d * 2 + static_cast<uint32_t>(kt0) * 128u;
  const uint64_t hbase = reinterpret_cast<uint64_t>(a.h) + static_cast<uint64_t>(h0) * d * 2 + static_cast<uint32_t>(kt0) * 128u;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)lds));
  const uint32_t ldsW = lds0 + wave * WL * 1024, ldsH = lds0 + SW * K::WB + wave * HL * 1024;

  // Loads of the next k-tile of h and of W, one piece at a time (h first).  With one wavefront per SIMD a
  // k-tile of the small tiles is bound by instruction issue, so a piece is three instructions; COND: not
  // past the end of the walk.
  struct Walk {
    uint64_t at;          // the k-tile's column of the operand
    uint32_t lds;         // the stage it goes to
    int k, n;             // its index; tiles issued before it
  };
  Walk hw{hbase + static_cast<uint32_t>(rot) * 128u, ldsH, rot, 0}, ww{wbase + static_cast<uint32_t>(rot) * 128u, ldsW, rot, 0};
  auto advance = [&](Walk& w, uint64_t base, uint32_t first, uint32_t bytes, int stages) {
    w.k = w.k + 1 == KT ? 0 : w.k + 1;
    w.at = base + static_cast<uint32_t>(w.k) * 128u;
    w.lds = w.lds + bytes == first + bytes * stages ? first : w.lds + bytes;
    ++w.n;
  };
  auto piece = [&](auto qq, auto cond) {
    constexpr int q = decltype(qq)::value;
    constexpr bool COND = decltype(cond)::value;
    if constexpr (q < HL) {
      if (!COND || hw.n < KT) load_lds16<false, q * 1024>(hw.at, ho[q], hw.lds);
      if constexpr (q == HL - 1) advance(hw, hbase, ldsH, K::HB, SH);
    } else {
      if (!COND || ww.n < KT) load_lds16<NT, (q - HL) * 1024>(ww.at, wo[q - HL], ww.lds);
      if constexpr (q == HL + WL - 1) advance(ww, wbase, ldsW, K::WB, SW);
    }
  };
  auto load_h = [&]() { static_for<HL>([&](auto i) { piece(i, TrueT{}); }); };
  auto load_w = [&]() { static_for<WL>([&](auto i) { piece(IntT<HL + decltype(i)::value>{}, TrueT{}); }); };

  f32x16 acc[NC][NB], whole[NC][NB];                 // partial sums, and the sum of the finished ones
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      acc[c][i] = f32x16{};
      if constexpr (K::PARTS) whole[c][i] = f32x16{};
    }
  // step(t) for the k-tiles from t up to `last`, one partial sum after the other
  int t = 0, complete = per;                         // the partial sums are complete before this k-tile
  auto walk = [&](int last, auto&& step) {
    while (t < last) {
      const int stop = K::PARTS ? min(last, complete) : last;
#pragma unroll 1
      for (; t < stop; ++t) step(t);
      if constexpr (K::PARTS) {
        if (t < complete) return;
        complete += per;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            whole[c][i] += acc[c][i];
            acc[c][i] = f32x16{};
          }
      }
    }
  };
  // Operand sets in registers.  FLAT: one per k-step of a tile, each refilled from the next tile right after
  // its MFMAs, so that the LDS round trip is covered by three k-steps (two MFMAs each in these small tiles);
  // it takes a stage more.  Otherwise (tiles that fill LDS with three stages) two sets, one k-step ahead.
  constexpr bool FLAT = S >= 4;
  u32x4 bq[FLAT ? 4 : 2][NC], aq[FLAT ? 4 : 2][NB];
  auto fetch = [&](int q, uint32_t sw, uint32_t sh, int kk) {
    const uint32_t slot = ((kk * 2 + lg) ^ ((ln >> 1) & 7)) * 16;
    const unsigned char* const Wt = lds + sw + (wc * K::CW + ln) * 128 + slot;
    const unsigned char* const Ht = lds + SW * K::WB + sh + (wr * K::RW + ln) * 128 + slot;
#pragma unroll
    for (int c = 0; c < NC; ++c) bq[q][c] = *reinterpret_cast<const u32x4*>(Wt + c * 4096);
#pragma unroll
    for (int i = 0; i < NB; ++i) aq[q][i] = *reinterpret_cast<const u32x4*>(Ht + i * 4096);
  };
  // the MFMAs of one k-step on operand set q, with quarter Q of a k-tile's loads between them (Q = 4: none)
  constexpr int NM = NC * NB, NP = HL + WL;
  auto mma = [&](int q, auto quarter, auto cond) {
    constexpr int Q = decltype(quarter)::value;
    constexpr int P0 = Q < 4 ? NP * Q / 4 : 0, P1 = Q < 4 ? NP * (Q + 1) / 4 : 0;
    static_for<NM>([&](auto ii) {
      constexpr int I = decltype(ii)::value, c = I / NB, i = I % NB;
      acc[c][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, aq[q][i]),
                                                          __builtin_bit_cast(bf16x8, bq[q][c]), acc[c][i], 0, 0, 0);
      constexpr int A = P0 + (P1 - P0) * I / NM, E = P0 + (P1 - P0) * (I + 1) / NM;
      if constexpr (E > A) {
        __builtin_amdgcn_sched_barrier(0);
        static_for<E - A>([&](auto k) { piece(IntT<A + decltype(k)::value>{}, cond); });
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    __builtin_amdgcn_sched_barrier(0);
  };

  uint32_t sw = 0, sh = 0;                           // stages of the tile whose operands are read next
  auto next_stage = [&]() {
    sw = sw + K::WB == SW * K::WB ? 0 : sw + K::WB;
    sh = sh + K::HB == SH * K::HB ? 0 : sh + K::HB;
  };
  if constexpr (FLAT) {
    // Tile t: the barrier at its top says that tile t + 1 is in LDS and that every wavefront holds tile t's
    // operands, hence is done with the stage of tile t - 1, which takes the loads of tile t + S - 1.
    // wait_tile(left): until the tile that `left` tiles follow is there; of those S - 3 have been issued.
    auto wait_tile = [&](int left) {
      bool done = false;
      static_for<S - 2>([&](auto k) {
        constexpr int N = S - 3 - decltype(k)::value;
        if (!done && left >= N) {
          wait_loads<N * NP>();
          done = true;
        }
      });
    };
    static_for<S - 2>([&](auto) {
      load_h();
      load_w();
    });
    wait_tile(KT - 1);
    load_h();
    load_w();
    __builtin_amdgcn_s_barrier();
    hard_fence();
    static_for<4>([&](auto kk) { fetch(decltype(kk)::value, 0, 0, decltype(kk)::value); });
    hard_fence();
    auto tile = [&](auto quarter_of) {
      __builtin_amdgcn_s_barrier();
      hard_fence();
      next_stage();
      static_for<4>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        mma(k, IntT<decltype(quarter_of)::value ? k : 4>{}, FalseT{});
        fetch(k, sw, sh, k);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    walk(KT - S + 1, [&](int) {
      wait_loads<(S - 3) * NP>();
      tile(TrueT{});
    });
    walk(KT - 1, [&](int t) {                        // everything is on its way
      wait_tile(KT - 2 - t);
      tile(FalseT{});
    });
    static_for<4>([&](auto kk) { mma(decltype(kk)::value, IntT<4>{}, FalseT{}); });
  } else {
    // Window t of the loads ends at the barrier of tile t; it brings W of tile t + 2 and h of tile
    // t + SH - 1, h first (a stage is free once the barrier of the tile that it held is passed).  At the
    // barrier of tile t both parts of tile t + 1 have to be in LDS; what was issued after them may be in flight.
    constexpr int AHEAD = WL + (SH == 3 ? HL : 0);
    load_h();
    load_w();
    if constexpr (SH == 3) load_h();
    load_w();
    if (KT > 1) wait_loads<AHEAD>();
    else wait_loads<0>();
    __builtin_amdgcn_s_barrier();
    hard_fence();
    static_for<NP / 4>([&](auto i) { piece(i, TrueT{}); });
    fetch(0, 0, 0, 0);
    hard_fence();
    auto tile = [&](auto cond, bool more, bool next) {   // loads go on past this tile's barrier; a tile follows
      fetch(1, sw, sh, 1);
      __builtin_amdgcn_sched_barrier(0);
      mma(0, IntT<1>{}, cond);
      fetch(0, sw, sh, 2);
      __builtin_amdgcn_sched_barrier(0);
      mma(1, IntT<2>{}, cond);
      fetch(1, sw, sh, 3);
      __builtin_amdgcn_sched_barrier(0);
      mma(0, IntT<3>{}, cond);
      hard_fence();
      if (more) wait_loads<AHEAD>();
      else wait_loads<0>();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this tile's operands are in registers
      __builtin_amdgcn_s_barrier();
      hard_fence();
      next_stage();
      if (next) fetch(0, sw, sh, 0);
      hard_fence();
      mma(1, IntT<0>{}, cond);
      hard_fence();
    };
    walk(KT - 3, [&](int) { tile(FalseT{}, true, true); });
    walk(KT, [&](int t) { tile(TrueT{}, t + 2 < KT, t + 1 < KT); });
  }
  if (dtail != 0) {
    // the ragged k-tile on its own: chunks past the end read the last one of the row and are zeroed in h
    // (finite weights) by the wavefront that loaded them
    const int nch = dtail / 8;
    __syncthreads();                                 // every wavefront has its operands: the stages are free
#pragma unroll
    for (int i = 0; i < HL; ++i) {
      const int ch = piece_chunk(piece_row(HL, i));
      load_lds16<false, 0>(hbase + static_cast<uint32_t>(KT) * 128u, ho[i] - max(ch - (nch - 1), 0) * 16, ldsH + i * 1024);
    }
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int ch = piece_chunk(piece_row(WL, i));
      load_lds16<NT, 0>(wbase + static_cast<uint32_t>(KT) * 128u, wo[i] - max(ch - (nch - 1), 0) * 16, ldsW + i * 1024);
    }
    wait_loads<0>();
#pragma unroll
    for (int i = 0; i < HL; ++i)
      if (piece_chunk(piece_row(HL, i)) >= nch)
        *reinterpret_cast<u32x4*>(lds + SW * K::WB + (wave * HL + i) * 1024 + lane * 16) = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    for (int kk = 0; kk * 2 < nch; ++kk) {
      fetch(0, 0, 0, kk);
      mma(0, IntT<4>{}, FalseT{});
    }
  }

  if constexpr (K::PARTS) {
    if (per <= KT) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[c][i] += whole[c][i];
    }
  }

  if constexpr (K::SPLITS) {
    if (a.part) {                                    // uniform
      // ---- sums of this part of k, for the row kernel -----------------------------------------------
      float* const part = a.part + static_cast<int64_t>(kp) * C * rows * a.n;
      with_bool(through_lines(a), [&](auto through) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int row = p_base + (wr * K::RB + i / C) * 32 + (j >> 2) * 8 + lg * 4 + (j & 3);
            float* const to = part + (static_cast<int64_t>(i % C) * rows + row) * a.n + vt * BN + wc * K::CW + ln;
#pragma unroll
            for (int c = 0; c < NC; ++c)
              if (row < rows && wc * K::CW + c * 32 + ln < v_left) store_logit<decltype(through)::value>(to + c * 32, acc[c][i][j]);
          }
      });
      return;
    }
  }
  // ---- epilogue: guidance mix, temperature, z; then the per-tile candidates ---------------------------
  __syncthreads();                                   // every wavefront is done with the stages
  int* const table = reinterpret_cast<int*>(lds);    // (the stages take all of LDS: no table before)
  if (tid < K::WR) table[tid] = row_dest(a, mine);
  __syncthreads();
  // element j of a block: window row 8 * (j / 4) + 4 * lg + j % 4 of its 32, column ln
  if (a.cand == nullptr) {                           // uniform
    with_bool(NT && through_lines(a), [&](auto through) {
#pragma unroll
      for (int r = 0; r < K::RB; ++r) {
        int4 to[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) to[g] = *reinterpret_cast<const int4*>(&table[(wr * K::RB + r) * 32 + g * 8 + lg * 4]);
        const int v = wc * K::CW + ln;                // column of the tile
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int4 t = to[j >> 2];
          const int row = (j & 3) == 0 ? t.x : (j & 3) == 1 ? t.y : (j & 3) == 2 ? t.z : t.w;
          float* const zr = a.z + (static_cast<int64_t>(row) * a.n + vt * BN + v);
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const float z = processed_logit<C>(a, acc[c][r * C][j], acc[c][r * C + C - 1][j]);
            if (row >= 0 && v + c * 32 < v_left) store_logit<decltype(through)::value>(&zr[c * 32], z);
          }
        }
      }
    });
    return;
  }
  // the processed logits replace the cond sums; tile_candidates stores them from the tile in LDS, 16 bytes per lane
#pragma unroll
  for (int r = 0; r < K::RB; ++r)
#pragma unroll
    for (int j = 0; j < 16; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        acc[c][r * C][j] = processed_logit<C>(a, acc[c][r * C][j], acc[c][r * C + C - 1][j]);
  float* const zt = reinterpret_cast<float*>(lds + K::TABLE);
  uint32_t* const hist = reinterpret_cast<uint32_t*>(zt + K::ZROWS * K::PITCH_Z) + wave * (kTileHist / 4);
  constexpr int PASSES = K::WR / K::ZROWS;           // 128 window rows at a time
  constexpr int WROW_PASS = K::WROW / PASSES;        // wavefront rows that hold them
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    if (pass > 0) __syncthreads();
    if (wr / WROW_PASS == pass) {
#pragma unroll
      for (int r = 0; r < K::RB; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int j = 0; j < 16; ++j)
            zt[(((wr % WROW_PASS) * K::RB + r) * 32 + (j >> 2) * 8 + lg * 4 + (j & 3)) * K::PITCH_Z + wc * K::CW + c * 32 + ln] =
                acc[c][r * C][j];
    }
    __syncthreads();
    constexpr int PER_WAVE = K::ZROWS / K::NW;
    static_assert(PER_WAVE % kTileRows == 0, "rows per wavefront");
#pragma unroll 1
    for (int q0 = wave * PER_WAVE; q0 < (wave + 1) * PER_WAVE; q0 += kTileRows) {
      const int row = pass * K::ZROWS + q0 + lane / kTileLanes;
      const int dest = table[row];
      if (__builtin_amdgcn_ballot_w64(dest >= 0) == 0ull) continue;
      tile_candidates<BN, true>(a, zt, hist, lane, q0, dest, p_base + row, vt * BN, vt, VT);
    }
  }
}

// ---- narrow vocabularies: k split over the wavefronts of a workgroup ---------------------
template <int RBW, int C, int KS>
struct SplitCfg {
  static constexpr int NW = KS;
  static constexpr int THREADS = NW * 64;
  static constexpr int NBLK = RBW * C;
  static constexpr int HROWS = NBLK * 32;
  static constexpr int D = KS == 8 ? 2 : 4;       // W tiles in flight per wavefront
  static constexpr int DH = 2;                    // h tiles in flight per wavefront
  static constexpr int STAGE_BYTES = NW * (32 + HROWS) * PITCH * 2;
  static constexpr int RED_BYTES = NW * NBLK * 16 * 64 * 4;
  static constexpr int LDS_BYTES = STAGE_BYTES > RED_BYTES ? STAGE_BYTES : RED_BYTES;
};

template <int RBW, int C, int KS>
__global__ __launch_bounds__((SplitCfg<RBW, C, KS>::THREADS)) void lm_head_splitk_kernel(
    // plain leading arguments: the hardware preloads them into SGPRs at wavefront launch, so the
    // first loads do not wait for a fetch of the kernel-argument segment
    const uint16_t* const W_, const uint16_t* const h_, const int d_, const int n_, const int L_,
    const int rows, const int MT, const int rm_gshift, const int rm_rot, const LmHeadArgs a) {
  const RowMap rm{rm_gshift, rm_rot};
  using K = SplitCfg<RBW, C, KS>;
  constexpr int NBLK = K::NBLK, HROWS = K::HROWS, D = K::D, DH = K::DH, NWAVE = K::NW;
  __shared__ __attribute__((aligned(16))) unsigned char lds_raw[K::LDS_BYTES];
  const int id = blockIdx.x;
  const int xcd = id % 8, jt = id / (8 * MT);
  const int vt = jt * 8 + xcd;
  const int mt = (id / 8) % MT;
  if (mapped_row(rm, xcd, jt, 32, 0) >= n_) return;   // no row left for this tile
  const int p_base = mt * RBW * 32;                   // first window row
  __shared__ __attribute__((aligned(16))) int table[RBW * 32];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int ln = lane & 31, lg = lane >> 5, chunk = lane & 7, lrow = lane >> 3;
  const int d = d_;
  const int KT = (d + BK - 1) / BK;
  const int ktq = (KT + NWAVE - 1) / NWAVE;
  const int kt_begin = wave * ktq;
  const int ntiles = max(0, min(KT, kt_begin + ktq) - kt_begin);
  // the cyclic walk covers exactly the wavefront's tiles: the last pass of the loop below runs
  // only as many tiles as are left (C1: 5 tiles per wavefront are one pass of 4 and one of 1)
  const int rot = ntiles > 0 ? (vt * 5 + wave * 3) % ntiles : 0;
  auto ktile = [&](int t, bool& valid) {     // see lm_head_kernel: loads are never predicated
    int r = t + rot;
    if (r >= ntiles) r -= ntiles;
    valid = t < ntiles;
    return valid ? kt_begin + r : 0;
  };
  uint16_t* const Ws = reinterpret_cast<uint16_t*>(lds_raw) + wave * (32 + HROWS) * PITCH;
  uint16_t* const Hs = Ws + 32 * PITCH;

  const char* const Wb = reinterpret_cast<const char*>(W_);
  const char* const Hb = reinterpret_cast<const char*>(h_);
  const uint32_t kclamp = static_cast<uint32_t>(d - 8) * 2u;
  uint32_t woff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int v = mapped_row(rm, xcd, jt, 32, lrow + 8 * i);
    woff[i] = static_cast<uint32_t>(min(v, n_ - 1)) * static_cast<uint32_t>(d) * 2u;
  }
  u32x4 wreg[D][4];
  auto wload = [&](int slot, int t) {
    bool valid;
    const int kt = ktile(t, valid);
    const uint32_t kb = min(static_cast<uint32_t>(kt * BK + chunk * 8) * 2u, kclamp);
#pragma unroll
    for (int i = 0; i < 4; ++i) wreg[slot][i] = load_w<false>(reinterpret_cast<const u32x4*>(Wb + (woff[i] + kb)));
  };
  static_assert(D % DH == 0, "register stages of h must be static in the unrolled body");
#pragma unroll
  for (int j = 0; j < D; ++j) wload(j, j);      // on their way while the addresses of h are worked out
  constexpr int HL = HROWS / 8;                  // loads per lane per h tile
  uint32_t hoff[HL];
#pragma unroll
  for (int i = 0; i < HL; ++i) {
    const int rr = lrow + 8 * i, blk = rr >> 5;
    hoff[i] = static_cast<uint32_t>(h_row(min(p_base + (blk / C) * 32, rows - 1), rr & 31, blk % C, C, L_, rows)) *
              static_cast<uint32_t>(d) * 2u;
  }
  u32x4 hreg[DH][HL];
  bool hkok[DH];
  auto hload = [&](int slot, int t) {
    bool valid;
    const int kt = ktile(t, valid);
    const int k = kt * BK + chunk * 8;
    const bool kok = valid && k < d;
    const uint32_t kb = min(static_cast<uint32_t>(k) * 2u, kclamp);
#pragma unroll
    for (int i = 0; i < HL; ++i) hreg[slot][i] = *reinterpret_cast<const u32x4*>(Hb + (hoff[i] + kb));
    hkok[slot] = kok;
  };
  f32x16 acc[NBLK];
#pragma unroll
  for (int i = 0; i < NBLK; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;

#pragma unroll
  for (int j = 0; j < DH; ++j) hload(j, j);
  const RowState mine = row_state(a, p_base + tid);
  // one pass over CNT <= D tiles; PF false: the last pass, no loads past the end
  auto body = [&](int t0, auto pf, auto cnt) {
    constexpr bool PF = decltype(pf)::value;
    constexpr int CNT = decltype(cnt)::value;
#pragma unroll
    for (int j = 0; j < CNT; ++j) {
      compiler_fence();
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<u32x4*>(&Ws[(lrow + 8 * i) * PITCH + chunk * 8]) = wreg[j][i];
#pragma unroll
      for (int i = 0; i < HL; ++i) {          // zeroing here: at the load it would wait for it
        const u32x4 t4 = hreg[j % DH][i];
        *reinterpret_cast<u32x4*>(&Hs[(lrow + 8 * i) * PITCH + chunk * 8]) =
            (hkok[j % DH] ? t4 : u32x4{0u, 0u, 0u, 0u});
      }
      if (PF) wload(j, t0 + j + D);
      if (PF || j + DH < CNT) hload(j % DH, t0 + j + DH);
      compiler_fence();
#pragma unroll
      for (int kk = 0; kk < BK / 16; ++kk) {
        const u32x4 braw = *reinterpret_cast<const u32x4*>(&Ws[ln * PITCH + kk * 16 + lg * 8]);
        const bf16x8 bfrag = __builtin_bit_cast(bf16x8, braw);
#pragma unroll
        for (int i = 0; i < NBLK; ++i) {
          const u32x4 araw = *reinterpret_cast<const u32x4*>(&Hs[(i * 32 + ln) * PITCH + kk * 16 + lg * 8]);
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, araw), bfrag,
                                                           acc[i], 0, 0, 0);
        }
      }
      compiler_fence();
    }
  };
  {
    const int full = ntiles / D * D, rem = ntiles - full;
    const int prefetching = rem == 0 ? full - D : full;      // tiles of the passes that load ahead
    for (int t0 = 0; t0 < prefetching; t0 += D) body(t0, TrueT{}, IntT<D>{});
    if (rem == 0) {
      if (full > 0) body(full - D, FalseT{}, IntT<D>{});
    } else if (rem == 1) {
      body(full, FalseT{}, IntT<1>{});
    } else if constexpr (D > 2) {
      if (rem == 2) body(full, FalseT{}, IntT<2>{});
      else body(full, FalseT{}, IntT<3>{});
    }
  }
  // the partial accumulators meet in LDS
  if (tid < RBW * 32) table[tid] = row_dest(a, mine);
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds_raw);
#pragma unroll
  for (int i = 0; i < NBLK; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) red[((wave * NBLK + i) * 16 + j) * 64 + lane] = acc[i][j];
  __syncthreads();
  // wavefront w adds up (partial sums in wavefront order 0, 1, 2, ...) and stores the
  // accumulator elements j = w, w + NWAVE, ... of every tile
  const int v = mapped_row(rm, xcd, jt, 32, ln);
  if (v >= a.n) return;
  with_bool(through_lines(a), [&](auto through) {
#pragma unroll
    for (int rbw = 0; rbw < RBW; ++rbw) {
#pragma unroll
      for (int jj = 0; jj < 16 / NWAVE; ++jj) {
        const int j = wave + jj * NWAVE;
        const int row = table[rbw * 32 + (j >> 2) * 8 + lg * 4 + (j & 3)];
        float c = red[((0 * NBLK + rbw * C) * 16 + j) * 64 + lane];
        float u = red[((0 * NBLK + rbw * C + C - 1) * 16 + j) * 64 + lane];
#pragma unroll
        for (int w = 1; w < NWAVE; ++w) {
          c += red[((w * NBLK + rbw * C) * 16 + j) * 64 + lane];
          u += red[((w * NBLK + rbw * C + C - 1) * 16 + j) * 64 + lane];
        }
        if (row >= 0)
          store_logit<decltype(through)::value>(&a.z[static_cast<int64_t>(row) * a.n + v], processed_logit<C>(a, c, u));
      }
    }
  });
}

// Row map for these operands and the number of workgroup tiles per XCD it needs.
RowMap make_row_map(const LmHeadArgs& a, int BN, int VT, int* tiles_per_xcd) {
  RowMap m{-1, 0};
  *tiles_per_xcd = (VT + 7) / 8;
  const size_t row_bytes = static_cast<size_t>(a.d) * 2;
  constexpr size_t kBlock = 128 * 1024;
  if (kBlock % row_bytes != 0) return m;
  const int G = static_cast<int>(kBlock / row_bytes);
  if ((G & (G - 1)) != 0) return m;
  int gs = 0;
  while ((1 << gs) < G) ++gs;
  m.gshift = gs;
  // block (mod 8) that holds the middle of group 0
  m.rot = static_cast<int>(((reinterpret_cast<uintptr_t>(a.W) + kBlock / 2) / kBlock) % 8);
  const long groups = (static_cast<long>(a.n) + G - 1) / G;
  const long rows_per_xcd = (groups + 7) / 8 * G;
  *tiles_per_xcd = static_cast<int>((rows_per_xcd + BN - 1) / BN);
  return m;
}

// Optional timing of the launch: the runtime attaches the two events to the dispatch itself
// (start and stop time of the kernel), so no marker packets of their own enter the stream.
struct LaunchEvents {
  hipEvent_t start, stop;
};
template <class Kern, class... Args>
void launch_kernel(Kern kernel, dim3 grid, dim3 block, hipStream_t s, const LaunchEvents& ev, Args... args) {
  if (ev.start && ev.stop) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev.start, ev.stop, 0, args...);
  else hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
}

// W is streamed past the caches when its slice cannot stay in the memory-side cache anyway
bool stream_w(const LmHeadArgs& a) { return 2.0 * a.d * a.n > 192.0 * 1024 * 1024; }

template <int RBW, int C, int NWV>
hipError_t launch_wide(const LmHeadArgs& a, hipStream_t s, const LaunchEvents& ev) {
  using K = Cfg<RBW, C, NWV>;
  const int VT = (a.n - 1) / K::BN + 1;
  const int MT = (a.B * a.L + 32 * RBW - 1) / (32 * RBW);
  // The wavefronts of this kernel walk k in step (shared h tile): with all rows of a workgroup
  // in one residue class (RowMap) its requests would pile onto one channel at a time (measured: 124 us
  // against 94 us for the full vocabulary), so rows stay consecutive here.
  const dim3 grid((VT + 7) / 8 * 8 * MT);
  if (stream_w(a)) launch_kernel(lm_head_kernel<RBW, C, NWV, true>, grid, dim3(K::THREADS), s, ev, a, VT, MT);
  else launch_kernel(lm_head_kernel<RBW, C, NWV, false>, grid, dim3(K::THREADS), s, ev, a, VT, MT);
  return hipGetLastError();
}

template <int RBW, int C, int KS>
hipError_t launch_split(const LmHeadArgs& a, hipStream_t s, const LaunchEvents& ev) {
  using K = SplitCfg<RBW, C, KS>;
  const int VT = (a.n + 31) / 32;
  const int MT = (a.B * a.L + 32 * RBW - 1) / (32 * RBW);
  int JT;
  const RowMap rm = make_row_map(a, 32, VT, &JT);
  launch_kernel(lm_head_splitk_kernel<RBW, C, KS>, dim3(JT * 8 * MT), dim3(K::THREADS), s, ev, a.W, a.h, a.d, a.n,
                a.L, a.B * a.L, MT, rm.gshift, rm.rot, a);
  return hipGetLastError();
}

// In how many partial sums the k of a logit is added up outside the split kernel.  The rounding error of one
// chain of 32-bit additions grows with its length: against 64 bits, over d = 4096 4.0e-7 of the logits' size in one
// chain, 1.9e-7 in 4 parts, 1.4e-7 in 8.  Calls of up to 96 rows and 49024 ids have it at the lower levels (the
// lines of the split kernel, which served them all at first); larger ones load the matrix pipe most, and take
// one chain in every kernel.
int k_parts(const LmHeadArgs& a) {
  const int rows = a.B * a.L, KT = (a.d + BK - 1) / BK;
  if (rows > 96 || a.n > 49024 || KT < 16) return 1;
  return rows <= 32 && KT >= 48 ? 8 : 4;
}

template <int C, int HR, int BN, int S>
hipError_t launch_tile(const LmHeadArgs& a, hipStream_t s, const LaunchEvents& ev) {
  using K = TileCfg<C, HR, BN, S>;
  const int VT = (a.n - 1) / BN + 1, MT = (a.B * a.L + K::WR - 1) / K::WR;
  const int KS = K::SPLITS && a.part ? a.ksplit : 1;
  const dim3 grid((VT + 7) / 8 * 8 * MT * KS);
  // (a part of k in KS is added up in its share of the partial sums)
  const int KT = a.d / 64 / KS, parts = (k_parts(a) + KS - 1) / KS, per = parts > 1 ? (KT + parts - 1) / parts : KT + 2;
  if (stream_w(a)) launch_kernel(lm_head_tile_kernel<C, HR, BN, S, true>, grid, dim3(K::THREADS), s, ev, a, VT, MT, KS, per);
  else launch_kernel(lm_head_tile_kernel<C, HR, BN, S, false>, grid, dim3(K::THREADS), s, ev, a, VT, MT, KS, per);
  return hipGetLastError();
}

// Which kernel serves a problem shape.
struct Variant {
  bool split;   // lm_head_splitk_kernel (else lm_head_kernel)
  int rbw, nw;  // row blocks per workgroup; wavefronts (= k parts for the split kernel)
  int hr, bn;   // hr > 0: lm_head_tile_kernel with tiles of hr h rows x bn columns ...
  int stages;   // ... and as many stages of W
};
// The lines were drawn by timing every kernel on 32 to 512 window rows x 1000 to 65536 ids over d = 64 to
// 4096 (us; the rows' W not in a cache).
Variant choose(const LmHeadArgs& a) {
  const int nRB = (a.B * a.L + 31) / 32;
  const int KT = (a.d + BK - 1) / BK;
  const long m = static_cast<long>(a.B) * a.L * a.C;
  if (a.d < 64) return {false, 1, 4, 0, 0, 0};           // no whole k-tile
  const int columns32 = (a.n - 1) / 32 + 1;
  const bool reach = 2L * a.d * a.n < 1L << 32;          // the split kernel's offsets into W have 32 bits
  // Few rows and columns: 32-column workgroups with k split, as long as all of them run at once (LDS: one
  // per CU with guidance, two without).  32 rows x 8192 ids over 4096: 16 : 20 of the best tile; x 11000,
  // two rounds, 29 : 30; without guidance x 16384 28 : 33, x 22000 39 : 36; over d = 320 the two are even.
  if (reach && KT >= 8 && nRB == 1 && columns32 <= (a.C == 2 ? 256 : 512)) return {true, 1, 8, 0, 0, 0};
  // 33 to 128 rows without guidance: 64 x 8192 over 4096 17.5 : 21, x 11000 31 : 32; 128 x 2048 15 : 20,
  // x 6000 (two rounds) 23 : 21
  if (reach && KT >= 8 && a.C == 1 && nRB > 1 && nRB <= 4 && (nRB + 1) / 2 * columns32 <= 256)
    return {true, 2, 4, 0, 0, 0};
  // 32 rows without guidance: half of a tile's MFMAs would be wasted on the longest streams, 84 : 85 at 65536
  // ids, even at 45000 (44 : 44 at 32768, where 128-column tiles still run at once)
  const bool chain = k_parts(a) == 1;
  if (a.C == 1 && nRB == 1 && a.n > 32768 && chain) return {false, 1, 8, 0, 0, 0};
  // otherwise tiles: rounds of one workgroup per CU, times what a round takes (us over d = 4096 with 64
  // or fewer workgroups, when neither memory nor power is short)
  struct Shape { int hr, bn, stages, cost; };
  constexpr Shape shapes[] = {{64, 128, 6, 20}, {64, 256, 4, 28}, {128, 128, 5, 27}, {128, 256, 3, 41},
                              {256, 128, 3, 40}, {256, 256, 3, 73}};
  const Shape* best = nullptr;
  long least = 0;
  for (const Shape& t : shapes) {
    // no registers for partial sums: 96 rows with guidance x 49024 ids over 1280 take two rounds of 256 x 128,
    // 41 us for 35
    if (t.hr * t.bn == 256 * 256 && !chain) continue;
    const long g = (m + t.hr - 1) / t.hr * ((a.n - 1) / t.bn + 1);
    const long cost = (g + 255) / 256 * t.cost;
    if (!best || cost < least) {
      best = &t;
      least = cost;
    }
  }
  return {false, 0, 0, best->hr, best->bn, best->stages};
}

template <int C>
hipError_t launch_c(const LmHeadArgs& a, hipStream_t s, const LaunchEvents& ev) {
  const Variant v = choose(a);
  if (v.hr == 256) return v.bn == 256 ? launch_tile<C, 256, 256, 3>(a, s, ev) : launch_tile<C, 256, 128, 3>(a, s, ev);
  if (v.hr == 128) return v.bn == 256 ? launch_tile<C, 128, 256, 3>(a, s, ev) : launch_tile<C, 128, 128, 5>(a, s, ev);
  if (v.hr == 64) return v.bn == 256 ? launch_tile<C, 64, 256, 4>(a, s, ev) : launch_tile<C, 64, 128, 6>(a, s, ev);
  if constexpr (C == 1) {
    if (v.split) return v.rbw == 2 ? launch_split<2, 1, 4>(a, s, ev) : launch_split<1, 1, 8>(a, s, ev);
    if (v.nw == 8) return launch_wide<1, 1, 8>(a, s, ev);
  } else {
    if (v.split) return launch_split<1, 2, 8>(a, s, ev);
  }
  return launch_wide<1, C, 4>(a, s, ev);
}

}  // namespace

hipError_t launch_lm_head(const LmHeadArgs& a, hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const LaunchEvents ev{ev_start, ev_stop};
  if (a.part) return a.C == 2 ? launch_tile<2, 64, 128, 6>(a, s, ev) : launch_tile<1, 64, 128, 6>(a, s, ev);
  return a.C == 2 ? launch_c<2>(a, s, ev) : launch_c<1>(a, s, ev);
}

// Few tiles leave most of the chip idle: k is dealt over as many workgroups per 64 x 128 tile as make 128 of them (with
// 256 the row kernel's reads cost more than is won), no part below four k-tiles.  What it saves grows with d and with
// the rows; what it costs, with the arrays that a row reads.  One step, LM head and rows, in one part : in the parts taken
// here (us): 64 rows with guidance x 1024 ids over 4096 28.8 : 18.7, over 1280 19.4 : 16.8; x 4096 30.3 : 24.6, 20.9 : 19.6;
// 128 rows without x 2048 23.8 : 19.9, 18.1 : 17.8; 256 x 2048 30.2 : 24.4, 22.1 : 20.0.  Not taken: d of 512 (64 rows with
// guidance x 2048 16.4 : 16.5); two parts where the split kernel runs in one round (128 rows without guidance x 4096 over 1280
// 19.8 : 20.0, 64 x 8192 20.9 : 21.9); up to 32 rows, whose kernel fills more CUs, but for d of 4096 on few ids (with
// guidance x 2048 20.4 : 18.8, x 8192 26.6 : 27.9; without x 1024 16.5 : 16.2, x 4096 18.9 : 20.2).
int lm_head_ksplit(const LmHeadArgs& a) {
  const long rows = static_cast<long>(a.B) * a.L;
  const long tiles = (rows * a.C + 63) / 64 * ((a.n - 1) / 128 + 1);
  const int KT = a.d / 64;
  if (a.n < 256 || a.n > kRowPartsMaxN || tiles > 64) return 1;
  int ks = a.n <= kRowPartsMaxN / 2 ? kMaxKSplit : 4;
  while (ks > 1 && (tiles * ks > 128 || KT < 4 * ks)) ks /= 2;
  const int least = rows <= 32 ? (KT < 64 ? kMaxKSplit + 1 : a.C == 2 ? 4 : 8)
                    : KT < 20 ? kMaxKSplit + 1 : a.C == 1 && rows <= 128 ? 4 : 2;
  return ks >= least ? ks : 1;
}

int lm_head_tiles(const LmHeadArgs& a) {
  const Variant v = choose(a);
  const int bn = v.hr > 0 ? v.bn : (!v.split && v.nw == 8) ? 256 : 0;
  if (bn == 0) return 0;
  const int tiles = (a.n - 1) / bn + 1;
  return tiles <= kRowMaxTiles ? tiles : 0;
}

int lm_head_kernel_name(const LmHeadArgs& a, char* buf, size_t cap) {
  const Variant v = a.ksplit > 1 ? Variant{false, 0, 0, 64, 128, 6} : choose(a);
  const char* nt = stream_w(a) ? "true" : "false";
  if (v.hr > 0) return snprintf(buf, cap, "lm_head_tile_kernel<%d, %d, %d, %d, %s>", a.C, v.hr, v.bn, v.stages, nt);
  if (v.split) return snprintf(buf, cap, "lm_head_splitk_kernel<%d, %d, %d>", v.rbw, a.C, v.nw);
  return snprintf(buf, cap, "lm_head_kernel<%d, %d, %d, %s>", v.rbw, a.C, v.nw, nt);
}

}  // namespace scd
