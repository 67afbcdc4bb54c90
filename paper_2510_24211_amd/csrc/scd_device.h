// Device-side helpers shared by the gfx950 kernels of the SCD step:
// Philox4x32-10 (Salmon et al., SC'11), the 23-bit uniform mapping, the
// order-preserving float <-> uint32 key map used by the radix select, and
// block-wide reductions for 64-lane wavefronts.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scd {

constexpr int kWave = 64;

enum : uint32_t {
  kStreamInit = 0, kStreamAccept = 1, kStreamResid = 2, kStreamGumbel = 3, kStreamAlpha = 4, kStreamIndep = 5
};

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);     // one instruction on gfx950
}
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint2 k) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // one widening multiply per product (v_mad_u64_u32) instead of a high and a low one
    const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c.x;
    const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c.z;
    c = make_uint4(xor3(static_cast<uint32_t>(p1 >> 32), c.y, k.x), static_cast<uint32_t>(p1),
                   xor3(static_cast<uint32_t>(p0 >> 32), c.w, k.y), static_cast<uint32_t>(p0));
    k.x += 0x9E3779B9u;
    k.y += 0xBB67AE85u;
  }
  return c;
}

// ((bits >> 9) + 1/2) * 2^-23: every step is exact in fp32, result in (0,1).
__device__ __forceinline__ float u01(uint32_t bits) {
  return (static_cast<float>(bits >> 9) + 0.5f) * 1.1920928955078125e-07f;
}

// e^x for x up to about 88, as of differences of a logit and a maximum or a log normaliser: x log2(e), to twice the
// precision, is split into an integer and a rest of at most a half, whose power of two the exponential unit takes
// (1 ulp).  (The two-part product is the usual one: log2(e) split at 24 bits, the first product's rounding error taken from
// a fused multiply-add.)  11 instructions where the general function, which also has large arguments to look after, takes 14,
// with the same error (largest 1.39, root mean square 0.43 of 2^-24, over -100 .. 0).  Far below the smallest float's
// logarithm, -inf included: 0.  NaN: NaN.
__device__ __forceinline__ float exp_of(float x) {
  const float y = x < -150.f ? -150.f : x;
  const float t = __fmul_rn(y, 1.44269502f);
  const float rest = __fmaf_rn(y, 1.92596303e-8f, __fmaf_rn(y, 1.44269502f, -t));   // log2(e) less its 24-bit part
  const float k = __builtin_rintf(t);
  return __builtin_ldexpf(__builtin_amdgcn_exp2f((t - k) + rest), static_cast<int>(k));
}
// -ln(u) of a uniform of u01 (2^-24 and more: no denormals): the logarithm unit's log2 (1 ulp) times ln 2 in two
// parts, the product's rounding error made good: the general function's result bit for bit, over all 2^23 uniforms,
// without its care for denormals and infinity.
__device__ __forceinline__ float neg_log(float u) {
  const float y = __builtin_amdgcn_logf(u);
  const float h = __fmul_rn(y, 0.693147182f);
  const float l = __fmaf_rn(y, -1.90465430e-9f, __fmaf_rn(y, 0.693147182f, -h));
  return -(h + l);
}

__device__ __forceinline__ uint2 seed_key(uint64_t seed) {
  return make_uint2(static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32));
}

// Uniform initial draft of a never-evaluated position: floor(r64 * n / 2^64).
__device__ __forceinline__ int32_t init_token(uint64_t seed, int b, int pos, int n) {
  const uint4 r = philox4x32_10(make_uint4(0u, static_cast<uint32_t>(pos), 0u,
                                           (static_cast<uint32_t>(b) << 8) | kStreamInit),
                                seed_key(seed));
  const uint64_t r64 = (static_cast<uint64_t>(r.x) << 32) | r.y;
  return static_cast<int32_t>(__umul64hi(r64, static_cast<uint64_t>(n)));
}

// Larger float <-> larger key (total order; -0 < +0; NaNs sort above +inf or
// below -inf by sign).
__device__ __forceinline__ uint32_t float_to_key(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_to_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
// key with -0 folded onto +0, so that key order == float order for non-NaNs
__device__ __forceinline__ uint32_t zkey(float f) { return float_to_key(f == 0.f ? 0.f : f); }

// Four neighbouring floats in one 16-byte load from any 4-byte-aligned address (rows of odd length
// start at such addresses): global memory needs dword alignment only.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load4(const float* p) {
  const f32x4_u v = *reinterpret_cast<const f32x4_u*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store4(float* p, float a, float b, float c, float d) {
  *reinterpret_cast<f32x4_u*>(p) = f32x4_u{a, b, c, d};
}

// The same into a row of n floats (short enough for 32-bit byte offsets), written through the L2: what a kernel leaves in it is
// written back behind its last workgroup, 1 us and more for 8 MB, before the next kernel starts.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(float* row, int n) {
  return __builtin_amdgcn_make_buffer_rsrc(row, 0, 4 * n, 0x00020000);       // raw, bounds in bytes
}
__device__ __forceinline__ void store4_through(__amdgpu_buffer_rsrc_t row, int at, float a, float b, float c, float d) {
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  constexpr int kSc1 = 16;                                                    // agent scope
  __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{__float_as_uint(a), __float_as_uint(b), __float_as_uint(c), __float_as_uint(d)},
                                         row, 4 * at, 0, kSc1);
}

// Three-way maximum / minimum of floats; a NaN operand is ignored.  As builtins they would come with a
// quieting instruction per operand.
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float min3(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// ---- wavefront collectives ---------------------------------------------------------
// Lane exchanges through the vector ALU's data-parallel primitives (DPP): no round trip through
// the LDS crossbar, which a shuffle costs.  All of them must be called with the whole wavefront active.
enum : int {
  kDppXor1 = 0xB1,        // quad_perm [1,0,3,2]: lane ^ 1
  kDppXor2 = 0x4E,        // quad_perm [2,3,0,1]: lane ^ 2
  kDppHalfMirror = 0x141, // lane i <-> 7 - i inside groups of 8
  kDppMirror = 0x140,     // lane i <-> 15 - i inside rows of 16
  kDppRowShl = 0x100,     // + n: lane i reads lane i + n of its row of 16 (0 if there is none)
  kDppRowShr = 0x110,     // + n: lane i reads lane i - n of its row of 16 (0 if there is none)
  kDppBcast15 = 0x142,    // rows 1 and 3 read the last lane of the row before
  kDppBcast31 = 0x143,    // rows 2 and 3 read the last lane of row 1
};
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return static_cast<uint32_t>(dpp_i32<CTRL>(static_cast<int>(v)));
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(dpp_i32<CTRL>(__float_as_int(v)));
}
// What the rows named by MASK read of another row; `rest` in the other rows.
template <int CTRL, int MASK>
__device__ __forceinline__ int dpp_row_i32(int rest, int v) {
  return __builtin_amdgcn_update_dpp(rest, v, CTRL, MASK, 0xF, false);
}
template <int CTRL, int MASK>
__device__ __forceinline__ float dpp_row_f32(float rest, float v) {
  return __int_as_float(dpp_row_i32<CTRL, MASK>(__float_as_int(rest), __float_as_int(v)));
}
__device__ __forceinline__ float readlane_f32(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Reductions: pairs, quads, eights, rows of 16, the rows two by two, the halves -- a fixed order; the result
// as a scalar.
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f32<kDppXor1>(v);
  v += dpp_f32<kDppXor2>(v);
  v += dpp_f32<kDppHalfMirror>(v);
  v += dpp_f32<kDppMirror>(v);
  v += dpp_row_f32<kDppBcast15, 0xA>(0.f, v);
  v += dpp_row_f32<kDppBcast31, 0xC>(0.f, v);
  return readlane_f32(v, 63);
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t u) {
  auto mx = [](uint32_t a, int b) { return a > static_cast<uint32_t>(b) ? a : static_cast<uint32_t>(b); };
  uint32_t v = u;
  v = mx(v, dpp_i32<kDppXor1>(static_cast<int>(v)));
  v = mx(v, dpp_i32<kDppXor2>(static_cast<int>(v)));
  v = mx(v, dpp_i32<kDppHalfMirror>(static_cast<int>(v)));
  v = mx(v, dpp_i32<kDppMirror>(static_cast<int>(v)));
  v = mx(v, dpp_row_i32<kDppBcast15, 0xA>(0, static_cast<int>(v)));
  v = mx(v, dpp_row_i32<kDppBcast31, 0xC>(0, static_cast<int>(v)));
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 63));
}
// Largest / smallest value over the wavefront (NaNs are ignored unless every lane holds one).
__device__ __forceinline__ float wave_max_f32(float v) {
  v = fmaxf(v, dpp_f32<kDppXor1>(v));
  v = fmaxf(v, dpp_f32<kDppXor2>(v));
  v = fmaxf(v, dpp_f32<kDppHalfMirror>(v));
  v = fmaxf(v, dpp_f32<kDppMirror>(v));
  v = fmaxf(v, dpp_row_f32<kDppBcast15, 0xA>(v, v));
  v = fmaxf(v, dpp_row_f32<kDppBcast31, 0xC>(v, v));
  return readlane_f32(v, 63);
}
__device__ __forceinline__ float wave_min_f32(float v) {
  v = fminf(v, dpp_f32<kDppXor1>(v));
  v = fminf(v, dpp_f32<kDppXor2>(v));
  v = fminf(v, dpp_f32<kDppHalfMirror>(v));
  v = fminf(v, dpp_f32<kDppMirror>(v));
  v = fminf(v, dpp_row_f32<kDppBcast15, 0xA>(v, v));
  v = fminf(v, dpp_row_f32<kDppBcast31, 0xC>(v, v));
  return readlane_f32(v, 63);
}
// Inclusive prefix sum over the lanes of the wavefront; lane 63 holds the total.
__device__ __forceinline__ int wave_inclusive_sum_i32(int v) {
  v += dpp_i32<kDppRowShr + 1>(v);
  v += dpp_i32<kDppRowShr + 2>(v);
  v += dpp_i32<kDppRowShr + 4>(v);
  v += dpp_i32<kDppRowShr + 8>(v);
  v += dpp_row_i32<kDppBcast15, 0xA>(0, v);
  v += dpp_row_i32<kDppBcast31, 0xC>(0, v);
  return v;
}
__device__ __forceinline__ int wave_sum_i32(int v) {
  return __builtin_amdgcn_readlane(wave_inclusive_sum_i32(v), 63);
}

// ---- folds over the wavefronts of a workgroup ----------------------------------------------
// Of W = 4, 8 or 16 entries in LDS, one per wavefront, every lane reads one (lane modulo W) and the lanes of a
// row exchange them: ten instructions, where reading all of them in every lane takes three per entry, in
// every wavefront (a row kernel has about eight such folds; with them, the DPP-only reductions above and the
// shorter selection, four steps on supplied logits of 32 x 65536 take 96 us instead of 111).  The caller's
// barrier stands between the writes and these.
template <int W>
__device__ __forceinline__ int fold_entry() {
  static_assert(W == 4 || W == 8 || W == 16, "wavefronts");
  return threadIdx.x & (W - 1);
}
__device__ __forceinline__ int wave_index() {        // as a scalar
  return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
}
// Sum of the entries of the wavefronts before this one, and of all.
template <int W>
__device__ __forceinline__ int fold_before(const int* ex, int wave, int& total) {
  int v = ex[fold_entry<W>()];
  v += dpp_i32<kDppRowShr + 1>(v);
  v += dpp_i32<kDppRowShr + 2>(v);
  if constexpr (W >= 8) v += dpp_i32<kDppRowShr + 4>(v);
  if constexpr (W == 16) v += dpp_i32<kDppRowShr + 8>(v);
  total = __builtin_amdgcn_readlane(v, W - 1);
  return wave > 0 ? __builtin_amdgcn_readlane(v, wave > 0 ? wave - 1 : 0) : 0;
}
template <int W>
__device__ __forceinline__ uint32_t fold_max(const uint32_t* ex) {
  auto mx = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
  uint32_t v = ex[fold_entry<W>()];
  v = mx(v, dpp_u32<kDppXor1>(v));
  v = mx(v, dpp_u32<kDppXor2>(v));
  if constexpr (W >= 8) v = mx(v, dpp_u32<kDppHalfMirror>(v));
  if constexpr (W == 16) v = mx(v, dpp_u32<kDppMirror>(v));
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}
template <int W>
__device__ __forceinline__ float fold_sum(const float* ex) {       // a fixed tree
  float v = ex[fold_entry<W>()];
  v += dpp_f32<kDppXor1>(v);
  v += dpp_f32<kDppXor2>(v);
  if constexpr (W >= 8) v += dpp_f32<kDppHalfMirror>(v);
  if constexpr (W == 16) v += dpp_f32<kDppMirror>(v);
  return readlane_f32(v, 0);
}

// Lexicographic minimum of (score, id) over the wavefront, in every lane; scores and ids are not negative
// (and no NaN), so both compare as integers.
__device__ __forceinline__ void wave_min_score_id(float& score, int& id) {
  const uint32_t mine = __float_as_uint(score);
  const uint32_t least = ~wave_max_u32(~mine);
  id = static_cast<int>(~wave_max_u32(~(mine == least ? static_cast<uint32_t>(id) : 0xFFFFFFFFu)));
  score = __uint_as_float(least);
}

// Guidance mix and temperature of one logit (cond sum c, uncond sum u): three fp32 roundings
// for the mix, one for the division (skipped for tau = 1, where it changes nothing).
template <int C>
__device__ __forceinline__ float processed_logit(float lam, float one_plus_lam, float tau, float c, float u) {
  float z = c;
  if (C == 2) z = __fsub_rn(__fmul_rn(one_plus_lam, c), __fmul_rn(lam, u));
  return tau == 1.0f ? z : __fdiv_rn(z, tau);
}

}  // namespace scd
