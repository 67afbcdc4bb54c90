// Division by the window length L as a multiplication, for the row kernels (a division is about thirty
// instructions, in every wavefront).  Plain C++: host code and kernels share it.
#pragma once
#include <cstdint>

namespace scd {

// ceil(2^32 / L), which gives v / L exactly for every v with v L < 2^32 (its excess over 2^32 / L is below 1), where the
// largest dividend of these sizes lies within that: a row of the launch, or a position in the window or behind it.  Else 0.
constexpr uint32_t window_reciprocal(int rows, int N, int L) {
  const int64_t behind = static_cast<int64_t>(N) + 2 * L, most = rows > behind ? rows : behind;
  return L > 1 && most * L < (1ll << 32) ? static_cast<uint32_t>(((1ull << 32) + L - 1) / L) : 0u;
}
// v / L for 0 <= v.
constexpr int div_window(int v, int L, uint32_t recip) {
  return recip != 0u ? static_cast<int>(static_cast<uint64_t>(static_cast<uint32_t>(v)) * recip >> 32) : v / L;
}

}  // namespace scd
