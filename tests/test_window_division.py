"""The row kernels divide by the window length L with a multiplication by its reciprocal where the launcher finds that exact
(csrc/window_division.h, compiled here by itself): every L, at the sizes where the launcher's line lies and at the multiples of
L around which a quotient could slip, up to the largest dividend of those sizes."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_24211_amd", "csrc")
PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "window_division.h"
int main() {
  long checked = 0, by_product = 0, refused = 0;
  for (int L = 1; L <= 256; ++L) {
    const int line = static_cast<int>(std::min((1ll << 32) / L - 2 * L, 0x7fffffffll));     // about the largest N
    for (int N : {1, 2304, line - 2, line - 1, line, std::min(line, 0x7ffffff0) + 1, 0x7fffffff - 2 * L})
      for (int rows : {L, 37 * L, (1 << 20) * L}) {
        const unsigned recip = scd::window_reciprocal(rows, N, L);
        (recip ? by_product : refused) += 1;
        const long most = std::max<long>(rows - 1, std::min<long>(N + 2l * L - 1, 0x7fffffff));
        auto check = [&](long v) {
          if (v < 0 || v > most) return true;
          ++checked;
          if (scd::div_window(static_cast<int>(v), L, recip) == v / L) return true;
          std::printf("%ld / %d, N %d, %d rows\n", v, L, N, rows);
          return false;
        };
        for (long q = 0; q <= most / L; q += q < 300 || q > most / L - 300 ? 1 : 1 + most / L / 997)
          if (!check(q * L - 1) || !check(q * L) || !check(q * L + L - 1)) return 1;
        if (!check(most)) return 1;
      }
  }
  std::printf("%ld %ld %ld\n", checked, by_product, refused);
  return 0;
}
"""


def test_division_by_the_window_length_is_exact(tmp_path):
    (tmp_path / "division.cpp").write_text(PROGRAM)
    exe = tmp_path / "division"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(tmp_path / "division.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    checked, by_product, refused = map(int, r.stdout.split())
    assert checked > 1_000_000 and by_product > 1000 and refused > 500      # both ways, on each side of the line
