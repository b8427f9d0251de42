"""Guard offsets of the buffer loads of few rows, by constant evaluation: a compiler refuses an expression that overflows."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_04557_amd", "csrc")

PROGRAM = r"""
#include "offsets.h"
using namespace sprinter;
// the last unit that a pass over K asks for: K itself, the loads in flight (8 groups of 8 waves) and the units of a group beyond it
constexpr int last_unit(int K, int ku) { return (K + ku - 1) / ku + 2 * 8 * 8 * 4; }
constexpr bool beyond(int K, int ku, int bytes, unsigned lane, unsigned size) {
  for (int u = 0; u <= last_unit(K, ku); ++u)
    if (unit_offset(false, lane, u, bytes) < size || unit_offset(true, NOWHERE, u, bytes) < size) return false;
  return true;
}
constexpr int KS[] = {8, 96, 8192, 32768, FEW_ROWS_MAX_K};
static_assert(64LL * FEW_ROWS_MAX_K < NOWHERE, "a buffer reaches NOWHERE");
constexpr bool all() {
  for (int K : KS) {
    const int kt = (K + 31) / 32;
    if (!beyond(K, 32, 1024, 1023 * 16u, 2u * kt * 1024)) return false;         // float16 operand tiles, two of them
    if (!beyond(K, 16, 64, 15u * K * 4 + 48, 16u * K * 4)) return false;        // float32 rows
  }
  return true;
}
static_assert(all(), "an absent load reaches a buffer");
static_assert(unit_offset(true, 48, 3, 64) == 240 && unit_offset(true, 16, 5, 1024) == 5136, "");
"""


def test_offsets_of_absent_loads_stay_beyond_the_buffer(tmp_path):
    src = tmp_path / "offsets.cpp"
    src.write_text(PROGRAM)
    r = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-Wall", "-Werror", "-I", CSRC, str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_every_guard_uses_them():
    """No buffer load of the kernels of few rows adds to NOWHERE by itself."""
    with open(os.path.join(CSRC, "k_gemm_norm.hip")) as f:
        lines = [l for l in f if "raw_buffer_load" in l]
    assert lines and all("unit_offset(" in l and "NOWHERE" not in l for l in lines), lines
