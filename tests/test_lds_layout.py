"""The aggregation's LDS layout, checked at compile time (no GPU needed).

The kernel reads the one-hot rows, partial sums, staged octets and key list
as 16-byte vectors, so each of these areas must start on a multiple of 16
bytes, whatever fields lie before it.
"""
import subprocess

from paper_2607_12789_amd import build

CHECK = """
#include "avq_aggregate.hip"
#include <cstddef>
namespace avq {
template <typename T, int D, int NT, int MODE, bool SMALL>
constexpr bool layout_ok() {
  using C = AggCfg<T, D, NT, MODE, SMALL>;
  using L = typename C::Tables;
  static_assert(offsetof(L, onehot) % 16 == 0, "one-hot rows");
  static_assert(sizeof(L::onehot[0][0]) % 16 == 0, "one-hot rows of a wave");
  static_assert(C::OFF_SLOT % 16 == 0 && C::SLOT_BYTES % 16 == 0, "partial sums");
  static_assert(C::OFF_STAGE % 16 == 0 && C::STAGE_BYTES % 16 == 0, "staged octets");
  static_assert(C::OFF_SLOT >= (int)sizeof(L), "the tables end before the partial sums");
  for (int F = 1; F <= kMaxFamilies; ++F)
    if (C::off_list(F) % 16 != 0) return false;
  return true;
}
template <typename T, int D>
constexpr bool all_ok() {
  return layout_ok<T, D, 1, kAggCodes, false>() && layout_ok<T, D, 2, kAggCodes, false>() &&
         layout_ok<T, D, 1, kAggFlat, false>() && layout_ok<T, D, 1, kAggFlatFew, false>() &&
         layout_ok<T, D, 1, kAggFused, false>() && layout_ok<T, D, 2, kAggFused, false>() &&
         layout_ok<T, D, 1, kAggCodes, true>() && layout_ok<T, D, 1, kAggFlat, true>() &&
         layout_ok<T, D, 1, kAggFlatFew, true>() && layout_ok<T, D, 1, kAggFused, true>();
}
static_assert(all_ok<bf16, 64>() && all_ok<bf16, 128>() && all_ok<float, 64>() &&
                  all_ok<float, 128>(), "key list");
}
"""


def test_vector_read_areas_are_aligned(tmp_path):
    src = tmp_path / "check.hip"
    src.write_text(CHECK)
    r = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-host-only",
                        "-fsyntax-only", f"-I{build.CSRC}", str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
