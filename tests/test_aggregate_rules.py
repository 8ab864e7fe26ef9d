"""How the aggregation divides a head among workgroups (compile time, no GPU
needed): a flat codebook's families hold fewer parents where 16 of them would
leave compute units idle, and still cover every parent in whole octets; heads
of few keys take the small workgroups, several per compute unit.
"""
import subprocess

from paper_2607_12789_amd import build

CHECK = """
#include "avq_aggregate.hip"
namespace avq {
constexpr bool covers() {
  for (int M0 = 1; M0 <= 512; ++M0)
    for (int rsh = 0; rsh <= 4; ++rsh) {
      const int parents = flat_families(M0, rsh) << rsh;
      const int octets = (M0 + 63) / 64 * 8;  // as packed_layout
      if (parents < M0 || parents % 8 != 0 || parents > 8 * octets) return false;
    }
  return true;
}
static_assert(covers(), "whole octets, every parent, none past the padding");
// workgroups of (heads, N, M0): enough for every slot, while the parents last
constexpr long long families(long long BH, int N, int M0, long long slots) {
  return BH * flat_families(M0, flat_shift(BH, N, M0, slots));
}
static_assert(families(1, 1 << 20, 256, 256) == 256);
static_assert(families(4, 65536, 128, 256) == 256);
static_assert(families(1, 65536, 8, 256) == 8);
static_assert(families(32, 8192, 64, 512) == 512);
static_assert(flat_shift(48, 16384, 512, 256) == 4);
static_assert(flat_shift(1, 512, 512, 256) == 4);  // few keys: 16 parents
// heads of few keys share a compute unit with others, whatever the type
static_assert(kSmallKeys<bf16, 64> > 4096 && kSmallKeys<bf16, 128> > 512 &&
              kSmallKeys<float, 64> > 512 && kSmallKeys<float, 128> > 512);
constexpr int C = 256;  // compute units
static_assert(small_workgroups<bf16, 64, kAggCodes>(48, 4096, 64, C) &&
              small_workgroups<float, 128, kAggCodes>(1, 700, 64, C) &&
              small_workgroups<bf16, 128, kAggFused>(1, 700, 64, C) &&
              small_workgroups<float, 128, kAggFlat>(96, 700, 512, C));
// up to 2048 keys also others that would take more than one round
static_assert(small_workgroups<float, 64, kAggCodes>(300, 2000, 64, C) &&
              small_workgroups<bf16, 128, kAggFused>(214, 1040, 256, C) &&
              !small_workgroups<bf16, 128, kAggFused>(64, 1040, 256, C) &&
              !small_workgroups<float, 64, kAggCodes>(96, 4096, 256, C) &&
              !small_workgroups<float, 64, kAggFlat>(214, 1040, 256, C) &&
              small_workgroups<float, 128, kAggFlat>(304, 1504, 12, C));
// few families of fp32 products at d = 128
static_assert(!small_workgroups<float, 128, kAggFlat>(26, 872, 64, C) &&
              !small_workgroups<float, 128, kAggFlat>(88, 876, 2, C) &&
              small_workgroups<float, 128, kAggFlat>(71, 301, 5, C) &&
              small_workgroups<float, 64, kAggFlat>(26, 872, 64, C) &&
              small_workgroups<bf16, 128, kAggFlat>(26, 872, 64, C));
// heads of many keys do not
static_assert(kSmallKeys<bf16, 64> <= 16384 && kSmallKeys<bf16, 128> <= 4096 &&
              kSmallKeys<float, 64> <= 4096 && kSmallKeys<float, 128> <= 4096);
}
"""


def test_flat_families(tmp_path):
    src = tmp_path / "check.hip"
    src.write_text(CHECK)
    r = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-host-only",
                        "-fsyntax-only", "-fconstexpr-steps=10000000", f"-I{build.CSRC}",
                        str(src)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
