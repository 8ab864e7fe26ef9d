"""Which launches of the attention put two query tiles in a workgroup (compile
time, no GPU needed): the pair's child sweep takes whole octets of children,
so with 2 or 4 children it is taken only where few parents are refined.
"""
import subprocess

from paper_2607_12789_amd import build

CHECK = """
#include "avq_attention.hip"
namespace avq {
constexpr int C = 256;  // compute units
// 8, 16, 1 and no children: by the number of tiles alone
static_assert(pair_tiles<bf16, 64>(64, 400, C, 256, 8, 256));
static_assert(pair_tiles<bf16, 64>(48, 500, C, 64, 16, 64));
static_assert(pair_tiles<bf16, 64>(64, 400, C, 256, 1, 256));
static_assert(pair_tiles<bf16, 128>(32, 513, C, 256, 0, 0));
static_assert(!pair_tiles<bf16, 128>(32, 512, C, 256, 0, 0));
static_assert(!pair_tiles<bf16, 64>(64, 256, C, 256, 8, 32));
static_assert(!pair_tiles<bf16, 64>(64, 513, C, 256, 8, 32));
static_assert(!pair_tiles<bf16, 64>(64, 768, C, 256, 8, 32));
static_assert(pair_tiles<bf16, 64>(64, 769, C, 256, 8, 32));
static_assert(!pair_tiles<bf16, 64>(65, 4096, C, 256, 8, 32));
template <int Ch>
constexpr bool few_children() {
  // measured slower: one round of tiles, large shares where the pairs begin
  // their second round
  return !pair_tiles<bf16, 64>(64, 400, C, 256, Ch, 85) &&
         !pair_tiles<bf16, 128>(64, 400, C, 256, Ch, 85) &&
         !pair_tiles<bf16, 64>(48, 500, C, 64, Ch, 64) &&
         !pair_tiles<bf16, 128>(48, 500, C, 512, Ch, 170) &&
         !pair_tiles<bf16, 64>(64, 500, C, 256, Ch, 48) &&
         !pair_tiles<bf16, 64>(32, 1600, C, 256, Ch, 85) &&
         !pair_tiles<bf16, 64>(32, 1600, C, 256, Ch, 48) &&
         !pair_tiles<bf16, 128>(32, 1200, C, 256, Ch, 40) &&
         !pair_tiles<bf16, 128>(32, 1500, C, 128, Ch, 32) &&
         // measured faster
         pair_tiles<bf16, 64>(64, 500, C, 256, Ch, 24) &&
         pair_tiles<bf16, 128>(64, 300, C, 256, Ch, 16) &&
         pair_tiles<bf16, 64>(32, 800, C, 256, Ch, 85) &&
         pair_tiles<bf16, 64>(64, 800, C, 256, Ch, 85) &&
         pair_tiles<bf16, 64>(64, 1000, C, 64, Ch, 64) &&
         pair_tiles<bf16, 64>(32, 1600, C, 256, Ch, 32) &&
         pair_tiles<bf16, 64>(32, 4000, C, 256, Ch, 60) &&
         pair_tiles<bf16, 64>(64, 2000, C, 256, Ch, 75) &&
         pair_tiles<bf16, 128>(32, 1600, C, 256, Ch, 64) &&
         pair_tiles<bf16, 128>(32, 4000, C, 256, Ch, 75) &&
         pair_tiles<bf16, 128>(64, 1000, C, 64, Ch, 64) &&
         pair_tiles<float, 64>(32, 1200, C, 256, Ch, 170) &&
         pair_tiles<float, 128>(32, 600, C, 64, Ch, 64);
}
static_assert(few_children<2>() && few_children<4>());
static_assert(!pair_tiles<float, 64>(33, 4096, C, 256, 8, 32));
static_assert(!pair_tiles<float, 64>(32, 512, C, 256, 8, 32));
}
"""


def test_pair_rule(tmp_path):
    src = tmp_path / "check.hip"
    src.write_text(CHECK)
    r = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-host-only",
                        "-fsyntax-only", f"-I{build.CSRC}", str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
