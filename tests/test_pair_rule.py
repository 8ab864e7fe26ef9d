"""Which launches of the attention put two query tiles in a workgroup (compile
time, no GPU needed): the pair's child sweep takes whole octets of children,
so with 2 or 4 children it is taken only where few parents are refined; and a
pair's tiles are of one head, so few tiles per head, if odd, stay single.
"""
import subprocess

from paper_2607_12789_amd import build

CHECK = """
#include "avq_attention.hip"
namespace avq {
constexpr int C = 256;  // compute units
// 8, 16, 1 and no children: by the number of tiles alone
static_assert(pair_tiles<bf16, 64>(64, 2, 200, C, 256, 8, 256));
static_assert(pair_tiles<bf16, 64>(48, 2, 250, C, 64, 16, 64));
static_assert(pair_tiles<bf16, 64>(64, 2, 200, C, 256, 1, 256));
static_assert(pair_tiles<bf16, 128>(32, 513, 1, C, 256, 0, 0));
static_assert(!pair_tiles<bf16, 128>(32, 2, 256, C, 256, 0, 0));
static_assert(!pair_tiles<bf16, 64>(64, 2, 128, C, 256, 8, 32));
static_assert(!pair_tiles<bf16, 64>(64, 513, 1, C, 256, 8, 32));
static_assert(!pair_tiles<bf16, 64>(64, 2, 384, C, 256, 8, 32));
static_assert(pair_tiles<bf16, 64>(64, 769, 1, C, 256, 8, 32));
static_assert(!pair_tiles<bf16, 64>(65, 2, 2048, C, 256, 8, 32));
template <int Ch>
constexpr bool few_children() {
  // measured slower: one round of tiles, large shares where the pairs begin
  // their second round
  return !pair_tiles<bf16, 64>(64, 2, 200, C, 256, Ch, 85) &&
         !pair_tiles<bf16, 128>(64, 2, 200, C, 256, Ch, 85) &&
         !pair_tiles<bf16, 64>(48, 2, 250, C, 64, Ch, 64) &&
         !pair_tiles<bf16, 128>(48, 2, 250, C, 512, Ch, 170) &&
         !pair_tiles<bf16, 64>(64, 2, 250, C, 256, Ch, 48) &&
         !pair_tiles<bf16, 64>(32, 2, 800, C, 256, Ch, 85) &&
         !pair_tiles<bf16, 64>(32, 2, 800, C, 256, Ch, 48) &&
         !pair_tiles<bf16, 128>(32, 2, 600, C, 256, Ch, 40) &&
         !pair_tiles<bf16, 128>(32, 2, 750, C, 128, Ch, 32) &&
         // measured faster
         pair_tiles<bf16, 64>(64, 2, 250, C, 256, Ch, 24) &&
         pair_tiles<bf16, 128>(64, 2, 150, C, 256, Ch, 16) &&
         pair_tiles<bf16, 64>(32, 2, 400, C, 256, Ch, 85) &&
         pair_tiles<bf16, 64>(64, 2, 400, C, 256, Ch, 85) &&
         pair_tiles<bf16, 64>(64, 2, 500, C, 64, Ch, 64) &&
         pair_tiles<bf16, 64>(32, 2, 800, C, 256, Ch, 32) &&
         pair_tiles<bf16, 64>(32, 2, 2000, C, 256, Ch, 60) &&
         pair_tiles<bf16, 64>(64, 2, 1000, C, 256, Ch, 75) &&
         pair_tiles<bf16, 128>(32, 2, 800, C, 256, Ch, 64) &&
         pair_tiles<bf16, 128>(32, 2, 2000, C, 256, Ch, 75) &&
         pair_tiles<bf16, 128>(64, 2, 500, C, 64, Ch, 64) &&
         pair_tiles<float, 64>(32, 2, 600, C, 256, Ch, 170) &&
         pair_tiles<float, 128>(32, 2, 300, C, 64, Ch, 64);
}
// a head's tiles: one is never paired, an odd number only in fewer rounds
static_assert(!pair_tiles<bf16, 64>(64, 1, 400, C, 256, 8, 128));
static_assert(!pair_tiles<bf16, 128>(64, 1, 5000, C, 256, 8, 128));
static_assert(!pair_tiles<float, 64>(32, 1, 5000, C, 256, 8, 128));
static_assert(pair_tiles<bf16, 64>(32, 3, 300, C, 256, 8, 128));
static_assert(!pair_tiles<bf16, 64>(32, 3, 512, C, 256, 8, 128));
static_assert(!pair_tiles<bf16, 128>(32, 3, 300, C, 256, 8, 128));
static_assert(!pair_tiles<bf16, 128>(32, 3, 512, C, 256, 8, 128));
static_assert(!pair_tiles<bf16, 64>(32, 5, 300, C, 256, 8, 128));
static_assert(pair_tiles<bf16, 64>(32, 5, 512, C, 256, 8, 128));
static_assert(pair_tiles<bf16, 128>(32, 5, 300, C, 256, 8, 128));
static_assert(!pair_tiles<bf16, 64>(64, 3, 512, C, 256, 8, 128));
static_assert(pair_tiles<bf16, 64>(64, 3, 300, C, 256, 8, 128));
static_assert(pair_tiles<bf16, 64>(64, 5, 300, C, 256, 8, 128));
static_assert(pair_tiles<bf16, 128>(64, 3, 300, C, 256, 8, 128));
static_assert(pair_tiles<float, 64>(32, 3, 512, C, 256, 8, 128));
static_assert(few_children<2>() && few_children<4>());
static_assert(!pair_tiles<float, 64>(33, 2, 2048, C, 256, 8, 32));
static_assert(!pair_tiles<float, 64>(32, 2, 256, C, 256, 8, 32));
}
"""


def test_pair_rule(tmp_path):
    src = tmp_path / "check.hip"
    src.write_text(CHECK)
    r = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-host-only",
                        "-fsyntax-only", f"-I{build.CSRC}", str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
