"""Query blocks of at most 64: two tiles per workgroup.

Many tiles (so that the launcher pairs them), with an odd number of tiles per
head (the last workgroup has one), ragged last tiles, blocks of one and two
waves, every number of children, and a tile that differs from its neighbour
in its selection. Compared with the oracle as the edge cases of
test_gpu_parity, and bit for bit with the same queries in larger launches.
"""
import pytest
import torch

from paper_2607_12789_amd import inputs
from tests import parity
from tests.test_gpu_parity import banner, report, small

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_12789_amd import avq
    avq.lib()


# 2 x 3 heads of N / block_q tiles: more than 3 per CU of a 256-CU device
# (pairs for any block), or 300 .. 500 in all (pairs for blocks above 32)
CASES = {
    "bq32": small(N=32 * 136 + 5, block_q=32, M0=70, Ch=8, P=9),
    "bq17_d128": small(N=17 * 139 - 3, block_q=17, M0=40, Ch=4, P=7, d=128),
    "bq64_odd": small(N=64 * 67 + 1, block_q=64, M0=100, Ch=8, P=13),
    "bq64_ch16_d128": small(N=64 * 59, block_q=64, M0=66, Ch=16, P=5, d=128),
    "bq33_ch2": small(N=33 * 131 + 32, block_q=33, M0=40, Ch=2, P=9),
    "bq48_fp32": small(N=48 * 61 + 7, block_q=48, M0=70, Ch=8, P=6, dtype="f32"),
    "bq64_fp32_d128": small(N=64 * 55 + 9, block_q=64, M0=70, Ch=4, P=6, dtype="f32", d=128),
    "bq32_fp32_d128": small(N=32 * 91 + 9, block_q=32, M0=40, Ch=16, P=3, dtype="f32", d=128),
    "bq64_flat": small(N=64 * 61 + 30, block_q=64, Ch=0, P=0),
    "bq40_p_full": small(N=40 * 53, block_q=40, P=40),
    "bq1": small(N=150, block_q=1, P=2),
}


@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_small_blocks(name, tiled):
    w = CASES[name]
    if tiled and w.Ch == 0:
        pytest.skip("no importance with a flat codebook")
    banner(name, w)
    report(parity.compare(inputs.generate(w), w, tiled=tiled))


@pytest.mark.parametrize("block_q,d", [(32, 64), (64, 128), (50, 64)])
def test_pairs_equal_single_tiles(block_q, d):
    """The output and selection of a tile do not depend on whether another
    tile shares its workgroup: a launch of one head (single tiles) against the
    same head among many (pairs)."""
    from paper_2607_12789_amd import avq
    w = small(N=block_q * 9 + 5, block_q=block_q, d=d, M0=70, Ch=8, P=9, B=1, H=2)
    x = parity.to_gpu(inputs.generate(w))
    _, _, packed, _, _ = avq.assign_aggregate(x["K"], x["V"], x["Cp"], x["Cc"])
    one = avq.attention_fwd(x["Q"], x["Cp"], x["Cc"], packed, w.P, block_q, debug=True)
    rep = 64  # 64 x 2 heads of 10 tiles
    many = avq.attention_fwd(x["Q"].repeat(rep, 1, 1, 1), x["Cp"], x["Cc"],
                             packed.repeat(rep, 1, 1), w.P, block_q, debug=True)
    for a, b in zip(one, many):
        for i in (0, rep // 2, rep - 1):
            assert torch.equal(a[0], b[i])
