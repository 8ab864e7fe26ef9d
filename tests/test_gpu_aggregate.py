"""The aggregation's key list: heads whose keys crowd into few families.

A workgroup lists the keys of its families in LDS. These cases give one
workgroup more keys than the list holds, so that it takes its families in
batches, and one family more than the list holds, so that the family's keys
come in segments; families before, between and after it are small, of whole
groups of 32 keys and one key more or less, or empty. Sums are compared with
64-bit ones within the fp32 summation bound, counts exactly.
"""
import pytest
import torch

from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_12789_amd import avq
    avq.lib()


def crowded(M0, per_family, g):
    """Parents of a head's keys: per_family[p] keys of parent p, shuffled."""
    par = torch.repeat_interleave(torch.arange(M0), torch.tensor(per_family))
    return par[torch.randperm(len(par), generator=g)]


# keys per parent of a 16-parent head: one family of 30000 (past every list)
# among small ones, and 16 of about 3000 (together past every list)
GIANT = [31, 32, 33, 0, 1, 30000, 0, 64, 65, 5, 0, 0, 17, 96, 2, 0]
BATCHES = [3000 + 37 * (p % 3) for p in range(16)]
# families of every size up to a whole group of keys and past it
SIZES = list(range(40))
KEYS = {"giant": GIANT, "batches": BATCHES, "sizes": SIZES}


def reference(V, par, code, M0, Ch):
    """64-bit sums and counts, and the sums of |v| (of one head)."""
    Mtot = M0 * (1 + Ch)
    n = torch.bincount(code, minlength=Mtot)
    n[:M0] = torch.bincount(par, minlength=M0)
    out = []
    for v in (V.double(), V.double().abs()):
        s = torch.zeros(Mtot, V.shape[1], dtype=torch.float64, device=V.device)
        s.index_add_(0, par, v)
        moved = code >= M0
        s.index_add_(0, code[moved], v[moved])
        out.append(s)
    return n, out[0], out[1]


def check(V, par, code, M0, Ch, packed, counts, Vbar):
    n, s, mag = reference(V, par, code, M0, Ch)
    assert torch.equal(counts.long(), n)
    tol = torch.from_numpy(parity.gamma(n.clamp(min=1).cpu().numpy())).to(s)[:, None] * mag + 1e-30
    assert ((Vbar.double() - s).abs() <= tol).all()
    dt = {torch.float32: "f32", torch.bfloat16: "bf16"}[V.dtype]
    means, n_pk, _, pad = parity.unpack_packed(packed[None, None].cpu().numpy(), M0, Ch,
                                               V.shape[1], dt)
    assert (pad["means"] == 0).all() and (pad["n"] == 0).all()
    assert (n_pk[0, 0] == n.cpu().numpy()).all()
    r_store = 2.0 ** -8 if dt == "bf16" else parity.U
    nn = n.clamp(min=1)[:, None]
    mean = (s / nn).cpu().numpy()
    tol_m = (tol / nn).cpu().numpy() + (3 * parity.U + r_store) * abs(mean) + 1e-30
    assert (abs(means[0, 0] - mean) <= tol_m).all()


@pytest.mark.parametrize("heads", [1, 256])  # 256: all 16 families in one workgroup
@pytest.mark.parametrize("keys", list(KEYS))
@pytest.mark.parametrize("dtype,d,Ch", [(torch.bfloat16, 128, 8), (torch.bfloat16, 64, 16),
                                        (torch.float32, 64, 2), (torch.bfloat16, 128, 0),
                                        (torch.float32, 128, 0)])
def test_crowded_codes(dtype, d, Ch, keys, heads):
    from paper_2607_12789_amd import avq
    M0 = len(KEYS[keys])
    g = torch.Generator().manual_seed(7)
    par = crowded(M0, KEYS[keys], g).cuda()
    N = len(par)
    if heads * N * d >= 2 ** 30:
        heads = 128
    child = torch.randint(-1, max(Ch, 1), (N,), generator=g).cuda()
    code = torch.where(child < 0, par, M0 + par * Ch + child) if Ch else par
    V1 = torch.randn(N, d, generator=g).to(dtype).cuda()
    V = V1.expand(1, heads, N, d).contiguous()
    codes = code.to(torch.int32).expand(1, heads, N).contiguous()
    packed, counts, Vbar = avq.aggregate(V, codes, M0, Ch, sums=True)
    for h in {0, heads // 2, heads - 1}:
        check(V1, par, code, M0, Ch, packed[0, h], counts[0, h], Vbar[0, h])


@pytest.mark.parametrize("keys", list(KEYS))
@pytest.mark.parametrize("dtype,d,Ch", [(torch.bfloat16, 128, 8), (torch.bfloat16, 64, 4),
                                        (torch.bfloat16, 128, 16), (torch.float32, 64, 16),
                                        (torch.float32, 128, 8)])
def test_crowded_fused(dtype, d, Ch, keys):
    """The fused pass on the same crowds: the codes of avq_assign exactly, and
    the sums of those codes."""
    from paper_2607_12789_amd import avq
    M0, heads = len(KEYS[keys]), 128
    g = torch.Generator().manual_seed(9)
    par = crowded(M0, KEYS[keys], g)
    N = len(par)
    Cp = torch.randn(M0, d, generator=g)
    Cc = Cp[:, None] + 0.1 * torch.randn(M0, Ch, d, generator=g)
    pick = torch.randint(0, Ch + 1, (N,), generator=g)
    rows = torch.cat([Cp[:, None], Cc], 1)[par, pick]
    K1 = (rows + 0.05 * torch.randn(N, d, generator=g)).to(dtype).cuda()
    V1 = torch.randn(N, d, generator=g).to(dtype).cuda()
    K, V = (x.expand(1, heads, N, d).contiguous() for x in (K1, V1))
    cp = Cp.to(dtype).cuda().expand(heads, M0, d).contiguous()
    cc = Cc.to(dtype).cuda().expand(heads, M0, Ch, d).contiguous()
    p_idx, c_idx, packed, counts, Vbar = avq.assign_aggregate(K, V, cp, cc, sums=True)
    p_ref, c_ref = avq.assign(K[:, :2].contiguous(), cp[:2].contiguous(), cc[:2].contiguous())
    assert torch.equal(p_idx[:, :2], p_ref) and torch.equal(c_idx[:, :2], c_ref)
    for h in {0, heads // 2, heads - 1}:
        assert torch.equal(c_idx[0, h], c_idx[0, 0])
        check(V1, p_idx[0, h].long(), c_idx[0, h].long(), M0, Ch, packed[0, h], counts[0, h],
              Vbar[0, h])


# a head of at most 12000 keys: one family past the list of a small workgroup
# (about 6000 keys), and 16 or 64 families that are past it together
SMALL_GIANT = [31, 32, 33, 0, 1, 11000, 0, 64, 65, 5, 0, 0, 17, 96, 2, 0]
SMALL_BATCHES = {16: [740 + 7 * (p % 3) for p in range(16)],
                 64: [180 + 7 * (p % 3) for p in range(64)]}


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("keys", ["giant", "batches"])
@pytest.mark.parametrize("Ch", [0, 4, 8])
def test_crowded_small_workgroups(Ch, keys, fused):
    """The same crowds in the small workgroups, whose lists are the shortest
    (bf16, d = 64, below 16384 keys), with so many heads that a workgroup holds
    all the families."""
    from paper_2607_12789_amd import avq
    dtype, d, heads = torch.bfloat16, 64, 1024
    per = SMALL_GIANT if keys == "giant" else SMALL_BATCHES[16 if Ch else 64]
    M0 = len(per)
    g = torch.Generator().manual_seed(17)
    par = crowded(M0, per, g)
    N = len(par)
    assert 6500 < N < 16384
    V1 = torch.randn(N, d, generator=g).to(dtype).cuda()
    V = V1.expand(1, heads, N, d).contiguous()
    if fused:
        Cp = torch.randn(M0, d, generator=g)
        Cc = Cp[:, None] + 0.1 * torch.randn(M0, Ch, d, generator=g)
        pick = torch.randint(0, Ch + 1, (N,), generator=g)
        rows = torch.cat([Cp[:, None], Cc], 1)[par, pick]
        K1 = (rows + 0.05 * torch.randn(N, d, generator=g)).to(dtype).cuda()
        K = K1.expand(1, heads, N, d).contiguous()
        cp = Cp.to(dtype).cuda().expand(heads, M0, d).contiguous()
        cc = Cc.to(dtype).cuda().expand(heads, M0, Ch, d).contiguous()
        p_idx, c_idx, packed, counts, Vbar = avq.assign_aggregate(K, V, cp, cc, sums=True)
        p_ref, c_ref = avq.assign(K[:, :2].contiguous(), cp[:2].contiguous(), cc[:2].contiguous())
        assert torch.equal(p_idx[:, :2], p_ref) and torch.equal(c_idx[:, :2], c_ref)
        assert (c_idx == c_idx[:, :1]).all()
        par, code = p_idx[0, 0].long(), c_idx[0, 0].long()
    else:
        child = torch.randint(-1, max(Ch, 1), (N,), generator=g)
        code = (torch.where(child < 0, par, M0 + par * Ch + child) if Ch else par).cuda()
        par = par.cuda()
        codes = code.to(torch.int32).expand(1, heads, N).contiguous()
        packed, counts, Vbar = avq.aggregate(V, codes, M0, Ch, sums=True)
    for h in (0, heads // 2, heads - 1):
        check(V1, par, code, M0, Ch, packed[0, h], counts[0, h], Vbar[0, h])


@pytest.mark.parametrize("dtype,d,Ch", [(torch.bfloat16, 128, 0), (torch.bfloat16, 128, 4),
                                        (torch.float32, 64, 8), (torch.float32, 128, 0),
                                        (torch.float32, 128, 8)])
@pytest.mark.parametrize("N,M0,heads", [(1, 3, 5), (130, 16, 600), (1023, 100, 300),
                                        (1023, 512, 3), (2047, 70, 270), (2048, 70, 270)])
def test_short_heads(dtype, d, Ch, N, M0, heads):
    """Heads of fewer than 1024 keys (2048 where they are many): the small
    workgroups, two per compute unit, of the other types and widths; codes and (Ch
    >= 1) the fused pass."""
    from paper_2607_12789_amd import avq
    g = torch.Generator(device="cuda").manual_seed(19)

    def randn(*s):
        return torch.randn(*s, device="cuda", generator=g)

    par = torch.randint(0, M0, (heads, N), device="cuda", generator=g)
    V = randn(heads, N, d).to(dtype)
    if Ch == 0:
        packed, counts, Vbar = avq.aggregate(V[None], par[None].to(torch.int32), M0, 0, sums=True)
        for h in sorted({0, heads // 2, heads - 1}):
            check(V[h], par[h], par[h], M0, 0, packed[0, h], counts[0, h], Vbar[0, h])
        return
    Cp = randn(heads, M0, d)
    Cc = Cp[:, :, None] + 0.1 * randn(heads, M0, Ch, d)
    pick = torch.randint(0, Ch, (heads, N), device="cuda", generator=g)
    hh = torch.arange(heads, device="cuda")[:, None]
    K = (Cc[hh, par, pick] + 0.05 * randn(heads, N, d)).to(dtype)[None]
    cp, cc = Cp.to(dtype), Cc.to(dtype)
    p_idx, c_idx, packed, counts, Vbar = avq.assign_aggregate(K, V[None], cp, cc, sums=True)
    p_ref, c_ref = avq.assign(K, cp, cc)
    assert torch.equal(p_idx, p_ref) and torch.equal(c_idx, c_ref)
    packed2, counts2, Vbar2 = avq.aggregate(V[None], c_idx, M0, Ch, sums=True)
    assert torch.equal(counts, counts2)
    for h in sorted({0, heads // 2, heads - 1}):
        p, c = p_idx[0, h].long(), c_idx[0, h].long()
        check(V[h], p, c, M0, Ch, packed[0, h], counts[0, h], Vbar[0, h])
        check(V[h], p, c, M0, Ch, packed2[0, h], counts2[0, h], Vbar2[0, h])


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 64), (torch.bfloat16, 128),
                                     (torch.float32, 64), (torch.float32, 128)])
@pytest.mark.parametrize("Ch", [0, 1, 8, 16])
@pytest.mark.parametrize("N,M0,heads", [(1, 200, 70), (70, 203, 300)])
def test_fewer_keys_than_codes(dtype, d, Ch, N, M0, heads):
    """Most families have no keys: before, between and after those that do."""
    test_short_heads(dtype, d, Ch, N, M0, heads)


@pytest.mark.parametrize("N", [2 ** 21 - 3, 2 ** 21 + 5])
def test_long_head(N):
    """More keys than a compacted entry's key field holds (2^21), and the
    longest ragged head below that."""
    from paper_2607_12789_amd import avq
    M0, Ch, d = 24, 4, 64
    g = torch.Generator(device="cuda").manual_seed(11)
    par = torch.randint(0, M0, (N,), device="cuda", generator=g)
    child = torch.randint(-1, Ch, (N,), device="cuda", generator=g)
    code = torch.where(child < 0, par, M0 + par * Ch + child)
    V = torch.randn(N, d, device="cuda", generator=g).to(torch.bfloat16)
    packed, counts, Vbar = avq.aggregate(V.view(1, 1, N, d), code.to(torch.int32).view(1, 1, N),
                                         M0, Ch, sums=True)
    check(V, par, code, M0, Ch, packed[0, 0], counts[0, 0], Vbar[0, 0])


@pytest.mark.parametrize("heads", [1, 13, 26, 52, 103, 171])
@pytest.mark.parametrize("M0", [37, 100])
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 64), (torch.bfloat16, 128),
                                     (torch.float32, 64), (torch.float32, 128)])
def test_flat_families(dtype, d, M0, heads):
    """Flat codebooks with 1, 2, 4, 8 and 16 parents per family: at M0 = 37 the
    number of heads at which a 256-CU device goes from one to the next; the
    last family and octet are partly padding."""
    from paper_2607_12789_amd import avq
    N = 1100
    g = torch.Generator(device="cuda").manual_seed(13)
    # a skewed head: the last parent empty, one parent with a quarter of the keys
    code = torch.randint(0, M0 - 1, (heads, N), device="cuda", generator=g)
    code[:, ::4] = 7
    V = torch.randn(heads, N, d, device="cuda", generator=g).to(dtype)
    packed, counts, Vbar = avq.aggregate(V[None], code[None].to(torch.int32), M0, 0, sums=True)
    for h in sorted({0, heads // 2, heads - 1}):
        check(V[h], code[h], code[h], M0, 0, packed[0, h], counts[0, h], Vbar[0, h])
