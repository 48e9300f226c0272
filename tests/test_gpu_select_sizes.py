"""The selection at the edges of its paths: rows that stay in registers, rows whose workgroup lists its own
candidates, rows thinned out by the whole chip, and the rows that neither can serve.  Whole numbers: every
result equals a stable full sort."""
import pytest
import torch

import paper_2501_15383_amd as vs

pytestmark = pytest.mark.gpu

SIZES = [64, 65, 1000, 8192, 8193, 16384, 16385, 32768, 32769, 49152, 49153, 131071, 700001]


def _want(sc, budget, keep):
    hq, n = sc.shape
    k = min(budget, n)
    s = sc.clone()
    s[:, :min(keep, k)] = float("inf")
    idx = torch.full((hq, budget), -1, dtype=torch.int32, device=sc.device)
    idx[:, :k] = torch.sort(s, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values.int()
    return idx, torch.full((hq,), k, dtype=torch.int32, device=sc.device)


def _scores(kind, hq, n, g):
    dev = torch.device("cuda:0")
    if kind == "spread":      # what an estimate leaves
        return (torch.randn((hq, n), generator=g, device=dev) * 0.4).exp() / n
    if kind == "ties":        # thousands of equal scores at every threshold
        return torch.randint(0, 23, (hq, n), generator=g, device=dev).float() / 32
    if kind == "equal":
        return torch.full((hq, n), 0.25, device=dev)
    if kind == "sparse":      # mostly zeros: the threshold may be zero itself
        return torch.where(torch.rand((hq, n), generator=g, device=dev) < 0.002, torch.rand((hq, n), generator=g, device=dev), 0.0)
    if kind == "crowded":     # the best entries side by side at one end
        x = torch.rand((hq, n), generator=g, device=dev)
        x[:, n // 3:n // 3 + max(1, n // 20)] += 1.0
        return x
    return torch.randn((hq, n), generator=g, device=dev)   # "signed": beyond what the interface asks for


@pytest.mark.parametrize("kind", ["spread", "ties", "equal", "sparse", "crowded", "signed"])
@pytest.mark.parametrize("n", SIZES)
def test_select_equals_a_full_sort(n, kind):
    g = torch.Generator(device="cuda:0").manual_seed(100 + n)
    hq = 3
    vsc, ssc = _scores(kind, hq, n, g), _scores(kind, hq, n, g)
    # ordinary budgets; one line; more lines than any list in LDS holds; everything
    for bv, bs, keep in ((1000, 6096, 64), (1, 70, 64), (40, 30000, 0), (n, n + 3, 64)):
        c = min(64, n)
        ck = vs.Chunk(hq, 1, 128, c, n - c, 0.1, vertical_budget=bv, slash_budget=bs, keep_first_cols=1, keep_local_band=keep)
        want = (*_want(vsc, bv, 1), *_want(ssc, bs, keep))
        for sets in (vs.select(ck, vsc, ssc), vs.select_static(ck, vsc, ssc, vs.alloc_index_sets(ck, vsc.device))):
            for a, b, nm in zip(sets, want, ("v_idx", "v_cnt", "s_idx", "s_cnt")):
                assert torch.equal(a, b), f"{nm}: n {n}, {kind}, budgets {bv} / {bs}"


# lists in registers: 8, 12 and 16 candidates per lane, numbers of slices (2,048 scores behind the forced ones) around a power of two, the
# most that are placed at once (2,048) and one more
@pytest.mark.parametrize("kind", ["spread", "ties", "crowded"])
@pytest.mark.parametrize("bs", [300, 6500, 9500, 13000])
@pytest.mark.parametrize("n", [32 * 2048 + 64, 32 * 2048 + 65, 64 * 2048 + 63, 2048 * 2048 + 64, 2048 * 2048 + 65])
def test_lists_in_registers(n, bs, kind):
    g = torch.Generator(device="cuda:0").manual_seed(200 + n)
    vsc, ssc = _scores(kind, 2, n, g), _scores(kind, 2, n, g)
    ck = vs.Chunk(2, 1, 128, 64, n - 64, 0.1, vertical_budget=1000, slash_budget=bs, keep_first_cols=1, keep_local_band=64)
    for a, b in zip(vs.select(ck, vsc, ssc), (*_want(vsc, 1000, 1), *_want(ssc, bs, 64))):
        assert torch.equal(a, b), f"n {n}, {kind}, {bs} offsets"


# (heads, keys, offsets kept): lists in the workspace that fit the LDS, that do not, and that are not made (slices); of the
# static entry point, whose scratch holds 12 MB, the first as well, rows that list their own candidates, and slices
@pytest.mark.parametrize("kind", ["spread", "ties", "sparse", "signed"])
@pytest.mark.parametrize("hq,n,bs", [(3, 131071, 9000), (3, 131071, 20000), (3, 131071, 26000), (128, 100000, 6096),
                                     (64, 100000, 16000), (2, 3000001, 40000)])
def test_every_route_of_long_rows(hq, n, bs, kind):
    g = torch.Generator(device="cuda:0").manual_seed(200 + n + bs)
    vsc, ssc = _scores(kind, hq, n, g), _scores(kind, hq, n, g)
    ck = vs.Chunk(hq, 1, 128, 64, n - 64, 0.1, vertical_budget=700, slash_budget=bs, keep_first_cols=1, keep_local_band=64)
    want = (*_want(vsc, 700, 1), *_want(ssc, bs, 64))
    for sets in (vs.select(ck, vsc, ssc), vs.select_static(ck, vsc, ssc, vs.alloc_index_sets(ck, vsc.device))):
        for a, b, nm in zip(sets, want, ("v_idx", "v_cnt", "s_idx", "s_cnt")):
            assert torch.equal(a, b), f"{nm}: {hq} heads, n {n}, {kind}, {bs} offsets"


def _few(hq, n, g):
    """Every score one to five times: thresholds fall on short lists, between equal scores of several waves and of one."""
    dev = torch.device("cuda:0")
    return torch.randint(1, n // 2 + 2, (hq, n), generator=g, device=dev).float() / n


@pytest.mark.parametrize("n", [200, 4095, 4096, 4097, 8191, 12288, 12289, 16384, 24576, 24577, 32768, 40960, 40961, 49151, 49152])
def test_rows_in_registers_at_every_length(n):
    g = torch.Generator(device="cuda:0").manual_seed(300 + n)
    hq = 4
    for vsc, ssc in ((_few(hq, n, g), _few(hq, n, g)), (_scores("sparse", hq, n, g), _scores("ties", hq, n, g))):
        for bv, bs, keep in ((2, 70, 64), (n // 7 + 2, n // 3 + 2, 64), (n - 1, n // 2, 0)):
            ck = vs.Chunk(hq, 1, 128, 64, n - 64, 0.1, vertical_budget=bv, slash_budget=bs, keep_first_cols=1, keep_local_band=keep)
            want = (*_want(vsc, bv, 1), *_want(ssc, bs, keep))
            for a, b, nm in zip(vs.select(ck, vsc, ssc), want, ("v_idx", "v_cnt", "s_idx", "s_cnt")):
                assert torch.equal(a, b), f"{nm}: n {n}, budgets {bv} / {bs}"


# Rows in registers from one counter per bin to four, and scores of a few values: every lane of a wave adds to the same bin, the
# threshold falls on a crowd (of the largest value, of one in the middle, at the end of one), and crowds lie side by side or scattered.
@pytest.mark.parametrize("n", [16384, 16385, 32769, 40961, 49152])
@pytest.mark.parametrize("values", [2, 5, 50])
def test_crowds_in_registers(n, values):
    g = torch.Generator(device="cuda:0").manual_seed(400 + n + values)
    hq = 4
    crowd = lambda: torch.randint(0, values, (hq, n), generator=g, device="cuda").float() / 32 + 1  # noqa: E731
    half = torch.where(torch.rand((hq, n), generator=g, device="cuda") < 0.5, 1.5, _scores("spread", hq, n, g) * n)
    for vsc, ssc in ((crowd(), crowd().sort(1, descending=True).values), (half, -crowd())):
        for bv, bs, keep in ((128, 256, 64), (n // 2, n // values, 0), (1000, n - n // values, 0)):
            ck = vs.Chunk(hq, 1, 128, 64, n - 64, 0.1, vertical_budget=bv, slash_budget=bs, keep_first_cols=1, keep_local_band=keep)
            want = (*_want(vsc, bv, 1), *_want(ssc, bs, keep))
            for a, b, nm in zip(vs.select(ck, vsc, ssc), want, ("v_idx", "v_cnt", "s_idx", "s_cnt")):
                assert torch.equal(a, b), f"{nm}: n {n}, {values} values, budgets {bv} / {bs}"
