"""Batches of single tokens and longer requests in one launch (caches of 64 MB and more): against one call per request, with all of the
workspace and with the smallest that is taken (whose tokens and longer requests are launches of their own)."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2501_15383_amd as vs
from paper_2501_15383_amd import binding

pytestmark = pytest.mark.gpu


# (rows, keys, sparse) of the requests: tokens that go two KV heads side by side (none sparse, 8,192 blocks and more) and that do not, no
# token, nothing but tokens (under bounds of more rows), a token of one key, longer requests of few pieces and of several rounds
@pytest.mark.parametrize("hq,hkv,d,specs", [
    (28, 4, 128, [(1, 100003, False), (64, 70000, True), (1, 90000, False), (17, 30001, False), (1, 1, False), (200, 1000, True)]),
    (28, 4, 128, [(1, 60000, True), (1, 60001, False), (5, 64, False), (129, 40000, True)]),
    (12, 2, 128, [(40, 140000, False), (40, 130000, True), (3, 70, False)]),
    (8, 2, 64, [(1, 200000, True), (1, 190000, False), (1, 63, True), (1, 64, False)]),
    (8, 2, 64, [(1, 150001, False), (1000, 150000, True), (1, 64, True), (33, 90000, False)] * 2),
    (40, 8, 128, [(1, 3000 + 17 * i, bool(i % 3)) if i % 2 else (1 + i % 20, 2000 + 31 * i, bool(i % 4)) for i in range(36)])])
def test_tokens_beside_longer_requests(hq, hkv, d, specs):
    gen = torch.Generator(device="cuda").manual_seed(5400 + len(specs) + d)
    rnd = lambda *size: torch.randn(size, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    bv, bs = 100, 300
    reqs, want = [], []
    most_rows, most_keys = max(max(r for r, _, _ in specs), 2), max(n for _, n, _ in specs)
    scale = 1.0 / np.sqrt(d)
    for rows, n, sparse in specs:
        q, k, v = rnd(rows, hq, d), rnd(n, hkv, d), rnd(n, hkv, d)
        sets = None
        if sparse:
            pick = lambda m, far: torch.stack([torch.randperm(far, generator=gen, device="cuda")[:m].sort().values for _ in range(hq)]).int()  # noqa: E731
            nv, ns = min(bv, n), min(bs, n)
            pad = lambda t, m: torch.nn.functional.pad(t, (0, m - t.shape[1]), value=-1).contiguous()  # noqa: E731
            cnt = lambda m: torch.full((hq,), m, dtype=torch.int32, device="cuda")  # noqa: E731
            sets = (pad(pick(nv, n), bv), cnt(nv), pad(pick(ns, n), bs), cnt(ns))
        ck = vs.Chunk(hq, hkv, d, rows, n - rows, scale, vertical_budget=bv, slash_budget=bs)
        one = vs.sparse_attn_prefill(ck, q, k, v, *sets, want_lse=True) if sparse else vs.dense_causal_prefill(ck, q, k, v, want_lse=True)
        want.append(one)
        reqs.append(dict(q=q, k=k, v=v, out=torch.empty_like(q), lse=torch.empty(hq, rows, device="cuda"), q_start=n - rows, sets=sets))
    ck = vs.Chunk(hq, hkv, d, most_rows, most_keys - most_rows, scale, vertical_budget=bv, slash_budget=bs)
    skipped = dict(reqs[0], v=reqs[0]["v"], out=torch.full_like(reqs[0]["out"], 7.0))
    table = vs.request_table(reqs + [skipped], "cuda")
    table[-1, 2] = 0   # no values: not taken
    p = ck.params(q=reqs[0]["q"], k=reqs[0]["k"], v=reqs[0]["v"], out=reqs[0]["out"])
    L = binding.lib()
    full = int(L.vs_batch_workspace_bytes(C.byref(p), len(reqs) + 1))
    room = torch.empty(full + 4096, dtype=torch.uint8, device="cuda")

    def call(size):
        return L.vs_attn_batch(C.byref(p), C.c_void_p(table.data_ptr()), len(reqs) + 1, C.c_void_p(room.data_ptr()), C.c_size_t(size),
                               C.c_void_p(torch.cuda.current_stream().cuda_stream))

    def check(size, byte):
        room.fill_(byte)
        for r in reqs:
            r["out"].fill_(3.0); r["lse"].fill_(3.0)
        assert call(size) == vs.VS_OK
        torch.cuda.synchronize()
        assert (room[size:] == byte).all() and (skipped["out"] == 7.0).all()
        for r, (o, l), spec in zip(reqs, want, specs):
            a, b = r["out"].float(), o.float()
            # bf16 probabilities and outputs on either side: 2^-9 each, unbiased, about 6e-3 between the two
            assert ((a - b).norm(dim=2) <= 2e-2 * b.norm(dim=2) + 1e-30).all(), spec
            np.testing.assert_allclose(r["lse"].cpu().numpy(), l.cpu().numpy(), rtol=2e-5, atol=5e-5, err_msg=str(spec))
        return [(r["out"].clone(), r["lse"].clone()) for r in reqs]
    first, again = check(full, 0x5A), check(full, 0xA5)
    for x, y in zip(first, again):
        assert torch.equal(x[0].view(torch.int16), y[0].view(torch.int16)) and torch.equal(x[1], y[1])
    lo, hi = 0, full // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        rc = call(256 * mid)
        assert rc in (vs.VS_OK, vs.VS_ERR_WORKSPACE)
        lo, hi = (lo, mid) if rc == vs.VS_OK else (mid, hi)
    if 256 * hi < full:
        check(256 * hi, 0x5A)


# A sparse token beside longer requests whose list takes several windows of diagonals: 4,096 of groups of 9 to 16 heads (262,144 keys), 8,192 of smaller
# ones (524,288), fewer than a call of its own has.  Offsets and columns crowd on both sides of the windows' edges, other ones for every head; a
# column is gathered where its head lacks the diagonal.
@pytest.mark.parametrize("hq,hkv,d,n", [(16, 1, 128, 270000), (12, 1, 64, 2 * 262144 + 777), (24, 2, 128, 262144 + 64), (8, 1, 64, 530001), (28, 4, 128, 525000)])
def test_lists_of_tokens_in_windows(hq, hkv, d, n):
    gen = torch.Generator(device="cuda").manual_seed(5700 + n)
    rnd = lambda *size: torch.randn(size, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    draw = lambda lo, hi, count: torch.randint(max(lo, 0), hi, (count,), generator=gen, device="cuda")  # noqa: E731
    window = 64 * (8192 if hq // hkv <= 8 else 4096)
    bv, bs = 200, 300
    edges = [e for e in range(window, n, window)]

    def lines(budget, m, spots):
        idx = torch.full((hq, budget), -1, dtype=torch.int32, device="cuda")
        cnt = torch.zeros(hq, dtype=torch.int32, device="cuda")
        for h in range(hq):
            x = torch.cat([draw(0, m, 40)] + [draw(lo, min(hi, m), 60) for lo, hi in spots]).unique()
            idx[h, :len(x)] = x.int()
            cnt[h] = len(x)
        return idx, cnt
    k, v = rnd(n, hkv, d), rnd(n, hkv, d)
    specs = [(1, n), (40, 5000), (1, n - 70)]
    reqs, want = [], []
    for r, m in specs:
        q = rnd(r, hq, d)
        # (offset o of the token is key m - 1 - o)
        sets = (*lines(bv, m, [(m - e - 700, m - e + 700) for e in edges]), *lines(bs, m, [(e - 700, e + 700) for e in edges])) if r == 1 else None
        ck = vs.Chunk(hq, hkv, d, r, m - r, 1.0 / np.sqrt(d), vertical_budget=bv, slash_budget=bs)
        one = vs.sparse_attn_prefill(ck, q, k[:m], v[:m], *sets, want_lse=True) if sets else vs.dense_causal_prefill(ck, q, k[:m], v[:m], want_lse=True)
        want.append(one)
        reqs.append(dict(q=q, k=k, v=v, out=torch.empty_like(q), lse=torch.empty(hq, r, device="cuda"), q_start=m - r, sets=sets))
    ck = vs.Chunk(hq, hkv, d, 40, n - 40, 1.0 / np.sqrt(d), vertical_budget=bv, slash_budget=bs)
    table = vs.request_table(reqs, "cuda")
    vs.attn_batch(ck, table, len(reqs), reqs[0]["q"], k, v, reqs[0]["out"])
    torch.cuda.synchronize()
    for r, (o, l), spec in zip(reqs, want, specs):
        a, b = r["out"].float(), o.float()
        # bf16 probabilities and outputs on either side: 2^-9 each, unbiased, about 6e-3 between the two
        assert ((a - b).norm(dim=2) <= 2e-2 * b.norm(dim=2) + 1e-30).all(), spec
        np.testing.assert_allclose(r["lse"].cpu().numpy(), l.cpu().numpy(), rtol=2e-5, atol=5e-5, err_msg=str(spec))
