"""Single tokens at the edges of the decode kernel: positions around the 32- and 64-key boundaries, group sizes from one
head to a full MFMA tile, shares that end inside a KV head or span several requests, tokens without any line, and more
requests than a workgroup has threads.  Against the fp64 oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import paper_2501_15383_amd as vs
from gpu_util import assert_attn_close, chunk_of, dev
from helpers import rand_bf16
from test_gpu_attention import _rand_sets, _t

pytestmark = pytest.mark.gpu


def _problem(rng, hq, hkv, d, s, bv, bs, lines):
    q, k, v = rand_bf16(rng, (1, hq, d)), rand_bf16(rng, (s + 1, hkv, d)), rand_bf16(rng, (s + 1, hkv, d))
    pb = oracle.Problem(hq, hkv, d, 1, s, 1.0 / np.sqrt(d), vertical_budget=bv, slash_budget=bs, keep_first_cols=0, keep_local_band=0)
    if lines == "none":
        sets = (np.full((hq, bv), -1, np.int32), np.zeros(hq, np.int32), np.full((hq, bs), -1, np.int32), np.zeros(hq, np.int32))
    elif lines == "columns":   # no diagonal: the union list is empty
        sets = list(_rand_sets(rng, pb, min(bv, s + 1), 0))
    elif lines == "both":
        sets = _rand_sets(rng, pb, min(bv, max(1, (s + 1) // 4)), min(bs, max(1, (s + 1) // 50)), force_cols=[0], force_offs=[0])
    else:
        sets = None
    return pb, q, k, v, sets


@pytest.mark.parametrize("hq,hkv,d", [(7, 1, 128), (5, 5, 128), (32, 2, 64), (16, 1, 128)])
@pytest.mark.parametrize("s", [0, 1, 30, 31, 32, 63, 64, 95, 127, 128, 4159, 9000])
def test_single_tokens_at_every_boundary(hq, hkv, d, s):
    rng = np.random.default_rng(2000 + s)
    for lines in ("dense", "both", "columns", "none"):
        pb, q, k, v, sets = _problem(rng, hq, hkv, d, s, 150, 90, lines)
        if sets is None:
            ref = oracle.dense_attention(pb, q, k, v)
            got = vs.dense_causal_prefill(chunk_of(pb), dev(q), dev(k), dev(v), want_lse=True)
        else:
            ref = oracle.sparse_attention(pb, q, k, v, *sets)
            got = vs.sparse_attn_prefill(chunk_of(pb), dev(q), dev(k), dev(v), *[_t(x) for x in sets], want_lse=True)
        torch.cuda.synchronize()
        assert_attn_close(*got, *ref, f"{lines} {hq}/{hkv} D={d} s={s}")


@pytest.mark.parametrize("n_req", [2, 37, 300])
def test_shares_over_many_requests(n_req):
    hq, hkv, d, bv, bs = 6, 2, 64, 40, 30
    rng = np.random.default_rng(2100 + n_req)
    reqs, gpu = [], []
    for i in range(n_req):
        s = int(rng.choice([0, 5, 63, 64, 200, 3000 if n_req < 100 else 700]))
        pb, q, k, v, sets = _problem(rng, hq, hkv, d, s, bv, bs, ("dense", "both", "none", "dense")[i % 4])
        reqs.append((pb, q, k, v, sets))
        gpu.append(dict(q=dev(q), k=dev(k), v=dev(v), q_start=s, out=torch.full((1, hq, d), -3.0, dtype=torch.bfloat16, device="cuda"),
                        lse=torch.full((hq, 1), 7.0, device="cuda"), sets=None if sets is None else tuple(_t(x) for x in sets)))
    ck = vs.Chunk(hq, hkv, d, 1, max(p.q_start for p, *_ in reqs), 1.0 / np.sqrt(d), vertical_budget=bv, slash_budget=bs)
    table = vs.request_table(gpu, "cuda")
    skipped = n_req // 2
    table[skipped, 10] = 0   # a request outside the bounds, between two others
    first = None
    for _ in range(2):
        vs.attn_batch(ck, table, n_req, gpu[0]["q"], gpu[0]["k"], gpu[0]["v"], gpu[0]["out"])
        torch.cuda.synchronize()
        now = [(g["out"].clone(), g["lse"].clone()) for g in gpu]
        assert first is None or all(torch.equal(a[0].view(torch.int16), b[0].view(torch.int16)) and torch.equal(a[1], b[1])
                                    for a, b in zip(first, now)), "not run-to-run identical"
        first = now
    for i, ((pb, q, k, v, sets), g) in enumerate(zip(reqs, gpu)):
        if i == skipped:
            assert (g["out"].float() == -3.0).all() and (g["lse"] == 7.0).all()
            continue
        ref = oracle.dense_attention(pb, q, k, v) if sets is None else oracle.sparse_attention(pb, q, k, v, *sets)
        assert_attn_close(g["out"], g["lse"], *ref, f"request {i} of {n_req}, s={pb.q_start}")


@pytest.mark.parametrize("hq,hkv,s", [(14, 2, 262143), (24, 8, 65599), (21, 3, 180000)])
def test_long_token_of_neighbouring_heads(hq, hkv, s):
    """8,192 blocks and more: two KV heads side by side where their number is even."""
    rng = np.random.default_rng(2200 + hkv)
    pb, q, k, v, _ = _problem(rng, hq, hkv, 128, s, 1, 1, "dense")
    kd, vd = dev(k), dev(v)
    ref = oracle.dense_attention(pb, q, k, v)
    for major in (False, True):   # caches of [keys][KV heads][128], and of [KV heads][keys][128], whose heads go by themselves
        if major:
            kd, vd = (x.permute(1, 0, 2).contiguous().permute(1, 0, 2) for x in (kd, vd))
        got = vs.dense_causal_prefill(chunk_of(pb), dev(q), kd, vd, want_lse=True)
        torch.cuda.synchronize()
        assert_attn_close(*got, *ref, f"{hq}/{hkv} s={s} major={major}")


def test_neighbouring_heads_of_many_requests():
    """A table whose bounds take the path of neighbouring heads: dense and sparse tokens, the heads' lists of different lengths (and
    without any line), shares that hold several requests."""
    hq, hkv, d, bv, bs, n_req = 6, 2, 128, 40, 30, 300
    rng = np.random.default_rng(2300)
    reqs, gpu = [], []
    for i in range(n_req):
        s = int(rng.choice([0, 5, 63, 64, 200, 940]))
        pb, q, k, v, sets = _problem(rng, hq, hkv, d, s, bv, bs, ("dense", "both", "none", "both")[i % 4])
        if sets is not None and i % 4 == 3:   # the second KV head keeps a line of each kind, or only a column
            sets = tuple(x.copy() for x in sets)
            sets[1][3:] = np.minimum(sets[1][3:], 1)
            sets[3][3:] = np.minimum(sets[3][3:], i // 4 % 2)
        reqs.append((pb, q, k, v, sets))
        gpu.append(dict(q=dev(q), k=dev(k), v=dev(v), q_start=s, out=torch.full((1, hq, d), -3.0, dtype=torch.bfloat16, device="cuda"),
                        lse=torch.full((hq, 1), 7.0, device="cuda"), sets=None if sets is None else tuple(_t(x) for x in sets)))
    ck = vs.Chunk(hq, hkv, d, 1, 940, 1.0 / np.sqrt(d), vertical_budget=bv, slash_budget=bs)
    vs.attn_batch(ck, vs.request_table(gpu, "cuda"), n_req, gpu[0]["q"], gpu[0]["k"], gpu[0]["v"], gpu[0]["out"])
    torch.cuda.synchronize()
    for i, ((pb, q, k, v, sets), g) in enumerate(zip(reqs, gpu)):
        ref = oracle.dense_attention(pb, q, k, v) if sets is None else oracle.sparse_attention(pb, q, k, v, *sets)
        assert_attn_close(g["out"], g["lse"], *ref, f"request {i}, s={pb.q_start}")


@pytest.mark.parametrize("lens,mode", [([12000], "dense"), ([3000, 12000, 70, 5000, 64, 1, 900, 2500], "dense"), ([12000, 3000], "both"),
                                       ([70000, 61000], "both")])
def test_bounds_beyond_the_requests(lens, mode):
    """What a table's tokens are is decided by their lengths and index sets, not by the table's bounds: the same bits (where
    the fold has as many waves: it goes by the bounds)."""
    hq, hkv, d, bv, bs = 14, 2, 128, 100, 300
    rng = np.random.default_rng(2400)
    gpu = []
    for i, n in enumerate(lens):
        pb, q, k, v, sets = _problem(rng, hq, hkv, d, n - 1, bv, bs, "both" if mode == "both" and i == 0 else "dense")
        gpu.append(dict(q=dev(q), k=dev(k), v=dev(v), q_start=n - 1, out=torch.zeros((1, hq, d), dtype=torch.bfloat16, device="cuda"),
                        lse=torch.zeros((hq, 1), device="cuda"), sets=None if sets is None else tuple(_t(x) for x in sets)))
    got = []
    table = vs.request_table(gpu, "cuda")
    for bound in (max(lens), 1 << 20):
        ck = vs.Chunk(hq, hkv, d, 1, bound - 1, 1.0 / np.sqrt(d), vertical_budget=bv, slash_budget=bs)
        vs.attn_batch(ck, table, len(lens), gpu[0]["q"], gpu[0]["k"], gpu[0]["v"], gpu[0]["out"])
        torch.cuda.synchronize()
        got.append([(g["out"].clone(), g["lse"].clone()) for g in gpu])
    for a, b in zip(*got):
        assert torch.equal(a[0].view(torch.int16), b[0].view(torch.int16)) and torch.equal(a[1], b[1])


def test_workspaces_without_room_for_neighbouring_heads():
    """Three long tokens, one with index sets of heads that have every diagonal, in the workspace of heads by themselves."""
    hq, hkv, d, bv, bs, n = 6, 2, 128, 100, 1400, 88000
    rng = np.random.default_rng(2500)
    gpu = []
    for i in range(3):
        pb, q, k, v, _ = _problem(rng, hq, hkv, d, n - 1 - 40 * i, bv, bs, "dense")
        sets = None
        if i == 1:
            si = np.full((hq, bs), -1, np.int32)
            si[:, :1375] = 64 * np.arange(1375)
            si[2:4, 700:1375] = np.append(si[2:4, 701:1375], np.full((2, 1), -1), axis=1)   # two heads lack a diagonal
            sets = (np.tile(np.arange(bv, dtype=np.int32) * 7, (hq, 1)), np.full(hq, bv, np.int32), si, (si >= 0).sum(1).astype(np.int32))
        gpu.append(dict(q=dev(q), k=dev(k), v=dev(v), q_start=pb.q_start, out=torch.zeros((1, hq, d), dtype=torch.bfloat16, device="cuda"),
                        lse=torch.zeros((hq, 1), device="cuda"), sets=None if sets is None else tuple(_t(x) for x in sets)))
    ck = vs.Chunk(hq, hkv, d, 1, n - 1, 1.0 / np.sqrt(d), vertical_budget=bv, slash_budget=bs)
    table = vs.request_table(gpu, "cuda")
    apart = ck.params()
    apart.k_stride_tok, apart.k_stride_head = d, d * n   # (heads by themselves)
    least, full = (vs.lib().vs_batch_workspace_bytes(C.byref(p), 3) for p in (apart, ck.params()))
    got = []
    for size in (full, least):
        buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        vs.attn_batch(ck, table, 3, gpu[0]["q"], gpu[0]["k"], gpu[0]["v"], gpu[0]["out"], ws=buf[:size])
        torch.cuda.synchronize()
        assert (buf[size:] == 0x5A).all()
        got.append([(g["out"].clone().float(), g["lse"].clone()) for g in gpu])
    assert least < full
    for a, b in zip(*got):   # bf16 probabilities relative to other references, sums of other parts
        assert (a[0] - b[0]).norm() <= 2e-2 * b[0].norm() and (a[1] - b[1]).abs().max() < 1e-4


def test_as_many_sparse_tokens_as_a_table_takes():
    """4,096 tokens with index sets, 8,192 units: none of them may be taken for one without."""
    hq, hkv, d, n, n_req = 4, 2, 128, 150, 4096
    gen = torch.Generator(device="cuda").manual_seed(2600)
    q, k, v = (torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16) for s in ((1, hq, d), (n, hkv, d), (n, hkv, d)))
    ck = vs.Chunk(hq, hkv, d, 1, n - 1, 1.0 / np.sqrt(d), vertical_budget=20, slash_budget=3)
    si = np.array([[0, -1, -1], [64, -1, -1], [0, 128, -1], [0, 64, 128]], np.int32)   # (the last head has every diagonal)
    vi = np.tile(np.arange(20, dtype=np.int32) * 3, (hq, 1))
    sets = tuple(_t(x) for x in (vi, np.full(hq, 20, np.int32), si, (si >= 0).sum(1).astype(np.int32)))
    want, lse = vs.sparse_attn_prefill(ck, q, k, v, *sets, want_lse=True)
    out = torch.zeros((n_req, 1, hq, d), dtype=torch.bfloat16, device="cuda")
    lses = torch.zeros((n_req, hq, 1), device="cuda")
    table = vs.request_table([dict(q=q, k=k, v=v, q_start=n - 1, out=out[i], lse=lses[i], sets=sets) for i in range(n_req)], "cuda")
    vs.attn_batch(ck, table, n_req, q, k, v, out[0])
    torch.cuda.synchronize()
    assert ((out.float() - want.float()).flatten(1).norm(dim=1) <= 2e-2 * want.float().norm()).all()
    assert (lses - lse).abs().max() < 1e-4
