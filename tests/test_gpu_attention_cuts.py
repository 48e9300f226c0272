"""The ways the tile kernel cuts a launch into units and pieces: heads that share a tile (rows of one query block, at every
place in it and at 32 / 33 rows, where two or four heads fit), whole units next to cut ones (with and without pace
keeping), and plans over batches of more requests than a wave, and than a workgroup, looks at in one go.  Against the fp64
oracle, at the largest sizes on a sample of rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_15383_amd as vs
from gpu_util import assert_attn_close, chunk_of, dev, f64
from helpers import rand_bf16
from test_gpu_attention import _rand_sets, _t
from test_gpu_batch import _check, _make_requests, _run_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d", [(7, 1, 128), (6, 3, 64), (5, 1, 64), (3, 3, 128)])
@pytest.mark.parametrize("c,place", [(2, 0), (31, 33), (32, 32), (32, 33), (33, 31), (33, 0), (63, 1), (64, 0)])
@pytest.mark.parametrize("blocks", [1, 40, 70])   # key blocks before the chunk's: one range, a few, a second batch of entries
def test_heads_that_share_a_tile(hq, hkv, d, c, place, blocks):
    s = 64 * blocks + place
    rng = np.random.default_rng(3000 + s + c)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (s + c, hkv, d)); v = rand_bf16(rng, (s + c, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d), vertical_budget=160, slash_budget=90, keep_first_cols=0, keep_local_band=0)
    ref = oracle.dense_attention(pb, q, k, v)
    got = vs.dense_causal_prefill(chunk_of(pb), dev(q), dev(k), dev(v), want_lse=True)
    torch.cuda.synchronize()
    assert_attn_close(*got, *ref, f"dense {hq}/{hkv} C={c} s={s}")
    for nv, ns in ((150, 6), (65, 0), (0, 20)):   # no diagonal, no column: rows without any key among them
        sets = _rand_sets(rng, pb, nv, ns)
        for h in range(0, hq, 2):   # heads of a tile with lists of different lengths
            keep = int(sets[1][h]) // 2
            sets[0][h, keep:] = -1; sets[1][h] = keep
        ref = oracle.sparse_attention(pb, q, k, v, *sets)
        got = vs.sparse_attn_prefill(chunk_of(pb), dev(q), dev(k), dev(v), *[_t(x) for x in sets], want_lse=True)
        torch.cuda.synchronize()
        assert_attn_close(*got, *ref, f"sparse {hq}/{hkv} C={c} s={s} {nv} columns {ns} offsets")


@pytest.mark.parametrize("blocks", [4, 11, 12, 22, 23])   # 160 columns: four heads of a tile from 24 blocks on, two from 12
def test_heads_that_share_a_tile_as_the_columns_let_them(blocks):
    test_heads_that_share_a_tile(7, 1, 128, 20, 5, blocks)


# Dense calls of few pieces have no block list and no cleared counters: one, two and four heads per tile, one range and many, walks
# of less and more than a batch of 64 entries, with a workspace of another call's bytes.
@pytest.mark.parametrize("hq,hkv,d,c,s", [(4, 1, 64, 130, 64 * 130 + 5), (7, 1, 128, 65, 64 * 66), (8, 2, 128, 20, 64 * 129 + 3),
                                          (6, 3, 64, 64, 64 * 63), (1, 1, 128, 300, 10), (5, 1, 128, 2, 61), (40, 8, 128, 129, 64 * 16 + 1)])
def test_dense_calls_without_a_list(hq, hkv, d, c, s):
    rng = np.random.default_rng(3050 + s + c)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (s + c, hkv, d)); v = rand_bf16(rng, (s + c, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d))
    ck = chunk_of(pb)
    for byte in (0, 0xA5):
        ws = torch.full((max(256, vs.workspace_bytes(ck, vs.VS_WS_DENSE)),), byte, dtype=torch.uint8, device="cuda")
        got = vs.dense_causal_prefill(ck, dev(q), dev(k), dev(v), want_lse=True, ws=ws)
        torch.cuda.synchronize()
        assert_attn_close(*got, *oracle.dense_attention(pb, q, k, v), f"dense {hq}/{hkv} C={c} s={s}")


# Ranges of two and three key blocks, the last of them of one key, and lists shorter than the ranges that are cut from them.
@pytest.mark.parametrize("hq,hkv,d", [(7, 1, 128), (4, 2, 64)])
@pytest.mark.parametrize("c,n", [(3, 4 * 64 - 1), (3, 4 * 64), (33, 5 * 64 + 1), (65, 17 * 64), (140, 9 * 64 + 1)])
def test_ranges_of_a_few_blocks(hq, hkv, d, c, n):
    s = n - c
    rng = np.random.default_rng(3080 + n + c)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (n, hkv, d)); v = rand_bf16(rng, (n, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d), vertical_budget=70, slash_budget=90, keep_first_cols=0, keep_local_band=0)
    got = vs.dense_causal_prefill(chunk_of(pb), dev(q), dev(k), dev(v), want_lse=True)
    torch.cuda.synchronize()
    assert_attn_close(*got, *oracle.dense_attention(pb, q, k, v), f"dense {hq}/{hkv} C={c} n={n}")
    for nv, ns in ((70, 3), (1, 0), (0, 1)):
        sets = _rand_sets(rng, pb, min(nv, n), ns)
        got = vs.sparse_attn_prefill(chunk_of(pb), dev(q), dev(k), dev(v), *[_t(x) for x in sets], want_lse=True)
        torch.cuda.synchronize()
        assert_attn_close(*got, *oracle.sparse_attention(pb, q, k, v, *sets), f"sparse {hq}/{hkv} C={c} n={n} {nv} columns {ns} offsets")


# A call's ranges, however short, are as near to 64 bits as its walk in one piece: the probabilities of a range are rounded to bf16
# relative to a reference of its own, by 2^-9 at most all the same.  Other roundings, so the two differ by about sqrt(2) of either's
# error; the error itself is the same but for chance.  Squared errors of n independent values give their root mean to 1 / sqrt(2 n):
# 0.3 % for the 532 rows of 128 of the smallest call, 3 % if all values of a row moved as one; 5 % are allowed.
@pytest.mark.parametrize("hq,hkv,d,c,n", [(28, 4, 128, 138, 2869), (28, 4, 128, 214, 2337), (8, 2, 64, 234, 14394), (40, 8, 128, 35, 954),
                                          (28, 4, 128, 19, 22035), (4, 1, 64, 191, 1866)])
def test_ranges_lose_no_precision(hq, hkv, d, c, n):
    rng = np.random.default_rng(3090 + n)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (n, hkv, d)); v = rand_bf16(rng, (n, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, n - c, 1.0 / np.sqrt(d))
    ref = oracle.dense_attention(pb, q, k, v)[0].transpose(1, 0, 2)
    err, size = [], []
    for split in (0, 1):
        try:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, split)
            size.append(vs.workspace_bytes(chunk_of(pb), vs.VS_WS_DENSE))
            got = vs.dense_causal_prefill(chunk_of(pb), dev(q), dev(k), dev(v))[0]
            torch.cuda.synchronize()
        finally:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 0)
        err.append(np.linalg.norm(f64(got) - ref) / np.linalg.norm(ref))
    assert size[0] > size[1]   # (it was cut)
    assert err[0] <= 1.05 * err[1], err


@pytest.mark.parametrize("c,s", [(66 * 128 - 5, 70), (66 * 128 - 5, 4100 * 64 + 1)])   # 528 units: 512 whole, 16 cut
def test_whole_units_and_cut_ones(c, s):
    hq, hkv, d = 8, 1, 64
    rng = np.random.default_rng(3100)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (s + c, hkv, d)); v = rand_bf16(rng, (s + c, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d), vertical_budget=300, slash_budget=400)
    out, lse = vs.dense_causal_prefill(chunk_of(pb), dev(q), dev(k), dev(v), want_lse=True)
    sets = _rand_sets(rng, pb, 290, 300, force_cols=[0], force_offs=range(64))
    out_s, lse_s = vs.sparse_attn_prefill(chunk_of(pb), dev(q), dev(k), dev(v), *[_t(x) for x in sets], want_lse=True)
    torch.cuda.synchronize()
    # rows of the first, of the last whole and of the cut tiles
    for rows in ([0, 57, 58, 191], [c - 1, c - 128, c // 2]):
        at = torch.tensor(rows, device="cuda")
        ref = oracle.dense_attention(pb, q, k, v, rows=rows)
        assert_attn_close(out[at], lse[:, at], *ref, f"dense C={c} s={s} rows {rows}")
        ref = oracle.sparse_attention(pb, q, k, v, *sets, rows=rows)
        assert_attn_close(out_s[at], lse_s[:, at], *ref, f"sparse C={c} s={s} rows {rows}")
    # all rows against the kernel that cuts nothing: both within the rounding of bf16 probabilities and outputs
    vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 1)
    try:
        p, lp = vs.dense_causal_prefill(chunk_of(pb), dev(q), dev(k), dev(v), want_lse=True)
        ps, lps = vs.sparse_attn_prefill(chunk_of(pb), dev(q), dev(k), dev(v), *[_t(x) for x in sets], want_lse=True)
        torch.cuda.synchronize()
    finally:
        vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 0)
    for a, b, la, lb in ((out, p, lse, lp), (out_s, ps, lse_s, lps)):
        a, b = a.float(), b.float()
        assert ((a - b).norm(dim=2) <= 2e-2 * b.norm(dim=2)).all() and (la - lb).abs().max().item() < 1e-4


# the same with Dual Chunk Attention: chunk boundaries inside the rows and the window's end inside key blocks, sampled around
# both and in whole and cut tiles
@pytest.mark.parametrize("c,s,chunk,window", [(66 * 128 - 5, 70, 3200, 320), (66 * 128 - 5, 4100 * 64 + 1, 4130 * 64, 576)])
def test_whole_units_and_cut_ones_with_dca(c, s, chunk, window):
    hq, hkv, d = 8, 1, 64
    rng = np.random.default_rng(3110)
    qs = [rand_bf16(rng, (c, hq, d)) for _ in range(3)]
    k = rand_bf16(rng, (s + c, hkv, d)); v = rand_bf16(rng, (s + c, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d), vertical_budget=300, slash_budget=400)
    ref_dca = oracle.Dca(chunk, window, qs[1], qs[2])
    gpu_dca = (dev(qs[1]), dev(qs[2]), chunk, window)
    out, lse = vs.dense_causal_prefill(chunk_of(pb), dev(qs[0]), dev(k), dev(v), want_lse=True, dca=gpu_dca)
    sets = _rand_sets(rng, pb, 290, 300, force_cols=[0], force_offs=range(64))
    out_s, lse_s = vs.sparse_attn_prefill(chunk_of(pb), dev(qs[0]), dev(k), dev(v), *[_t(x) for x in sets], want_lse=True,
                                          dca=gpu_dca)
    torch.cuda.synchronize()
    bound = chunk - s % chunk   # the first row of the next chunk
    for rows in ([0, 57, 58, 191], [bound - 1, bound, bound + 40, bound + window], [c - 1, c - 128, c // 2]):
        at = torch.tensor(rows, device="cuda")
        ref = oracle.dense_attention(pb, qs[0], k, v, rows=rows, dca=ref_dca)
        assert_attn_close(out[at], lse[:, at], *ref, f"dense dca C={c} s={s} rows {rows}")
        ref = oracle.sparse_attention(pb, qs[0], k, v, *sets, rows=rows, dca=ref_dca)
        assert_attn_close(out_s[at], lse_s[:, at], *ref, f"sparse dca C={c} s={s} rows {rows}")


# block lists of more diagonals than their builders hold at a time: 16 heads of a token (8,192), packed heads (16,448), one head (65,792)
@pytest.mark.parametrize("hq,c,win", [(16, 1, 8192), (7, 1, 16384), (4, 2, 16448), (2, 70, 65792)])
def test_lists_of_several_windows(hq, c, win):
    d, n = 64, 64 * win + 1000
    gen = torch.Generator(device="cuda").manual_seed(3140)
    q = torch.randn((c, hq, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    k = torch.randn((n, 1, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    v = torch.randn((n, 1, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    rng = np.random.default_rng(3141)
    ck = vs.Chunk(hq, 1, d, c, n - c, 0.125, vertical_budget=40, slash_budget=1500)
    vi = np.full((hq, 40), -1, np.int32); si = np.full((hq, 1500), -1, np.int32)
    sc = np.zeros(hq, np.int32)
    for h in range(hq):
        vi[h] = np.sort(rng.choice(n - c, 40, replace=False))
        edge = 64 * win - 64 * (h % 3) + np.arange(-1, 2 + 100 * (h % 2))   # both sides of the window's end
        offs = np.unique(np.concatenate([np.arange(3), edge, [n - 1], rng.choice(n, 40 * (1 + h), replace=False)]))
        sc[h] = len(offs); si[h, :sc[h]] = offs
    _check_by_gathering(ck, q, k, v, vi, si, sc)


# the two ways to make bitmaps: 4,096 diagonals and one more, of four heads and of one, an odd word and a part of one behind them
@pytest.mark.parametrize("n", [64 * 4096, 64 * 4096 + 1, 64 * 4128 + 17])
@pytest.mark.parametrize("hq,c", [(7, 2), (2, 70)])
def test_lists_at_the_line_between_ballots_and_lanes(hq, c, n):
    d = 64
    gen = torch.Generator(device="cuda").manual_seed(3170)
    q, k, v = (torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16) for s in ((c, hq, d), (n, 1, d), (n, 1, d)))
    rng = np.random.default_rng(3171)
    ck = vs.Chunk(hq, 1, d, c, n - c, 0.125, vertical_budget=40, slash_budget=4500)
    vi = np.full((hq, 40), -1, np.int32); si = np.full((hq, 4500), -1, np.int32)
    sc = np.zeros(hq, np.int32)
    for h in range(hq):
        vi[h] = np.sort(rng.choice(n - c, 40, replace=False))
        offs = 64 * np.arange((n + 63) // 64) if h % 3 == 1 else np.unique(np.concatenate([[0, n - 1], rng.choice(n, 30 * (1 + h), replace=False)]))
        if h == 4: offs = offs[:-1]   # all but the last diagonal
        sc[h] = len(offs); si[h, :sc[h]] = offs
    _check_by_gathering(ck, q, k, v, vi, si, sc)


# heads that have every diagonal, whose columns nobody gathers, beside heads that lack one diagonal (the first, one inside, the last) and
# have columns in its key block: single tokens, packed heads, tiles of two query blocks
@pytest.mark.parametrize("hq,c,n", [(3, 1, 1000), (7, 1, 64), (4, 2, 1000), (5, 40, 2048), (3, 130, 1000), (2, 300, 4999)])
def test_columns_of_heads_that_have_every_diagonal(hq, c, n):
    d, n_blk = 64, (n + 63) // 64
    gen = torch.Generator(device="cuda").manual_seed(3150)
    q, k, v = (torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16) for s in ((c, hq, d), (n, 1, d), (n, 1, d)))
    rng = np.random.default_rng(3151)
    ck = vs.Chunk(hq, 1, d, c, n - c, 0.125, vertical_budget=70, slash_budget=n_blk)
    vi = np.full((hq, 70), -1, np.int32); si = np.full((hq, n_blk), -1, np.int32)
    sc = np.zeros(hq, np.int32)
    for h in range(hq):
        n_col = min(70, n)
        vi[h, :n_col] = np.sort(rng.choice(n, n_col, replace=False))
        offs = 64 * np.arange(n_blk)
        if h % 4: offs = np.delete(offs, [0, n_blk // 2, n_blk - 1][h % 4 - 1])
        sc[h] = len(offs); si[h, :sc[h]] = offs
    _check_by_gathering(ck, q, k, v, vi, si, sc)
    if c > 1: return
    # the same token in a batch beside one without index sets
    sets = [_t(x) for x in (vi, (vi >= 0).sum(1).astype(np.int32), si, sc)]
    outs = [torch.empty_like(q) for _ in range(2)]
    reqs = [dict(q=q, k=k, v=v, out=outs[x], q_start=n - c, lse=None, sets=tuple(sets) if x == 0 else None) for x in range(2)]
    vs.attn_batch(ck, vs.request_table(reqs, q.device), 2, q, k, v, outs[0])
    one = vs.sparse_attn_prefill(ck, q, k, v, *sets)
    torch.cuda.synchronize()
    assert (outs[0].float() - (one[0] if isinstance(one, tuple) else one).float()).norm() <= 2e-2 * outs[0].float().norm()


def _check_by_gathering(ck, q, k, v, vi, si, sc):
    """Outputs of one KV head against fp32 softmax over the keys that the sets name, gathered."""
    (c, hq, _), n = q.shape, k.shape[0]
    out = vs.sparse_attn_prefill(ck, q, k, v, *[_t(x) for x in (vi, (vi >= 0).sum(1).astype(np.int32), si, sc)])
    out = out[0] if isinstance(out, (tuple, list)) else out
    for h in range(hq):
        offs = torch.as_tensor(si[h, :sc[h]], device="cuda").long()
        ad = torch.cat([offs // 64, (offs + 63) // 64]).unique()
        for r in {0, c // 2, c - 1}:
            pos = n - c + r
            blocks = pos // 64 - ad[ad <= pos // 64]
            keys = (64 * blocks[:, None] + torch.arange(64, device="cuda")).flatten()
            keys = torch.cat([keys, torch.as_tensor(vi[h][vi[h] >= 0], device="cuda").long()]).unique()
            keys = keys[keys <= pos]
            p = torch.softmax((k[keys, 0].float() @ q[r, h].float()) * 0.125, 0)
            ref = p @ v[keys, 0].float()
            # as everywhere: probabilities and outputs are rounded to bf16
            assert (out[r, h].float() - ref).norm() <= 2e-2 * ref.norm(), (h, r)


def test_ranges_that_are_asked_for_of_many_units():
    hq, hkv, d, c, s = 1100, 10, 64, 512, 2048 + 33   # 5,500 units, 41 key blocks: two ranges of each
    rng = np.random.default_rng(3120)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (s + c, hkv, d)); v = rand_bf16(rng, (s + c, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d))
    got = []
    for n in (0, 2):
        vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, n)
        try:
            got.append((vs.workspace_bytes(chunk_of(pb), vs.VS_WS_DENSE),
                        *vs.dense_causal_prefill(chunk_of(pb), dev(q), dev(k), dev(v), want_lse=True)))
            torch.cuda.synchronize()
        finally:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 0)
    assert got[1][0] - got[0][0] == 2 * 5500 * 128 * (d + 2) * 4
    heads, rows = [0, 109, 110, 700, 1099], [0, 94, 95, 300, 511]
    at = torch.tensor(rows, device="cuda")
    ref = oracle.dense_attention(pb, q, k, v, heads=heads, rows=rows)
    for _, out, lse in got:
        assert_attn_close(out[at][:, heads], lse[heads][:, at], *ref, f"{hq} heads")
    (_, a, la), (_, b, lb) = got
    assert ((a.float() - b.float()).norm(dim=2) <= 2e-2 * b.float().norm(dim=2)).all() and (la - lb).abs().max().item() < 1e-4


def _guarded(n):
    """A workspace of n bytes and the bytes behind it."""
    buf = torch.full((n + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    return buf[:n], buf[n:]


def test_workspaces_without_room_for_uneven_ranges():
    """448 units that are whole with even ranges: a workspace that holds nothing of partial results is taken (and not left), for a
    sparse call and for a chunk; one byte less is refused."""
    ck = vs.Chunk(32, 2, 64, 1792, 66000, 0.125, vertical_budget=100, slash_budget=500)
    gen = torch.Generator(device="cuda").manual_seed(3160)
    q, k, v = (torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16) for s in ((1792, 32, 64), (ck.n_k, 2, 64), (ck.n_k, 2, 64)))
    sets = vs.select(ck, *vs.estimate(ck, q, k)[:2])
    calls = ((vs.VS_WS_SPARSE, lambda ws: vs.sparse_attn_prefill(ck, q, k, v, *sets, want_lse=True, ws=ws)),
             (vs.VS_WS_CHUNK, lambda ws: vs.prefill_chunk(ck, q, k, v, want_lse=True, ws=ws)))
    for which, call in calls:
        full = vs.workspace_bytes(ck, which)
        try:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 1)
            least = vs.workspace_bytes(ck, which)
            want = call(_guarded(least)[0])
        finally:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 0)
        assert full - least > 50e6
        ws, behind = _guarded(least)
        got = call(ws)
        torch.cuda.synchronize()
        assert torch.equal(got[0].view(torch.int16), want[0].view(torch.int16)) and torch.equal(got[1], want[1])
        assert (behind == 0x5A).all()
        with pytest.raises(vs.VsError) as e:
            call(_guarded(least)[0][:-1])
        assert e.value.status == vs.VS_ERR_WORKSPACE


def _uneven_pieces(ws):
    """What k_attn_pieces left in the workspace of a sparse call: the number of pieces of an uneven cut, 0 where the even one stayed.  Behind
    it, at the end of the workspace, lie 256 bytes less one word, 2,048 units (8 bytes) and 2,048 pieces (32 bytes)."""
    at = ws.numel() - 256 - 2048 * (8 + 32)
    torch.cuda.synchronize()
    return int(ws[at:at + 4].view(torch.int32).item())


@pytest.mark.parametrize("differ", [0, 1])
def test_lists_of_about_one_length_keep_even_ranges(differ):
    hq, c, s = 32, 450, 20007
    ck = vs.Chunk(hq, 2, 64, c, s, 0.125, vertical_budget=100, slash_budget=2000)
    gen = torch.Generator(device="cuda").manual_seed(3180)
    q, k, v = (torch.randn(x, generator=gen, device="cuda", dtype=torch.bfloat16) for x in ((c, hq, 64), (s + c, 2, 64), (s + c, 2, 64)))
    si = np.full((hq, 2000), -1, np.int32); sc = np.full(hq, 150, np.int32)
    for h in range(hq):
        sc[h] -= differ * (h % 3)
        si[h, :sc[h]] = 128 * np.arange(sc[h])
    ws = torch.zeros(vs.workspace_bytes(ck, vs.VS_WS_SPARSE), dtype=torch.uint8, device="cuda")
    vi = np.tile(np.arange(100, dtype=np.int32), (hq, 1))
    vs.sparse_attn_prefill(ck, q, k, v, *[_t(x) for x in (vi, np.full(hq, 100, np.int32), si, sc)], ws=ws)
    assert _uneven_pieces(ws) == 0


# heads whose lists differ by a factor of ten, and one with everything selected: ranges by the lists' own lengths (k_attn_pieces), of
# units in several ranges (128 units), of units that are whole with even ranges (448), and of 528 of which 512 are whole units in front
@pytest.mark.parametrize("hq,hkv,c,s,chunk", [(32, 2, 450, 20007, 0), (32, 2, 1792, 66000, 0), (8, 1, 65 * 128 - 9, 140009, 0),
                                              (32, 2, 450, 20007, 6400)])
def test_ranges_by_the_lists_own_lengths(hq, hkv, c, s, chunk):
    d, n = 64, s + c
    rng = np.random.default_rng(3130)
    qs = [rand_bf16(rng, (c, hq, d)) for _ in range(3 if chunk else 1)]
    k = rand_bf16(rng, (n, hkv, d)); v = rand_bf16(rng, (n, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d), vertical_budget=100, slash_budget=2500)
    vi = np.full((hq, 100), -1, np.int32); si = np.full((hq, 2500), -1, np.int32)
    vc = rng.integers(1, 101, hq).astype(np.int32); sc = np.zeros(hq, np.int32)
    for h in range(hq):
        vi[h, :vc[h]] = np.sort(np.concatenate([[0], 1 + rng.choice(n - 1, vc[h] - 1, replace=False)]))
        far = n // 16 if h % 4 == 1 else n   # (clustered)
        offs = np.union1d(np.arange(64), rng.choice(far, 1900 if h % 4 == 2 else 20 + 5 * h, replace=False))
        if h == 3: offs = np.minimum(np.arange(0, n + 63, 64), n - 1)   # every diagonal
        sc[h] = len(offs)
        si[h, :sc[h]] = offs
    dca = (dev(qs[1]), dev(qs[2]), chunk, 640) if chunk else None
    args = (chunk_of(pb), dev(qs[0]), dev(k), dev(v), *[_t(x) for x in (vi, vc, si, sc)])
    ws = torch.zeros(vs.workspace_bytes(chunk_of(pb), vs.VS_WS_SPARSE), dtype=torch.uint8, device="cuda")
    out, lse = vs.sparse_attn_prefill(*args, want_lse=True, dca=dca, ws=ws)
    pieces = _uneven_pieces(ws)
    # by length: more than one a unit, and not a multiple of the units as with the same number of ranges for all
    n_cut = hq * ((c + s % 64 + 127) // 128) % 512
    assert n_cut < pieces <= 2048 and pieces % n_cut, (pieces, n_cut)
    again, lse_again = vs.sparse_attn_prefill(*args, want_lse=True, dca=dca)
    vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 1)
    try:
        one, lse_one = vs.sparse_attn_prefill(*args, want_lse=True, dca=dca)
    finally:
        vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 0)
    torch.cuda.synchronize()
    assert torch.equal(out, again) and torch.equal(lse, lse_again)
    # both within the rounding of bf16 probabilities and outputs
    a, b = out.float(), one.float()
    assert ((a - b).norm(dim=2) <= 2e-2 * b.norm(dim=2)).all() and (lse - lse_one).abs().max().item() < 1e-4
    rows, heads = [0, 127, 128, c // 2, c - 1], [0, 1, 2, 3, hq - 1]
    at = torch.tensor(rows, device="cuda")
    ref = oracle.sparse_attention(pb, qs[0], k, v, vi, vc, si, sc, heads=heads, rows=rows,
                                  **(dict(dca=oracle.Dca(chunk, 640, qs[1], qs[2])) if chunk else {}))
    assert_attn_close(out[at][:, heads], lse[heads][:, at], *ref, f"C={c} s={s}")


# one KV head, 64 rows and as many keys as whole units keep pace from: 515 tiles of two heads, 512 of them whole and the last
# three cut; and the same heads behind a start inside a block (two query blocks: no sharing, 1,030 units)
@pytest.mark.parametrize("s", [4095 * 64, 4096 * 64 + 9])
def test_whole_tiles_of_shared_heads_at_long_contexts(s):
    hq, hkv, d, c = 1030, 1, 64, 64
    rng = np.random.default_rng(3150)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (s + c, hkv, d)); v = rand_bf16(rng, (s + c, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d), vertical_budget=100, slash_budget=90)
    heads = [0, 1, 255, 511, 512, 513, 700, 1022, 1023, 1024, 1029]   # both heads of a tile; whole and cut tiles
    rows = [0, 31, 32, 63]
    at = torch.tensor(rows, device="cuda")
    few = oracle.Problem(7, 1, d, c, s, 1.0 / np.sqrt(d), vertical_budget=100, slash_budget=90)
    sets = [x[np.arange(hq) % 7] for x in _rand_sets(rng, few, 90, 20, force_cols=[0], force_offs=range(64))]
    for name, call, want in (
            ("dense", lambda o: vs.dense_causal_prefill(chunk_of(pb), dev(q), dev(k), dev(v), want_lse=True, out=o),
             lambda: oracle.dense_attention(pb, q, k, v, heads=heads, rows=rows)),
            ("sparse", lambda o: vs.sparse_attn_prefill(chunk_of(pb), dev(q), dev(k), dev(v), *[_t(x) for x in sets],
                                                        want_lse=True, out=o),
             lambda: oracle.sparse_attention(pb, q, k, v, *sets, heads=heads, rows=rows))):
        o = torch.full((c, hq, d), 7.0, dtype=torch.bfloat16, device="cuda")
        out, lse = call(o)
        torch.cuda.synchronize()
        assert not (out == 7.0).all(dim=2).any(), f"{name}: rows that nobody wrote"
        assert_attn_close(out[at][:, heads], lse[heads][:, at], *want(), f"{name}, {hq} heads, s={s}")


@pytest.mark.parametrize("n_req", [70, 1030])
def test_plans_over_many_requests(n_req):
    hq, hkv, d, bv, bs = 4, 2, 64, 40, 90
    rng = np.random.default_rng(3200 + n_req)
    specs = [(int(rng.integers(2, 5)), int(rng.integers(0, 150)), bool(i % 3 == 0)) for i in range(n_req)]
    specs[n_req // 2] = (130, 9000, False)   # one that is cut, between short ones
    specs[-1] = (40, 5000, True)
    reqs = _make_requests(rng, hq, hkv, d, specs, bv, bs)
    skipped = n_req // 2 + 1

    def poison(table):
        table[skipped, 2] = 0   # no values: skipped, between two that are taken
    a = _run_batch(reqs, hq, hkv, d, bv, bs, poison=poison)
    b = _run_batch(reqs, hq, hkv, d, bv, bs, poison=poison)
    for x, y in zip(a, b):
        assert torch.equal(x["out"].view(torch.int16), y["out"].view(torch.int16)) and torch.equal(x["lse"], y["lse"])
    assert (a[skipped]["out"].float() == -3.0).all() and (a[skipped]["lse"] == 7.0).all()
    _check(reqs, a, skip=(skipped,))


def test_more_lists_than_a_launch_takes_along_y():
    hq, hkv, d, bv, bs, n_req = 24, 1, 64, 20, 70, 4096   # 98,304 lists (the y axis of a launch takes 65,535)
    rng = np.random.default_rng(3250)
    specs = [(int(rng.integers(1, 4)), int(rng.integers(0, 130)), i % 16 == 5) for i in range(n_req)]
    reqs = _make_requests(rng, hq, hkv, d, specs, bv, bs)
    got = _run_batch(reqs, hq, hkv, d, bv, bs)
    lse = torch.cat([g["lse"].reshape(-1) for g in got])
    assert not (lse == 7.0).any(), "rows that nobody wrote"
    some = [0, 5, 2729, 2730, 2731, 4085, 4095] + rng.integers(0, n_req, 60).tolist()   # 65,536 / 24 = 2,730.7
    _check([reqs[i] for i in some], [got[i] for i in some])


def test_a_batch_without_any_request_to_take():
    hq, hkv, d, bv, bs = 4, 2, 64, 40, 90
    reqs = _make_requests(np.random.default_rng(3300), hq, hkv, d, [(20, 300, False), (5, 100, True)], bv, bs)

    def poison(table):
        table[:, 0] = 0   # no queries
    for g in _run_batch(reqs, hq, hkv, d, bv, bs, poison=poison):
        assert (g["out"].float() == -3.0).all() and (g["lse"] == 7.0).all()
