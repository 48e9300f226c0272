"""The kernel of short calls (one round of short ranges, two sets of waves): where its ranges, its tiles' stages and its lists end, and
against the general kernel over the forms of input that both take."""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_15383_amd as vs
from gpu_util import assert_attn_close, chunk_of, dev, f64
from helpers import rand_bf16
from test_gpu_attention import _rand_sets, _t

pytestmark = pytest.mark.gpu


# One tile and two (a set without any), as many as the stages of either head size hold and one more, ranges of one and of many blocks, 64
# distances; one, two and four heads per tile, a last tile of one query block, rows that start and end inside a block.
@pytest.mark.parametrize("hq,hkv,d,c,n", [
    (1, 1, 64, 3, 3), (2, 1, 64, 70, 70), (4, 1, 64, 130, 130), (1, 1, 64, 65, 4 * 64 + 1), (8, 2, 64, 1024, 1025), (8, 2, 64, 100, 9 * 64),
    (200, 50, 64, 17, 8 * 64 + 3), (4, 1, 64, 1, 17 * 64), (4, 1, 64, 129, 511 * 64 + 5),
    (1, 1, 128, 5, 5), (7, 1, 128, 64, 128), (7, 1, 128, 63, 2 * 64 + 1), (3, 3, 128, 200, 5 * 64), (28, 4, 128, 33, 40 * 64 + 1),
    (28, 4, 128, 500, 14 * 64), (40, 8, 128, 31, 64 * 64 - 1), (6, 2, 128, 66, 512 * 64)])
def test_ranges_stages_and_lists_of_short_calls(hq, hkv, d, c, n):
    s = n - c
    rng = np.random.default_rng(5000 + n + c)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (n, hkv, d)); v = rand_bf16(rng, (n, hkv, d))
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d), vertical_budget=min(n, 200), slash_budget=min(n, 130), keep_first_cols=0,
                        keep_local_band=0)
    ck = chunk_of(pb)
    rows = sorted({0, c // 2, c - 1, min(c - 1, 64), min(c - 1, 127)}) if n * c > 100000 else None
    at = torch.tensor(rows if rows else list(range(c)), device="cuda")

    def close(got, ref, what):
        assert_attn_close(got[0][at], got[1][:, at], *ref, f"{what} {hq}/{hkv} D={d} C={c} n={n}")
    got = vs.dense_causal_prefill(ck, dev(q), dev(k), dev(v), want_lse=True)
    torch.cuda.synchronize()
    close(got, oracle.dense_attention(pb, q, k, v, rows=rows), "dense")
    for nv, ns in ((min(n, 200), min(n, 7)), (1, 0), (0, 1), (min(n, 65), min(n, 130))):
        sets = _rand_sets(rng, pb, nv, ns)
        for h in range(0, hq, 2):   # heads of a tile with lists of different lengths
            keep = int(sets[1][h]) // 2
            sets[0][h, keep:] = -1; sets[1][h] = keep
        for byte in (0, 0xA5):
            ws = torch.full((max(256, vs.workspace_bytes(ck, vs.VS_WS_SPARSE)),), byte, dtype=torch.uint8, device="cuda")
            got = vs.sparse_attn_prefill(ck, dev(q), dev(k), dev(v), *[_t(x) for x in sets], want_lse=True, ws=ws)
            torch.cuda.synchronize()
            close(got, oracle.sparse_attention(pb, q, k, v, *sets, rows=rows), f"sparse, {nv} columns {ns} offsets")


# Caches by token and by KV head, a slice of a fused buffer; offsets in any order (no order is asked of them), scores that outrun
# the reference by more than 2^64 in a later tile.  The general kernel is what a split that is asked for takes (1: none).
@pytest.mark.parametrize("hq,hkv,d,c,n,pack_kv", [(8, 2, 64, 300, 3000, False), (28, 4, 128, 40, 2500, True), (4, 1, 128, 100, 1900, True)])
def test_short_calls_against_the_general_kernel(hq, hkv, d, c, n, pack_kv):
    gen = torch.Generator(device="cuda").manual_seed(5100 + n)
    rnd = lambda *size: torch.randn(size, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    q = rnd(c, hq + 2 * hkv, d)[:, hkv:hkv + hq]
    kv = rnd(2, hkv, n, d).transpose(1, 2) if pack_kv else rnd(2, n, hkv, d)
    k, v = kv[0], kv[1]
    k[:64] *= 40.0   # the far end: met last
    ck = vs.Chunk(hq, hkv, d, c, n - c, 1.0 / np.sqrt(d), vertical_budget=150, slash_budget=90)
    v_idx = torch.stack([torch.randperm(n, generator=gen, device="cuda")[:150].sort().values for _ in range(hq)]).int()
    s_idx = torch.stack([torch.randperm(n, generator=gen, device="cuda")[:90] for _ in range(hq)]).int()
    cnt = lambda m: torch.full((hq,), m, dtype=torch.int32, device="cuda")  # noqa: E731
    sets = (v_idx, cnt(150), s_idx, cnt(90))
    got = {}
    for split in (0, 1):
        try:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, split)
            got[split] = (*vs.dense_causal_prefill(ck, q, k, v, want_lse=True), *vs.sparse_attn_prefill(ck, q, k, v, *sets, want_lse=True))
            torch.cuda.synchronize()
        finally:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 0)
    for i in (0, 2):
        a, b = got[0][i].float(), got[1][i].float()
        # bf16 probabilities and outputs on either side: 2^-9 each, unbiased, about 6e-3 between the two
        assert ((a - b).norm(dim=2) <= 2e-2 * b.norm(dim=2) + 1e-30).all()
        la, lb = f64(got[0][i + 1]), f64(got[1][i + 1])
        np.testing.assert_allclose(la, lb, rtol=2e-5, atol=2e-5)
