"""With every offset selected a sparse call runs the tiles of the dense one in the same order: the same bits, whichever kernel takes the shape
and wherever its diagonals come from."""
import numpy as np
import pytest
import torch

import paper_2501_15383_amd as vs

pytestmark = pytest.mark.gpu


# Offsets that a workgroup of the short kernel collects by itself, up to 65,536 of a tile's 4, 2 or 1 heads, and more of them, which come from
# lists (from 16,385 keys on with four heads per tile, the last of which is not full; the most keys); rows that start inside a block, a few and 64
# key blocks per range; the general kernel (33,000 keys, 2,000 rows); whole units that keep pace where those of the dense call do not
@pytest.mark.parametrize("hq,hkv,d,c,n", [
    (28, 4, 128, 16, 1024), (28, 4, 128, 16, 8000), (28, 4, 128, 4, 5000), (28, 4, 128, 32, 12000), (28, 4, 128, 32, 16384), (28, 4, 128, 32, 16385),
    (28, 4, 128, 9, 20009), (28, 4, 128, 8, 30000), (28, 4, 128, 32, 32768), (8, 1, 64, 32, 32768), (5, 1, 64, 20, 18000), (40, 8, 128, 64, 16000),
    (7, 1, 128, 50, 9000), (3, 1, 128, 300, 16400), (4, 1, 64, 300, 20000), (8, 2, 64, 100, 17000), (8, 2, 64, 64, 25024), (4, 1, 64, 1000, 18000),
    (4, 1, 64, 200, 16000), (2, 1, 64, 70, 32768), (1, 1, 64, 500, 32767), (4, 1, 64, 17, 33000), (28, 4, 128, 2000, 3000),
    (8, 2, 64, 16512, 262272)])
def test_all_offsets_give_the_bits_of_the_dense_call(hq, hkv, d, c, n):
    gen = torch.Generator(device="cuda").manual_seed(5500 + n + c)
    rnd = lambda *size: torch.randn(size, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    q, k, v = rnd(c, hq, d), rnd(n, hkv, d), rnd(n, hkv, d)
    ck = vs.Chunk(hq, hkv, d, c, n - c, 1.0 / np.sqrt(d), vertical_budget=3, slash_budget=n)
    full = lambda m: torch.full((hq,), m, dtype=torch.int32, device="cuda")  # noqa: E731
    offsets = torch.stack([torch.randperm(n, generator=gen, device="cuda") for _ in range(hq)]).int()
    columns = torch.tensor([[0, 1, n - 1]] * hq, dtype=torch.int32, device="cuda")
    want = vs.dense_causal_prefill(ck, q, k, v, want_lse=True)
    for byte in (0, 0xA5):
        ws = torch.full((vs.workspace_bytes(ck, vs.VS_WS_SPARSE),), byte, dtype=torch.uint8, device="cuda")
        got = vs.sparse_attn_prefill(ck, q, k, v, columns, full(3), offsets, full(n), want_lse=True, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(got[0].view(torch.int16), want[0].view(torch.int16)) and torch.equal(got[1], want[1])


# Diagonals from lists of some of the offsets, in any order, beside gathered columns: the kernel that a split that is asked for takes (1: none)
@pytest.mark.parametrize("hq,hkv,d,c,n,bs,used", [(28, 4, 128, 32, 20000, 18000, 400), (5, 1, 64, 20, 32768, 32768, 70), (28, 4, 128, 3, 30011, 30000, 9000),
                                                  (8, 1, 64, 31, 17000, 16500, 1)])
def test_lists_of_some_offsets(hq, hkv, d, c, n, bs, used):
    gen = torch.Generator(device="cuda").manual_seed(5600 + n)
    rnd = lambda *size: torch.randn(size, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    q, k, v = rnd(c, hq, d), rnd(n, hkv, d), rnd(n, hkv, d)
    ck = vs.Chunk(hq, hkv, d, c, n - c, 1.0 / np.sqrt(d), vertical_budget=150, slash_budget=bs)
    columns = torch.stack([torch.randperm(n, generator=gen, device="cuda")[:150].sort().values for _ in range(hq)]).int()
    offsets = torch.stack([torch.randperm(n, generator=gen, device="cuda")[:bs] for _ in range(hq)]).int()
    counts = torch.tensor([used if h % 3 else max(1, used // 2) for h in range(hq)], dtype=torch.int32, device="cuda")
    sets = (columns, torch.full((hq,), 150, dtype=torch.int32, device="cuda"), offsets, counts)
    got = {}
    for split in (0, 1):
        try:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, split)
            got[split] = vs.sparse_attn_prefill(ck, q, k, v, *sets, want_lse=True)
            torch.cuda.synchronize()
        finally:
            vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 0)
    a, b = got[0][0].float(), got[1][0].float()
    # bf16 probabilities and outputs on either side: 2^-9 each, unbiased, about 6e-3 between the two
    assert ((a - b).norm(dim=2) <= 2e-2 * b.norm(dim=2) + 1e-30).all()
    np.testing.assert_allclose(got[0][1].cpu().numpy(), got[1][1].cpu().numpy(), rtol=2e-5, atol=2e-5)
