"""Long chunks whose query tiles are not whole rounds: the walk that keeps pace and the pieces behind it in one kernel, with as many pieces
as the workspace has room for, against the kernel that cuts nothing."""
import numpy as np
import pytest
import torch

import paper_2501_15383_amd as vs

pytestmark = pytest.mark.gpu


# units beyond whole rounds of 512: 20 (many ranges each), 504 (a few), 8 of heads of 64 (which keep no pace) and the last of their full rounds,
# rows that start inside a block; and, too short to keep pace, 488; of full rounds the last, of more than 4,096 units what is over (64); 4,608 in full rounds, which stay whole
@pytest.mark.parametrize("hq,hkv,d,c,n,dca", [(28, 4, 128, 2400, 264000, False), (28, 4, 128, 2432, 262144 + 2433, True),
                                              (8, 2, 64, 8320, 300001, False), (8, 1, 64, 8300, 264007, True), (127, 1, 64, 1000, 262200, False),
                                              (16, 2, 64, 8192, 262400, False), (8, 2, 64, 15950, 16384, False), (8, 2, 128, 15950, 16385, True),
                                              (16, 2, 128, 8192, 8192, False), (16, 4, 64, 8192, 9024, True), (64, 1, 64, 8320, 8391, False),
                                              (72, 1, 64, 8192, 8256, True)])
def test_pieces_behind_whole_units(hq, hkv, d, c, n, dca):
    gen = torch.Generator(device="cuda").manual_seed(5200 + c)
    rnd = lambda *size: torch.randn(size, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    q, k, v = rnd(c, hq, d), rnd(n, hkv, d), rnd(n, hkv, d)
    rot = (rnd(c, hq, d), rnd(c, hq, d), 131072, 4096) if dca else None
    ck = vs.Chunk(hq, hkv, d, c, n - c, 1.0 / np.sqrt(d), vertical_budget=200, slash_budget=300)
    # lists of different lengths: offsets of head h within the last n / (h % 5 + 1)
    s_idx = torch.stack([(torch.rand(300, generator=gen, device="cuda") * (n // (h % 5 + 1))).int().sort().values for h in range(hq)])
    v_idx = torch.stack([torch.randint(0, n, (200,), generator=gen, device="cuda").int().sort().values for _ in range(hq)])
    s_idx[:, :2] = 0   # (a diagonal twice)
    v_idx = torch.stack([torch.cat([u := x.unique(), torch.full((200 - len(u),), -1, dtype=torch.int32, device="cuda")]) for x in v_idx])
    cnt = lambda x: (x >= 0).sum(dim=1).int()  # noqa: E731
    sets = (v_idx.contiguous(), cnt(v_idx), s_idx.contiguous(), cnt(s_idx))
    call = lambda ws=None: vs.sparse_attn_prefill(ck, q, k, v, *sets, want_lse=True, dca=rot, ws=ws)  # noqa: E731
    full = vs.workspace_bytes(ck, vs.VS_WS_SPARSE)
    try:
        vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 1)
        want, uncut = call(), vs.workspace_bytes(ck, vs.VS_WS_SPARSE)
    finally:
        vs.set_option(vs.VS_OPT_ATTN_KEY_SPLIT, 0)

    def close(got):
        a, b = got[0].float(), want[0].float()
        # bf16 probabilities and outputs on either side: 2^-9 each, unbiased, about 6e-3 between the two
        assert ((a - b).norm(dim=2) <= 2e-2 * b.norm(dim=2)).all() and (got[1] - want[1]).abs().max().item() < 1e-4
    room = torch.empty(full + 4096, dtype=torch.uint8, device="cuda")

    def guarded(size):
        room.fill_(0x5A)
        got = call(room[:size])
        torch.cuda.synchronize()
        assert (room[size:] == 0x5A).all()
        return got
    got = guarded(full)
    close(got)
    again = call()
    torch.cuda.synchronize()
    assert torch.equal(got[0].view(torch.int16), again[0].view(torch.int16)) and torch.equal(got[1], again[1])
    if full == uncut:   # (no pieces: the workspace is as small as it can be)
        assert hq == 72
        return
    # the smallest workspace that is taken (what a call needed when its pieces were fewer)
    lo, hi = uncut // 256 - 1, full // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            call(room[:256 * mid])
            hi = mid
        except vs.VsError:
            lo = mid
    assert 256 * hi < full
    close(guarded(256 * hi))


# heads of 64 that keep pace for all that: two whole rounds and 16, 8, 128 units (whose walks the budgets make short), and, as before, none of them (16 heads)
@pytest.mark.parametrize("hq,hkv,d,c,n,dca", [(8, 2, 64, 16500, 262144 + 13, False), (8, 8, 64, 16512, 262272, True), (4, 1, 64, 36864, 270016, False),
                                              (16, 2, 64, 8320, 262272, False)])
def test_few_heads_of_64_keep_pace(hq, hkv, d, c, n, dca):
    test_pieces_behind_whole_units(hq, hkv, d, c, n, dca)
