"""Selections of long rows by the floor of a sample: 4,096, 8,192 and 16,384 of them, with all of the workspace and with the smallest that
is taken, and scores whose neighbours are alike, which a sample meets all or none of."""
import ctypes as C

import pytest
import torch

import paper_2501_15383_amd as vs
from paper_2501_15383_amd import binding
from test_gpu_select_sizes import _scores, _want

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,n,bv,bs", [(3, 49153, 300, 700), (28, 100003, 1000, 6096), (2, 300001, 1000, 6096), (28, 300001, 1000, 9000),
                                        (4, 1048576, 1000, 6096), (1, 2000003, 128, 2000)])
@pytest.mark.parametrize("kind", ["spread", "crowded", "runs"])
def test_samples_and_workspaces(hq, n, bv, bs, kind):
    g = torch.Generator(device="cuda:0").manual_seed(5300 + n)
    if kind == "runs":   # 16 neighbours within a thousandth of one another
        one = lambda: (torch.randn((hq, n // 16 + 1), generator=g, device="cuda").exp().repeat_interleave(16, dim=1)[:, :n] *  # noqa: E731
                       (1.0 + 1e-3 * torch.rand((hq, n), generator=g, device="cuda"))).contiguous()
        vsc, ssc = one(), one()
    else:
        vsc, ssc = _scores(kind, hq, n, g), _scores(kind, hq, n, g)
    ck = vs.Chunk(hq, 1, 128, 64, n - 64, 0.1, vertical_budget=bv, slash_budget=bs, keep_first_cols=1, keep_local_band=64)
    want = (*_want(vsc, bv, 1), *_want(ssc, bs, 64))
    full = vs.workspace_bytes(ck, vs.VS_WS_SELECT)
    room = torch.empty(full + 4096, dtype=torch.uint8, device="cuda")
    p = ck.params()

    def call(size):
        sets = vs.alloc_index_sets(ck, vsc.device)
        rc = binding.lib().vs_select(C.byref(p), *[C.c_void_p(t.data_ptr()) for t in (vsc, ssc, *sets)], C.c_void_p(room.data_ptr()),
                                     C.c_size_t(size), C.c_void_p(torch.cuda.current_stream().cuda_stream))
        return rc, sets
    lo, hi = 0, full // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        rc, _ = call(256 * mid)
        assert rc in (vs.VS_OK, vs.VS_ERR_WORKSPACE)
        lo, hi = (lo, mid) if rc == vs.VS_OK else (mid, hi)
    assert (256 * hi < full) == (n <= 300001 and bs < 9000)   # (the others' lists of 4,096 samples are too long: one size)
    for size in (full, 256 * hi):
        room.fill_(0x5A)
        rc, sets = call(size)
        torch.cuda.synchronize()
        assert rc == vs.VS_OK and (room[size:] == 0x5A).all()
        for a, b, nm in zip(sets, want, ("v_idx", "v_cnt", "s_idx", "s_cnt")):
            assert torch.equal(a, b), f"{nm}: {hq} heads, n {n}, {kind}, {size} bytes"
