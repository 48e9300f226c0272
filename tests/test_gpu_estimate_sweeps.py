"""The two sweeps of the estimate at the edges of their cut: one tile of keys, ragged last tiles, windows shorter than 64 rows
(whose last offsets lie behind the last tile), groups of one head to more than a workgroup takes, several tiles per wave (their
seams add two parts), rotations that change between and inside blocks.  Against the fp64 oracle: element-wise at the rule of the other estimate tests, and 1e-5 of the norm
(sums of up to 64 fp32 exponentials, whose arguments carry a few 2^-24 of scores below 32)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_15383_amd as vs
from gpu_util import chunk_of, dev, f64, host_u16
from helpers import rand_bf16

pytestmark = pytest.mark.gpu


def _check(hq, hkv, d, c, s, seed, dca=None, ramp=None, norm=1e-5):
    rng = np.random.default_rng(seed)
    q = rand_bf16(rng, (c, hq, d)); k = rand_bf16(rng, (s + c, hkv, d))
    if ramp is not None:   # keys whose length goes from ramp[0] to ramp[1] along the cache
        kf = (k.astype(np.uint32) << 16).view(np.float32) * np.linspace(*ramp, s + c, dtype=np.float32)[:, None, None]
        k = host_u16(torch.from_numpy(kf).bfloat16())
    succ, inter = (rand_bf16(rng, (c, hq, d)) for _ in range(2))   # unlike q: a wrong choice of rotation shows
    pb = oracle.Problem(hq, hkv, d, c, s, 1.0 / np.sqrt(d))
    rvs, rss, rlse = oracle.estimate(pb, q, k, dca=None if dca is None else oracle.Dca(dca[0], dca[1], succ, inter))
    gd = None if dca is None else (dev(succ), dev(inter), dca[0], dca[1])
    ck = chunk_of(pb)
    poison = lambda: torch.full((hq, s + c), float("nan"), device="cuda")  # noqa: E731  every score is written
    vsc, ssc, lse = vs.estimate(ck, dev(q), dev(k), want_lse=True, vscore=poison(), sscore=poison(), dca=gd)
    again = vs.estimate(ck, dev(q), dev(k), want_lse=True, vscore=poison(), sscore=poison(), dca=gd)
    torch.cuda.synchronize()
    assert torch.equal(vsc, again[0]) and torch.equal(ssc, again[1]) and torch.equal(lse, again[2])
    for got, ref in ((vsc, rvs), (ssc, rss)):
        got = f64(got)
        np.testing.assert_allclose(got, ref, rtol=2e-4, atol=1e-7)
        assert np.linalg.norm(got - ref) <= norm * np.linalg.norm(ref)
    np.testing.assert_allclose(f64(lse).reshape(rlse.shape), rlse, rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("c,s", [(1, 0), (1, 63), (1, 64), (5, 59), (63, 1), (64, 0), (64, 64), (65, 63), (100, 933), (3, 4094)])
@pytest.mark.parametrize("hq,hkv,d", [(1, 1, 128), (7, 1, 128), (6, 2, 64), (9, 1, 64), (16, 2, 128)])
def test_edges(hq, hkv, d, c, s):
    _check(hq, hkv, d, c, s, 4000 + c + s)


@pytest.mark.parametrize("hq,hkv,d,c,s", [(16, 8, 64, 77, 140001), (14, 2, 128, 64, 30000), (4, 4, 128, 20, 200000)])
def test_several_tiles_and_workgroups(hq, hkv, d, c, s):
    _check(hq, hkv, d, c, s, 4100)


@pytest.mark.parametrize("c,s,dca", [
    (64, 1000, (64, 0)),          # the smallest chunk: rows on both sides of a boundary, no window
    (64, 1000, (128, 64)),
    (40, 2000, (512, 512)),       # a window as long as the chunk
    (64, 4064, (1024, 192)),      # rows on both sides; the window ends inside blocks
    (64, 3000, (1024, 4096)),     # longer than the chunk
    (3, 700, (4096, 64)),         # one chunk
    (200, 30000, (8192, 1024)),
])
@pytest.mark.parametrize("hq,hkv,d", [(7, 1, 128), (6, 2, 64), (5, 5, 128)])
def test_rotations(hq, hkv, d, c, s, dca):
    _check(hq, hkv, d, c, s, 4200 + s, dca)


def test_rotations_over_several_tiles_per_wave():
    _check(8, 8, 64, 64, 120000, 4300, (32768, 2048))


@pytest.mark.parametrize("hq,hkv,d,c,s,dca", [(8, 8, 64, 64, 120000, None), (14, 2, 128, 40, 30000, None), (8, 8, 64, 64, 120000, (32768, 2048))])
@pytest.mark.parametrize("ramp", [(0.05, 12.0), (12.0, 0.05)])
def test_scores_that_outrun_the_reference_of_a_wave(hq, hkv, d, c, s, dca, ramp):
    # Base-2 scores up to about 4.5 * 12 * log2(e) = 78 along a wave's tiles: references taken from a first tile are passed by far
    # more than 2^8 and taken again (rising), or leave nothing of the later tiles (falling).  Arguments below 128 are off by up to 2^-18
    # per rounding, of which there are three (the score, its product with the scale, the lse): 3 * 2^-18 * ln 2 = 8e-6 for a
    # single probability that all weight lies on, and as much again for the sum that the lse comes from.
    _check(hq, hkv, d, c, s, 4400, dca, ramp, norm=2e-5)


@pytest.mark.parametrize("hq,hkv,c,s", [(4, 2, 64, 2000), (8, 8, 40, 120000)])
def test_scores_of_tens_of_thousands(hq, hkv, c, s):
    # Base-2 scores of about -2^16 to 2^16, every second window row below zero throughout.  The products are whole numbers below 2^24,
    # so that scores are exact but for their factor; what is left is the rounding of an lse below 2^17, 2^-8 each when it is made and
    # when its maximum's product with the factor is: 2^-7 * ln 2 of a probability, and 2^-23 of the lse.
    rng = np.random.default_rng(4500)
    u = rng.choice([-64, 64], (1, 1, 64))
    k = u + rng.integers(-60, 61, (s + c, hkv, 64))
    q = u * np.where(np.arange(c) % 2, -1, 1)[:, None, None] + rng.integers(-60, 61, (c, hq, 64))
    k, q = (host_u16(torch.from_numpy(x.astype(np.float32)).bfloat16()) for x in (k, q))
    pb = oracle.Problem(hq, hkv, 64, c, s, 0.125)
    rvs, rss, rlse = oracle.estimate(pb, q, k)
    assert rlse.min() < -2.0 ** 13 and rlse.max() > 2.0 ** 15
    vsc, ssc, lse = vs.estimate(chunk_of(pb), dev(q), dev(k), want_lse=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(f64(lse).reshape(rlse.shape), rlse, rtol=2.0 ** -21)
    for got, ref in ((vsc, rvs), (ssc, rss)):
        np.testing.assert_allclose(f64(got), ref, rtol=2.0 ** -6, atol=1e-7)


@pytest.mark.parametrize("scale", [0.68, 1.0, 2.9])   # the largest base-2 scores lie past 2^17, 2^18 and 2^20
@pytest.mark.parametrize("every", [1, 2, 3])
@pytest.mark.parametrize("hq,hkv,d,c,s,dca", [(4, 2, 64, 64, 2000, None), (8, 8, 64, 40, 120000, None), (7, 1, 128, 64, 9000, None),
                                              (8, 8, 64, 40, 120000, (32768, 2048))])
def test_scores_past_the_range_of_a_half_word(hq, hkv, d, c, s, dca, every, scale):
    # As above, with factors that take the scores on; the keys of every 2nd or 3rd tile of 64 have only scores of a few
    # thousandths of that, so that the largest score of a row goes up past 2^17, and of the rows below zero back from there, on the
    # way through a wave's tiles.  Roundings as above: a probability is off by a factor of 2^(2^(b - 23)) for scores of 2^b.
    rng = np.random.default_rng(4600)
    u = rng.choice([-64, 64], (1, 1, 64))
    far = (np.arange(s + c) // 64 % 3 % every == 0)[:, None, None]
    k = np.zeros((s + c, hkv, d))
    k[..., :64] = far * u + rng.integers(-60, 61, (s + c, hkv, 64)) * np.where(far, 1, 1 / 64)
    qs = []
    for _ in range(3 if dca else 1):
        q = np.zeros((c, hq, d))
        q[..., :64] = u * np.where(np.arange(c) % 2, -1, 1)[:, None, None] + rng.integers(-60, 61, (c, hq, 64))
        qs.append(q)
    k, *qs = (host_u16(torch.from_numpy(x.astype(np.float32)).bfloat16()) for x in (k, *qs))
    pb = oracle.Problem(hq, hkv, d, c, s, scale)
    rvs, rss, rlse = oracle.estimate(pb, qs[0], k, dca=oracle.Dca(*dca, *qs[1:]) if dca else None)
    top = rlse.max() * np.log2(np.e)
    assert top > 2.0 ** {0.68: 17, 1.0: 18, 2.9: 20}[scale]
    ck = chunk_of(pb)
    n = vs.workspace_bytes(ck, vs.VS_WS_ESTIMATE)
    ws = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    vsc, ssc, lse = vs.estimate(ck, dev(qs[0]), dev(k), want_lse=True, ws=ws[:n], dca=(*map(dev, qs[1:]), *dca) if dca else None)
    torch.cuda.synchronize()
    assert bool((ws[n:] == 0xA5).all())
    # (rows below zero may end near it: there the rounding is that of their own largest products)
    np.testing.assert_allclose(f64(lse).reshape(rlse.shape), rlse, rtol=2.0 ** -21, atol=2.0 ** -10)
    for got, ref in ((vsc, rvs), (ssc, rss)):
        np.testing.assert_allclose(f64(got), ref, rtol=2.0 ** (np.floor(np.log2(top)) - 22), atol=1e-7)
