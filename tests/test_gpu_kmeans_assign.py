"""The k-means build's assignment by the product with split centres: the edges of its tiles (points, centres, depth), rows of
any length, ranges that cut tiles and ranges of whole ones, ties, and values that are no numbers.  The assignment shows in the
centres after one round, which are compared with means over the nearest centres by float64 distances."""
import numpy as np
import pytest
import torch

from paper_2002_02645_amd import binding

pytestmark = pytest.mark.gpu


def _nearest64(pts, cen):
    """Index of the nearest centre (equal distances: the lower), and the smallest relative gap to the second, float64."""
    p, c = torch.from_numpy(pts).double(), torch.from_numpy(cen).double()
    best, gap = [], np.inf
    for lo in range(0, p.shape[0], max(1, (1 << 24) // c.numel())):
        x = p[lo:lo + max(1, (1 << 24) // c.numel())]
        dist = ((x[:, None, :] - c[None]) ** 2).sum(2).numpy()
        best.append(dist.argmin(1))
        if c.shape[0] > 1:
            two = np.partition(dist, 1, axis=1)
            gap = min(gap, ((two[:, 1] - two[:, 0]) / np.maximum(two[:, 1], 1e-30)).min())
    return np.concatenate(best), gap


def _means(pts, assign, cen):
    out = cen.copy()
    for c in range(cen.shape[0]):
        rows = pts[assign == c].astype(np.float64)
        if rows.shape[0]:
            out[c] = (np.add.accumulate(rows, axis=0)[-1] / rows.shape[0]).astype(np.float32)
    return out


def _build(pts, cen, iters=1):
    fc = binding.FreezeCache(1)
    try:
        lab = torch.zeros(pts.shape[0], dtype=torch.int32, device="cuda")
        got = fc.build_kmeans_layer(0, torch.from_numpy(pts).cuda(), lab, 3, torch.from_numpy(cen).cuda(), iters)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in got.items()}
    finally:
        fc.close()


@pytest.mark.parametrize("n,d,kc", [
    (256, 32, 1),         # one tile of points, one k-step, one centre
    (257, 33, 16),        # the second tile reaches back over 255 rows of the first
    (300, 4, 64), (511, 100, 65), (1021, 31, 97),
    (300, 132, 80), (411, 33, 112), (290, 68, 131), (310, 65, 176),   # 5, 7, 9 and 11 column blocks: the waves of a pair differ
    (2051, 36, 200),      # 13
    (400, 70, 230),       # 15: as 16
    (700, 520, 256),      # the widest tile
    (900, 68, 257), (1500, 98, 512),       # two tiles of centres
    (600, 100, 343),      # ... of 11 column blocks
    (1300, 60, 513),      # more centres than the product takes
    (601, 4104, 13),      # re-scored by the whole workgroup, ranges that cut tiles in several places
    (600, 4099, 33),      # ... by waves, rows on any boundary
    (255, 64, 9),         # fewer points than a tile
])
def test_assignment_on_random_points(n, d, kc):
    rng = np.random.default_rng(n * 7 + d + kc)
    centre = 2.0 * rng.standard_normal((5, d))
    pts = (centre[rng.integers(0, 5, n)] + rng.standard_normal((n, d))).astype(np.float32)
    cen = pts[rng.permutation(n)[:kc]].copy() if kc <= n else pts[:kc].copy()
    want, gap = _nearest64(pts, cen)
    # an fp32 distance is good to (log2 d + 16) 2^-24 < 2e-6; no point of these inputs is that close to two centres
    assert gap > 4e-6
    got = _build(pts, cen)
    np.testing.assert_allclose(got["centers"], _means(pts, want, cen), rtol=1e-6, atol=1e-7)
    assert (got["fraction"][np.bincount(_nearest64(pts, got["centers"])[0], minlength=kc) == 0] == 0).all()


@pytest.mark.parametrize("n,d,kc", [
    (3000, 6, 40),
    (530000, 8, 5),       # so many tiles that ranges are whole ones
    (1200, 7, 300),
])
def test_assignment_with_ties(n, d, kc):
    # whole numbers that bf16 does not hold: every distance is exact, many are equal, and some centres are there twice
    rng = np.random.default_rng(n)
    pts = rng.integers(-2, 3, (n, d)).astype(np.float32) * 257.0
    cen = pts[:kc].copy()
    cen[kc // 2] = cen[kc // 3]
    want, _ = _nearest64(pts, cen)
    got = _build(pts, cen)
    np.testing.assert_allclose(got["centers"], _means(pts, want, cen), rtol=1e-6, atol=1e-4)
    assert np.array_equal(got["centers"][kc // 2], cen[kc // 2])      # its twin has the lower index and every point


def test_identical_points():
    # every centre is left for every point: all of them re-scored, all equal, the first one takes them
    pts = np.full((400, 40), 1.0039, dtype=np.float32)
    got = _build(pts, pts[:30].copy())
    assert np.array_equal(got["centers"], pts[:30]) and got["fraction"][0] == 1.0 and (got["fraction"][1:] == 0).all()


def test_points_that_are_no_numbers():
    # outside the contract, but nothing is read or written out of bounds and the other points are assigned as ever
    rng = np.random.default_rng(3)
    n, d, kc = 777, 45, 20
    pts = rng.standard_normal((n, d)).astype(np.float32)
    cen = pts[:kc].copy()
    want, gap = _nearest64(pts, cen)
    assert gap > 4e-6
    bad = [100, 300, 776]
    broken = pts.copy()
    broken[100, 7], broken[300, :], broken[776, 44] = np.nan, np.inf, -np.inf
    got = _build(broken, cen)["centers"]
    keep = np.ones(n, bool)
    keep[bad] = False
    exp = _means(pts[keep], want[keep], cen)
    hit = ~np.isfinite(got).all(axis=1)                               # centres that took one of the three
    assert hit.sum() <= 3
    np.testing.assert_allclose(got[~hit], exp[~hit], rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("n,d,kc,shape", [
    (32768, 65536, 512, "constant"),      # two tiles of centres, as many tiles as CUs: a sum runs over the whole row
    (16384, 65536, 100, "constant"),      # ... over a quarter of it
    (32768, 65536, 300, "blocks"),        # runs of equal values, every other run small: sums that grow evenly too
    (66000, 16384, 60, "constant"),
])
def test_rows_whose_sums_round_one_way(n, d, kc, shape):
    # The addends of a point's sums are all alike, so within a binade every addition rounds the same way and the errors
    # of a key add up over the row's length.  Centres close together in value: keys that are off by that are wrong.  With the
    # index of its nearest centre as every point's label, clusters that took no other points have a share of exactly 1.
    g = torch.Generator().manual_seed(n + d + kc)
    cval = torch.sort(0.5 + 1.5 * torch.rand(kc, generator=g, dtype=torch.float64))[0].float().double()
    gap = torch.minimum(torch.diff(cval, prepend=cval[:1] - 1), torch.diff(cval, append=cval[-1:] + 1))
    want = torch.randint(0, kc, (n,), generator=g)
    want[:kc] = torch.arange(kc)
    # at most 0.4 of the way to the next centre: squared distances 1 : 2.25 at least, where fp32 ones are good to 1e-3
    pval = (cval[want] + gap[want] * 0.8 * (torch.rand(n, generator=g, dtype=torch.float64) - 0.5)).float()
    keep = torch.ones(d, device="cuda")
    if shape == "blocks":
        keep = 1.0 - 0.9375 * ((torch.arange(d, device="cuda") // 512) % 2).float()
    pts = torch.empty(n, d, device="cuda")
    torch.mul(pval.cuda()[:, None], keep[None, :], out=pts)
    cen = cval.float().cuda()[:, None] * keep[None, :]
    fc = binding.FreezeCache(1)
    try:
        got = fc.build_kmeans_layer(0, pts, want.to(torch.int32).cuda(), kc, cen.contiguous(), 0)
        torch.cuda.synchronize()
        share, label = got["fraction"].cpu(), got["majority"].cpu()
    finally:
        fc.close()
    wrong = (share != 1.0) | (label != torch.arange(kc))
    assert not wrong.any(), (int(wrong.sum()), share[wrong][:5], torch.nonzero(wrong)[:5, 0])


def test_update_of_many_centres():
    # more centres than the update's grid has in one dimension; two points each to the last 7,000
    n, kc, d = 40000, 33000, 8
    pts = torch.zeros(n, d)
    i = torch.arange(kc)
    pts[:kc, 0], pts[:kc, 1] = 8.0 * (i % 200), 8.0 * (i // 200)
    pts[kc:] = pts[kc - (n - kc):kc] + 1.0
    cen = pts[:kc].clone()
    want = cen.clone()
    want[kc - (n - kc):] += 0.5
    assert np.array_equal(_build(pts.numpy(), cen.numpy())["centers"], want.numpy())


def test_centres_of_more_than_2_to_the_32_values():
    # more threads than a grid takes, were there one per value.  Every centre is a point and stays where it is.
    if torch.cuda.mem_get_info()[0] < 180e9:
        pytest.skip("needs 180 GB of device memory")
    n, d = 4097, 1 << 20
    fc = binding.FreezeCache(1)
    got = None
    try:
        pts = torch.empty(n, d, device="cuda")
        for i in range(0, n, 256):
            pts[i:i + 256].normal_()
        lab = torch.arange(n, dtype=torch.int32, device="cuda")
        got = fc.build_kmeans_layer(0, pts, lab, n, pts, 1)
        torch.cuda.synchronize()
        assert all(torch.equal(got["centers"][i:i + 256], pts[i:i + 256]) for i in range(0, n, 256))
        assert torch.equal(got["majority"], lab)
    finally:
        fc.close()
        del pts, got, fc
        torch.cuda.empty_cache()


@pytest.mark.parametrize("n,d,kc", [(600, 4100, 33), (700, 4099, 50), (900, 33, 20), (520, 36, 300), (513, 95, 70), (400, 64, 16)])
def test_large_first_value(n, d, kc):
    # The row's first values stand in for what lies past its end, and are taken off the sums of squares again: the bound of the
    # keys' errors must not fall short.  The large value is the same everywhere, so that distances are those of the others.
    rng = np.random.default_rng(n + d)
    centre = 2.0 * rng.standard_normal((5, d))
    pts = (centre[rng.integers(0, 5, n)] + rng.standard_normal((n, d))).astype(np.float32)
    pts[:, 0] = 3000.37
    cen = pts[rng.permutation(n)[:kc]].copy()
    want, gap = _nearest64(pts, cen)
    assert gap > 4e-6
    np.testing.assert_allclose(_build(pts, cen)["centers"], _means(pts, want, cen), rtol=1e-6, atol=1e-7)
