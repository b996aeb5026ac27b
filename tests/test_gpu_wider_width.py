"""Long rows whose re-scoring width is wider than k has by default (the default's candidates first, the others for the
queries that these do not confirm), on the route that materialises its keys, and on per-query lists, which small
workspaces get: a dense cloud, where the first step confirms nearly all queries and not all, and widths that leave a remainder of
one."""
import pytest
import torch

from paper_2002_02645_amd import binding, synth
from tests import parity
from tests.test_gpu_lists import _lookup_on_the_smallest_workspace
from tests.test_gpu_parity import _host_entries

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,b,k,r,offset,dtype", [
    (3000, 4096, 200, 10, 64, 0.0, torch.bfloat16),    # materialised keys: 16 first, then 48
    (3000, 4096, 200, 10, 64, 3.0, torch.float32),
    (1500, 16384, 40, 10, 33, 0.0, torch.bfloat16),    # ... 16, then 17; rows by all 1,024 threads; few queries
    (3000, 4104, 90, 1, 17, 2.0, torch.bfloat16),      # ... 16, then one
    (3000, 4096, 90, 24, 64, 0.0, torch.bfloat16),     # ... 32, then 32
    (3000, 4096, 130, 40, 0, 0.0, torch.bfloat16),     # ... 48, then 16 (the default width)
    (22000, 4096, 1100, 10, 64, 1.0, torch.bfloat16),  # more queries than materialise their keys: block minima
    (14000, 4096, 1100, 30, 0, 1.0, torch.bfloat16),   # ...
])
def test_wider_width(n, d, b, k, r, offset, dtype):
    g = torch.Generator().manual_seed(77 + n + d + b + k)
    ent = (torch.randn(n, d, generator=g) + offset).to(dtype)
    lab = torch.randint(0, 10, (n,), generator=g, dtype=torch.int32)
    q = torch.randn(b, d, generator=g) * 0.7 + offset
    thr = max(1, k - 3)
    fc = binding.FreezeCache(1)
    try:
        counters = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_lookup_stats_attach(fc.ctx, counters)
        fc.build_layer(0, ent.cuda(), lab.cuda(), 10)
        out = fc.lookup(0, q.cuda(), k, thr, r)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
        c = counters.cpu().numpy()
    finally:
        fc.close()
    some = torch.arange(b) if b < 300 else torch.arange(0, b, 9)   # (the oracle is slow)
    got = {key: v[some.numpy()] for key, v in got.items()}
    e_h, l_h, q_h = _host_entries(ent), lab.numpy(), q[some].numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, thr)
    # fp32 sums of d squares: as the other long rows' tests
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, thr, rel=1e-5, dist_rel=1e-5)
    assert c.sum() == b, c


@pytest.mark.parametrize("n,d,b,k,r,offset,dtype", [
    (3000, 4096, 1100, 10, 64, 0.0, torch.bfloat16),   # 48 first, then 16
    (3000, 4104, 1030, 30, 0, 1.0, torch.float32),     # ... the default width of k = 30
    (2500, 4096, 1030, 10, 33, 0.0, torch.bfloat16),   # 17, then 16
    (1500, 16384, 300, 10, 64, 0.0, torch.bfloat16),   # rows by 1,024 threads
    (3000, 4096, 1030, 20, 0, 0.0, torch.float32),     # 24, then eight
])
def test_wider_width_on_lists(n, d, b, k, r, offset, dtype):
    g = torch.Generator().manual_seed(7 + n + d + b + k)
    ent = (torch.randn(n, d, generator=g) + offset).to(dtype)
    lab = torch.randint(0, 10, (n,), generator=g, dtype=torch.int32)
    q = torch.randn(b, d, generator=g) * 0.7 + offset
    thr = max(1, k - 3)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, ent.cuda(), lab.cuda(), 10)
        got = _lookup_on_the_smallest_workspace(fc, q.cuda(), k, thr, r)
        whole = fc.lookup(0, q.cuda(), k, thr, r)
        torch.cuda.synchronize()
        for key in ("idx", "dist", "label", "votes", "hit"):
            assert (whole[key].cpu().numpy() == got[key]).all(), key
    finally:
        fc.close()
    some = torch.arange(0, b, 13)   # (the oracle is slow)
    got = {key: v[some.numpy()] for key, v in got.items()}
    e_h, l_h, q_h = _host_entries(ent), lab.numpy(), q[some].numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, thr)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, thr, rel=1e-5, dist_rel=1e-5)


def _by_1024_threads(q, c):
    """fp32 distances of the rows of q to those of c, added up by 1,024 threads: chains of every 1,024th piece of eight values, a
    butterfly over a wave's, four waves' at a time.  (Inputs: squares of 24 bits, so that float64 rounds like a fused step.)"""
    x = (q - c).view(q.shape[0], -1, 1024, 8).double()
    acc = torch.zeros(q.shape[0], 1024, device=q.device)
    for s in range(x.shape[1]):
        for e in range(8):
            acc = (acc.double() + x[:, s, :, e] ** 2).float()
    acc, lane = acc.view(-1, 16, 64), torch.arange(64, device=q.device)
    for off in (32, 16, 8, 4, 2, 1):
        acc = acc + acc[:, :, lane ^ off]
    wave, t = acc[:, :, 0], torch.zeros(q.shape[0], device=q.device)
    for w in range(0, 16, 4):
        t = t + ((wave[:, w] + wave[:, w + 1]) + (wave[:, w + 2] + wave[:, w + 3]))
    return t


@pytest.mark.parametrize("points,copies,b,k,stage", [
    (256, 2, 512, 1, 1),      # a workgroup per query that the first candidates do not confirm
    (256, 2, 16, 1, 1),       # ... several, that meet
    (1, 600, 12, 5, 2),       # the exact scan
])
def test_longest_rows_have_one_order_of_additions(points, copies, b, k, stage):
    """Entries as far from a query as each other but for the roundings of the sums: permutations of the same differences.  Up to
    1,024 queries on 16,384 values: what re-scores later candidates adds up like what re-scores the first ones."""
    d = 16384
    g = torch.Generator().manual_seed(points + b)
    at = torch.randint(-32, 33, (points, d), generator=g) / 16.0
    off = torch.randint(-4095, 4096, (points, d), generator=g) / 4096.0
    ent = torch.stack([at + off[:, torch.randperm(d, generator=g)] for _ in range(copies)], 1).view(points * copies, d).cuda()
    q = at[torch.arange(b) % points].cuda().contiguous()
    fc = binding.FreezeCache(1)
    try:
        stats = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_lookup_stats_attach(fc.ctx, stats)
        fc.build_layer(0, ent, torch.zeros(points * copies, dtype=torch.int32, device="cuda"), 2)
        got = fc.lookup(0, q, k, 1)
        torch.cuda.synchronize()
        binding.freeze_lookup_stats_attach(fc.ctx, None)
    finally:
        fc.close()
    assert stats[stage] > 0, stats
    dist = torch.stack([_by_1024_threads(q, ent[torch.arange(b, device="cuda") % points * copies + j]) for j in range(copies)], 1)
    want, place = torch.sort(dist, dim=1, stable=True)
    assert torch.equal(got["dist"], want[:, :k])
    assert torch.equal(got["idx"].long(), (torch.arange(b, device="cuda") % points * copies)[:, None] + place[:, :k])
