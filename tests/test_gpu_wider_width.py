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
