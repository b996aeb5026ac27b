"""Caches whose neighbours the coarse key cannot tell apart by the dozen: every entry present many times, clusters
tighter than the key's rounding, 0 / 1 entries.  The answer is the oracle's, and the 256 best candidates by the
coarse key are enough for (nearly) all queries: the scan of the whole cache, many times as expensive, stays out."""
import pytest
import torch

from paper_2002_02645_amd import binding
from tests import parity
from tests.test_gpu_parity import TIGHT, _host_entries

pytestmark = pytest.mark.gpu


def _data(kind, n, d, b, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    cent = torch.randn(10, d, generator=g)
    lab = torch.randint(0, 10, (n,), generator=g, dtype=torch.int32)
    cq = cent[torch.randint(0, 10, (b,), generator=g)]
    if kind == "copies":                       # 21 copies of every entry, far apart
        m = (n + 20) // 21
        lab = lab[:m].repeat(21)[:n].contiguous()
        e = (cent[lab[:m].long()] + 0.8 * torch.randn(m, d, generator=g)).repeat(21, 1)[:n]
        q = cq + 0.8 * torch.randn(b, d, generator=g)
    elif kind == "neighbours":                 # ... next to each other
        m = (n + 20) // 21
        lab = lab[:m].repeat_interleave(21)[:n].contiguous()
        e = (cent[lab[::21].long()] + 0.8 * torch.randn(m, d, generator=g)).repeat_interleave(21, 0)[:n]
        q = cq + 0.8 * torch.randn(b, d, generator=g)
    else:                                      # clusters whose spread is that small against their distance from the mean
        e = cent[lab.long()] + kind * torch.randn(n, d, generator=g)
        q = cq + kind * torch.randn(b, d, generator=g)
    return e.contiguous().to(dtype), lab, q


def _check(kind, n, d, b, k, dtype, most_scanned):
    ent, lab, q = _data(kind, n, d, b, dtype, 11 + n + b)
    thr = max(1, k - 2)
    fc = binding.FreezeCache(1)
    try:
        c = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_lookup_stats_attach(fc.ctx, c)
        fc.build_layer(0, ent.cuda(), lab.cuda(), 10)
        out = fc.lookup(0, q.cuda(), k, thr)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
        c = c.tolist()
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(ent), lab.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, thr)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, thr, rel=TIGHT, dist_rel=TIGHT)
    assert sum(c) == b and c[2] <= most_scanned * b, c


@pytest.mark.parametrize("kind,n,d,b,k,dtype,most_scanned", [
    ("copies", 6000, 4096, 300, 10, torch.bfloat16, 0.0),
    ("copies", 10000, 3100, 40, 10, torch.float32, 0.0),     # (fewer than 128 queries)
    ("copies", 9001, 8200, 260, 10, torch.bfloat16, 0.0),    # 256-query keys-out kernel
    ("neighbours", 10000, 4100, 300, 5, torch.bfloat16, 0.0),
    (0.05, 3000, 4096, 300, 10, torch.bfloat16, 0.1),
])
def test_materialised_keys(kind, n, d, b, k, dtype, most_scanned):
    _check(kind, n, d, b, k, dtype, most_scanned)


@pytest.mark.parametrize("kind,n,d,b,k,dtype,most_scanned", [
    ("copies", 10000, 512, 300, 10, torch.bfloat16, 0.0),
    ("copies", 10000, 517, 1100, 10, torch.float32, 0.0),     # more flagged queries than workgroups
    ("copies", 20000, 1030, 300, 20, torch.bfloat16, 0.0),    # R = 32, odd rows
    ("neighbours", 10000, 256, 300, 5, torch.bfloat16, 0.0),
    ("neighbours", 4000, 100, 260, 1, torch.float32, 0.0),
    ("copies", 300000, 64, 140, 10, torch.bfloat16, 0.05),    # more minima than the group minima's first round
    (0.02, 5000, 256, 600, 10, torch.bfloat16, 0.1),
    (0.05, 3000, 512, 300, 40, torch.float32, 0.1),           # R = 64
])
def test_block_minima(kind, n, d, b, k, dtype, most_scanned):
    _check(kind, n, d, b, k, dtype, most_scanned)


def test_few_flagged_queries_share_workgroups():
    """Block minima with seven queries among entries present 21 times, the others among ordinary ones: sixteen workgroups
    share the wider re-scoring of each of the seven."""
    n, d, b, k = 6000, 256, 300, 10
    ent, lab, q = _data("copies", n, d, b, torch.float32, 5)
    g = torch.Generator().manual_seed(6)
    ent = torch.cat([3.0 * ent, torch.randn(n, d, generator=g)]).to(torch.bfloat16)
    lab = torch.cat([lab, lab])
    q = 3.0 * q
    q[7:] = 0.7 * torch.randn(b - 7, d, generator=g)
    c = torch.zeros(3, dtype=torch.int64, device="cuda")
    fc = binding.FreezeCache(1)
    try:
        binding.freeze_lookup_stats_attach(fc.ctx, c)
        binding.freeze_set_centring(fc.ctx, 0)
        fc.build_layer(0, ent.cuda(), lab.cuda(), 10)
        out = fc.lookup(0, q.cuda(), k, 8)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(ent), lab.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, 8)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, 8, rel=TIGHT, dist_rel=TIGHT)
    c = c.tolist()
    assert sum(c) == b and 7 <= c[1] <= 20 and c[2] == 0, c
