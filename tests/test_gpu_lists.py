"""Routes that a look-up reaches only at some sizes: the fused kernel's per-query lists (all three widths, ragged
and balanced, the live count on the device, the follow-up of unconfirmed queries), which most batches on short rows
leave to block minima, but which every such batch takes when its workspace is small; the 256-query
keys-out kernel with one and several query tiles, whole and cut along the depth; the finishing kernel's re-scoring
by groups of waves; and the k-means rounds that take the points in grouped order.  All against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import freeze_oracle as fo
from paper_2002_02645_amd import binding, synth
from tests import parity
from tests import test_gpu_guard_bands as guard_bands
from tests import test_gpu_kmeans as kmeans
from tests.test_gpu_parity import TIGHT, _host_entries, check_case
from tests.test_gpu_sweep import _cases as sweep_cases

pytestmark = pytest.mark.gpu


def _layer(n, d, b, k, dtype, seed, relu=True):
    wl = synth.scaled(synth.WORKLOADS["c2_batched"], n=n, batch=b)
    spec = synth.LayerSpec(n, d, 10, wl.layers[0].sigma, relu=relu, store_bf16=(dtype == torch.bfloat16))
    data = synth.make_workload(type(wl)(wl.name, (spec,), b, k, (max(1, k - 2),), 0, seed))
    return data.layers[0], data.queries[0]


def _lookup_on_the_smallest_workspace(fc, q, k, thr, r):
    """The result on the smallest workspace the look-up accepts, which holds per-query lists for these shapes."""
    b = q.shape[0]
    hi = binding.freeze_lookup_workspace_bytes(fc.ctx, 0, b, k, r) // 256
    ws = torch.empty(hi * 256, dtype=torch.uint8, device="cuda")
    out = fc.alloc_outputs(b, k)

    def served(blocks):
        try:
            binding.freeze_lookup(fc.ctx, 0, q, k, thr, r, out["label"], out["hit"], out["votes"], out["idx"], out["dist"],
                                  ws[:blocks * 256])
            return True
        except binding.FreezeError as e:
            assert e.code == binding.FREEZE_EWORKSPACE
            return False

    lo = 0
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if served(mid) else (mid, hi)
    for t in out.values():
        t.fill_(99)
    assert served(hi)
    torch.cuda.synchronize()
    return {key: v.cpu().numpy() for key, v in out.items()}


@pytest.mark.parametrize("n,d,b,k,r,dtype", [
    (50000, 64, 10000, 10, 0, torch.bfloat16),   # balanced decomposition, workgroups that serve two query tiles
    (33000, 96, 4100, 20, 0, torch.float32),     # ... lists of 32
    (33000, 96, 4100, 30, 0, torch.bfloat16),    # ... lists of 64, 128-query tiles
    (3000, 64, 100000, 10, 0, torch.bfloat16),   # 391 query tiles
    (2000000, 64, 300, 48, 0, torch.bfloat16),   # two million entries
    (5000, 1024, 600, 10, 0, torch.bfloat16),    # 3 query tiles (ragged), 20 cache tiles, several splits
    (4000, 512, 300, 5, 12, torch.bfloat16),     # lists shorter than the kernel variant's 16 slots
    (2901, 1500, 300, 20, 24, torch.float32),    # ... than its 32; ragged depth
    (600, 16392, 300, 10, 0, torch.float32),     # long rows, depth not a multiple of 64
    (3000, 4096, 300, 10, 0, torch.bfloat16),    # two-step re-scoring
    (1500, 3080, 1030, 10, 0, torch.bfloat16),   # (lists with any workspace from here on)
    (1501, 3100, 1100, 20, 0, torch.float32),
    (1300, 3080, 1100, 40, 0, torch.bfloat16),
    (257, 3333, 1281, 4, 0, torch.bfloat16),     # one entry and one query past a tile
])
def test_lists(n, d, b, k, r, dtype):
    L, q = _layer(n, d, b, k, dtype, 41 + n + d)
    thr = max(1, k - 2)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        got = _lookup_on_the_smallest_workspace(fc, q.cuda(), k, thr, r)
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(L.entries), L.labels.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, thr)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, thr, rel=TIGHT, dist_rel=TIGHT)


@pytest.mark.parametrize("kind,n,d,b,k,r,bf16,relu,seed", [c for c in sweep_cases() if c[0] in ("tiled", "wide", "balanced")])
def test_random_shape_on_the_smallest_workspace(kind, n, d, b, k, r, bf16, relu, seed):
    L, q = _layer(n, d, b, k, torch.bfloat16 if bf16 else torch.float32, seed, relu)
    thr = max(1, k - 2)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        got = _lookup_on_the_smallest_workspace(fc, q.cuda(), k, thr, r)
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(L.entries), L.labels.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, thr)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, thr, rel=TIGHT, dist_rel=TIGHT)


@pytest.mark.parametrize("n,d,k,offset,dtype", [
    (3000, 4096, 10, 0.0, torch.bfloat16),   # lists of 16: twelve candidates first, four more when unconfirmed
    (3000, 4096, 10, 3.0, torch.float32),
    (2500, 4104, 20, 1.0, torch.bfloat16),   # lists of 32: 24 first, then 8
])
def test_two_steps_on_lists(n, d, k, offset, dtype):
    """One dense Gaussian cloud, so that the first step does not confirm every query (test_gpu_parity.py has the same
    inputs on materialised keys)."""
    g = torch.Generator().manual_seed(4242 + n + d + k)
    ent = (torch.randn(n, d, generator=g) + offset).to(dtype)
    lab = torch.randint(0, 10, (n,), generator=g, dtype=torch.int32)
    q = torch.randn(300, d, generator=g) * 0.7 + offset
    thr = max(1, k - 3)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, ent.cuda(), lab.cuda(), 10)
        got = _lookup_on_the_smallest_workspace(fc, q.cuda(), k, thr, 0)
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(ent), lab.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, thr)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, thr, rel=TIGHT, dist_rel=TIGHT)


@pytest.mark.parametrize("n,d,b,k,r,dtype", [
    (4000, 512, 300, 5, 12, torch.bfloat16),
    (5000, 1024, 600, 10, 0, torch.float32),
    (1500, 3080, 1030, 20, 0, torch.bfloat16),
    (1300, 3100, 1030, 30, 30, torch.float32),   # k = R: no spare candidate
])
def test_lists_on_clusters_far_from_the_origin(n, d, b, k, r, dtype):
    """Without centring the coarse keys cannot rank entries this far from the origin: the lists go through the wider
    re-scoring and the exact scan."""
    L, q = _layer(n, d, b, k, dtype, 77 + n, relu=False)
    ent, q = (L.entries.float() + 100.0).to(dtype), q + 100.0
    thr = max(1, k - 2)
    fc = binding.FreezeCache(1)
    try:
        counters = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_set_centring(fc.ctx, 0)
        fc.build_layer(0, ent.cuda(), L.labels.cuda(), 10)
        _lookup_on_the_smallest_workspace(fc, q.cuda(), k, thr, r)
        binding.freeze_lookup_stats_attach(fc.ctx, counters)
        got = _lookup_on_the_smallest_workspace(fc, q.cuda(), k, thr, r)
        c = counters.cpu().numpy()
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(ent), L.labels.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, thr)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, thr, rel=TIGHT, dist_rel=TIGHT)
    assert c.sum() % b == 0 and c[1] + c[2] > 0, "this input is meant to defeat the coarse ranking"


@pytest.mark.parametrize("offset", [0.0, 100.0])
def test_lists_in_a_cascade(offset):
    """Layers of 8,192 and 4,096 values: from the second on the lists' splits follow the live count on the device; with
    the offset (and no centring) so does their follow-up."""
    wl = synth.scaled(synth.WORKLOADS["c4_cascade_noisy"], n=1500, d_div=8, batch=600)
    wl = type(wl)(wl.name, wl.layers[:2], wl.batch, wl.k, (9, 9), wl.rescore_r, wl.seed)
    data = synth.make_workload(wl)
    ents = [(L.entries.float() + offset).to(L.entries.dtype) for L in data.layers]
    qs = [q + offset for q in data.queries]
    fc = binding.FreezeCache(2)
    try:
        counters = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_lookup_stats_attach(fc.ctx, counters)
        binding.freeze_set_centring(fc.ctx, 0)
        for l, L in enumerate(data.layers):
            fc.build_layer(l, ents[l].cuda(), L.labels.cuda(), L.spec.num_classes)
        out = fc.lookup_cascade([0, 1], [q.cuda() for q in qs], wl.k, list(wl.vote_thresholds), wl.rescore_r)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
        c = counters.cpu().numpy()
    finally:
        fc.close()
    exp_l, exp_x, exp_h, _ = fo.cascade([q.numpy() for q in qs], [_host_entries(e) for e in ents],
                                        [L.labels.numpy() for L in data.layers],
                                        [L.spec.num_classes for L in data.layers], wl.k, wl.vote_thresholds)
    assert np.array_equal(got["exit_layer"], exp_x) and np.array_equal(got["label"], exp_l)
    assert got["hits_per_layer"].tolist() == exp_h.tolist()
    assert (exp_x == 1).any() and (exp_x == -1).any() and (offset == 0.0 or c[1] + c[2] > 0)


@pytest.mark.parametrize("n,d,b,k,r,dtype", [
    (2999, 3100, 1030, 7, 0, torch.bfloat16),    # lists, nothing a multiple of a tile
    (1301, 3333, 1030, 20, 0, torch.float32),    # ... of 32
    (1300, 3080, 1100, 40, 0, torch.bfloat16),   # ... of 64
    (2100, 8200, 300, 10, 0, torch.bfloat16),    # keys-out kernel, two query tiles cut along the depth
    (16300, 3080, 1000, 5, 0, torch.bfloat16),   # ... four, whole
    (3900, 4100, 200, 20, 0, torch.float32),     # ... one, cut
    (3000, 100, 300, 5, 0, torch.bfloat16),      # block minima
    (16500, 2100, 100, 10, 0, torch.bfloat16),   # streaming kernel, cut tiles
])
def test_buffers_of_these_routes(n, d, b, k, r, dtype):
    guard_bands.test_lookup_stays_inside_its_buffers(n, d, b, k, r, dtype)


@pytest.mark.parametrize("n,d,b,k,r,dtype", [
    (2000, 8200, 257, 10, 0, torch.bfloat16),    # several query tiles cut along the depth, the first batch size ...
    (2100, 8200, 700, 20, 0, torch.float32),
    (2000, 8192, 1024, 10, 0, torch.bfloat16),   # ... and the last of this route
    (1024, 16500, 512, 10, 64, torch.bfloat16),  # full tiles, the widest re-scoring
    (16300, 3080, 1024, 5, 0, torch.bfloat16),   # whole tiles that fill the chip
    (20000, 1900, 200, 10, 0, torch.bfloat16),   # one query tile, whole
    (3900, 4100, 129, 20, 0, torch.float32),     # one query tile, cut; ragged depth
    (300, 32768, 256, 10, 0, torch.bfloat16),
])
def test_keys_out_kernel(n, d, b, k, r, dtype):
    L, q = _layer(n, d, b, k, dtype, 61 + n + b)
    check_case(L.entries, L.labels, q, 10, k, max(1, k - 2), r)


@pytest.mark.parametrize("n,d,b,k,r,dtype", [
    (2500, 4104, 40, 20, 0, torch.bfloat16),     # 17 to 32 candidates of 4,096 to 16,383 values: one step
    (2500, 4104, 40, 20, 0, torch.float32),
    (2500, 4104, 100, 20, 0, torch.bfloat16),    # ... two steps
    (2500, 4104, 100, 20, 0, torch.float32),
    (2500, 8200, 600, 24, 0, torch.bfloat16),
    (600, 16384, 40, 20, 0, torch.bfloat16),     # by the whole workgroup
    (600, 16392, 70, 20, 0, torch.float32),
])
def test_rescoring_by_groups_of_waves(n, d, b, k, r, dtype):
    L, q = _layer(n, d, b, k, dtype, 71 + n + b)
    check_case(L.entries, L.labels, q, 10, k, max(1, k - 2), r)


@pytest.mark.parametrize("n,d,kc", [
    (3000, 4104, 260),      # 4.3 MB of centres: grouped order from the second round on
    (1301, 4100, 250),      # d a multiple of 4 only
    (1100, 3333, 310),      # odd rows
])
def test_kmeans_in_grouped_order(n, d, kc):
    kmeans.test_kmeans_build_and_lookup_against_oracle(n, d, kc, 7, 2, False)


def _distance_in_order(q, row):
    """sum (q_i - c_i)^2 in fp32 as the library adds it up for rows whose length is no multiple of eight: chain l of 64 takes
    elements l, l + 64, .. with fused multiply-adds, then the chains 32, 16, 8, 4, 2 and 1 apart are added.  q, row [m, d]."""
    m, d = q.shape
    pad = -d % 64
    diff = np.pad(q - row, ((0, 0), (0, pad))).reshape(m, -1, 64)        # fp32; padding adds zeros
    acc = np.zeros((m, 64), dtype=np.float32)
    for s in range(diff.shape[1]):
        x = diff[:, s].astype(np.float64)
        acc = (x * x + acc.astype(np.float64)).astype(np.float32)        # the product is exact in fp64
    lane = np.arange(64)
    for off in (32, 16, 8, 4, 2, 1):
        acc = acc + acc[:, lane ^ off]
    return acc[:, 0]


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (3000, 517, 300, 10, torch.bfloat16),     # block minima
    (3000, 517, 300, 10, torch.float32),
    (3000, 517, 100, 20, torch.bfloat16),     # keys: one or two rows per wave
    (3000, 517, 100, 40, torch.float32),      # ... four
    (3000, 517, 100, 1, torch.bfloat16),      # fewer rows than waves
    (3000, 517, 9, 10, torch.bfloat16),       # keys, few queries
    (3000, 117, 9, 10, torch.bfloat16),       # small-batch kernel
    (1500, 4101, 1030, 10, torch.bfloat16),   # lists: four rows per wave
    (1500, 4101, 1030, 20, torch.float32),    # ... eight
    (1500, 4101, 1030, 40, torch.bfloat16),   # ... sixteen
    (700, 62, 300, 5, torch.float32),         # shorter than a wave
])
def test_order_of_additions(n, d, b, k, dtype):
    """Distances bit for bit, whichever kernel formed them."""
    L, q = _layer(n, d, b, k, dtype, 3 + n + d + b)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        out = fc.lookup(0, q.cuda(), k, max(1, k - 2))
        torch.cuda.synchronize()
        idx, dist = out["idx"].cpu().numpy(), out["dist"].cpu().numpy()
    finally:
        fc.close()
    ent, q = L.entries.float().numpy(), q.numpy()
    for j in (0, k // 2, k - 1):
        assert np.array_equal(_distance_in_order(q, ent[idx[:, j]]), dist[:, j]), j


@pytest.mark.parametrize("n,d,b,k", [(20000, 2, 1, 1), (20000, 2, 3, 2), (20000, 2, 1, 3), (500, 1, 5, 2)])
def test_merge_of_the_exact_scan(n, d, b, k):
    """Dense points on a line or plane, which the coarse key cannot rank: every query is scanned, and the lists of up to 512
    workgroups meet, few enough in all to be sorted at once or not."""
    g = torch.Generator().manual_seed(n + d + k)
    ent, q = torch.rand(n, d, generator=g), torch.rand(b, d, generator=g)
    lab = torch.randint(0, 10, (n,), generator=g, dtype=torch.int32)
    fc = binding.FreezeCache(1)
    try:
        c = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_lookup_stats_attach(fc.ctx, c)
        fc.build_layer(0, ent.cuda(), lab.cuda(), 10)
        out = fc.lookup(0, q.cuda(), k, 1)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
    finally:
        fc.close()
    ref = parity.oracle_reference(q.numpy(), ent.numpy(), lab.numpy(), 10, k, 1)
    parity.assert_lookup_matches(got, ref, q.numpy(), ent.numpy(), lab.numpy(), 10, k, 1, rel=TIGHT, dist_rel=TIGHT)
    assert n < 1000 or c.tolist()[2] > 0


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (1, 3100, 1030, 1, torch.bfloat16),
    (7, 3333, 1100, 3, torch.float32),
    (30, 4104, 1030, 20, torch.bfloat16),
])
def test_lists_that_hold_the_whole_cache(n, d, b, k, dtype):
    """Nothing is left out of the lists of a cache that small: no query needs more than the first re-scoring of all entries."""
    g = torch.Generator().manual_seed(n + d)
    ent, q = torch.randn(n, d, generator=g).to(dtype), torch.randn(b, d, generator=g)
    lab = torch.randint(0, 10, (n,), generator=g, dtype=torch.int32)
    fc = binding.FreezeCache(1)
    try:
        c = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_lookup_stats_attach(fc.ctx, c)
        fc.build_layer(0, ent.cuda(), lab.cuda(), 10)
        out = fc.lookup(0, q.cuda(), k, 1)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(ent), lab.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, 1)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, 1, rel=TIGHT, dist_rel=TIGHT)
    assert c.tolist()[2] == 0
