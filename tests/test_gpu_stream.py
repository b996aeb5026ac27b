"""The streaming distance kernel (batches of at most 128 queries, up to 1,024 on small caches): every query tile,
tiles cut by the ends of ranges and whole ones, first and last sizes of its range, against the CPU
oracle; the later layers of a small cascade, whose live count is on the device; and the entry point
with the fixed workspace, which has to fall back to ranges of whole tiles."""
import numpy as np
import pytest
import torch

from oracle import freeze_oracle as fo
from paper_2002_02645_amd import binding, synth
from tests import parity
from tests.test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


def _inputs(n, d, b, k, dtype, seed):
    wl = synth.scaled(synth.WORKLOADS["c2_batched"], n=n, batch=b)
    spec = synth.LayerSpec(n, d, 10, wl.layers[0].sigma, relu=True, store_bf16=(dtype == torch.bfloat16))
    data = synth.make_workload(type(wl)(wl.name, (spec,), b, k, (max(1, k - 2),), 0, seed))
    return data.layers[0], data.queries[0]


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (256, 1030, 1, 3, torch.bfloat16),       # one cache tile, one query, 33 k-steps cut over several workgroups
    (257, 8200, 16, 5, torch.float32),       # the second tile holds one entry; a full tile of 16 queries
    (5000, 1030, 16, 10, torch.bfloat16),
    (20000, 2100, 17, 10, torch.bfloat16),   # 32-query tile, cut tiles
    (20000, 2100, 32, 1, torch.float32),
    (16640, 2048, 33, 20, torch.bfloat16),   # 64-query tile
    (16640, 2048, 64, 10, torch.bfloat16),
    (16500, 2100, 65, 10, torch.bfloat16),   # 128-query tile
    (16500, 2100, 128, 30, torch.bfloat16),  # k = 30: R = 64
    (27000, 1200, 12, 5, torch.float32),     # tiles long enough to be cut (38 k-steps), whole because that is faster,
    (27000, 1200, 28, 10, torch.bfloat16),   # at every size of the query tile
    (27000, 1100, 70, 10, torch.bfloat16),
    (33393, 1100, 120, 10, torch.bfloat16),
    (70000, 500, 33, 10, torch.bfloat16),    # short activation: whole tiles
    (140000, 64, 100, 10, torch.float32),    # the shortest tile: two k-steps, fewer than the ring's stages
    (2000, 512, 256, 5, torch.float32),      # small cache, several query tiles
    (300, 65, 130, 4, torch.bfloat16),
])
def test_stream_shapes(n, d, b, k, dtype):
    L, q = _inputs(n, d, b, k, dtype, 900 + n + b)
    check_case(L.entries, L.labels, q, 10, k, max(1, k - 2))


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (2900, 4100, 257, 10, torch.bfloat16),   # three query tiles cut along the depth
    (2900, 4100, 600, 20, torch.float32),
    (1500, 2048, 1024, 10, torch.bfloat16),  # (block minima)
    (1500, 2048, 1025, 10, torch.bfloat16),  # (block minima)
    (5000, 1024, 640, 5, torch.bfloat16),    # ten query tiles, whole (32 k-steps), in place of block minima
])
def test_keys_out_for_several_query_tiles(n, d, b, k, dtype):
    L, q = _inputs(n, d, b, k, dtype, 900 + n + b)
    check_case(L.entries, L.labels, q, 10, k, max(1, k - 2))


@pytest.mark.parametrize("n,k,r", [
    (2000, 20, 0),     # 64 blocks of 32 entries: half of them, the width itself, are let in and not all
    (1280, 20, 0),     # 40: the width is more than half
    (1025, 20, 0),     # ... the last eight of which hold one entry
    (1024, 20, 0),     # 32, as many as the width: groups of entries in their place
    (2000, 40, 0),     # ... width 64, two entries per thread
    (40, 10, 0), (17, 10, 0),   # ... hardly more entries than the width
    (2000, 20, 33),    # a width beyond half
    (700, 10, 0),      # 24 blocks, width 16
    (500, 1, 0),       # 16, width 8
])
def test_keys_of_few_blocks(n, k, r):
    L, q = _inputs(n, 512, 40, k, torch.bfloat16, 40 + n + k + r)
    check_case(L.entries, L.labels, q, 10, k, max(1, k - 2), r)


@pytest.mark.parametrize("batch,thresholds", [(1, (8, 8, 8, 8)), (40, (10, 10, 10, 10)), (128, (8, 8, 8, 8))])
def test_small_cascade(batch, thresholds):
    """All layers by the streaming kernel; with thresholds of 10 of 10 many requests go all the way."""
    wl = synth.scaled(synth.WORKLOADS["c4_cascade_noisy"], n=3000, d_div=32, batch=batch)
    data = synth.make_workload(wl)
    nl = len(wl.layers)
    fc = binding.FreezeCache(nl)
    try:
        for l, L in enumerate(data.layers):
            fc.build_layer(l, L.entries.cuda(), L.labels.cuda(), L.spec.num_classes)
        qs = [q.cuda().contiguous() for q in data.queries]
        out = fc.lookup_cascade(list(range(nl)), qs, wl.k, list(thresholds), 0)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
    finally:
        fc.close()
    exp_l, exp_x, exp_h, _ = fo.cascade([q.numpy() for q in data.queries], [synth.bf16_bits(L.entries) for L in data.layers],
                                        [L.labels.numpy() for L in data.layers], [L.spec.num_classes for L in data.layers],
                                        wl.k, thresholds)
    assert np.array_equal(got["label"], exp_l) and np.array_equal(got["exit_layer"], exp_x)
    assert np.array_equal(got["hits_per_layer"], exp_h)


def test_fixed_workspace_takes_whole_tiles():
    n, d, b, k = 20000, 1984, 100, 10
    L, q = _inputs(n, d, b, k, torch.bfloat16, 77)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        assert binding.freeze_lookup_workspace_bytes(fc.ctx, 0, b, k) > binding.FREEZE_STATIC_SCRATCH_BYTES
        out = fc.alloc_outputs(b, k)
        binding.freeze_lookup_static(fc.ctx, 0, q.cuda().contiguous(), k, 8, 0, out["label"], out["hit"], out["votes"],
                                     out["idx"], out["dist"])
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
    finally:
        fc.close()
    e_h, l_h, q_h = synth.bf16_bits(L.entries), L.labels.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, 8)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, 8, rel=1e-5, dist_rel=1e-5)
