"""Few queries on long rows: several workgroups share a query's re-scoring (materialised keys).  All ways a width divides, rows by
four waves and by sixteen, odd lengths, both types; in a cascade, whose live count is on the device; and replayed from a
captured graph."""
import numpy as np
import pytest
import torch

from oracle import freeze_oracle as fo
from paper_2002_02645_amd import binding, synth
from tests.test_gpu_blocks import _inputs
from tests.test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,b,k,r,dtype", [
    (1000, 16384, 1, 10, 0, torch.bfloat16),     # eight workgroups, two rows each
    (700, 16384, 4, 20, 0, torch.float32),       # ... four rows each
    (600, 20000, 3, 1, 0, torch.bfloat16),       # eight rows in all
    (600, 16392, 2, 10, 13, torch.bfloat16),     # thirteen rows: the last workgroup has one
    (1000, 4096, 2, 10, 0, torch.bfloat16),      # rows by four waves each; four workgroups
    (1000, 8200, 17, 10, 0, torch.float32),      # ... fp32, ragged depth
    (700, 8192, 60, 30, 0, torch.bfloat16),      # width 64; four workgroups of sixteen rows
    (700, 8192, 100, 10, 64, torch.bfloat16),    # the default's 16 rows shared by two, the other 48 by the last one
    (1000, 4099, 5, 10, 0, torch.bfloat16),      # odd length
    (1000, 9001, 5, 25, 0, torch.float32),
    (500, 66000, 128, 10, 0, torch.bfloat16),
    (14, 5000, 3, 10, 0, torch.float32),         # hardly more entries than neighbours
])
def test_shapes(n, d, b, k, r, dtype):
    L, q = _inputs(n, d, b, k, dtype, 40 + n + b)
    check_case(L.entries, L.labels, q, 10, k, max(1, k - 2), r)


def test_unconfirmed_queries():
    """One dense cloud: some queries are not confirmed by what the workgroups shared."""
    g = torch.Generator().manual_seed(11)
    ent = torch.randn(2000, 4096, generator=g).to(torch.bfloat16)
    lab = torch.randint(0, 10, (2000,), generator=g, dtype=torch.int32)
    q = torch.randn(60, 4096, generator=g)
    for r in (10, 11, 0):
        check_case(ent, lab, q, 10, 10, 5, r)


def test_in_a_cascade():
    wl = synth.scaled(synth.WORKLOADS["c4_cascade_noisy"], n=1500, d_div=8, batch=40)
    data = synth.make_workload(wl)
    nl = len(wl.layers)
    fc = binding.FreezeCache(nl)
    try:
        for l, L in enumerate(data.layers):
            fc.build_layer(l, L.entries.cuda(), L.labels.cuda(), L.spec.num_classes)
        qs = [q.cuda().contiguous() for q in data.queries]
        for _ in range(3):
            out = fc.lookup_cascade(list(range(nl)), qs, wl.k, [9] * nl, 0)
            torch.cuda.synchronize()
            got = {key: v.cpu().numpy() for key, v in out.items()}
            exp_l, exp_x, exp_h, _ = fo.cascade([q.numpy() for q in data.queries], [synth.bf16_bits(L.entries) for L in data.layers],
                                                [L.labels.numpy() for L in data.layers], [L.spec.num_classes for L in data.layers],
                                                wl.k, [9] * nl)
            assert np.array_equal(got["label"], exp_l) and np.array_equal(got["exit_layer"], exp_x)
            assert np.array_equal(got["hits_per_layer"], exp_h)
    finally:
        fc.close()


def test_replayed_from_a_graph():
    n, d, b, k = 1000, 8192, 8, 10
    L, q = _inputs(n, d, b, k, torch.bfloat16, 77)
    _, q2 = _inputs(n, d, b, k, torch.bfloat16, 78)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        q_dev = q.cuda()
        out = fc.alloc_outputs(b, k)
        fc.lookup(0, q_dev, k, 8, out=out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            fc.lookup(0, q_dev, k, 8, out=out)
        for i in range(4):
            q_dev.copy_(q if i % 2 else q2)
            want = {key: v.clone() for key, v in fc.lookup(0, q_dev.clone(), k, 8).items()}
            graph.replay()
            torch.cuda.synchronize()
            for key in ("idx", "dist", "label", "votes", "hit"):
                assert torch.equal(out[key], want[key]), (key, i)
    finally:
        fc.close()
