"""The block-minima route (batches on short activations): sizes at the edges of its tiles, groups and
selection, against the CPU oracle; its certificate on inputs the coarse key cannot rank; and the later
layers of a cascade, whose live count is on the device."""
import numpy as np
import pytest
import torch

from oracle import freeze_oracle as fo
from paper_2002_02645_amd import binding, synth
from tests import parity
from tests.test_gpu_parity import check_case, run_lookup

pytestmark = pytest.mark.gpu


def _inputs(n, d, b, k, dtype, seed, relu=True):
    wl = synth.scaled(synth.WORKLOADS["c2_batched"], n=n, batch=b)
    spec = synth.LayerSpec(n, d, 10, wl.layers[0].sigma, relu=relu, store_bf16=(dtype == torch.bfloat16))
    data = synth.make_workload(type(wl)(wl.name, (spec,), b, k, (max(1, k - 2),), 0, seed))
    return data.layers[0], data.queries[0]


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (300, 64, 257, 5, torch.bfloat16),       # two k-steps a tile: fewer than the ring's stages; 38 blocks with an entry
    (51, 48, 300, 1, torch.float32),         # a few blocks in all: taken at once
    (97, 60, 600, 5, torch.bfloat16),
    (256, 20, 513, 10, torch.float32),       # one cache tile, a third query tile with one row, d not a multiple of 8
    (2049, 100, 300, 1, torch.bfloat16),     # k = 1; d a multiple of 4 only; a tile with one entry
    (8200, 517, 300, 20, torch.float32),     # R = 32, odd d
    (20000, 260, 400, 40, torch.bfloat16),   # R = 64: every wave gives its 16th smallest
    (3000, 1000, 260, 64, torch.bfloat16),   # (the streaming kernel; k = 64 below)
    (3000, 300, 260, 64, torch.float32),     # k = 64: the first round takes all that may be taken
    (3000, 128, 1100, 64, torch.bfloat16),   # ... two waves per query
    (66000, 64, 1100, 10, torch.bfloat16),   # two waves per query; more blocks than the registers hold
    (9000, 1030, 1030, 7, torch.bfloat16),   # five query tiles, two per group
])
def test_block_shapes(n, d, b, k, dtype):
    L, q = _inputs(n, d, b, k, dtype, 700 + n + b)
    check_case(L.entries, L.labels, q, 10, k, max(1, k - 2))


@pytest.mark.parametrize("offset,copies", [(100.0, 1), (0.0, 40)])
def test_block_certificate(offset, copies):
    """Far from the origin without centring the key's rounding exceeds the neighbours' differences; with
    every entry present 40 times whole blocks tie.  Either way the result is the oracle's."""
    n, d, b, k = 4000, 128, 300, 10
    L, q = _inputs(n // copies, d, b, k, torch.bfloat16, 4242, relu=False)
    ent = (L.entries.float() + offset).to(torch.bfloat16).repeat(copies, 1)
    labels = L.labels.repeat(copies)
    q = q + offset
    e_h, l_h, q_h = synth.bf16_bits(ent), labels.numpy(), q.numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, 8)
    fc = binding.FreezeCache(1)
    try:
        counters = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_lookup_stats_attach(fc.ctx, counters)
        binding.freeze_set_centring(fc.ctx, 0)
        fc.build_layer(0, ent.cuda(), labels.cuda(), 10)
        out = fc.lookup(0, q.cuda(), k, 8)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
        c = counters.cpu().numpy()
    finally:
        fc.close()
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, 8, rel=1e-5, dist_rel=1e-5)
    assert c.sum() == b and c[1] + c[2] > 0, "this input is meant to defeat the coarse ranking"


def test_blocks_in_a_cascade():
    wl = synth.scaled(synth.WORKLOADS["c4_cascade_noisy"], n=2500, d_div=64, batch=900)
    data = synth.make_workload(wl)
    nl = len(wl.layers)
    fc = binding.FreezeCache(nl)
    try:
        for l, L in enumerate(data.layers):
            fc.build_layer(l, L.entries.cuda(), L.labels.cuda(), L.spec.num_classes)
        out = fc.lookup_cascade(list(range(nl)), [q.cuda().contiguous() for q in data.queries], wl.k, [9] * nl, 0)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
    finally:
        fc.close()
    exp_l, exp_x, exp_h, _ = fo.cascade([q.numpy() for q in data.queries], [synth.bf16_bits(L.entries) for L in data.layers],
                                        [L.labels.numpy() for L in data.layers], [L.spec.num_classes for L in data.layers],
                                        wl.k, [9] * nl)
    assert np.array_equal(got["label"], exp_l) and np.array_equal(got["exit_layer"], exp_x)
    assert np.array_equal(got["hits_per_layer"], exp_h)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_entries_whose_norm_overflows(dtype):
    """Finite values whose squares overflow in fp32: the distance is +inf, and such entries rank behind all
    others in the order of their indices.  Only five of 300 entries are nearer here, none of them
    in a block with the first indices."""
    n, d, b, k = 300, 64, 300, 10
    g = torch.Generator().manual_seed(99)
    ent = torch.randn(n, d, generator=g) * 1e25
    near = [100, 130, 200, 255, 290]
    ent[near] = torch.randn(5, d, generator=g)
    ent = ent.to(dtype)
    q = torch.randn(b, d, generator=g)
    labels = torch.randint(0, 10, (n,), generator=g, dtype=torch.int32)
    got = run_lookup(ent, labels, q, 10, k, 3)
    dist = ((q.double()[:, None, :] - ent[near].double()[None]) ** 2).sum(2)
    order = dist.argsort(dim=1)
    assert np.array_equal(got["idx"][:, :5], np.array(near)[order.numpy()])
    np.testing.assert_allclose(got["dist"][:, :5], dist.sort(dim=1).values.numpy(), rtol=1e-5)
    assert np.array_equal(got["idx"][:, 5:], np.broadcast_to(np.arange(5), (b, 5)))
    assert np.isposinf(got["dist"][:, 5:]).all()

@pytest.mark.parametrize("n,d,dtype", [
    (3000, 512, torch.bfloat16),
    (3000, 517, torch.float32),
    (3000, 517, torch.bfloat16),
    (3000, 100, torch.bfloat16),     # a multiple of 4 only
    (2500, 20, torch.float32),
    (20000, 1030, torch.float32),
    (20000, 2053, torch.bfloat16),
])
def test_distances_do_not_depend_on_the_batch(n, d, dtype):
    """The same queries in one batch (block minima), in batches of 100 and of 16 (other finishing kernels):
    the same distances bit for bit, which is also what the exact scan of an unconfirmed query gives."""
    b, k = 300, 10
    L, q = _inputs(n, d, b, k, dtype, 5 + n + d)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        q = q.cuda()
        whole = fc.lookup(0, q, k, 8)
        for step in (100, 16):
            for i in range(0, b, step):
                part = fc.lookup(0, q[i:i + step].contiguous(), k, 8)
                torch.cuda.synchronize()
                for key in ("idx", "dist"):
                    assert torch.equal(part[key], whole[key][i:i + step]), (key, step, i)
    finally:
        fc.close()
