"""GPU parity for the distance-weighted confidence rule (Sec. 3 heuristic), its cascade
(Pseudocode 1, FreezeInference with float thresholds) and ComputeThresholds, through the C ABI,
against the CPU oracle on the same seeded inputs."""
import numpy as np
import pytest
import torch

from oracle import freeze_oracle as fo
from paper_2002_02645_amd import binding, synth
from tests import parity

pytestmark = pytest.mark.gpu

TIGHT = 1e-5


def _host_entries(t: torch.Tensor) -> np.ndarray:
    return synth.bf16_bits(t) if t.dtype == torch.bfloat16 else t.detach().cpu().numpy()


def run_confidence(entries, labels, queries, num_classes, k, thr, r=0):
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, entries.cuda().contiguous(), labels.cuda().contiguous(), num_classes)
        out = fc.lookup_confidence(0, queries.cuda().contiguous(), k, thr, r)
        torch.cuda.synchronize()
        return {key: v.cpu().numpy() for key, v in out.items()}
    finally:
        fc.close()


def check_confidence(entries, labels, queries, num_classes, k, thr=None, r=0):
    e_h, l_h, q_h = _host_entries(entries), labels.cpu().numpy(), queries.cpu().numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, num_classes, k, 1)
    if thr is None:   # the oracle's median confidence: both outcomes occur
        _, conf = fo.confidence(l_h, ref["idx"], ref["sqdist"], num_classes)
        thr = float(np.float32(np.median(conf[np.isfinite(conf)])))
    got = run_confidence(entries, labels, queries, num_classes, k, thr, r)
    for rel in (TIGHT, parity.REL):
        near, amb, fails = parity.compare_confidence(got, ref, q_h, e_h, l_h, num_classes, k, thr, rel=rel)
        assert not fails, f"rel {rel}: {len(fails)} mismatching queries, first: {fails[:5]}"
    # the votes output is the winning label's share of the k neighbours
    for i in range(q_h.shape[0]):
        assert got["votes"][i] == (l_h[got["idx"][i]] == got["label"][i]).sum()
    return got, ref, thr


def test_hand_example_confidence_on_gpu():
    ent = torch.tensor([[0, 0], [1, 0], [0, 2], [3, 0], [1, 0], [4, 4]], dtype=torch.float32)
    lab = torch.tensor([0, 0, 1, 1, 1, 0], dtype=torch.int32)
    q = torch.tensor([[1, 1], [1, 0]], dtype=torch.float32)
    c1 = 0.6 * (1 + 1 / np.sqrt(2) + 1 / np.sqrt(5))
    for dt in (torch.float32, torch.bfloat16):
        got = run_confidence(ent.to(dt), lab, q, 2, 5, 1.0)
        assert got["label"][0] == 1 and got["votes"][0] == 3 and got["hit"][0] == 1
        assert got["conf"][0] == np.float32(c1)
        assert np.isposinf(got["conf"][1]) and got["hit"][1] == 1   # a cached copy of the query: always a hit
        # strict comparison: the confidence itself as threshold is a miss, the next float below is a hit
        got = run_confidence(ent.to(dt), lab, q, 2, 5, float(np.float32(c1)))
        assert got["hit"][0] == 0
        got = run_confidence(ent.to(dt), lab, q, 2, 5, float(np.nextafter(np.float32(c1), np.float32(0))))
        assert got["hit"][0] == 1
    # closeness beats plurality (two of label 0 at distance 1, three of label 1 at distance 10)
    ent = torch.tensor([[1, 0], [-1, 0], [10, 0], [-10, 0], [0, 10]], dtype=torch.float32)
    lab = torch.tensor([0, 0, 1, 1, 1], dtype=torch.int32)
    got = run_confidence(ent, lab, torch.zeros(1, 2), 2, 5, 0.5)
    assert got["label"][0] == 0 and got["votes"][0] == 2 and got["hit"][0] == 1
    assert got["conf"][0] == pytest.approx(0.8, rel=1e-6)
    # equal confidences: the smaller label id
    got = run_confidence(torch.tensor([[2., 0.], [-2., 0.]]), torch.tensor([5, 3], dtype=torch.int32),
                         torch.zeros(1, 2), 6, 2, 0.0)
    assert got["label"][0] == 3 and got["conf"][0] == np.float32(0.25)


def test_config1_confidence_full_batch():
    wl = synth.WORKLOADS["c1_tiny"]
    data = synth.make_workload(wl)
    L = data.layers[0]
    got, _, _ = check_confidence(L.entries, L.labels, data.queries[0], 10, wl.k)
    assert 0 < got["hit"].sum() < wl.batch


@pytest.mark.parametrize("n,d,b,k,r,dtype", [
    (777, 100, 37, 7, 0, torch.float32),       # streaming kernel, ragged everything
    (5000, 1024, 600, 10, 0, torch.bfloat16),  # ... ten query tiles
    (20000, 512, 8, 20, 0, torch.bfloat16),    # streaming kernel, few queries
    (250001, 512, 8, 20, 0, torch.bfloat16),   # small-batch kernel
    (3000, 2048, 100, 10, 0, torch.bfloat16),  # long rows
    (1500, 192, 9, 33, 0, torch.bfloat16),     # k > 24
    (300, 64, 1, 1, 0, torch.float32),         # k = 1: confidence = 1 / distance
    (1200, 4096, 300, 10, 0, torch.bfloat16),  # long activations: the two-step re-scoring in front of the rule
    (900, 4104, 40, 20, 0, torch.float32),     # ... width 32, few queries (one step), fp32 cache
])
def test_confidence_shapes_random_labels(n, d, b, k, r, dtype):
    wl = synth.scaled(synth.WORKLOADS["c2_batched"], n=n, batch=b)
    spec = wl.layers[0]
    spec = type(spec)(n, d, 10, spec.sigma, relu=True, store_bf16=(dtype == torch.bfloat16))
    data = synth.make_workload(type(wl)(wl.name, (spec,), b, k, (1,), r, 177 + n + d))
    L = data.layers[0]
    # labels independent of the geometry: several labels share the k neighbours of most queries
    lab = synth.random_labels(n, 4, 31 + n)
    got, _, _ = check_confidence(L.entries, lab, data.queries[0], 4, k, None, r)
    if k == 1:
        assert np.allclose(got["conf"], 1.0 / np.sqrt(got["dist"][:, 0]), rtol=1e-6)


def test_confidence_with_cached_copies_of_the_query():
    wl = synth.scaled(synth.WORKLOADS["c1_tiny"], n=900, batch=60)
    data = synth.make_workload(wl)
    L = data.layers[0]
    q = data.queries[0].clone()
    q[:15] = L.entries[200:215]
    lab = synth.random_labels(900, 4, 5)
    got, _, _ = check_confidence(L.entries, lab, q, 4, 7, 3.0)
    assert np.isposinf(got["conf"][:15]).all() and got["hit"][:15].all()
    assert (got["label"][:15] == lab[200:215].numpy()).all()
    assert np.isfinite(got["conf"][15:]).all()


def _cascade_problem(seed_shift=0, batch=300, val=200):
    from dataclasses import replace
    wl = synth.scaled(synth.WORKLOADS["c4_cascade_noisy"], n=3000, batch=batch + val, d_div=32)
    wl = replace(wl, seed=wl.seed + seed_shift)
    return wl, synth.make_workload(wl, device="cuda")


def test_compute_thresholds_and_confidence_cascade_against_oracle():
    val, batch = 200, 300
    wl, data = _cascade_problem(0, batch, val)
    nl = len(wl.layers)
    ents = [_host_entries(L.entries) for L in data.layers]
    labs = [L.labels.cpu().numpy() for L in data.layers]
    ncls = [L.spec.num_classes for L in data.layers]
    v_q = [q[:val].contiguous() for q in data.queries]
    t_q = [q[val:].contiguous() for q in data.queries]
    y = data.query_classes[:val].to(torch.int32).cpu().contiguous()   # the model's label for each validation item
    fc = binding.FreezeCache(nl)
    try:
        for l, L in enumerate(data.layers):
            fc.build_layer(l, L.entries, L.labels, L.spec.num_classes)
        thr = fc.compute_thresholds(list(range(nl)), v_q, wl.k, y.cuda())
        torch.cuda.synchronize()
        thr_h = thr.cpu().numpy()
        # zero validation error (Sec. 3.1): with its own thresholds no validation item freezes wrongly
        out_v = fc.lookup_cascade_confidence(list(range(nl)), v_q, wl.k, thr_h.tolist())
        torch.cuda.synchronize()
        xv, lv = out_v["exit_layer"].cpu().numpy(), out_v["label"].cpu().numpy()
        assert (lv[xv >= 0] == y.numpy()[xv >= 0]).all()
        # the cascade on fresh requests: thresholds as the library computed them, and stricter ones
        # (each layer's median confidence by the oracle) so that every exit, and none, occurs
        tq_h = [q.cpu().numpy() for q in t_q]
        med = [float(np.float32(np.median(fo.lookup_confidence(tq_h[l], ents[l], labs[l], ncls[l], wl.k, 0.0)["conf"])))
               for l in range(nl)]
        got = {}
        for name, th in (("computed", thr_h.tolist()), ("median", med)):
            out_t = fc.lookup_cascade_confidence(list(range(nl)), t_q, wl.k, th)
            torch.cuda.synchronize()
            got[name] = {key: v.cpu().numpy() for key, v in out_t.items()}
    finally:
        fc.close()
    exp_thr = fo.compute_thresholds([q.cpu().numpy() for q in v_q], ents, labs, ncls, wl.k, y.numpy())
    assert (exp_thr > 0).any(), "label noise must produce wrong look-ups"
    assert np.allclose(thr_h, exp_thr, rtol=TIGHT, atol=0), (thr_h, exp_thr)
    for name, th in (("computed", thr_h.tolist()), ("median", med)):
        g = got[name]
        exp_l, exp_x, exp_hits = fo.cascade_confidence(tq_h, ents, labs, ncls, wl.k, th)
        per = [fo.lookup_confidence(tq_h[l], ents[l], labs[l], ncls[l], wl.k, th[l]) for l in range(nl)]
        ambiguous = np.zeros(batch, dtype=bool)
        for l in range(nl):
            ambiguous |= np.abs(per[l]["conf"].astype(np.float64) - th[l]) <= parity.REL * th[l]
            ref = parity.oracle_reference(tq_h[l], ents[l], labs[l], ncls[l], wl.k, 1)
            # the k-th and the first excluded neighbour nearly equidistant: either may be reported
            # (swaps inside the first k do not change a confidence beyond rounding)
            D = ref["sqdist_ext"]
            ambiguous |= (D[:, wl.k] - D[:, wl.k - 1]) < parity.REL * D[:, wl.k]
        ok = ~ambiguous
        assert ok.sum() > batch // 2
        assert np.array_equal(g["exit_layer"][ok], exp_x[ok]), name
        assert np.array_equal(g["label"][ok], exp_l[ok]), name
        assert g["hits_per_layer"].sum() == (g["exit_layer"] >= 0).sum()
        for l in range(nl):
            assert g["hits_per_layer"][l] == (g["exit_layer"] == l).sum()
    assert set(got["median"]["exit_layer"].tolist()) == {-1, 0, 1, 2, 3}


def test_thresholds_are_zero_without_wrong_lookups_and_argument_errors():
    wl = synth.scaled(synth.WORKLOADS["c1_tiny"], n=600, batch=40)
    data = synth.make_workload(wl, device="cuda")
    L = data.layers[0]
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries, L.labels, 10)
        q = data.queries[0]
        # clean separable classes: every look-up agrees with the request's class
        thr = fc.compute_thresholds([0], [q], 5, data.query_classes.to(torch.int32).cuda())
        torch.cuda.synchronize()
        assert thr.cpu().tolist() == [0.0]
        out = fc.alloc_outputs(40, 5)
        out["conf"] = torch.empty(40, dtype=torch.float32, device="cuda")
        for bad_thr in (-1.0, float("nan")):
            with pytest.raises(binding.FreezeError):
                fc.lookup_confidence(0, q, 5, bad_thr)
            with pytest.raises(binding.FreezeError):
                fc.lookup_cascade_confidence([0], [q], 5, [bad_thr])
        with pytest.raises(binding.FreezeError):
            fc.lookup_confidence(0, q, 601, 0.5)
        # an empty batch is a no-op
        e = fc.lookup_confidence(0, q[:0], 5, 0.5)
        assert e["conf"].numel() == 0
        thr = fc.compute_thresholds([0], [q[:0]], 5, torch.empty(0, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        assert thr.cpu().tolist() == [0.0]
    finally:
        fc.close()
