"""The work that a user of the cache look-up library has it do, as cases for timing and comparison.

Every case is a dict of plain values; its "kind" says which public entry points a pass goes through:

  lookup    one layer's cache is resident, a batch of activations is looked up (vote rule or the
            distance-weighted confidence); with "rebuild" the missed requests' activations are then
            compacted into the next layer's input, as a program that runs the model layer by layer does
  cascade   the layers of a model in order, only the misses going on (one call)
  kmeans    the k-means cache of a layer is built from its points
  project   the dense layer in front of a look-up
  offline   caches of new activations are built and the layers' thresholds computed on a validation set

The sizes are those of the benchmark configurations (CIFAR ResNet-18 block outputs: 65,536, 32,768,
16,384, 8,192 and, pooled, 512 values; 50,000 training images; the serving case with 1,000,000 entries)
and odd sizes between them.  Inputs are the synthetic class-clustered activations of synth.py.
"""
import math

import torch

from paper_2002_02645_amd import binding, synth

DEV = "cuda:0"
NOISE = (0.35, 0.25, 0.15, 0.05)   # share of deviating cache labels by depth: early layers agree less


def listed():
    return [
        # one request against a large cache of pooled activations: the latency a freeze decision adds
        dict(name="serve_b1_pooled", kind="lookup", n=1000000, d=512, b=1, k=20, r=0, bf16=True, relu=False,
             sigma=0.7, classes=100, flip=0.0, conf=False, rebuild=False),
        # one request at a middle block of the network (256 x 8 x 8 outputs)
        dict(name="serve_b1_block", kind="lookup", n=50000, d=16384, b=1, k=10, r=0, bf16=True, relu=True,
             sigma=0.8, classes=10, flip=0.15, conf=False, rebuild=False),
        # a serving batch under the paper's confidence rule, then the next layer's input from the misses
        dict(name="serve_b32_block", kind="lookup", n=50000, d=8192, b=32, k=10, r=0, bf16=True, relu=True,
             sigma=0.8, classes=10, flip=0.25, conf=True, rebuild=True),
        # the smallest look-ups: a small fp32 cache, launches and latencies count
        dict(name="small_cache", kind="lookup", n=2000, d=512, b=256, k=5, r=0, bf16=False, relu=False,
             sigma=0.5, classes=10, flip=0.0, conf=False, rebuild=False),
        # a whole evaluation batch at a block's output
        dict(name="batch_block", kind="lookup", n=50000, d=8192, b=10000, k=10, r=0, bf16=True, relu=True,
             sigma=0.8, classes=10, flip=0.0, conf=False, rebuild=False),
        # the widest block output, a moderate batch, the caller's own re-scoring width
        dict(name="wide_b256", kind="lookup", n=50000, d=65536, b=256, k=10, r=64, bf16=True, relu=False,
             sigma=1.5, classes=10, flip=0.0, conf=False, rebuild=False),
        # an evaluation batch at the pooled output
        dict(name="batch_pooled", kind="lookup", n=50000, d=512, b=4096, k=10, r=0, bf16=True, relu=False,
             sigma=0.3, classes=10, flip=0.05, conf=False, rebuild=False),
        # a serving batch through the caches of all blocks
        dict(name="cascade_b32", kind="cascade", n=50000, dims="65536,32768,16384,512", b=32, k=10),
        # an evaluation batch through the caches of all blocks: the largest case
        dict(name="cascade_b4096", kind="cascade", n=50000, dims="65536,32768,16384,512", b=4096, k=10),
        # the k-means cache of a block (200 centres)
        dict(name="kmeans_block", kind="kmeans", n=50000, d=8192, centres=200, iters=2),
        # the dense layer of 1,024 units in front of a look-up
        dict(name="project_block", kind="project", b=10000, d=8192, m=1024, bf16=True, relu=True),
        # the offline phase on activations of odd sizes handed over in fp32: build two layers, thresholds
        dict(name="offline_odd", kind="offline", n=20011, dims="4104,517", b=1537, k=20, bf16=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["serve", "serve", "serve", "batch", "batch", "batch", "cascade", "kmeans", "project", "offline"])
    if kind in ("serve", "batch"):
        bf16 = rng.random() < 0.7
        d = rng.choice([512, 1024, 8192, 16384, _log(rng, 200, 65536), _log(rng, 200, 65536) // 8 * 8])
        most = 3.2e9 if bf16 else 6e8            # values in the cache
        n = _log(rng, 2000, max(4000, min(1000000, most / d)))
        b = _log(rng, 1, 64) if kind == "serve" else _log(rng, 65, max(130, min(10000, 4e12 / (n * d))))
        k = rng.choice([1, 5, 10, 10, 20, rng.randint(2, 30)])
        return dict(kind="lookup", n=n, d=d, b=b, k=k, r=0, bf16=bf16, relu=rng.random() < 0.5, sigma=0.8,
                    classes=rng.choice([10, 100]), flip=rng.choice([0.0, 0.15, 0.25]), conf=rng.random() < 0.4,
                    rebuild=rng.random() < 0.3)
    if kind == "cascade":
        dims = [65536, 32768, 16384, 8192, 512][rng.randint(0, 2):]
        n = _log(rng, 2000, 50000)
        return dict(kind="cascade", n=n, dims=",".join(str(x) for x in dims[:4]), b=_log(rng, 1, 2048),
                    k=rng.choice([5, 10]))
    if kind == "kmeans":
        return dict(kind="kmeans", n=_log(rng, 3000, 50000), d=rng.choice([512, 2048, _log(rng, 300, 8192)]),
                    centres=_log(rng, 20, 400), iters=rng.randint(1, 3))
    if kind == "project":
        return dict(kind="project", b=_log(rng, 1, 10000), d=rng.choice([8192, 16384, _log(rng, 500, 32768)]),
                    m=rng.choice([1024, 256, rng.randint(100, 1500)]), bf16=rng.random() < 0.5, relu=rng.random() < 0.5)
    d0 = _log(rng, 600, 8192)
    return dict(kind="offline", n=_log(rng, 3000, 30000), dims="%d,%d" % (d0, rng.choice([512, d0 // 4])),
                b=_log(rng, 200, 2000), k=rng.choice([5, 10, 20]), bf16=rng.random() < 0.5)


class State:
    pass


def _dims(case):
    return [int(x) for x in case["dims"].split(",")]


def _classes(b, classes, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(0, classes, (b,), generator=g, dtype=torch.int64).to(torch.int32)


def _lookup_inputs(case, seed):
    spec = synth.LayerSpec(case["n"], case["d"], case["classes"], case["sigma"], relu=case["relu"],
                           store_bf16=case["bf16"], label_flip_p=case["flip"])
    layer = synth.make_layer(spec, 1000 * seed + 1, DEV)
    return layer, synth.make_queries(layer, _classes(case["b"], case["classes"], seed), 1000 * seed + 50)


def _layer_stack(case, seed, sigma, bf16):
    """The layers of a cascade or of the offline phase, one at a time: (layer, its queries)."""
    dims = _dims(case)
    cls = _classes(case["b"], 10, seed)
    for i, d in enumerate(dims):
        spec = synth.LayerSpec(case["n"], d, 10, sigma[i], store_bf16=bf16, label_flip_p=NOISE[len(NOISE) - len(dims) + i])
        layer = synth.make_layer(spec, 1000 * seed + 100 * i + 1, DEV)
        yield layer, synth.make_queries(layer, cls, 1000 * seed + 100 * i + 50)


def _model_labels(case, seed):
    # what the model itself predicts for the validation items: one in ten is not the items' class
    g = torch.Generator().manual_seed(seed + 7)
    other = torch.randint(1, 10, (case["b"],), generator=g, dtype=torch.int64).to(torch.int32)
    wrong = torch.rand(case["b"], generator=g) < 0.1
    cls = _classes(case["b"], 10, seed)
    return torch.where(wrong, (cls + other) % 10, cls).to(torch.int32).to(DEV)


def _cascade_sigma(dims):
    return [{65536: 1.5, 32768: 1.0, 16384: 0.6, 8192: 0.8}.get(d, 0.3) for d in dims]


def _conf_threshold(case):
    # what about 80 % agreement amounts to at the typical distance between two items of a class
    return 0.8 * 0.8 * case["k"] / (case["sigma"] * math.sqrt(2.0 * case["d"] * (0.5 if case["relu"] else 1.0)))


def _kmeans_inputs(case, seed):
    layer = synth.make_layer(synth.LayerSpec(case["n"], case["d"], 10, 0.8, store_bf16=False), 1000 * seed + 1, DEV)
    return layer.entries, layer.labels, layer.entries[: case["centres"]].clone()


def _project_inputs(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn(case["b"], case["d"], device=DEV, generator=g).clamp_(min=0.0)
    w = torch.randn(case["m"], case["d"], device=DEV, generator=g) / case["d"] ** 0.5
    bias = 0.1 * torch.randn(case["m"], device=DEV, generator=g)
    return x, w.to(torch.bfloat16) if case["bf16"] else w, bias


def prepare(case, seed):
    s = State()
    s.case, kind = case, case["kind"]
    if kind == "lookup":
        layer, s.q = _lookup_inputs(case, seed)
        s.fc = binding.FreezeCache(1, DEV)
        s.fc.build_layer(0, layer.entries, layer.labels, case["classes"])
        s.out = s.fc.alloc_outputs(case["b"], case["k"])
        if case["conf"]:
            s.out["conf"] = torch.empty(case["b"], dtype=torch.float32, device=DEV)
        if case["rebuild"]:
            s.out["sel"] = torch.full((case["b"],), -1, dtype=torch.int32, device=DEV)
            s.out["missed"] = torch.zeros(1, dtype=torch.int32, device=DEV)
            s.out["next"] = torch.zeros_like(s.q)
    elif kind == "cascade":
        dims = _dims(case)
        s.fc, s.q = binding.FreezeCache(len(dims), DEV), []
        for i, (layer, q) in enumerate(_layer_stack(case, seed, _cascade_sigma(dims), True)):
            s.fc.build_layer(i, layer.entries, layer.labels, 10)
            s.q.append(q)
            del layer
        s.out = dict(label=torch.empty(case["b"], dtype=torch.int32, device=DEV),
                     exit_layer=torch.empty(case["b"], dtype=torch.int32, device=DEV),
                     hits_per_layer=torch.empty(len(dims), dtype=torch.int64, device=DEV))
    elif kind == "kmeans":
        s.fc = binding.FreezeCache(1, DEV)
        s.points, s.labels, s.init = _kmeans_inputs(case, seed)
    elif kind == "project":
        s.fc = binding.FreezeCache(1, DEV)
        s.x, w, bias = _project_inputs(case, seed)
        s.fc.build_projection(0, w, bias)
    else:
        dims = _dims(case)
        s.fc, s.entries, s.labels, s.q = binding.FreezeCache(len(dims), DEV), [], [], []
        for layer, q in _layer_stack(case, seed, [0.8] * len(dims), case["bf16"]):
            s.entries.append(layer.entries)
            s.labels.append(layer.labels)
            s.q.append(q)
        s.model_labels = _model_labels(case, seed)
    return s


def run(s):
    c, kind = s.case, s.case["kind"]
    if kind == "lookup":
        if c["conf"]:
            s.fc.lookup_confidence(0, s.q, c["k"], _conf_threshold(c), c["r"], out=s.out)
        else:
            s.fc.lookup(0, s.q, c["k"], max(1, int(0.8 * c["k"])), c["r"], out=s.out)
        if c["rebuild"]:
            binding.freeze_compact_misses(s.out["hit"], None, s.out["sel"], s.out["missed"])
            binding.freeze_gather_rows(s.q, s.out["sel"], s.out["missed"], s.out["next"])
        return s.out
    if kind == "cascade":
        layers = list(range(len(s.q)))
        return s.fc.lookup_cascade(layers, s.q, c["k"], [max(1, int(0.8 * c["k"]))] * len(layers), 0, out=s.out)
    if kind == "kmeans":
        return s.fc.build_kmeans_layer(0, s.points, s.labels, 10, s.init, c["iters"])
    if kind == "project":
        return s.fc.project(0, s.x, c["relu"])
    for i in range(len(s.q)):
        s.fc.build_layer(i, s.entries[i], s.labels[i], 10)
    return s.fc.compute_thresholds(list(range(len(s.q))), s.q, c["k"], s.model_labels)


def _share_on(k, need, p):
    """Share of requests with at least `need` of k neighbours carrying the right label."""
    return sum(math.comb(k, i) * (1 - p) ** i * p ** (k - i) for i in range(need, k + 1))


def work(case):
    kind = case["kind"]
    if kind == "lookup":
        n, d, b, k = case["n"], case["d"], case["b"], case["k"]
        # (the vote needs the cache once; the stored values of the neighbours are part of it)
        more = 2 * b * d * 4 * (1 - _share_on(k, max(1, int(0.8 * k)), case["flip"])) if case["rebuild"] else 0
        return {"bytes": n * d * 2 + b * d * 4 + b * (8 * k + 9) + more, "flops": 2.0 * b * n * d}
    if kind == "cascade":
        dims, live, total, flops = _dims(case), float(case["b"]), 0.0, 0.0
        for i, d in enumerate(dims):
            total += case["n"] * d * 2 + live * d * 4
            flops += 2.0 * live * case["n"] * d
            live *= 1 - _share_on(case["k"], max(1, int(0.8 * case["k"])), NOISE[len(NOISE) - len(dims) + i])
        return {"bytes": total, "flops": flops}
    if kind == "kmeans":
        n, d, c = case["n"], case["d"], case["centres"]
        # every round reads the points to assign them and, but for the last, to average them
        return {"bytes": (2 * case["iters"] + 1) * n * d * 4 + 2 * c * d * 4, "flops": 2.0 * (case["iters"] + 1) * n * c * d}
    if kind == "project":
        b, d, m = case["b"], case["d"], case["m"]
        return {"bytes": b * d * 4 + m * d * 2 + b * m * 4, "flops": 2.0 * b * d * m}
    size = 2 if case["bf16"] else 4
    return {"bytes": sum(case["n"] * d * (2 * size + 4) + case["b"] * d * 4 for d in _dims(case)),
            "flops": sum(2.0 * case["n"] * d * case["b"] for d in _dims(case))}


def tolerance(case):
    if case["kind"] == "kmeans":
        # a point between two centres may go to either; the mean of a cluster then moves
        return {"rel": 1e-3, "max": 0.05, "differ": 0.01}
    # 32-bit sums (measured against 64 bits: 5e-8 for a distance, 3e-7 for the projection, whose large
    # products cancel); neighbours closer than their rounding may change places
    return {"rel": 2e-6, "max": 2e-5, "differ": 0.01}


def _knn64(q, entries, k):
    """The k nearest entries of every query in 64 bits: (squared distances, indices), nearest first."""
    n, d = entries.shape
    qd = q.double()
    best_d = best_i = None
    rows = max(64, min((1 << 28) // d, (1 << 30) // q.shape[0]))
    for lo in range(0, n, rows):
        e = entries[lo:lo + rows].double()
        dist = (e * e).sum(1)[None, :] - 2.0 * (qd @ e.t())
        v, i = dist.topk(min(k + 6, e.shape[0]), dim=1, largest=False)
        i = i + lo
        if best_d is not None:
            v, i = torch.cat([best_d, v], 1), torch.cat([best_i, i], 1)
            v, at = v.topk(min(k + 6, v.shape[1]), dim=1, largest=False)
            i = i.gather(1, at)
        best_d, best_i = v, i
        del e, dist
    out_d, out_i = [], []
    step = max(1, (1 << 26) // (d * best_i.shape[1]))
    for lo in range(0, q.shape[0], step):
        i = best_i[lo:lo + step]
        diff = qd[lo:lo + step, None, :] - entries[i].double()
        dist = (diff * diff).sum(2)
        i, at = i.sort(dim=1)
        dist = dist.gather(1, at)
        dist, at = dist.sort(dim=1, stable=True)
        out_d.append(dist[:, :k])
        out_i.append(i.gather(1, at)[:, :k])
    return torch.cat(out_d), torch.cat(out_i)


def _confidence64(dist, labels):
    """Confidence of the winning label and that label (shares of the label times its summed 1 / distance)."""
    k = labels.shape[1]
    same = (labels[:, :, None] == labels[:, None, :]).double()
    c = same.sum(2) / k * (same * (1.0 / dist.sqrt())[:, None, :]).sum(2)
    top = c.max(1).values
    return top, torch.where(c == top[:, None], labels, 1 << 30).min(1).values


def exact(case, seed):
    kind = case["kind"]
    if kind == "lookup":
        layer, q = _lookup_inputs(case, seed)
        dist, idx = _knn64(q, layer.entries, case["k"])
        out = dict(dist=dist, idx=idx.to(torch.int32))
        if case["conf"]:
            out["conf"] = _confidence64(dist, layer.labels[idx])[0]
        return out
    if kind == "project":
        x, w, bias = _project_inputs(case, seed)
        out = []
        wd = w.to(torch.bfloat16).double().t()
        for lo in range(0, case["b"], 2048):
            out.append(x[lo:lo + 2048].to(torch.bfloat16).double() @ wd + bias.double())
        y = torch.cat(out)
        return y.clamp_(min=0.0) if case["relu"] else y
    if kind == "kmeans":
        points, labels, cen = _kmeans_inputs(case, seed)
        cen, assign = cen.double(), None
        for it in range(case["iters"] + 1):
            assign = []
            for lo in range(0, case["n"], 4096):
                p = points[lo:lo + 4096].double()
                assign.append(((cen * cen).sum(1)[None, :] - 2.0 * (p @ cen.t())).argmin(1))
            assign = torch.cat(assign)
            size = torch.bincount(assign, minlength=case["centres"])
            if it < case["iters"]:
                total = torch.zeros_like(cen)
                for lo in range(0, case["n"], 4096):
                    total.index_add_(0, assign[lo:lo + 4096], points[lo:lo + 4096].double())
                cen = torch.where(size[:, None] > 0, total / size.clamp(min=1)[:, None], cen).float().double()
        votes = torch.zeros(case["centres"], 10, dtype=torch.int64, device=DEV)
        votes.index_put_((assign, labels.long()), torch.ones_like(assign), accumulate=True)
        return dict(centers=cen, majority=None, fraction=votes.max(1).values.double() / size.clamp(min=1))
    if kind == "offline":
        thr = []
        model = _model_labels(case, seed)
        for layer, q in _layer_stack(case, seed, [0.8] * len(_dims(case)), case["bf16"]):
            dist, idx = _knn64(q, layer.entries, case["k"])
            conf, label = _confidence64(dist, layer.labels[idx])
            thr.append(torch.where(label != model, conf, torch.zeros_like(conf)).max())
        return torch.stack(thr)
    return None   # a cascade returns whole numbers only
