"""Workspaces smaller than the preferred decomposition wants: the entry point with the fixed buffer, and a
buffer sized once for a full batch that serves the smaller ones too.  The decomposition changes the speed,
never the result, so every output equals that of a call with its own workspace, bit for bit."""
import pytest
import torch

from paper_2002_02645_amd import binding, synth
from tests.test_gpu_guard_bands import Guarded

pytestmark = pytest.mark.gpu


def _layer(n, d, b, k, dtype, seed):
    wl = synth.scaled(synth.WORKLOADS["c2_batched"], n=n, batch=b)
    spec = synth.LayerSpec(n, d, 10, wl.layers[0].sigma, relu=True, store_bf16=(dtype == torch.bfloat16))
    data = synth.make_workload(type(wl)(wl.name, (spec,), b, k, (max(1, k - 2),), 0, seed))
    return data.layers[0], data.queries[0]


def _equal(got, want):
    torch.cuda.synchronize()
    for key in want:
        assert torch.equal(got[key], want[key]), key


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (2000, 8192, 200, 10, torch.bfloat16),    # 2,048 k-steps per query tile: the preferred plan cuts tiles
    (800, 16384, 200, 5, torch.bfloat16),
    (3900, 4100, 129, 20, torch.float32),     # ragged depth, the first batch size past the streaming kernel's
    (300, 32768, 256, 10, torch.bfloat16),
])
def test_fixed_buffer_serves_whole_tiles_of_the_batched_kernel(n, d, b, k, dtype):
    L, q = _layer(n, d, b, k, dtype, 31 + n)
    thr = max(1, k - 2)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        assert binding.freeze_lookup_workspace_bytes(fc.ctx, 0, b, k) > binding.FREEZE_STATIC_SCRATCH_BYTES
        q = q.cuda().contiguous()
        want = fc.lookup(0, q, k, thr)
        got = fc.alloc_outputs(b, k)
        binding.freeze_lookup_static(fc.ctx, 0, q, k, thr, 0, got["label"], got["hit"], got["votes"], got["idx"], got["dist"])
        _equal(got, want)
    finally:
        fc.close()


@pytest.mark.parametrize("n,d,dtype,full,last,k", [
    (2900, 4104, torch.bfloat16, 1100, 700, 10),   # lists; 700 queries would rather have keys and accumulator slots
    (2900, 4100, torch.float32, 1100, 300, 20),
    (124, 23, torch.float32, 62, 5, 45),           # the streaming kernel; five queries are the small-batch kernel's
    (5000, 260, torch.bfloat16, 4096, 250, 10),    # block minima; 250 queries materialise their keys
])
def test_buffer_sized_for_the_full_batch_serves_the_last(n, d, dtype, full, last, k):
    L, q = _layer(n, d, full, k, dtype, 17 + n)
    thr = max(1, k - 2)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        ws = Guarded(binding.freeze_lookup_workspace_bytes(fc.ctx, 0, full, k))
        q = q.cuda()
        for b in (full, last):
            part = q[full - b:].clone()      # (a slice need not start on 16 bytes)
            want = fc.lookup(0, part, k, thr)
            got = fc.alloc_outputs(b, k)
            binding.freeze_lookup(fc.ctx, 0, part, k, thr, 0, got["label"], got["hit"], got["votes"], got["idx"], got["dist"],
                                  ws.payload)
            _equal(got, want)
            assert ws.intact()
    finally:
        fc.close()


@pytest.mark.parametrize("n,d,b,k,r,dtype", [
    (2900, 4104, 700, 10, 0, torch.bfloat16),    # keys and slots -> lists of 16
    (2901, 1500, 300, 20, 0, torch.float32),     # ... of 32, ragged depth
    (3000, 2050, 333, 40, 64, torch.bfloat16),   # ... of 64
    (20000, 517, 1300, 10, 0, torch.bfloat16),   # block minima -> lists
    (50000, 2048, 64, 10, 0, torch.bfloat16),    # cut tiles -> whole tiles, 64 queries per tile
    (36000, 2080, 200, 10, 64, torch.float32),   # ... of the 256-query kernel
    (300, 40, 1, 1, 0, torch.float32),
    (700, 16384, 900, 10, 0, torch.bfloat16),    # the longest rows, whose distances 1,024 threads add up on every route
])
def test_smaller_buffers_give_the_same_result_or_are_refused(n, d, b, k, r, dtype):
    L, q = _layer(n, d, b, k, dtype, 23 + n)
    thr = max(1, k - 2)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        q = q.cuda()
        want = fc.lookup(0, q, k, thr, r)
        size, served = binding.freeze_lookup_workspace_bytes(fc.ctx, 0, b, k, r), 0
        while True:
            ws = Guarded(size)
            got = fc.alloc_outputs(b, k)
            for t in got.values():
                t.fill_(7)
            try:
                binding.freeze_lookup(fc.ctx, 0, q, k, thr, r, got["label"], got["hit"], got["votes"], got["idx"], got["dist"],
                                      ws.payload)
            except binding.FreezeError as e:
                assert e.code == binding.FREEZE_EWORKSPACE
                torch.cuda.synchronize()
                assert all(bool((t == 7).all()) for t in got.values())    # a refused call writes nothing
                break
            _equal(got, want)
            assert ws.intact()
            served += 1
            size -= max(256, size // (256 if d == 16384 else 6))   # (there the routes' buffers differ by little)
        assert served >= 1
    finally:
        fc.close()


@pytest.mark.parametrize("n,d,b,k,r", [(3000, 8192, 100, 10, 16), (3000, 512, 128, 1, 8), (5000, 16384, 70, 20, 32)])
def test_materialised_keys_on_the_smallest_buffer(n, d, b, k, r):
    """Few queries take no more than their bf16 copy, the keys, block minima, candidates, and the exact scan's lists."""
    L, q = _layer(n, d, b, k, torch.bfloat16, 41 + n)
    thr = max(1, k - 2)
    rows, n_pad, cus = 128, (n + 255) // 256 * 256, torch.cuda.get_device_properties(0).multi_processor_count
    parts = [rows * d * 2, rows * n_pad * 4, rows * (n_pad // 32) * 8, rows * 4, rows * min(32 * r, 512) * 8, 16, b * 4, b * 4, b * 4,
             max(b, 2 * cus) * k * 8]
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        q = q.cuda()
        want = fc.lookup(0, q, k, thr)
        ws = Guarded(sum((x + 255) // 256 * 256 for x in parts))
        got = fc.alloc_outputs(b, k)
        binding.freeze_lookup(fc.ctx, 0, q, k, thr, 0, got["label"], got["hit"], got["votes"], got["idx"], got["dist"], ws.payload)
        _equal(got, want)
        assert ws.intact()
    finally:
        fc.close()


def test_cascade_and_thresholds_on_a_buffer_sized_for_the_full_batch():
    wl = synth.scaled(synth.WORKLOADS["c4_cascade_noisy"], n=2600, d_div=8, batch=1100)
    data = synth.make_workload(wl)
    nl, k = len(wl.layers), wl.k
    layers = list(range(nl))
    fc = binding.FreezeCache(nl)
    try:
        for l, L in enumerate(data.layers):
            fc.build_layer(l, L.entries.cuda(), L.labels.cuda(), L.spec.num_classes)
        full, last = 1100, 700
        ws = Guarded(binding.freeze_cascade_workspace_bytes(fc.ctx, layers, full, k))
        assert binding.freeze_cascade_workspace_bytes(fc.ctx, layers, last, k) > ws.nbytes
        model = torch.randint(0, 10, (full,), dtype=torch.int32).cuda()
        for b in (full, last, 20):
            qs = [q[full - b:].cuda().contiguous() for q in data.queries]
            want = fc.lookup_cascade(layers, qs, k, [9] * nl)
            got = {key: torch.empty_like(t) for key, t in want.items()}
            binding.freeze_lookup_cascade(fc.ctx, layers, qs, k, [9] * nl, 0, got["label"], got["exit_layer"],
                                          got["hits_per_layer"], ws.payload)
            _equal(got, want)
            thr = fc.compute_thresholds(layers, qs, k, model[:b])
            out = torch.empty_like(thr)
            binding.freeze_compute_thresholds(fc.ctx, layers, qs, k, 0, model[:b], out, ws.payload)
            torch.cuda.synchronize()
            assert torch.equal(out, thr) and ws.intact()
    finally:
        fc.close()


def test_projection_on_a_buffer_sized_for_the_full_batch():
    d, m, full = 1500, 1000, 600
    g = torch.Generator().manual_seed(8)
    x, w = torch.randn(full, d, generator=g), (torch.randn(m, d, generator=g) / d ** 0.5).to(torch.bfloat16)
    bias = torch.randn(m, generator=g) * 0.1
    ref = x.to(torch.bfloat16).double() @ w.double().t() + bias.double()
    scale = x.to(torch.bfloat16).double().abs() @ w.double().abs().t() + bias.double().abs()
    fc = binding.FreezeCache(1)
    try:
        fc.build_projection(0, w.cuda(), bias.cuda())
        ws = Guarded(binding.freeze_project_workspace_bytes(fc.ctx, 0, full))
        assert binding.freeze_project_workspace_bytes(fc.ctx, 0, 256) > ws.nbytes
        for b in (full, 400, 256, 17, 1):
            out = torch.empty(b, m, device="cuda")
            binding.freeze_project(fc.ctx, 0, x[:b].cuda(), False, out, ws.payload)
            torch.cuda.synchronize()
            # fp32 accumulation of exact products in blocks: (log2(d) + 16) * 2^-24 of the magnitude sum
            assert ((out.cpu().double() - ref[:b]).abs() <= 4e-6 * scale[:b]).all() and ws.intact()
    finally:
        fc.close()


@pytest.mark.parametrize("n,d,kc,twins", [
    (3000, 520, 300, False),
    (512, 16384, 512, True), (512, 16392, 500, True),   # the longest rows of few points, whose distances 1,024 threads add up
    (1030, 16384, 400, True), (600, 4104, 200, True), (700, 515, 260, True),
])
def test_kmeans_build_on_smaller_buffers(n, d, kc, twins):
    iters = 2
    g = torch.Generator().manual_seed(12)
    pts, lab = torch.randn(n, d, generator=g).cuda(), torch.randint(0, 7, (n,), generator=g, dtype=torch.int32).cuda()
    init = pts[:kc].clone()
    if twins:
        # two centres for every point, whose distances are sums of the same squares in another order: the nearer one is
        # a matter of the roundings
        iters = 0
        at = torch.randint(-32, 33, (kc // 2, d), generator=g) / 16.0
        off = torch.randint(-4095, 4096, (kc // 2, d), generator=g) / 4096.0
        init = torch.stack([at + off, at + off[:, torch.randperm(d, generator=g)]], 1).view(kc, d).cuda()
        pts = at[torch.arange(n) % (kc // 2)].cuda()
    fc = binding.FreezeCache(1)
    try:
        want = fc.build_kmeans_layer(0, pts, lab, 7, init, iters)
        storage = torch.empty(binding.freeze_kmeans_storage_bytes(kc, d), dtype=torch.uint8, device="cuda")
        size, served = binding.freeze_kmeans_workspace_bytes(fc.ctx, n, d, kc), 0
        while True:
            ws = Guarded(size)
            try:
                binding.freeze_kmeans_build(fc.ctx, 0, pts, lab, 7, init, iters, storage, ws.payload)
            except binding.FreezeError as e:
                assert e.code == binding.FREEZE_EWORKSPACE
                break
            got = dict(centers=torch.empty(kc, d, device="cuda"), majority=torch.empty(kc, dtype=torch.int32, device="cuda"),
                       fraction=torch.empty(kc, device="cuda"))
            binding.freeze_kmeans_read(fc.ctx, 0, got["centers"], got["majority"], got["fraction"])
            _equal(got, want)
            assert ws.intact()
            served += 1
            size -= max(256, size // 32)
        assert served >= 2
    finally:
        fc.close()


def test_buffers_without_room_for_the_bf16_copy_are_refused():
    """Also where the call would not make the copy of its inputs: what a buffer has to hold does not depend on the kernel."""
    b, d, m = 4096, 8192, 1024
    x = torch.randn(b, d, device="cuda")
    small = torch.empty(b * d * 2 - 4096, dtype=torch.uint8, device="cuda")
    fc = binding.FreezeCache(2)
    try:
        fc.build_projection(0, torch.randn(m, d, device="cuda"), torch.zeros(m, device="cuda"))
        out = torch.full((b, m), 7.0, device="cuda")
        with pytest.raises(binding.FreezeError) as e:
            binding.freeze_project(fc.ctx, 0, x, False, out, small)
        assert e.value.code == binding.FREEZE_EWORKSPACE
        st = torch.empty(binding.freeze_kmeans_storage_bytes(20, d), dtype=torch.uint8, device="cuda")
        with pytest.raises(binding.FreezeError) as e:
            binding.freeze_kmeans_build(fc.ctx, 1, x, torch.zeros(b, dtype=torch.int32, device="cuda"), 3, x[:20].clone(), 1, st, small)
        assert e.value.code == binding.FREEZE_EWORKSPACE
        torch.cuda.synchronize()
        assert bool((out == 7.0).all())
    finally:
        fc.close()
