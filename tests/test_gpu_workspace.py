"""Workspaces smaller than the preferred decomposition wants: the entry point with the fixed buffer, and a
buffer sized once for a full batch that serves the smaller ones too.  The decomposition changes the speed,
never the result, so every output equals that of a call with its own workspace, bit for bit."""
import pytest
import torch

from paper_2002_02645_amd import binding, synth

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
