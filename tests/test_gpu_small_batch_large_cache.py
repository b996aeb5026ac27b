"""The small-batch kernel on the caches that take it from rows of 193 values on, 250,000 entries and more: both of its
configurations (rows up to 512 and up to 1,024 values), both dtypes, ragged lengths, and the widths of its selection."""
import pytest
import torch

from paper_2002_02645_amd import binding, synth
from tests import parity
from tests.test_gpu_parity import _host_entries

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (250001, 193, 4, 10, torch.bfloat16),     # the shortest rows of the rule; a tile with one entry
    (250001, 250, 8, 20, torch.float32),
    (250112, 512, 2, 40, torch.bfloat16),     # R = 64 and k > 32
    (250001, 513, 4, 20, torch.float32),      # the configuration for longer rows, at its shortest
    (250001, 700, 8, 10, torch.float32),      # eight queries: up to 768 values
    (250000, 768, 8, 10, torch.bfloat16),
    (250001, 1000, 4, 10, torch.bfloat16),
    (260000, 1023, 1, 1, torch.bfloat16),     # odd length, one neighbour
    (500001, 500, 16, 10, torch.bfloat16),    # sixteen queries: up to 512 values from 500,000 entries on
    (500000, 257, 9, 24, torch.bfloat16),
])
def test_large_caches(n, d, b, k, dtype):
    spec = synth.LayerSpec(n, d, 10, 0.8, relu=True, store_bf16=(dtype == torch.bfloat16))
    L = synth.make_layer(spec, 50 + n + d, "cuda")
    q = synth.make_queries(L, (torch.arange(b) % 10).to(torch.int32), 7 + d)
    thr = max(1, k - 2)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries, L.labels.cuda(), 10)
        # this kernel leaves no keys, which 16 rows of the streaming kernel's would need
        assert binding.freeze_lookup_workspace_bytes(fc.ctx, 0, b, k) < 16 * n * 4
        assert binding.freeze_lookup_workspace_bytes(fc.ctx, 0, 17, k) > 16 * n * 4
        out = fc.lookup(0, q, k, thr)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy() for key, v in out.items()}
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(L.entries.cpu()), L.labels.cpu().numpy(), q.cpu().numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, thr)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, thr, rel=1e-5, dist_rel=1e-5)
