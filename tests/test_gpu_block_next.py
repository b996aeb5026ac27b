"""Block minima that carry the place of the smallest key and a bound of the block's other entries: rows long enough for
the other kernels to add them up by four waves, blocks whose entries have to be re-scored after all because several of
the nearest lie in them, and equal entries."""
import pytest
import torch

from paper_2002_02645_amd import binding, synth
from tests import parity
from tests.test_gpu_blocks import _inputs
from tests.test_gpu_parity import _host_entries, check_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (3000, 4096, 1100, 10, torch.bfloat16),
    (3000, 4104, 1030, 20, torch.float32),    # R = 32
    (3100, 5001, 1030, 10, torch.bfloat16),   # rows of odd length, longer than 4,096
    (2000, 4099, 1030, 30, torch.float32),    # R = 64
    (2500, 4096, 700, 20, torch.bfloat16),    # four waves per query
])
def test_long_rows(n, d, b, k, dtype):
    L, q = _inputs(n, d, b, k, dtype, 900 + n + b)
    some = torch.arange(0, b, 8)              # (the oracle is slow)
    fc = binding.FreezeCache(1)
    try:
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        q_dev = q.cuda()
        out = fc.lookup(0, q_dev, k, k - 2)
        torch.cuda.synchronize()
        got = {key: v[some.to(v.device)].cpu().numpy() for key, v in out.items()}
        # the same queries in small batches (other kernels): the same distances bit for bit
        for i in range(0, 200, 100):
            part = fc.lookup(0, q_dev[i:i + 100].contiguous(), k, k - 2)
            torch.cuda.synchronize()
            for key in ("idx", "dist"):
                assert torch.equal(part[key], out[key][i:i + 100]), (key, i)
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(L.entries), L.labels.numpy(), q[some].numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, k - 2)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, k - 2, rel=1e-5, dist_rel=1e-5)


@pytest.mark.parametrize("n,d,copies,noise,k,dtype", [
    (4096, 512, 4, 0.02, 10, torch.bfloat16),    # the four entries a lane holds in a row of a block are near one another
    (4096, 512, 32, 0.02, 20, torch.float32),    # ... all of a block, and of its neighbour
    (4096, 512, 4, 0.0, 10, torch.bfloat16),     # equal entries: no lead within a block
    (4096, 512, 32, 0.0, 10, torch.float32),
    (700, 512, 2, 0.5, 64, torch.bfloat16),      # few blocks, k = 64
])
def test_near_entries_share_blocks(n, d, copies, noise, k, dtype):
    g = torch.Generator().manual_seed(3 + n + copies + k)
    base = torch.randn(n // copies, d, generator=g)
    ent = base.repeat_interleave(copies, 0)
    ent = (ent + noise * torch.randn(ent.shape, generator=g)).to(dtype)
    lab = torch.randint(0, 10, (ent.shape[0],), generator=g, dtype=torch.int32)
    q = base[torch.randint(0, n // copies, (300,), generator=g)] + 0.3 * torch.randn(300, d, generator=g)
    check_case(ent, lab, q, 10, k, max(1, k - 3))
