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


@pytest.mark.parametrize("n,d,copies,k,dtype", [
    (4200, 512, 21, 10, torch.bfloat16),     # ten of 21 equal entries in 21 blocks: too few distances for a certificate in 64 blocks
    (4200, 1024, 21, 20, torch.float32),
    (2600, 4096, 13, 10, torch.bfloat16),
    (4200, 512, 21, 64, torch.bfloat16),
])
def test_copies_in_many_blocks(n, d, copies, k, dtype):
    """Every query needs the 256 blocks with the smallest keys, and more queries than the follow-up takes."""
    g = torch.Generator().manual_seed(n + d + k)
    ent = torch.randn(n // copies, d, generator=g).repeat(copies, 1).to(dtype)
    lab = torch.randint(0, 10, (n,), generator=g, dtype=torch.int32)
    q = torch.randn(1100 if d == 4096 else 300, d, generator=g)
    some = torch.arange(0, q.shape[0], 5)
    fc = binding.FreezeCache(1)
    try:
        counters = torch.zeros(3, dtype=torch.int64, device="cuda")
        binding.freeze_lookup_stats_attach(fc.ctx, counters)
        fc.build_layer(0, ent.cuda(), lab.cuda(), 10)
        out = fc.lookup(0, q.cuda(), k, 1)
        torch.cuda.synchronize()
        got = {key: v.cpu().numpy()[some.numpy()] for key, v in out.items()}
        c = counters.tolist()
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(ent), lab.numpy(), q[some].numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, 1)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, 1, rel=1e-5, dist_rel=1e-5)
    assert sum(c) == q.shape[0] and c[1] + c[2] > 32, c
