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


def _entries_of_blocks(n_pad):
    """[n_pad / 8, 8]: entry e of block blk."""
    blk, e = torch.arange(n_pad // 8)[:, None], torch.arange(8)[None, :]
    return (blk >> 5) * 256 + ((blk >> 3) & 3) * 64 + (blk & 1) * 32 + ((blk >> 1) & 3) * 4 + (e & 3) + (e >> 2) * 16


def _what_the_matrix_kernel_left(ws, ent, q):
    """"places", "minima" (alone) or None, by what lies in the workspace after a look-up on a cache that is not centred: the first
    and the last query's block minima, and behind the minima the places of these."""
    n, d = ent.shape
    n_pad, b = -(-n // 256) * 256, q.shape[0]
    b_pad, nb = -(-b // 256) * 256, n_pad // 8
    c, x = ent.to(torch.bfloat16).double(), q[[0, b - 1]].to(torch.bfloat16).double()
    key = torch.full((2, n_pad), float("inf"), dtype=torch.float64)
    key[:, :n] = ((c * c).sum(1)[None] - 2.0 * (x @ c.t())).cpu()
    of = _entries_of_blocks(n_pad)
    low, at = key[:, of].min(2)
    real = torch.isfinite(low[0])
    tol = 1e-4 * float((c * c).sum(1).max() + 2.0 * (x.norm(dim=1).max() * c.norm(dim=1).max()))
    f = ws[:ws.numel() // 4 * 4].view(torch.float32).cpu()
    for i in torch.nonzero((f - low[0, 0]).abs() < tol).flatten().tolist():
        last = i + (b - 1) * nb
        if last + nb > f.numel() or not ((f[i:i + nb] - low[0])[real].abs() < tol).all() or not ((f[last:last + nb] - low[1])[real].abs() < tol).all():
            continue
        start = (i + b_pad * nb) * 4          # (a multiple of 256: whole tiles of rows)
        found = ws[start:start + b * nb * 2]
        if found.numel() == b * nb * 2:
            place = (found.view(torch.int16).view(b, nb)[[0, b - 1]].cpu().int() & 7).long()
            if ((place == at)[:, real].float().mean(1) > 0.9).all():     # (but for keys that are equal up to rounding)
                return "places"
        return "minima"
    return None


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (1000, 12000, 700, 10, torch.bfloat16),
    (3000, 9000, 1030, 10, torch.float32),
    (1500, 16384, 1100, 10, torch.bfloat16),   # the longest rows on this route, with more queries than 1,024 threads each add up for
    (3000, 16384, 1030, 10, torch.float32),
])
def test_rows_beyond_8192_values(n, d, b, k, dtype):
    L, q = _inputs(n, d, b, k, dtype, 17 + n + b)
    some = torch.arange(0, b, 16)             # (the oracle is slow)
    fc = binding.FreezeCache(1)
    try:
        binding.freeze_set_centring(fc.ctx, 0)
        fc.build_layer(0, L.entries.cuda(), L.labels.cuda(), 10)
        q_dev = q.cuda()
        out = fc.lookup(0, q_dev, k, k - 2)
        torch.cuda.synchronize()
        assert _what_the_matrix_kernel_left(fc._ws, L.entries.cuda(), q_dev) == "places"
        got = {key: v[some.to(v.device)].cpu().numpy() for key, v in out.items()}
        if d < 16384:   # the same queries in small batches (other kernels): the same distances bit for bit
            part = fc.lookup(0, q_dev[:100].contiguous(), k, k - 2)
            torch.cuda.synchronize()
            for key in ("idx", "dist"):
                assert torch.equal(part[key], out[key][:100]), key
    finally:
        fc.close()
    e_h, l_h, q_h = _host_entries(L.entries), L.labels.numpy(), q[some].numpy()
    ref = parity.oracle_reference(q_h, e_h, l_h, 10, k, k - 2)
    parity.assert_lookup_matches(got, ref, q_h, e_h, l_h, 10, k, k - 2, rel=1e-5, dist_rel=1e-5)


@pytest.mark.parametrize("n,d,b,k,dtype", [
    (4096, 512, 300, 10, torch.bfloat16),
    (20011, 517, 700, 20, torch.float32),
    (2500, 4104, 1100, 10, torch.bfloat16),
])
def test_buffers_without_room_for_the_places(n, d, b, k, dtype):
    """Smaller and smaller buffers: minima with the places, minima alone (where they pay on rows of this length), then lists
    where these need less."""
    L, q = _inputs(n, d, b, k, dtype, 31 + n + b)
    fc = binding.FreezeCache(1)
    routes = []
    try:
        binding.freeze_set_centring(fc.ctx, 0)
        ent, q = L.entries.cuda(), q.cuda()
        fc.build_layer(0, ent, L.labels.cuda(), 10)
        want = fc.lookup(0, q, k, k - 2)
        size = binding.freeze_lookup_workspace_bytes(fc.ctx, 0, b, k)
        step = -(-b // 256) * 256 * (-(-n // 256) * 256) // 16 * 4 // 3 // 256 * 256   # a third of the places
        while size > 0:
            ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
            got = fc.alloc_outputs(b, k)
            try:
                binding.freeze_lookup(fc.ctx, 0, q, k, k - 2, 0, got["label"], got["hit"], got["votes"], got["idx"], got["dist"], ws)
            except binding.FreezeError as e:
                assert e.code == binding.FREEZE_EWORKSPACE
                break
            torch.cuda.synchronize()
            for key in want:
                assert torch.equal(got[key], want[key]), (key, size)
            routes.append(_what_the_matrix_kernel_left(ws, ent, q))
            size -= step
    finally:
        fc.close()
    assert routes[0] == "places" and routes == sorted(routes, key=["places", "minima", None].index), routes
    assert ("minima" in routes) == (d <= 3072), routes
