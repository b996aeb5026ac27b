"""The projection of small batches (streaming kernel, tiles cut along the depth): edges of its query tiles
and of the output tiles, odd output widths, and nothing written outside the output."""
import numpy as np
import pytest
import torch

from oracle import freeze_oracle as fo
from paper_2002_02645_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,d,m,wdtype,relu", [
    (1, 4100, 1024, torch.bfloat16, True),    # one input, every output tile cut over many workgroups
    (16, 64, 1, torch.float32, False),        # one whole tile, one column
    (17, 1100, 257, torch.bfloat16, False),   # the second output tile holds one column; odd rows
    (64, 2050, 1023, torch.float32, True),
    (129, 2048, 250, torch.bfloat16, True),
    (512, 1030, 510, torch.float32, False),   # the last batch size of this route
    (513, 1030, 510, torch.float32, False),   # ... and the first beyond it
    (700, 8200, 700, torch.bfloat16, True),   # fewer than 16 k-steps per CU, deep enough to be cut
    (1000, 2295, 4, torch.float32, False),    # ... and not
])
def test_small_projection(b, d, m, wdtype, relu):
    g = torch.Generator().manual_seed(77 + b + d + m)
    x = torch.randn(b, d, generator=g)
    w = (torch.randn(m, d, generator=g) / d ** 0.5).to(wdtype)
    bias = torch.randn(m, generator=g) * 0.1
    fc = binding.FreezeCache(1)
    try:
        fc.build_projection(0, w.cuda(), bias.cuda())
        guard = 1024
        raw = torch.full((guard + b * m + guard,), 123.0, device="cuda")
        out = raw[guard:guard + b * m].view(b, m)
        ws = torch.empty(binding.freeze_project_workspace_bytes(fc.ctx, 0, b), dtype=torch.uint8, device="cuda")
        binding.freeze_project(fc.ctx, 0, x.cuda(), relu, out, ws)
        torch.cuda.synchronize()
        assert (raw[:guard] == 123.0).all() and (raw[guard + b * m:] == 123.0).all()
        got = out.cpu().numpy()
    finally:
        fc.close()
    w_h = synth.bf16_bits(w) if wdtype == torch.bfloat16 else w.numpy()
    ref = fo.project(x.numpy(), w_h, bias.numpy(), relu)
    xr, wr = x.to(torch.bfloat16).double(), w.to(torch.bfloat16).double()
    scale = (xr.abs() @ wr.abs().t()).numpy() + np.abs(bias.numpy())[None, :]
    # fp32 accumulation of exact products in blocks: (log2(d) + 16) * 2^-24 of the magnitude sum
    assert (np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= 4e-6 * scale + 1e-30).all()
