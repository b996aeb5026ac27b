"""The projection straight from its fp32 inputs: tiles of 192 and of 256 rows, cut along the depth and whole, all widths of
a column tile, a last row tile that reaches back, depths that end within a k-step or are no multiple of four, and inputs that
are no finite numbers."""
import pytest
import torch

from paper_2002_02645_amd import binding

pytestmark = pytest.mark.gpu


def _project(x, w, bias, relu):
    fc = binding.FreezeCache(1)
    try:
        fc.build_projection(0, w.cuda(), bias.cuda())
        y = fc.project(0, x, relu)
        torch.cuda.synchronize()
        return y
    finally:
        fc.close()


@pytest.mark.parametrize("b,d,m,relu", [
    (257, 8192, 1024, False),      # the second tile of 192 rows reaches back over most of the first
    (300, 30020, 300, True),       # a k-step with four elements at the end; column tiles of 192
    (512, 16384, 1024, True),      # tiles of 256 rows
    (2000, 16384, 200, False),     # ... cut over many ranges; one column tile of which 56 columns are padding
    (700, 8191, 1001, True),       # neither rows nor output rows on 16 bytes
    (1100, 8193, 130, False),      # column tiles of 128; one element in the last k-step
    (10000, 500, 128, True),       # short depth: whole tiles and cut ones
    (10000, 1000, 1500, False),    # six column tiles
    (400000, 36, 64, True),        # whole tiles only
])
def test_rows(b, d, m, relu):
    g = torch.Generator(device="cuda").manual_seed(b + d + m)
    x = torch.randn(b, d, device="cuda", generator=g)
    w = (torch.randn(m, d, device="cuda", generator=g) / d ** 0.5).to(torch.bfloat16)
    bias = 0.1 * torch.randn(m, device="cuda", generator=g)
    y = _project(x, w, bias, relu)
    some = torch.arange(b, device="cuda") if b <= 2000 else torch.cat([torch.arange(300), torch.arange(b - 300, b), torch.randint(0, b, (1000,))]).cuda()
    xr, wr = x[some].to(torch.bfloat16).double(), w.double()
    ref = xr @ wr.t() + bias.double()
    scale = xr.abs() @ wr.abs().t() + bias.double().abs()
    if relu:
        ref = ref.clamp_(min=0.0)
    # fp32 accumulation of exact bf16 x bf16 products in blocks: (log2(d) + 16) * 2^-24 of the magnitude sum
    assert ((y[some].double() - ref).abs() <= 4e-6 * scale).all()


@pytest.mark.parametrize("d", [8190, 8193, 8196])
def test_no_finite_numbers(d):
    """Infinities and NaN anywhere in a row (its first element included, which stands in for what lies past its end) give
    what the same row gives in a small batch, which goes through a bf16 copy of the inputs."""
    b, m = 300, 1024
    g = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn(b, d, device="cuda", generator=g)
    x[0, 0] = float("inf")
    x[1, 0] = float("nan")
    x[2, d - 1] = float("-inf")
    x[3, 5000] = 3.4e38       # rounds to infinity
    x[299, 0] = float("-inf")
    w = (torch.randn(m, d, device="cuda", generator=g) / d ** 0.5).to(torch.bfloat16)
    bias = torch.zeros(m, device="cuda")
    whole = _project(x, w, bias, False)
    for rows in (slice(0, 100), slice(200, 300)):
        part = _project(x[rows].contiguous(), w, bias, False)
        a = whole[rows]
        assert torch.equal(a.isnan(), part.isnan()) and torch.equal(a.isinf(), part.isinf())
        assert torch.equal(a[a.isinf()], part[part.isinf()])
    assert whole[0].isinf().all() and whole[1].isnan().all() and whole[10].isfinite().all()


@pytest.mark.parametrize("b,d,m,most", [
    (6079, 8192, 1024, 2.56e-7),     # sums of 96 k-steps; of 128, as tiles of 192 rows have them, 3.2e-7
    (1500, 8192, 1024, 1.38e-7),
    (3000, 8192, 700, 1.58e-7),      # three column tiles: groups of workgroups across the XCDs
    (1050, 16384, 1190, 1.94e-7),    # five
    (766, 16384, 256, 1.43e-7),      # many slots per tile
    (544, 25600, 256, 1.62e-7),
])
def test_error_of_the_sums(b, d, m, most):
    # The length of a chain of fp32 additions, and of the sums of its pieces, is the error of the result.  most: relative error
    # (2-norm) on these inputs with tiles of 256 x 256 whose k-steps are dealt evenly to 256 CUs; 5 % for other random inputs.
    g = torch.Generator(device="cuda").manual_seed(b)
    x = torch.randn(b, d, device="cuda", generator=g).clamp_(min=0.0)
    w = (torch.randn(m, d, device="cuda", generator=g) / d ** 0.5).to(torch.bfloat16)
    bias = 0.1 * torch.randn(m, device="cuda", generator=g)
    y = _project(x, w, bias, False)
    ref = x.to(torch.bfloat16).double() @ w.double().t() + bias.double()
    assert ((y.double() - ref).norm() / ref.norm()).item() <= 1.05 * most


@pytest.mark.parametrize("b,d,m,first", [
    (700, 8192, 1024, 0),            # the outputs over the first inputs
    (700, 8192, 1024, 699 * 8192),   # ... over the last row and past it
    (400, 16384, 256, 12),
])
def test_outputs_over_inputs(b, d, m, first):
    g = torch.Generator(device="cuda").manual_seed(b + first)
    buf = torch.randn(b * d + b * m, device="cuda", generator=g)
    x, out = buf[:b * d].view(b, d), buf[first:first + b * m].view(b, m)
    w = (torch.randn(m, d, device="cuda", generator=g) / d ** 0.5).to(torch.bfloat16)
    bias = 0.1 * torch.randn(m, device="cuda", generator=g)
    xr = x.to(torch.bfloat16).double()
    ref = xr @ w.double().t() + bias.double()
    scale = xr.abs() @ w.double().abs().t() + bias.double().abs()
    fc = binding.FreezeCache(1)
    try:
        fc.build_projection(0, w, bias)
        ws = torch.empty(binding.freeze_project_workspace_bytes(fc.ctx, 0, b), dtype=torch.uint8, device="cuda")
        binding.freeze_project(fc.ctx, 0, x, False, out, ws)
        torch.cuda.synchronize()
    finally:
        fc.close()
    assert ((out.double() - ref).abs() <= 4e-6 * scale).all()   # as in test_rows
