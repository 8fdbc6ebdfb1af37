"""GELU and its derivative in the contractions' epilogues: against float64 beside the erf form in fp32,
and what is not finite."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2104_00237_amd import _lib as L  # noqa: E402

DEV = "cuda:0"


def _run(x):
    """GELU(x) and GELU'(x) through a 1 x 1 linear layer of weight 1."""
    n, s = x.numel(), torch.cuda.current_stream().cuda_stream
    w, one = torch.ones(1, 1, device=DEV), torch.ones(n, 1, device=DEV)
    z, y, dx = (torch.empty(n, 1, device=DEV) for _ in range(3))
    W = L.OfParam(w.data_ptr(), None, None, None, 1)
    d = L.OfLinearDesc(n, 1, 1, 0, 0, L.OF_F32, L.OF_ACT_GELU, 0, 0)
    e = L.OfLinearDesc(n, 1, 1, 0, 0, L.OF_F32, 0, 0, 0)
    ws = torch.empty(max(L.of_linear_workspace_size(d, 0), L.of_linear_workspace_size(e, 1)) // 4 + 16, device=DEV)
    L.of_linear_fwd(d, x.data_ptr(), W, None, z.data_ptr(), y.data_ptr(), ws.data_ptr(), ws.numel() * 4, s)
    L.of_linear_bwd_data(e, one.data_ptr(), W, x.data_ptr(), L.OF_ACT_GELU, dx.data_ptr(), ws.data_ptr(),
                         ws.numel() * 4, s)
    return y.reshape(-1), dx.reshape(-1)


def _erf_form(x):
    cdf = 0.5 * (1 + torch.erf(x * 0.70710678118654752))
    return x * cdf, cdf + x * (0.39894228040143268 * torch.exp(-0.5 * x * x))


@pytest.mark.parametrize("band", [(-0.1, 0.1), (-1, 0), (0, 1), (-5, -1), (1, 5), (-14, 14), 0.1, 1, 3])
def test_gelu_precision(band):
    """No band is further from float64 than the erf form in fp32, on average (5% for the sample) or at
    most; the value relative to x."""
    g, n = torch.Generator(device=DEV).manual_seed(0), 1 << 20
    x = (torch.rand(n, generator=g, device=DEV) * (band[1] - band[0]) + band[0] if isinstance(band, tuple)
         else torch.randn(n, generator=g, device=DEV) * band)
    x64 = x.double()
    cdf = torch.special.ndtr(x64)
    ref = x64 * cdf, cdf + x64 * torch.exp(-0.5 * x64 * x64) / math.sqrt(2 * math.pi)
    scale = x64.abs().clamp_min(1e-30), torch.ones_like(x64)
    for got, erf, r, sc in zip(_run(x), _erf_form(x), ref, scale):
        e, f = ((v.double() - r) / sc for v in (got, erf))
        print(band, *(f"{v.abs().max().item():.2e} {v.pow(2).mean().sqrt().item():.2e}" for v in (e, f)))
        assert e.pow(2).mean().sqrt() <= 1.05 * f.pow(2).mean().sqrt()
        assert e.abs().max() <= 1.05 * f.abs().max()


def test_gelu_not_finite():
    inf, big = float("inf"), torch.finfo(torch.float32).max
    y, dx = _run(torch.tensor([inf, -inf, float("nan"), big, -big, 0.0], device=DEV))
    assert y[0] == inf and y[3] == big and y[4] == 0 and y[5] == 0
    assert y[1:3].isnan().all() and dx[:3].isnan().all()
    assert dx[3] == 1 and dx[4] == 0 and dx[5] == 0.5
