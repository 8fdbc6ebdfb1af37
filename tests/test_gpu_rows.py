"""The row-panel forward of tall fp32 products with a short reduction and a large output: every number of MFMA steps, ragged
rows, columns and reductions, Z, activations and residuals against float64, and bit for bit against the
tiled kernel that a fused forward of the same layer takes."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2104_00237_amd import _lib as L  # noqa: E402

DEV = "cuda:0"

# at least 2^25 outputs; 8, 12, 16 and 32 steps, each with a reduction that fills them and one that does
# not; the fewest columns and the most of each; a last panel of one row and of 31
CASES = [(1016801, 33, 7), (231425, 145, 16), (131073, 256, 17), (335583, 100, 24), (134239, 250, 31),
         (559241, 60, 32), (223711, 150, 33), (209729, 160, 64), (349537, 96, 16)]


def _bufs(M, N, K, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    t = [torch.randn(*s, generator=g, device=DEV) for s in ((M, K), (N, K), (N,), (M, N))]
    ws = torch.empty(1 << 22, device=DEV)
    return *t, ws, (ws.data_ptr(), ws.numel() * 4), torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("M,N,K", CASES)
@pytest.mark.parametrize("act,res", [("gelu", 1), ("relu", 0), ("none", 1)])
def test_forward(M, N, K, act, res):
    x, w, b, r, keep, ws, s = _bufs(M, N, K, M + N + K)
    y, z = torch.full((M, N), math.nan, device=DEV), torch.full((M, N), math.nan, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, L.ACTS[act], 1, 0)
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    if res:
        L.of_linear_fwd_res(d, x.data_ptr(), W, b.data_ptr(), r.data_ptr(), z.data_ptr(), y.data_ptr(), None, *ws, s)
    else:
        L.of_linear_fwd(d, x.data_ptr(), W, b.data_ptr(), z.data_ptr(), y.data_ptr(), *ws, s)
    x64, w64 = x.double(), w.double().t()
    zr = x64 @ w64 + b.double()
    bound = (x64.abs() @ w64.abs() + b.double().abs()) * ((K + 2) * 2.0 ** -24)
    assert (z.double() - zr).abs().le(bound).all()
    yr = zr * torch.special.ndtr(zr) if act == "gelu" else zr.clamp_min(0) if act == "relu" else zr
    yr = yr + r.double() if res else yr
    # |gelu'| < 1.13
    assert (y.double() - yr).abs().le(1.13 * bound + (zr.abs() + yr.abs()) * 2.0 ** -22).all()


@pytest.mark.parametrize("M,N,K", CASES)
def test_fused_forward_bits(M, N, K):
    """The fused forward whose update leaves W as it is (no rate, no decay)."""
    x, w, b, r, keep, ws, s = _bufs(M, N, K, K)
    y, yf = torch.empty(M, N, device=DEV), torch.empty(M, N, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, L.OF_ACT_RELU, 0, 0)
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_linear_fwd(d, x.data_ptr(), W, None, None, y.data_ptr(), *ws, s)
    m, m2, g = (torch.zeros(N, K, device=DEV) for _ in range(3))
    o = L.make_opt(dict(kind="sgd", lr=0.0, momentum=0.0, weight_decay=0.0), 1)
    L.of_linear_fwd_fused(d, x.data_ptr(), L.OfParam(w.data_ptr(), m.data_ptr(), None, None, w.numel()),
                          L.param_of(torch.empty_like(w), m2), g.data_ptr(), None, None, None, o, None,
                          yf.data_ptr(), *ws, s)
    assert torch.equal(y, yf)
