"""fp32 contractions on the bf16 matrix cores (exact three-way operand splits): tile edges and
remainders against float64, and operands that are not finite or at the end of the range."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2104_00237_amd import _lib as L  # noqa: E402

DEV = "cuda:0"


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _ws(n):
    t = torch.empty((max(n, 16) + 15) // 16 * 4, device=DEV)
    return t, (t.data_ptr(), t.numel() * 4)


def _check(out, a, b, r):
    """out = a @ b with r reduction elements, element by element.  Products are exact; the three
    dropped partial products are below 2^-23 |ab| together, and the fp32 additions (one per 16
    elements, three times for the corrections, then splits, waves and the final sum) each round
    by at most 2^-24 of sum |ab|."""
    ref = a @ b
    bound = (a.abs() @ b.abs()) * ((r / 8 + 24) * 2.0 ** -24 + 2.0 ** -23)
    assert (out.double() - ref).abs().le(bound + 1e-30).all(), \
        ((out.double() - ref).abs() / (bound + 1e-30)).max().item()


# ragged in every dimension, scalar and vector loads, one and several splits, every tile
SHAPES = [(577, 1033, 1031), (640, 1000, 1004), (1300, 132, 4100), (129, 4100, 1300), (48, 4100, 4130),
          (2049, 520, 640), (160, 2052, 1300)]


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_linear(M, N, K):
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    x, w = torch.randn(M, K, generator=g, device=DEV), torch.randn(N, K, generator=g, device=DEV)
    dz = torch.randn(M, N, generator=g, device=DEV)
    y, dx, dw, db = (torch.empty(*s, device=DEV) for s in ((M, N), (M, K), (N, K), (N,)))
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, L.OF_ACT_NONE, 0, 0)
    keep, ws = _ws(max(L.of_linear_workspace_size(d, o) for o in (0, 1, 2)))
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_linear_fwd(d, x.data_ptr(), W, None, None, y.data_ptr(), *ws, _stream())
    L.of_linear_bwd_data(d, dz.data_ptr(), W, None, 0, dx.data_ptr(), *ws, _stream())
    L.of_linear_bwd_weight(d, dz.data_ptr(), x.data_ptr(), dw.data_ptr(), db.data_ptr(), 0, *ws, _stream())
    x64, w64, dz64 = x.double(), w.double(), dz.double()
    _check(y, x64, w64.t(), K)
    _check(dx, dz64, w64, N)
    _check(dw, dz64.t(), x64, M)
    _check(db.reshape(1, N), torch.ones(1, M, dtype=torch.float64, device=DEV), dz64, 8 * M)


@pytest.mark.parametrize("N,H,Wd,C,Co", [(9, 13, 11, 100, 217), (9, 13, 11, 101, 220), (70, 7, 5, 96, 130)])
def test_conv(N, H, Wd, C, Co):
    g = torch.Generator(device=DEV).manual_seed(C + Co)
    x, w = torch.randn(N, H, Wd, C, generator=g, device=DEV), torch.randn(Co, 3, 3, C, generator=g, device=DEV)
    dy = torch.randn(N, H, Wd, Co, generator=g, device=DEV)
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    d = L.OfConvDesc(N, H, Wd, C, Co, L.OF_ACT_NONE, 0, 1)
    keep, ws = _ws(max(L.of_conv_workspace_size(d, o) for o in (0, 1, 2)))
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_conv_fwd(d, x.data_ptr(), W, None, y.data_ptr(), *ws, _stream())
    L.of_conv_bwd_data(d, dy.data_ptr(), W, None, 0, dx.data_ptr(), *ws, _stream())
    L.of_conv_bwd_weight(d, dy.data_ptr(), x.data_ptr(), dw.data_ptr(), None, 0, *ws, _stream())

    def cols(t):   # [pixels, 9 * channels]: the 3x3 neighbourhood of every pixel
        p = torch.nn.functional.pad(t.double(), (0, 0, 1, 1, 1, 1))
        return torch.cat([p[:, i:i + H, j:j + Wd, :] for i in range(3) for j in range(3)], 3).reshape(
            N * H * Wd, -1)
    wk = w.double().reshape(Co, 9 * C)
    flip = w.double().flip(1, 2).permute(1, 2, 0, 3).reshape(9 * Co, C)
    _check(y.reshape(-1, Co), cols(x), wk.t(), 9 * C)
    _check(dx.reshape(-1, C), cols(dy), flip, 9 * Co)
    _check(dw.reshape(Co, -1), dy.double().reshape(-1, Co).t(), cols(x), N * H * Wd)


def test_not_finite():
    """An infinite, NaN or largest finite operand gives what an fp32 product sum gives."""
    M, N, K = 640, 1024, 1024
    g = torch.Generator(device=DEV).manual_seed(1)
    x, w = torch.randn(M, K, generator=g, device=DEV), torch.ones(N, K, device=DEV)
    w[::2] = -0.5
    inf, big = float("inf"), torch.finfo(torch.float32).max
    x[3, 5], x[70, 1000], x[130, 7], x[200, 0], x[333, 9] = inf, -inf, float("nan"), inf, inf
    x[200, 1] = -inf                 # inf - inf
    w[8, 9] = 0.0                    # inf * 0
    x[400], x[500] = 0.0, 0.0
    x[400, 17], x[500, 900] = big, -big
    y = torch.empty(M, N, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, L.OF_ACT_NONE, 0, 0)
    keep, ws = _ws(L.of_linear_workspace_size(d, 0))
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_linear_fwd(d, x.data_ptr(), W, None, None, y.data_ptr(), *ws, _stream())
    ref = x.cpu().double() @ w.cpu().double().t()
    y = y.cpu().double()
    assert torch.equal(torch.isnan(y), torch.isnan(ref))
    assert torch.equal(y[torch.isinf(ref)], ref[torch.isinf(ref)])
    ok = torch.isfinite(ref)
    assert (y[ok] - ref[ok]).abs().le(1e-4 + 1e-6 * ref[ok].abs()).all()
    assert torch.equal(y[400], ref[400]) and torch.equal(y[500], ref[500])
