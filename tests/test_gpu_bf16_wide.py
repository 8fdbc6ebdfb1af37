"""bf16-operand forward and data gradient on 256x256 tiles: ragged rows, columns and reductions,
both storage types of X and Y, activations and residuals, against float64."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2104_00237_amd import _lib as L  # noqa: E402

DEV = "cuda:0"


def _gelu(z):
    return 0.5 * z * (1 + torch.erf(z / math.sqrt(2)))


def _dgelu(z):
    return 0.5 * (1 + torch.erf(z / math.sqrt(2))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)


def _ws(n):
    t = torch.empty((max(n, 16) + 15) // 16 * 4, device=DEV)
    return t, (t.data_ptr(), t.numel() * 4)


def _bound(a, b, r):
    """Products of bf16 values are exact; each fp32 addition rounds by at most 2^-24 of sum |ab|."""
    return (a.abs() @ b.abs()) * ((r / 8 + 8) * 2.0 ** -24) + 1e-6


# at least 160 tiles of 256 x 256; one chunk, a partial one, an odd and an even number of them; rows of
# whole 128-byte lines and others, where a short reduction with plain fp32 outputs takes the general kernel
@pytest.mark.parametrize("M,N,K", [(3600, 2600, 64), (3601, 2601, 72), (3841, 2820, 200), (2561, 4098, 256),
                                   (3601, 2592, 72), (2561, 4128, 200), (2561, 4098, 1032), (3841, 2820, 1024)])
@pytest.mark.parametrize("x16,y16,act,res", [(1, 1, "gelu", 0), (0, 0, "relu", 1), (1, 0, "none", 1)])
def test_forward(M, N, K, x16, y16, act, res):
    g = torch.Generator(device=DEV).manual_seed(M + K)
    x, w = torch.randn(M, K, generator=g, device=DEV), torch.randn(N, K, generator=g, device=DEV) * 0.1
    b, r = torch.randn(N, generator=g, device=DEV), torch.randn(M, N, generator=g, device=DEV)
    xb, wb = x.bfloat16(), w.bfloat16()
    y = torch.zeros(M, N, device=DEV, dtype=torch.bfloat16 if y16 else torch.float32)
    z = torch.zeros(M, N, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_BF16, L.ACTS[act], 1, (1 if x16 else 0) | (2 if y16 else 0))
    keep, ws = _ws(L.of_linear_workspace_size(d, 0))
    W = L.OfParam(w.data_ptr(), None, None, wb.data_ptr(), w.numel())
    xp = (xb if x16 else x).data_ptr()
    s = torch.cuda.current_stream().cuda_stream
    if res:
        L.of_linear_fwd_res(d, xp, W, b.data_ptr(), r.data_ptr(), z.data_ptr(), y.data_ptr(), None, *ws, s)
    else:
        L.of_linear_fwd(d, xp, W, b.data_ptr(), z.data_ptr(), y.data_ptr(), *ws, s)
    a64, w64 = xb.double(), wb.double().t()
    zr = a64 @ w64 + b.double()
    bound = _bound(a64, w64, K)
    assert (z.double() - zr).abs().le(bound).all()
    yr = _gelu(zr) if act == "gelu" else zr.clamp_min(0) if act == "relu" else zr
    yr = yr + r.double() if res else yr
    slack = yr.abs() * 2.0 ** -8 if y16 else 0.0   # Y rounded to bf16
    # |gelu'| < 1.13
    assert (y.double() - yr).abs().le(1.13 * bound + (zr.abs() + yr.abs()) * 2.0 ** -22 + slack).all()


@pytest.mark.parametrize("M,N,K", [(3600, 64, 2600), (3601, 76, 2608), (3841, 200, 2824), (2561, 256, 4104),
                                   (3601, 76, 2592), (2561, 200, 4128), (3601, 388, 2608)])
@pytest.mark.parametrize("act,res", [("none", 0), ("gelu", 0), ("relu", 1), ("none", 1), ("gelu", 1)])
def test_data_gradient(M, N, K, act, res):
    g = torch.Generator(device=DEV).manual_seed(N + K)
    dz, w = torch.randn(M, N, generator=g, device=DEV), torch.randn(N, K, generator=g, device=DEV) * 0.1
    prev, r = torch.randn(M, K, generator=g, device=DEV), torch.randn(M, K, generator=g, device=DEV)
    wb, dx = w.bfloat16(), torch.zeros(M, K, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_BF16, 0, 0, 0)
    keep, ws = _ws(L.of_linear_workspace_size(d, 1))
    W = L.OfParam(w.data_ptr(), None, None, wb.data_ptr(), w.numel())
    pp = prev.data_ptr() if act != "none" else None
    s = torch.cuda.current_stream().cuda_stream
    if res:
        L.of_linear_bwd_data_res(d, dz.data_ptr(), W, pp, L.ACTS[act], r.data_ptr(), dx.data_ptr(), *ws, s)
    else:
        L.of_linear_bwd_data(d, dz.data_ptr(), W, pp, L.ACTS[act], dx.data_ptr(), *ws, s)
    a64, w64, p = dz.bfloat16().double(), wb.double(), prev.double()
    f = _dgelu(p) if act == "gelu" else (p > 0).double() if act == "relu" else torch.ones_like(p)
    c = a64 @ w64
    ref = c * f + (r.double() if res else 0.0)
    bound = 1.13 * _bound(a64, w64, N) + c.abs() * 2.0 ** -21 + ref.abs() * 2.0 ** -23
    assert (dx.double() - ref).abs().le(bound).all()


def test_gelu_tails():
    """GELU and its derivative over the whole range, through the fp32 path's epilogues."""
    n = 4096
    x = torch.linspace(-14, 14, n, device=DEV).reshape(n, 1).contiguous()
    x[0], x[1], x[2] = -200.0, 200.0, 0.0
    w, y, z, dx = torch.ones(1, 1, device=DEV), *(torch.empty(n, 1, device=DEV) for _ in range(3))
    d = L.OfLinearDesc(n, 1, 1, 0, 0, L.OF_F32, L.OF_ACT_GELU, 0, 0)
    keep, ws = _ws(max(L.of_linear_workspace_size(d, o) for o in (0, 1)))
    W = L.OfParam(w.data_ptr(), None, None, None, 1)
    s = torch.cuda.current_stream().cuda_stream
    L.of_linear_fwd(d, x.data_ptr(), W, None, z.data_ptr(), y.data_ptr(), *ws, s)
    one = torch.ones(n, 1, device=DEV)
    L.of_linear_bwd_data(d, one.data_ptr(), W, x.data_ptr(), L.OF_ACT_GELU, dx.data_ptr(), *ws, s)
    x64 = x.double()
    assert (y.double() - x64 * torch.special.ndtr(x64)).abs().le(x64.abs() * 1.2e-7).all()
    assert (dx.double() - _dgelu(x64)).abs().le(3e-7).all()


# 192 tiles of 128 x 128 and more; the last four on the kernel with direct loads: one row and one column
# past whole chunks and tiles, an odd number of chunks, the fewest rows
@pytest.mark.parametrize("M,N,K", [(64, 1540, 2056), (333, 3076, 1032), (200, 1800, 1800), (129, 2048, 1536),
                                   (1025, 2980, 2016), (1091, 4100, 1312), (1999, 2048, 2048), (1024, 3000, 1760)])
@pytest.mark.parametrize("opt,early", [("adamw", 0), ("sgd", 1), ("adagrad", 0)])
def test_weight_gradient(M, N, K, opt, early):
    """dW, db against float64, accumulation, and the fused update bit
    for bit against the eager gradient and optimizer step (with an earlier use's gradient too)."""
    g = torch.Generator(device=DEV).manual_seed(M + N)
    dz, x = torch.randn(M, N, generator=g, device=DEV), torch.randn(M, K, generator=g, device=DEV)
    xb, s = x.bfloat16(), torch.cuda.current_stream().cuda_stream
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_BF16, 0, 1, L.OF_IO_X_BF16)
    keep, ws = _ws(L.of_linear_workspace_size(d, 2))
    dw, db = torch.empty(N, K, device=DEV), torch.empty(N, device=DEV)
    L.of_linear_bwd_weight(d, dz.data_ptr(), xb.data_ptr(), dw.data_ptr(), db.data_ptr(), 0, *ws, s)
    a64, x64 = dz.bfloat16().double().t(), xb.double()
    assert (dw.double() - a64 @ x64).abs().le(_bound(a64, x64, M)).all()
    assert (db.double() - dz.double().sum(0)).abs().le(dz.double().abs().sum(0) * M * 2.0 ** -24).all()
    gw, gb = torch.randn(N, K, generator=g, device=DEV), torch.randn(N, generator=g, device=DEV)
    if early:
        dw2, db2 = gw.clone(), gb.clone()
        L.of_linear_bwd_weight(d, dz.data_ptr(), xb.data_ptr(), dw2.data_ptr(), db2.data_ptr(), 1, *ws, s)
        assert torch.equal(dw2, gw + dw) and torch.equal(db2, gb + db)
        dw, db = dw2, db2
    hyper = dict(kind=opt, lr=1e-2, momentum=0.9, beta1=0.9, beta2=0.99, eps=1e-8, weight_decay=1e-2)
    sets = []
    for _ in range(2):
        t = [torch.randn(N, K, generator=torch.Generator(device=DEV).manual_seed(5 + i), device=DEV).abs()
             for i in range(3)] + [torch.zeros(N, K, device=DEV, dtype=torch.bfloat16)]
        u = [torch.ones(N, device=DEV) * (i + 1) for i in range(3)]
        W, b = L.param_of(t[0], t[1], t[2], t[3]), L.param_of(*u)
        if opt == "adagrad":
            W.m = b.m = None
        sets.append((t, u, W, b))
    o = L.make_opt(hyper, 3)
    t, u, W, b = sets[0]
    L.of_optimizer_step(2, (L.OfParam * 2)(W, b), (L.c_void_p * 2)(dw.data_ptr(), db.data_ptr()), o, s)
    t2, u2, W2, b2 = sets[1]
    L.of_linear_bwd_fused(d, dz.data_ptr(), xb.data_ptr(), W2, b2, gw.data_ptr() if early else None,
                          gb.data_ptr() if early else None, o, None, 0, None, None, 0, *ws, s, None)
    for p, q in zip(t + u, t2 + u2):
        assert torch.equal(p, q)
