"""Which tiles a contraction takes: sizes at the edges of the rules, against float64 and between the
eager and the fused update; where a rule is about time, the time against plain stores of the output."""
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


def _us(f, n=20):
    """The best of five means over n passes."""
    f()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / n * 1e3)
    return best


@pytest.mark.parametrize("M,N,K", [(1, 4096, 4096), (37, 4101, 4099), (63, 4100, 4104), (63, 8192, 2048)])
def test_short_weight_gradient(M, N, K):
    """Fewer than 64 rows onto 1024 tiles of 128x128: the fused update bit for bit against the eager
    gradient and step, the gradient against float64 (at most M roundings of sum |ab|)."""
    g = torch.Generator(device=DEV).manual_seed(M)
    dz, x = torch.randn(M, N, generator=g, device=DEV), torch.randn(M, K, generator=g, device=DEV)
    dw, db = torch.empty(N, K, device=DEV), torch.empty(N, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, 0, 1, 0)
    keep, ws = _ws(L.of_linear_workspace_size(d, 2))
    s = _stream()
    L.of_linear_bwd_weight(d, dz.data_ptr(), x.data_ptr(), dw.data_ptr(), db.data_ptr(), 0, *ws, s)
    ref, mag = dz.double().t() @ x.double(), dz.double().abs().t() @ x.double().abs()
    assert (dw.double() - ref).abs().le(mag * M * 2.0 ** -24 + 1e-30).all()
    o = L.make_opt(dict(kind="adamw", lr=1e-2, beta1=0.9, beta2=0.99, eps=1e-8, weight_decay=1e-2), 3)
    sets = []
    for _ in range(2):
        h = torch.Generator(device=DEV).manual_seed(7)
        sets.append([torch.rand(n, generator=h, device=DEV) for n in (N * K, N * K, N * K, N, N, N)])
    W, b = L.param_of(*sets[0][:3]), L.param_of(*sets[0][3:])
    L.of_optimizer_step(2, (L.OfParam * 2)(W, b), (L.c_void_p * 2)(dw.data_ptr(), db.data_ptr()), o, s)
    W, b = L.param_of(*sets[1][:3]), L.param_of(*sets[1][3:])
    L.of_linear_bwd_fused(d, dz.data_ptr(), x.data_ptr(), W, b, None, None, o, None, 0, None, None, 0,
                          *ws, s, None)
    for p, q in zip(*sets):
        assert torch.equal(p, q)


@pytest.mark.parametrize("M,N,K", [(16, 8192, 8192), (16, 4096, 4096)])
def test_short_weight_gradient_time(M, N, K):
    """Storing dW is most of such a gradient: no slower than copying dW, which also reads as much
    (measured 0.9 of it; 1.5 to 2 on tiles that read each operand twice as often)."""
    dz, x, dw = (torch.randn(*s, device=DEV) for s in ((M, N), (M, K), (N, K)))
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, 0, 0, 0)
    keep, ws = _ws(L.of_linear_workspace_size(d, 2))
    s, src = _stream(), torch.randn(N, K, device=DEV)
    t = _us(lambda: L.of_linear_bwd_weight(d, dz.data_ptr(), x.data_ptr(), dw.data_ptr(), None, 0, *ws, s))
    copy = _us(lambda: dw.copy_(src))
    print(f"{M} x {N} x {K}: {t:.1f} us, copy {copy:.1f} us")
    assert t < 1.3 * copy



@pytest.mark.parametrize("N,K", [(3072, 1024), (3000, 1000), (2048, 1536)])
def test_bf16_weight_gradient_splits(N, K):
    """192 to 255 tiles of 128x128 over a long reduction: split in two (the fused update, plain and fused
    of X stored as fp32 gain 10 to 20%), whichever way X is stored."""
    for io in (0, L.OF_IO_X_BF16):
        d = L.OfLinearDesc(4096, N, K, 0, 0, L.OF_BF16, 0, 1, io)
        assert L.of_linear_workspace_size(d, 2) >= 2 * 4 * N * K


@pytest.mark.parametrize("M,N,K", [(1023, 2048, 2048), (1024, 2048, 2048), (1024, 2052, 2056), (1024, 3072, 1024),
                                   (1100, 4096, 1024)])
def test_bf16_weight_gradient_kernels(M, N, K):
    """Both sides of the rule for the kernel with direct loads: the bits of the general one, which takes a
    gradient whose dZ is not 16-byte aligned."""
    g, s = torch.Generator(device=DEV).manual_seed(M + N), _stream()
    dz, x = torch.randn(M, N, generator=g, device=DEV), torch.randn(M, K, generator=g, device=DEV).bfloat16()
    off = torch.empty(M * N + 4, device=DEV)[1:M * N + 1]
    off.copy_(dz.reshape(-1))
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_BF16, 0, 1, L.OF_IO_X_BF16)
    keep, ws = _ws(L.of_linear_workspace_size(d, 2))
    outs = []
    for p in (dz, off):
        dw, db = torch.empty(N, K, device=DEV), torch.empty(N, device=DEV)
        L.of_linear_bwd_weight(d, p.data_ptr(), x.data_ptr(), dw.data_ptr(), db.data_ptr(), 0, *ws, s)
        outs.append((dw, db))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])



# at least 160 tiles of 256x256 and more than 2048 reduction elements
@pytest.mark.parametrize("M,N,K", [(2561, 4098, 4104), (3600, 2600, 8200), (3601, 2601, 2056)])
@pytest.mark.parametrize("x16,y16,act,res", [(1, 0, "none", 0), (0, 0, "relu", 1), (1, 1, "gelu", 0)])
def test_bf16_long_forward(M, N, K, x16, y16, act, res):
    """No sum runs over more than 2048 products: the error against float64 stays that of such sums
    (measured 1.9e-7 to 2.8e-7; 4.0e-7 over 4100, 5.7e-7 over 8200), and the kernel with direct loads gives
    the bits of the general one, which takes the call when X is not 16-byte aligned."""
    g = torch.Generator(device=DEV).manual_seed(M + K)
    w = torch.randn(N, K, generator=g, device=DEV) * 0.1
    x, r = torch.randn(M, K, generator=g, device=DEV), torch.randn(M, N, generator=g, device=DEV)
    x = x.bfloat16() if x16 else x
    off = torch.empty(x.numel() + 4, device=DEV, dtype=x.dtype)[2 if x16 else 1:][:x.numel()]
    off.copy_(x.reshape(-1))
    wb, b, s = w.bfloat16(), torch.randn(N, generator=g, device=DEV), _stream()
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_BF16, L.ACTS[act], 1, (1 if x16 else 0) | (2 if y16 else 0))
    keep, ws = _ws(L.of_linear_workspace_size(d, 0))
    W, outs = L.OfParam(w.data_ptr(), None, None, wb.data_ptr(), w.numel()), []
    for xp in (x.data_ptr(), off.data_ptr()):
        y = torch.zeros(M, N, device=DEV, dtype=torch.bfloat16 if y16 else torch.float32)
        z = torch.zeros(M, N, device=DEV)
        if res:
            L.of_linear_fwd_res(d, xp, W, b.data_ptr(), r.data_ptr(), z.data_ptr(), y.data_ptr(), None, *ws, s)
        else:
            L.of_linear_fwd(d, xp, W, b.data_ptr(), z.data_ptr(), y.data_ptr(), *ws, s)
        outs.append((y, z))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    n = 512   # rows
    ref = x[:n].bfloat16().double() @ wb.double().t() + b.double()
    err = ((outs[0][1][:n].double() - ref).norm() / ref.norm()).item()
    assert err <= 3.2e-7, err


# sizes on the fp32 tiles again, beside ones like them on the bf16 matrix cores: a short weight gradient on
# few workgroups, split, just past one round of 256, past it in two splits, with single loads over few rows;
# a data gradient with single loads of W alone; a forward split in two
@pytest.mark.parametrize("M,N,K", [(993, 1424, 528), (1001, 1424, 528), (976, 440, 1000), (945, 504, 2108),
                                   (945, 504, 2560), (5439, 672, 912), (3390, 672, 912), (64, 4089, 4160),
                                   (375, 5304, 1302), (375, 5303, 1302), (512, 1277, 2000), (512, 1277, 2100)])
def test_fp32_rules(M, N, K):
    """Forward and gradients against float64 (at most r roundings of sum |ab|; the fp32 tiles' chains hold r / 2
    products), and the fused update bit for bit against the eager gradient and step."""
    g, s = torch.Generator(device=DEV).manual_seed(M + N + K), _stream()
    x, w, dz = (torch.randn(*n, generator=g, device=DEV) for n in ((M, K), (N, K), (M, N)))
    y, dx, dw = torch.empty(M, N, device=DEV), torch.empty(M, K, device=DEV), torch.empty(N, K, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, L.OF_ACT_NONE, 0, 0)
    keep, ws = _ws(max(L.of_linear_workspace_size(d, o) for o in (0, 1, 2)))
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_linear_fwd(d, x.data_ptr(), W, None, None, y.data_ptr(), *ws, s)
    L.of_linear_bwd_data(d, dz.data_ptr(), W, None, 0, dx.data_ptr(), *ws, s)
    L.of_linear_bwd_weight(d, dz.data_ptr(), x.data_ptr(), dw.data_ptr(), None, 0, *ws, s)
    x64, w64, z64 = x.double(), w.double(), dz.double()
    for out, a, b, r in ((y, x64, w64.t(), K), (dx, z64, w64, N), (dw, z64.t(), x64, M)):
        bound = (a.abs() @ b.abs()) * (r * 2.0 ** -24)
        assert (out.double() - a @ b).abs().le(bound).all()
    o = L.make_opt(dict(kind="adam", lr=1e-2, beta1=0.9, beta2=0.99, eps=1e-8, weight_decay=0.0), 2)
    sets = []
    for _ in range(2):
        h = torch.Generator(device=DEV).manual_seed(3)
        sets.append([torch.rand(N * K, generator=h, device=DEV) for _ in range(3)])
    P = L.param_of(*sets[0])
    L.of_optimizer_step(1, (L.OfParam * 1)(P), (L.c_void_p * 1)(dw.data_ptr()), o, s)
    L.of_linear_bwd_fused(d, dz.data_ptr(), x.data_ptr(), L.param_of(*sets[1]), None, None, None, o, None, 0, None,
                          None, 0, *ws, s, None)
    for p, q in zip(*sets):
        assert torch.equal(p, q)
