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
    """out = a @ b with r reduction elements, element by element.  The one dropped partial product is
    below 2^-29 |ab|; the fp32 additions (at most two per 16 elements for the leading products, then
    splits, waves and the final sum; the corrections' are 2^-6 of these) each round by at most 2^-24 of
    sum |ab|.  Such a bound grows with r past what the low planes contribute: test_one_product pins them."""
    ref = a @ b
    bound = (a.abs() @ b.abs()) * ((r / 8 + 24) * 2.0 ** -24 + 2.0 ** -29)
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


# outputs of one product each, on every tile and kind: 64x128 (forward and data gradient), 128x128 with
# and without splits, 64x64, each with whole float4s and with single loads; the fused forward's tiles
ONE = [(64, 4096, 4096), (300, 1500, 3000), (1024, 1024, 1024), (2048, 2048, 1024), (4096, 1000, 1000),
       (63, 4099, 4098), (301, 1501, 3003), (1001, 1023, 1021), (2047, 2049, 1023)]


def _random24(g, *shape):
    """24 random significant bits, exponents -4 to 4, both signs."""
    m = torch.randint(2 ** 23, 2 ** 24, shape, generator=g, device=DEV).double()
    e = torch.randint(-27, -18, shape, generator=g, device=DEV).double()
    s = torch.randint(0, 2, shape, generator=g, device=DEV).double() * 2 - 1
    return (s * m * 2.0 ** e).float()


def _one_hot(g, rows, cols):
    """One element per row, in a random column."""
    t = torch.zeros(rows, cols, device=DEV)
    c = torch.randint(0, cols, (rows,), generator=g, device=DEV)
    t[torch.arange(rows, device=DEV), c] = _random24(g, rows)
    return t


def _check_one(out, ref):
    """ref is one product of 24-bit operands: the leading partial product is exact, the corrections
    (below 2^-6 of it) round at most 7 times, then one rounding of their sum."""
    bound = ref.abs() * 2.0 ** -24 * (1 + 7 * 2.0 ** -6)
    assert (out.double() - ref).abs().le(bound).all(), \
        ((out.double() - ref).abs() / ref.abs().clamp_min(1e-300)).max().item() * 2.0 ** 24


@pytest.mark.parametrize("M,N,K", ONE)
def test_one_product(M, N, K):
    """Sparse operands: every product keeps the precision of an fp32 one."""
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    x, w, dzr = _one_hot(g, M, K), _random24(g, N, K), _one_hot(g, M, N)
    dzc, xd = _one_hot(g, N, M).t().contiguous(), _random24(g, M, K)
    y, yf, dx, dw = (torch.empty(*s, device=DEV) for s in ((M, N), (M, N), (M, K), (N, K)))
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, L.OF_ACT_NONE, 0, 0)
    keep, ws = _ws(max(L.of_linear_workspace_size(d, o) for o in (0, 1, 2)))
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_linear_fwd(d, x.data_ptr(), W, None, None, y.data_ptr(), *ws, _stream())
    L.of_linear_bwd_data(d, dzr.data_ptr(), W, None, 0, dx.data_ptr(), *ws, _stream())
    L.of_linear_bwd_weight(d, dzc.data_ptr(), xd.data_ptr(), dw.data_ptr(), None, 0, *ws, _stream())
    _check_one(y, x.double() @ w.double().t())
    _check_one(dx, dzr.double() @ w.double())
    _check_one(dw, dzc.double().t() @ xd.double())
    # the fused forward whose update leaves W as it is (no rate, no decay): the same bits
    t = [torch.zeros(N, K, device=DEV) for _ in range(3)]
    out = L.param_of(torch.empty_like(w), t[1]) if M > 64 else None
    o = L.make_opt(dict(kind="sgd", lr=0.0, momentum=0.0, weight_decay=0.0), 1)
    Wm = L.OfParam(w.data_ptr(), t[0].data_ptr(), None, None, w.numel())
    L.of_linear_fwd_fused(d, x.data_ptr(), Wm, out, t[2].data_ptr(), None, None, None, o, None, yf.data_ptr(),
                          *ws, _stream())
    assert torch.equal(y, yf)


@pytest.mark.parametrize("N,H,Wd,C,Co", [(64, 9, 12, 96, 160), (16, 15, 15, 256, 256), (64, 9, 12, 99, 100),
                                         (9, 15, 15, 254, 256), (64, 9, 12, 100, 99),
                                         (12, 15, 15, 254, 256), (64, 9, 12, 150, 150)])
def test_one_product_conv(N, H, Wd, C, Co):
    g = torch.Generator(device=DEV).manual_seed(C + Co)
    M = N * H * Wd

    def spread(ch):   # one channel of every third pixel each way: a window holds at most one
        t = _one_hot(g, M, ch).reshape(N, H, Wd, ch)
        keep = torch.zeros(H, Wd, device=DEV)
        keep[1::3, 1::3] = 1
        return t * keep[None, :, :, None]
    xs, dys, w = spread(C), spread(Co), _random24(g, Co, 3, 3, C)
    dyc, xd = _one_hot(g, Co, M).t().reshape(N, H, Wd, Co).contiguous(), _random24(g, N, H, Wd, C)
    y, dx, dw = torch.empty(M, Co, device=DEV), torch.empty(M, C, device=DEV), torch.empty(Co, 9 * C, device=DEV)
    d = L.OfConvDesc(N, H, Wd, C, Co, L.OF_ACT_NONE, 0, 1)
    keep, ws = _ws(max(L.of_conv_workspace_size(d, o) for o in (0, 1, 2)))
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_conv_fwd(d, xs.data_ptr(), W, None, y.data_ptr(), *ws, _stream())
    L.of_conv_bwd_data(d, dys.data_ptr(), W, None, 0, dx.data_ptr(), *ws, _stream())
    L.of_conv_bwd_weight(d, dyc.data_ptr(), xd.data_ptr(), dw.data_ptr(), None, 0, *ws, _stream())

    def cols(t):
        p = torch.nn.functional.pad(t.double(), (0, 0, 1, 1, 1, 1))
        return torch.cat([p[:, i:i + H, j:j + Wd, :] for i in range(3) for j in range(3)], 3).reshape(M, -1)
    flip = w.double().flip(1, 2).permute(1, 2, 0, 3).reshape(9 * Co, C)
    _check_one(y, cols(xs) @ w.double().reshape(Co, -1).t())
    _check_one(dx, cols(dys) @ flip)
    _check_one(dw, dyc.double().reshape(M, Co).t() @ cols(xd))


def test_same_sign():
    """Equal operands whose dropped product would add up: 1 + 2^-7 - 2^-23 everywhere."""
    M, N, K = 2048, 4096, 128
    v = 1 + 2.0 ** -7 - 2.0 ** -23
    x, w, y = torch.full((M, K), v, device=DEV), torch.full((N, K), v, device=DEV), torch.empty(M, N, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, L.OF_ACT_NONE, 0, 0)
    keep, ws = _ws(L.of_linear_workspace_size(d, 0))
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_linear_fwd(d, x.data_ptr(), W, None, None, y.data_ptr(), *ws, _stream())
    # the leading sums are whole numbers; the corrections (2^-6 of them) round at most 7 K / 16 times
    bound = 2.0 ** -24 * (2 + 7 * K / 16 * 2.0 ** -6)
    assert ((y.double() / (K * v * v)) - 1).abs().max().item() <= bound


@pytest.mark.parametrize("e", [-100, -110, -118, -126, -134, -142])
def test_tiny_operands(e):
    """Operands of 2^-110 and more keep all their bits; below, what lies under the smallest bf16
    (2^-133) is dropped, an absolute error of less than 2^-133 per operand."""
    M, N, K = 640, 1024, 1024
    g = torch.Generator(device=DEV).manual_seed(-e)
    x, w = _one_hot(g, M, K), _random24(g, N, K) * 2.0 ** 40
    x = (torch.frexp(x.double())[0] * 2.0 ** (e + 1)).float()    # exponent e (rounded when subnormal)
    y = torch.empty(M, N, device=DEV)
    d = L.OfLinearDesc(M, N, K, 0, 0, L.OF_F32, L.OF_ACT_NONE, 0, 0)
    keep, ws = _ws(L.of_linear_workspace_size(d, 0))
    W = L.OfParam(w.data_ptr(), None, None, None, w.numel())
    L.of_linear_fwd(d, x.data_ptr(), W, None, None, y.data_ptr(), *ws, _stream())
    ref = x.double() @ w.double().t()
    lost = (x != 0).double() @ w.double().abs().t() * 2.0 ** -133 if e < -110 else 0.0
    assert (y.double() - ref).abs().le(ref.abs() * 2.0 ** -24 * (1 + 7 * 2.0 ** -6) + lost).all()


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
