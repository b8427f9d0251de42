"""Products of the library called by themselves, through the launchers that a forward uses: their epilogues, element by element."""
import ctypes as C
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F32, BF16 = 0, 1                                             # dtype argument of the launchers
EPI_GELU, EPI_SWIGLU, EPI_PART = 2, 3, 4


def _lib():
    from paper_2502_04557_amd import binding
    return binding.load_library()


def _tile(epi, rows, N, K, max_shares):
    """(tile, K shares) of the launcher; tile 0: 256 x 256."""
    return divmod(_lib()["_ZN8sprinter16gemm_tile_choiceEiiiii"](epi, rows, N, K, max_shares), 16)


def _operand(x):
    """[rows, K] -> float16 operand tiles of 16 rows x 32 k, zero padded."""
    import torch
    m, k = x.shape
    p = torch.zeros(-(-m // 16) * 16, -(-k // 32) * 32, dtype=torch.float16, device="cuda")
    p[:m, :k] = x
    return p.view(p.shape[0] // 16, 16, p.shape[1] // 32, 4, 8).permute(0, 2, 3, 1, 4).contiguous()


def _rows(act, rows, N):
    """The first rows and columns of an activation in operand tiles."""
    return act.permute(0, 3, 1, 2, 4).reshape(act.shape[0] * 16, -1)[:rows, :N]


def _ptr(t):
    return C.c_void_p(None if t is None else t.data_ptr())


def _activation(dtype, epi, x, W, W2, bias, N, K):
    """epilogue(x W^T) as the library stores it, [rows, N]."""
    import torch
    rows = x.shape[0]
    X, Wd, W2d = (t if t is None or dtype == F32 else _operand(t) for t in (x, W, W2))
    out = torch.zeros(rows, N, device="cuda") if dtype == F32 else _operand(torch.zeros(rows, N, device="cuda"))
    n = torch.tensor([rows], dtype=torch.int32, device="cuda")
    _lib()["_ZN8sprinter11launch_gemmEiiPKvS1_S1_mPKiiiPKfPfiPviiP12ihipStream_t"](
        dtype, epi, _ptr(Wd), _ptr(W2d), _ptr(X), C.c_size_t(X.numel()), _ptr(n), N, K, _ptr(bias), _ptr(None), N, _ptr(out), N, rows,
        C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return (out if dtype == F32 else _rows(out, rows, N)).cpu().numpy()


def _pairs(v, N, one):
    """Rows whose product with [I | I] (K = 2 N and a column for `one`) is v: two float16 parts of each value, summed exactly in float32."""
    import torch
    v = v.view(-1, N)
    hi = v.half().float()
    lo = (v - hi).half().float()
    tail = torch.zeros(v.shape[0], 32, device="cuda")
    tail[:, 0] = one
    eye = torch.eye(N, device="cuda")
    W = torch.cat([eye, eye, torch.zeros(N, 32, device="cuda")], 1)
    W2 = torch.zeros_like(W)
    W2[:, 2 * N] = 1.0
    return torch.cat([hi, lo, tail], 1), W, W2, (hi.double() + lo.double()).cpu().numpy()


def _silu(x):
    with np.errstate(over="ignore", invalid="ignore"):
        return x / (1.0 + np.exp(-x))


def _gelu(x):
    """0.5 x (1 + tanh u) = x / (1 + exp(-2 u)), which does not cancel: 1 + tanh in 64 bits has no digit left from x = -6 on."""
    with np.errstate(over="ignore", invalid="ignore"):
        return x / (1.0 + np.exp(-2 * 0.7978845608028654 * (x + 0.044715 * x ** 3)))


def _gelu_bound(s):
    """Float32 error of x - x q (x > 0) or x q, q = e / (1 + e), e = exp(-|2 u|), 2 u = c (x + 0.044715 x^3).  Units of 2^-24: five roundings of 2 u are |2 u| times as much of
    e, whose own end is within 2; the sum, quotient and product one each, so 5 |2 u| + 5 of x q, and one of the result.  Below 2^-126 e may be zero."""
    with np.errstate(over="ignore", invalid="ignore"):
        t = np.abs(1.5957691216057308 * (s + 0.044715 * s ** 3))
        q = np.exp(-t) / (1 + np.exp(-t))
        return 2.0 ** -24 * (np.abs(s) * q * (5 * np.minimum(t, 200.0) + 5) + np.abs(_gelu(s))) + np.abs(s) * 2.0 ** -126


@pytest.mark.parametrize("rows, N, tile", [(4080, 2048, 0), (2032, 512, 2), (16, 512, None)])
@pytest.mark.parametrize("lo, hi", [(-3, 3), (-6, -3), (-12, -6), (-60, 60)])
def test_silu_is_rounded_once(rows, N, tile, lo, hi):
    """SiLU in float32, then one rounding to float16: of 8 thousand to 8 million values few differ from the correctly rounded one.  A
    relative error e moves a value over the middle between two float16 numbers with probability |e v| / spacing <= 2^11 |e|.  exp,
    the sum and the quotient, each within 1 ulp, have a root mean square below 2^-24 together: at most 2^-13 of the values, and
    four standard deviations of that count."""
    import torch
    K = 2 * N + 32
    if tile is not None:
        assert _tile(EPI_SWIGLU, rows, N, K, 1)[0] == tile
    g = torch.Generator(device="cuda").manual_seed(rows + 7 * hi)
    v = torch.empty(rows * N, device="cuda").uniform_(lo, hi, generator=g)
    x, W, W2, exact = _pairs(v, N, 1.0)
    got = _activation(BF16, EPI_SWIGLU, x, W, W2, None, N, K)
    want = _silu(exact).astype(np.float16)
    bad, expect = int((got != want).sum()), got.size * 2.0 ** -13
    print(rows, N, (lo, hi), "differ", bad, "of", got.size, "allowed", expect + 4 * expect ** 0.5, flush=True)
    assert bad <= expect + 4 * expect ** 0.5
    assert np.abs(got.astype(np.float64) - want).max() <= 2.0 ** -10 * max(abs(lo), abs(hi))       # neighbours at most


@pytest.mark.parametrize("rows, N, tile", [(4080, 3072, 0), (4080, 2048, 1), (2032, 512, 3), (16, 512, None)])
def test_gelu_stored_as_float16(rows, N, tile):
    """GELU (tanh) with a bias in float32, then one rounding to float16: half a spacing (2^-25 below the normal numbers) on top."""
    import torch
    K = 2 * N + 32
    if tile is not None:
        assert _tile(EPI_GELU, rows, N, K, 1)[0] == tile
    g = torch.Generator(device="cuda").manual_seed(rows)
    v = torch.cat([torch.empty(rows * N // 2, device="cuda").uniform_(a, b, generator=g) for a, b in ((-3, 3), (-60, 60))])
    x, W, _, exact = _pairs(v[torch.randperm(v.numel(), generator=g, device="cuda")], N, 0.0)
    bias = torch.empty(N, device="cuda").uniform_(-1, 1, generator=g)
    s = (exact.astype(np.float32) + bias.cpu().numpy()).astype(np.float64)
    got, want = _activation(BF16, EPI_GELU, x, W, None, bias, N, K).astype(np.float64), _gelu(s)
    bound = _gelu_bound(s) + np.maximum(np.abs(want) * 2.0 ** -11, 2.0 ** -25)
    print(rows, N, "worst share of the bound", float((np.abs(got - want) / bound).max()), flush=True)
    assert (np.abs(got - want) <= bound).all()


@pytest.mark.parametrize("rows", [16, 48])
def test_float32_activations_to_their_ends(rows):
    """Float32 mode: SiLU within 2^-21 down to where its float32 values end (exp(-x) overflows below -88.7), GELU within its own, which is
    relative on the negative side as well; infinities and NaN as the formulas give them."""
    import torch
    N = 256
    K = N + 4
    x = torch.zeros(rows, K, device="cuda")
    x[:, :N] = torch.linspace(-88.5, 88.5, rows * N, device="cuda").view(rows, N)
    x[0, :N] = torch.linspace(-88.5, -87, N, device="cuda")
    x[1, :N] = torch.linspace(-1e-3, 1e-3, N, device="cuda")
    x[:, N] = 1.0
    W = torch.cat([torch.eye(N, device="cuda"), torch.zeros(N, 4, device="cuda")], 1)
    W2 = torch.zeros_like(W)
    W2[:, N] = 1.0
    v = x[:, :N].cpu().numpy().astype(np.float64)
    got = _activation(F32, EPI_SWIGLU, x, W, W2, None, N, K)
    want = _silu(v)
    assert (np.abs(got - want) <= 2.0 ** -21 * np.abs(want)).all(), np.abs(got / want - 1).max()
    bias = torch.zeros(N, device="cuda")
    bias[:4] = torch.tensor([float("inf"), float("-inf"), float("nan"), 1e30], device="cuda")
    s = (x[:, :N].cpu().numpy() + bias.cpu().numpy()).astype(np.float64)
    got, want = _activation(F32, EPI_GELU, x, W, None, bias, N, K), _gelu(s)
    assert np.array_equal(got[:, :4], want[:, :4].astype(np.float32), equal_nan=True)
    got, want, s = got[:, 4:], want[:, 4:], s[:, 4:]
    off, bound = np.abs(got - want), _gelu_bound(s)
    low = (s > -6) & (s < -3)
    print(rows, "GELU, worst share of the bound", float((off[bound > 0] / bound[bound > 0]).max()), "on -6 .. -3", float((off[low] / bound[low]).max()), flush=True)
    assert (off <= bound).all()
    # x = 3e38 + 3e38 and the negative: infinite sums of the product itself, whose SiLU is infinity and NaN
    x[:, :N] = 0.0
    x[0, :2] = torch.tensor([3e38, -3e38], device="cuda")
    W[:2, :2] *= 2.0
    got = _activation(F32, EPI_SWIGLU, x, W, W2, None, N, K)
    assert got[0, 0] == np.inf and np.isnan(got[0, 1]) and (got[1:, :2] == 0).all()


@pytest.mark.parametrize("K", [520, 1024])
@pytest.mark.parametrize("with_bias", [True, False])
def test_last_round_in_halves_adds_itself(K, with_bias):
    """3561 rows of 5768 columns, which the 256 x 256 tile adds to the residual rows: 14 x 23 tiles, 66 of them beyond the first round of 256
    workgroups, in halves of 256 x 128; odd and even numbers of k tiles, a last one that is not full, neither rows nor columns a multiple of the
    tile.  Products of float16 values are exact in float32, their sum and the two additions off by at most 2^-24 of the absolute sums each."""
    import torch
    rows, live, N = 3568, 3561, 5768
    assert _tile(EPI_PART, rows, N, K, 8) == (0, 1) and 0 < -(-rows // 256) * -(-N // 256) - 256 <= 128
    g = torch.Generator(device="cuda").manual_seed(K)
    rnd = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
    x, w, h = rnd(rows, K).half().float(), (rnd(N, K) * 0.05).half().float(), rnd(rows, N)
    bias = rnd(N) if with_bias else None
    X, W, out = _operand(x), _operand(w), h.clone()
    n = torch.tensor([live], dtype=torch.int32, device="cuda")
    shares = _lib()["_ZN8sprinter16launch_gemm_partEiPKvS1_mPKiiiPfmiPKfS4_iP12ihipStream_t"](
        BF16, _ptr(W), _ptr(X), C.c_size_t(X.numel()), _ptr(n), N, K, _ptr(None), C.c_size_t(rows * N), 8, _ptr(bias), _ptr(out), rows,
        C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert shares == 0
    b = torch.zeros(N, device="cuda") if bias is None else bias
    want = h.double() + b.double() + x.double() @ w.double().T
    bound = 2.0 ** -24 * ((K + 2) * (x.abs().double() @ w.abs().double().T) + 2 * (h.abs() + b.abs()).double())
    worst = float(((out.double() - want).abs() / bound)[:live].max())
    print(K, with_bias, "worst share of the bound", round(worst, 4), flush=True)
    assert worst <= 1
    assert torch.equal(out[live:], h[live:])                 # rows beyond the count stay as they are
    # the bound tells a missing k tile in any element
    assert bool(((x[:, 32:64].double() @ w[:, 32:64].double().T).abs() > bound)[:live].float().mean() > 0.5)
