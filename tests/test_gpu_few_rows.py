"""The launches of a pass of few rows by themselves, every element against float64: the product that adds itself to the residual rows, and the product
that normalises those rows with the statistics the first one left."""
import ctypes as C
import numpy as np
import pytest
from test_gpu_products import BF16, F32, _lib, _operand, _ptr, _rows

pytestmark = pytest.mark.gpu
EPS = 1e-5


def _takes_norm(dtype, d, rows):
    return bool(_lib()["_ZN8sprinter15gemm_takes_normEiii"](dtype, d, rows) & 0xFF)


def _cases():
    # both sides of the lines in d (512, 1024, 2048) and of the rows a thread, a load or an operand takes; K: odd numbers of k tiles, a last one partly
    # filled, less than one round of the waves, several rounds of the loads in flight; columns beyond d: a part of a tile, two tiles per wave
    for d, K, rows in [(64, 64, (1, 9)), (512, 1344, (3, 8, 16)), (576, 72, (4, 5)), (768, 3072, (1, 4, 8, 9, 16)), (1024, 200, (12,)), (1088, 264, (1, 3, 8)),
                       (1600, 6400, (1, 2, 4, 5, 8)), (2048, 8192, (7,)), (2112, 2112, (1, 2, 3)), (4096, 14336, (1, 4, 5, 16, 17, 32)), (4160, 328, (25,)), (8192, 96, (13, 31))]:
        for r in rows:
            yield BF16, d, K, r, 40
    yield BF16, 1600, 1600, 4, 2520
    for r in (17, 24, 32):
        yield BF16, 1600, 1600, r, 0
        yield BF16, 576, 72, r, 0
    for d, K, rows in [(64, 72, (1, 16)), (256, 1024, (4, 5, 16)), (512, 2048, (1, 8)), (1024, 104, (3, 8)), (2048, 64, (4,))]:
        for r in rows:
            yield F32, d, K, r, 24


def _columns(dtype, d, rows):
    """Consecutive columns that a group of statistics covers."""
    return 16 if d > 2048 else 4 if dtype == F32 and d <= 1024 and rows <= 4 else 8


def _check_statistics(dtype, arch, h, stat):
    """The statistics that the product left, of every row and group, against those of the residual rows that it wrote."""
    rows, d = h.shape
    cols = _columns(dtype, d, rows)
    got = stat[:2 * rows * (d // cols)].view(rows, d // cols, 2).double()
    v = h.double().view(rows, d // cols, cols)
    size = v.abs().mean(2)
    off = 2.0 ** -24 * 5 * size if arch == 0 else 0 * size        # the mean: at most 4 additions, a power of two
    dv = v - v.mean(2, keepdim=True) if arch == 0 else v
    each = 2.0 ** -24 * dv.abs() + off[:, :, None]                              # of a distance, with its own rounding
    bound = (2 * dv.abs() * each + each ** 2).sum(2) + 6 * 2.0 ** -24 * (dv ** 2).sum(2)   # the square and at most 4 additions
    assert ((got[:, :, 1] - (dv ** 2).sum(2)).abs() <= bound).all()
    if arch == 0:
        assert ((got[:, :, 0] - v.sum(2)).abs() <= 2.0 ** -24 * 5 * cols * size).all()
    # in nearly every group the bound tells any one column's share
    assert ((dv ** 2) > bound[:, :, None]).double().mean() > 0.9


@pytest.mark.parametrize("arch", [0, 1])
@pytest.mark.parametrize("dtype,d,K,rows,more", list(_cases()))
def test_residual_rows_and_their_norm(dtype, d, K, rows, more, arch):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(d * 17 + rows + arch)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    store = (lambda t: t.contiguous()) if dtype == F32 else _operand
    x, W, bias = rnd(rows, K), rnd(d, K) * 0.1, rnd(d) if arch == 0 else None
    if dtype == BF16:
        x, W = x.half().float(), W.half().float()
    # residual rows as deep models have them: a mean, a few columns far out, rows of different sizes
    h = (rnd(rows, d) * 3 + 2) * (1 + torch.arange(rows, device="cuda")[:, None])
    h[:, 5::61] += 150
    Wd, X = store(W), store(x)                                              # (operand tiles: the rows of a tile that do not exist must have no effect)
    if dtype == BF16:
        X.view(-1, X.shape[1], 4, 16, 8)[:, :, :, rows:] = float("nan")
    hg, stat = h.clone(), torch.full((32 * d // 4,), float("nan"), device="cuda")
    _lib()["_ZN8sprinter17launch_gemm_residEiiPKvS1_iiPKfPfS4_iP12ihipStream_t"](
        dtype, arch, _ptr(Wd), _ptr(X), d, K, _ptr(bias), _ptr(hg), _ptr(stat), rows, stream)
    torch.cuda.synchronize()
    want = h.double() + x.double() @ W.double().T + (0 if bias is None else bias.double())
    # sums in float32: 32 products of an instruction, a wave's k tiles, 8 waves of at most 4 parts, residual and bias
    steps = 32 + K / 32 / 8 + 32 + 3
    bound = steps * 2.0 ** -24 * (h.double().abs() + x.double().abs() @ W.double().abs().T + (0 if bias is None else bias.double().abs()))
    assert ((hg.double() - want).abs() <= bound).all()
    _check_statistics(dtype, arch, hg, stat)
    if not _takes_norm(dtype, d, rows):
        assert _lib()["_ZN8sprinter14gemm_adds_rowsEiiii"](dtype, d, K, rows) & 0xFF
        return
    # a unit matrix shows the normalised rows themselves; the columns behind it are products
    gain, off = 1 + 0.1 * rnd(d), 0.1 * rnd(d) if arch == 0 else None
    V = torch.cat([torch.eye(d, device="cuda"), rnd(more, d)])
    if dtype == BF16:
        V = V.half().float()
    N, Vd = d + more, store(V)
    y = torch.full((rows, N), float("nan"), device="cuda")
    _lib()["_ZN8sprinter16launch_norm_gemmEiiiPKfS1_S1_S1_fPKNS_11EmbedSourceEPfPKvS7_iiS1_PviP12ihipStream_t"](
        dtype, arch, 0, _ptr(hg), _ptr(stat), _ptr(gain), _ptr(off), C.c_float(EPS), _ptr(None), _ptr(None), _ptr(Vd), _ptr(None), N, d, _ptr(None),
        _ptr(y), rows, stream)
    torch.cuda.synchronize()
    h64 = hg.double()
    mean = h64.mean(1, keepdim=True) if arch == 0 else torch.zeros(rows, 1, device="cuda", dtype=torch.float64)
    rstd = 1 / torch.sqrt(((h64 - mean) ** 2).mean(1, keepdim=True) + EPS)
    scaled = (h64 - mean) * rstd * gain.double()
    xn = scaled + (0 if off is None else off.double())
    # float32 arithmetic per element (the difference, three factors, the sum) and in the statistics (4 + 16 steps of their sums); float16 storage
    fine = 2.0 ** -24 * (24 * scaled.abs() + 24 * (mean * rstd * gain.double()).abs() + 4 * xn.abs())
    unit = fine + (2.0 ** -11 * 1.001 * xn.abs() + 2.0 ** -25 if dtype == BF16 else 0)
    assert ((y[:, :d].double() - xn).abs() <= unit).all()
    V64 = V[d:].double()
    steps = 32 + d / 32 / 8 + 8
    bound = unit @ V64.abs().T + steps * 2.0 ** -24 * (xn.abs() @ V64.abs().T)
    assert ((y[:, d:].double() - xn @ V64.T).abs() <= bound).all()


@pytest.mark.parametrize("d,K,rows", [(4096, 96, 24), (1088, 96, 24), (576, 72, 18)])
def test_rows_stay_apart(d, K, rows):
    """A row of infinities (activations beyond float16) has no effect on other rows, whichever operand it lies in, at an odd number of k tiles and fewer than the loads in flight."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(d)
    x, W, h = (torch.randn(*s, device="cuda", generator=g).half().float() for s in ((rows, K), (d, K), (rows, d)))
    assert _lib()["_ZN8sprinter14gemm_adds_rowsEiiii"](BF16, d, K, rows) & 0xFF
    out, Wd = [], _operand(W)
    for bad in (None, 2, 16):
        xb, hg = x.clone(), h.clone()
        if bad is not None:
            xb[bad] = float("inf")
        Xd = _operand(xb)
        _lib()["_ZN8sprinter17launch_gemm_residEiiPKvS1_iiPKfPfS4_iP12ihipStream_t"](
            BF16, 0, _ptr(Wd), _ptr(Xd), d, K, _ptr(None), _ptr(hg), _ptr(None), rows, C.c_void_p(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        out.append(hg)
        if bad is not None:
            assert not hg[bad].isfinite().any()
            keep = torch.arange(rows, device="cuda") != bad
            assert torch.equal(hg[keep], out[0][keep])


# gate + up with the norm inside: one and two column tiles per wave, the largest LDS of each
@pytest.mark.parametrize("d,N,rows", [(512, 1344, 16), (1024, 2816, 9), (2048, 4104, 8), (2048, 1000, 3), (4096, 520, 4)])
def test_gate_and_up(d, N, rows):
    import torch
    g = torch.Generator(device="cuda").manual_seed(d + N)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    h, gain, stat = rnd(rows, d) * 2, 1 + 0.1 * rnd(d), torch.zeros(8 * d, device="cuda")
    W, W2 = ((rnd(N, d) * d ** -0.5).half().float() for _ in range(2))
    Wd, W2d, Vd, none = _operand(W), _operand(W2), _operand(rnd(d, 64)), _operand(torch.zeros(rows, 64, device="cuda"))
    _lib()["_ZN8sprinter17launch_gemm_residEiiPKvS1_iiPKfPfS4_iP12ihipStream_t"](
        BF16, 1, _ptr(Vd), _ptr(none), d, 64, _ptr(None), _ptr(h), _ptr(stat), rows, stream)
    out = _operand(torch.zeros(rows, N, device="cuda"))
    _lib()["_ZN8sprinter16launch_norm_gemmEiiiPKfS1_S1_S1_fPKNS_11EmbedSourceEPfPKvS7_iiS1_PviP12ihipStream_t"](
        BF16, 1, 3, _ptr(h), _ptr(stat), _ptr(gain), _ptr(None), C.c_float(EPS), _ptr(None), _ptr(None), _ptr(Wd), _ptr(W2d), N, d, _ptr(None),
        _ptr(out), rows, stream)
    torch.cuda.synchronize()
    xn = h.double() * gain.double() / torch.sqrt((h.double() ** 2).mean(1, keepdim=True) + EPS)
    a, b = xn @ W.double().T, xn @ W2.double().T
    want, got = a / (1 + torch.exp(-a)) * b, _rows(out, rows, N).double()
    # every input of the sums is rounded by at most 2^-11, 2^-11 / sqrt(3) in the mean square, independently: so are the sums, relative to their spread of about 1; the
    # result moves by the factors' errors times at most 1.1 and 2.8 (SiLU's slope, and its values), then is rounded itself
    assert ((got - want).norm() / want.norm()).item() <= 2.0 ** -10
    spread = 2.0 ** -11 * 6 * (1.1 * b.abs() + a.abs() + 0.3)
    assert ((got - want).abs() <= spread + 2.0 ** -11 * want.abs() + 2.0 ** -25).all()


# widths and row counts at which the rule leaves the product in shares: one to eight of them, two column tiles per wave, tiles of 32 rows; workgroups for half the compute units and more than all
@pytest.mark.parametrize("d,K,rows", [(2112, 8448, 5), (2112, 3200, 16), (2112, 8448, 17), (3072, 5000, 32), (4352, 4352, 24), (5120, 5120, 32), (5120, 9000, 4), (6144, 6144, 16)])
def test_products_left_in_shares(d, K, rows):
    import torch
    assert not _lib()["_ZN8sprinter14gemm_adds_rowsEiiii"](BF16, d, K, rows) & 0xFF
    g = torch.Generator(device="cuda").manual_seed(d + rows)
    x, W = (torch.randn(*s, device="cuda", generator=g).half().float() for s in ((rows, K), (d, K)))
    h, bias = torch.randn(rows, d, device="cuda", generator=g), torch.randn(d, device="cuda", generator=g)
    X, Wd = torch.zeros(64, K, device="cuda"), _operand(W)                     # (activation buffers hold 64 rows)
    X[:rows] = x
    X, part, out = _operand(X), torch.full((8, rows, d), float("nan"), device="cuda"), h.clone()
    n = torch.tensor([rows], dtype=torch.int32, device="cuda")
    shares = _lib()["_ZN8sprinter16launch_gemm_partEiPKvS1_mPKiiiPfmiPKfS4_iP12ihipStream_t"](
        BF16, _ptr(Wd), _ptr(X), C.c_size_t(X.numel()), _ptr(n), d, K, _ptr(part), C.c_size_t(rows * d), 8, _ptr(bias), _ptr(out), rows,
        C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert 0 <= shares <= 8
    got = out.double() if shares == 0 else h.double() + bias.double() + part[:shares].double().sum(0)
    want = h.double() + bias.double() + x.double() @ W.double().T
    bound = 2.0 ** -24 * ((K + 2) * (x.double().abs() @ W.double().abs().T) + 2 * (h.double().abs() + bias.double().abs()))   # any order of the sum
    print(d, K, rows, "shares", shares, "worst share of the bound", float(((got - want).abs() / bound).max()), flush=True)
    assert ((got - want).abs() <= bound).all()
    # the bound tells a missing k tile
    assert ((x[:, 32:64].double() @ W[:, 32:64].double().T).abs() > bound).double().mean() > 0.5


@pytest.mark.parametrize("arch", [0, 1])
# every number of threads and rows per thread, fewer groups of statistics than lanes and as many as there can be
@pytest.mark.parametrize("dtype,d,rows", [(BF16, 64, 3), (BF16, 512, 9), (BF16, 576, 4), (BF16, 1024, 16), (BF16, 1088, 2), (BF16, 2048, 8), (BF16, 2112, 1), (BF16, 4096, 4),
                                          (F32, 512, 4), (F32, 512, 16), (F32, 1024, 4), (F32, 1024, 8), (F32, 2048, 4)])
def test_every_group_of_statistics_counts(dtype, d, rows, arch):
    """Rows of ones whose statistics say that one group's columns are far out - another group in every row and launch, each one once: the result is
    far from what it would be without that group, in float16 too."""
    import torch
    cols = _columns(dtype, d, rows)
    groups, dev = d // cols, "cuda"
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    h, gain, off, V = torch.ones(rows, d, device=dev), torch.ones(d, device=dev), torch.zeros(d, device=dev), torch.eye(d, device=dev)[:64].contiguous()
    Vd, y = (V if dtype == F32 else _operand(V)), torch.empty(rows, 64, device=dev)
    for at in range(0, groups, rows):
        big = (at + torch.arange(rows, device=dev)) % groups
        stat = torch.zeros(rows, groups, 2, device=dev)
        stat[:, :, 1] = 1.0
        stat[torch.arange(rows, device=dev), big, 1] = 1000.0 * groups
        if arch == 0:
            stat[torch.arange(rows, device=dev), big, 0] = 40.0 * d
        flat = torch.cat([stat.flatten(), torch.full((64,), float("nan"), device=dev)])
        _lib()["_ZN8sprinter16launch_norm_gemmEiiiPKfS1_S1_S1_fPKNS_11EmbedSourceEPfPKvS7_iiS1_PviP12ihipStream_t"](
            dtype, arch, 0, _ptr(h), _ptr(flat), _ptr(gain), _ptr(off if arch == 0 else None), C.c_float(EPS), _ptr(None), _ptr(None), _ptr(Vd), _ptr(None), 64, d, _ptr(None),
            _ptr(y), rows, stream)
        torch.cuda.synchronize()
        s = stat.double()
        mean = s[:, :, 0].sum(1, keepdim=True) / d if arch == 0 else torch.zeros(rows, 1, device=dev, dtype=torch.float64)
        m2 = (s[:, :, 1] + (cols * (s[:, :, 0] / cols - mean) ** 2 if arch == 0 else 0)).sum(1, keepdim=True)
        want = ((1 - mean) / torch.sqrt(m2 / d + EPS)).expand(rows, 64)
        # 16 additions of either sum, the difference, root, quotient and product, and float16
        assert ((y.double() - want).abs() <= want.abs() * ((2.0 ** -11 if dtype == BF16 else 0) + 64 * 2.0 ** -24)).all()


class _Rows(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("n_rows", "b", "tok", "pos", "slot")]


class _Embeddings(C.Structure):
    _fields_ = [("tok_emb", C.c_void_p), ("pos_emb", C.c_void_p), ("rows", _Rows), ("rope", C.c_void_p), ("theta", C.c_float), ("V", C.c_int), ("max_pos", C.c_int), ("dh", C.c_int)]


@pytest.mark.parametrize("arch", [0, 1])
@pytest.mark.parametrize("dtype,d,rows,N", [(BF16, 192, 16, 200), (BF16, 576, 9, 136), (BF16, 1024, 16, 1032), (BF16, 1088, 5, 264), (BF16, 1600, 8, 4808), (BF16, 2048, 7, 4096), (BF16, 4096, 3, 328),
                                            (F32, 64, 9, 40), (F32, 512, 16, 72), (F32, 1024, 8, 200), (F32, 2048, 4, 24)])
def test_first_product_of_a_pass(dtype, d, rows, N, arch):
    """The product that reads embeddings instead of residual rows: it starts the residual stream, normalises it and leaves the rotary factors."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(d + rows + arch)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    ints = lambda hi: torch.randint(hi, (rows,), device="cuda", generator=g, dtype=torch.int32)
    T, vocab, max_pos, dh, theta = torch.float32 if dtype == F32 else torch.bfloat16, 83, 301, 64, 10000.0
    tok_emb, pos_emb = (rnd(vocab, d) * 2 + 1).to(T), rnd(max_pos, d).to(T) if arch == 0 else None
    tok, pos = ints(vocab), ints(max_pos)
    pos[0] = max_pos - 1
    gain, off, bias = 1 + 0.1 * rnd(d), 0.1 * rnd(d) if arch == 0 else None, rnd(N) if arch == 0 else None
    V = rnd(N, d) if dtype == F32 else rnd(N, d).half().float()
    Vd = V if dtype == F32 else _operand(V)
    y, h, rope = (torch.full(s, float("nan"), device="cuda") for s in ((rows, N), (rows, d), (rows, dh)))
    n = torch.tensor([rows], dtype=torch.int32, device="cuda")
    emb = _Embeddings(_ptr(tok_emb), _ptr(pos_emb), _Rows(_ptr(n), None, _ptr(tok), _ptr(pos), None), _ptr(rope if arch == 1 else None), theta, vocab, max_pos, dh)
    _lib()["_ZN8sprinter16launch_norm_gemmEiiiPKfS1_S1_S1_fPKNS_11EmbedSourceEPfPKvS7_iiS1_PviP12ihipStream_t"](
        dtype, arch, 0, _ptr(None), _ptr(None), _ptr(gain), _ptr(off), C.c_float(EPS), C.byref(emb), _ptr(h), _ptr(Vd), _ptr(None), N, d, _ptr(bias),
        _ptr(y), rows, C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    row = tok_emb[tok.long()].float() + (pos_emb[pos.long()].float() if arch == 0 else 0)
    assert torch.equal(h, row)
    if arch == 1:
        ang = pos.double()[:, None] * theta ** (-2.0 * torch.arange(dh // 2, device="cuda", dtype=torch.float64) / dh)
        want = torch.stack([ang.cos(), ang.sin()], 2).view(rows, dh)
        assert ((rope.double() - want).abs() <= 2.0 ** -24).all()
    h64 = row.double()
    mean = h64.mean(1, keepdim=True) if arch == 0 else torch.zeros(rows, 1, device="cuda", dtype=torch.float64)
    rstd = 1 / torch.sqrt(((h64 - mean) ** 2).mean(1, keepdim=True) + EPS)
    scaled = (h64 - mean) * rstd * gain.double()
    xn = scaled + (0 if off is None else off.double())
    unit = 2.0 ** -24 * (24 * scaled.abs() + 24 * (mean * rstd * gain.double()).abs() + 4 * xn.abs())   # as in test_residual_rows_and_their_norm
    if dtype == BF16:
        unit = unit + 2.0 ** -11 * 1.001 * xn.abs() + 2.0 ** -25
    V64, b = V.double(), 0 if bias is None else bias.double()
    bound = unit @ V64.abs().T + (32 + d / 32 / 8 + 8) * 2.0 ** -24 * (xn.abs() @ V64.abs().T) + 2.0 ** -24 * (abs(b) if bias is None else b.abs())
    assert ((y.double() - (xn @ V64.T + b)).abs() <= bound).all()


@pytest.mark.parametrize("dtype,d,N,rows", [(BF16, 512, 1096, 16), (BF16, 1024, 200, 9), (BF16, 1600, 6400, 8), (BF16, 2048, 136, 5), (BF16, 4096, 520, 4), (F32, 512, 200, 16), (F32, 2048, 72, 4)])
def test_up_with_gelu(dtype, d, N, rows):
    """FFN-up of a GPT-shaped model with the norm inside."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(d + N)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    store = (lambda t: t.contiguous()) if dtype == F32 else _operand
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    h, gain, off, bias, stat = rnd(rows, d) * 2 + 1, 1 + 0.1 * rnd(d), 0.1 * rnd(d), rnd(N), torch.zeros(8 * d, device="cuda")
    W = rnd(N, d) * d ** -0.5
    if dtype == BF16:
        W = W.half().float()
    Wd, Vd, none = store(W), store(rnd(d, 64)), store(torch.zeros(rows, 64, device="cuda"))
    _lib()["_ZN8sprinter17launch_gemm_residEiiPKvS1_iiPKfPfS4_iP12ihipStream_t"](
        dtype, 0, _ptr(Vd), _ptr(none), d, 64, _ptr(None), _ptr(h), _ptr(stat), rows, stream)
    out = store(torch.zeros(rows, N, device="cuda"))
    _lib()["_ZN8sprinter16launch_norm_gemmEiiiPKfS1_S1_S1_fPKNS_11EmbedSourceEPfPKvS7_iiS1_PviP12ihipStream_t"](
        dtype, 0, 2, _ptr(h), _ptr(stat), _ptr(gain), _ptr(off), C.c_float(EPS), _ptr(None), _ptr(None), _ptr(Wd), _ptr(None), N, d, _ptr(bias),
        _ptr(out), rows, stream)
    torch.cuda.synchronize()
    h64 = h.double()
    xn = (h64 - h64.mean(1, keepdim=True)) / torch.sqrt(h64.var(1, unbiased=False, keepdim=True) + EPS) * gain.double() + off.double()
    a = xn @ W.double().T + bias.double()
    want = 0.5 * a * (1 + torch.tanh(0.7978845608028654 * (a + 0.044715 * a ** 3)))
    got = (out if dtype == F32 else _rows(out, rows, N)).double()
    if dtype == F32:
        # the norm's arithmetic (24 roundings of every factor), the sum over d, GELU's slope of at most 1.13 and its own 8 roundings
        bound = 1.13 * 2.0 ** -24 * ((52 + 32 + d / 16 / 8 + 8) * (xn.abs() @ W.double().abs().T) + 2 * bias.double().abs()) + 8 * 2.0 ** -24 * a.abs()
        assert ((got - want).abs() <= bound).all()
    else:
        # inputs rounded to 2^-11 each, independently: the sums move by 2^-11 of their spread of about 1 (6 times that at most), the result by 1.13 of it and its own rounding
        assert ((got - want).norm() / want.norm()).item() <= 2.0 ** -10
        assert ((got - want).abs() <= 2.0 ** -11 * 6 * 1.13 + 2.0 ** -11 * want.abs() + 2.0 ** -25).all()
