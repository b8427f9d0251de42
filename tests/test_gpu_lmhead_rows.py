"""The LM head at the row counts around its passes, launched by itself: the sampled key of every row does not depend on how many other
rows share the launch (up to 16 rows another kernel samples), and its logits are the product's."""
import ctypes as C
import numpy as np
import pytest
from test_gpu_prefill_attention import _Rows
from test_gpu_products import _lib, _operand, _ptr

pytestmark = pytest.mark.gpu


class _Sampler(C.Structure):
    _fields_ = [("seed_lo", C.c_uint), ("seed_hi", C.c_uint), ("stream", C.c_uint), ("inv_t", C.c_float)]


def _head(W, x, b, pos, V, K, n_wg):
    """(largest key per row, logits) of the rows of x."""
    import torch
    rows = x.shape[0]
    pad = -(-rows // 16) * 16
    X, n = _operand(x), torch.tensor([rows], dtype=torch.int32, device="cuda")
    part = torch.zeros(n_wg, pad, dtype=torch.int64, device="cuda")
    logits = torch.full((rows, V), float("nan"), device="cuda")
    r = _Rows(*(t.data_ptr() for t in (n, b, b, pos, pos)))
    sa = _Sampler(3, 4, 1, 1.0)
    _lib()["_ZN8sprinter13launch_lmheadEiPKvS1_mRKNS_7RowDescEiiRKNS_11SamplerArgsEPyiiPfiP12ihipStream_tPKNS_12VerifierArgsE"](
        1, _ptr(W), _ptr(X), C.c_size_t(X.numel()), C.byref(r), V, K, C.byref(sa), _ptr(part), n_wg, pad, _ptr(logits), rows,
        C.c_void_p(torch.cuda.current_stream().cuda_stream), _ptr(None))
    torch.cuda.synchronize()
    return part.cpu().numpy().view(np.uint64).max(0)[:rows], logits


# vocabularies with up to 8 and with more column tiles per workgroup (one and two per wave)
@pytest.mark.parametrize("V,K", [(1003, 200), (70001, 96)])
@pytest.mark.parametrize("rows", [17, 33, 64, 65, 80, 81, 96, 97, 128, 129, 160, 161, 193, 257])
def test_rows_of_a_pass(V, K, rows):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + V)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    x, w = rnd(rows, K).half().float(), (rnd(V, K) * 0.1).half().float()
    W, n_wg = _operand(w), _lib()["_ZN8sprinter13lmhead_num_wgEii"](1, V)
    b = torch.randint(0, 999, (rows,), generator=g, device="cuda", dtype=torch.int32)
    pos = torch.randint(0, 999, (rows,), generator=g, device="cuda", dtype=torch.int32)
    keys, logits = _head(W, x, b, pos, V, K, n_wg)
    ref = x.double() @ w.double().T
    # float32 sums of K exact products: K / 2 ulp of the sum of magnitudes at most
    bound = (x.abs().double() @ w.abs().double().T) * K * 2.0 ** -25
    assert ((logits.double() - ref).abs() <= bound).all()
    for at in range(0, rows, 16):
        part, small = _head(W, x[at:at + 16], b[at:at + 16].contiguous(), pos[at:at + 16].contiguous(), V, K, n_wg)
        assert torch.equal(small, logits[at:at + 16]) and (part == keys[at:at + 16]).all()   # (both add the k tiles in order)
