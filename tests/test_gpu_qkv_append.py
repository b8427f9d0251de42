"""The QKV projection that puts keys and values into the caches by itself, against the projection and the append launch: the same
queries and the same cache bits, at the row counts and widths that take each of the product's kernels."""
import ctypes as C
import numpy as np
import pytest
from test_gpu_prefill_attention import _Dims, _Rows
from test_gpu_products import _lib, _operand, _ptr

pytestmark = pytest.mark.gpu


class _Kv(C.Structure):
    _fields_ = [("k", C.c_void_p), ("v", C.c_void_p), ("b", C.c_void_p), ("slot", C.c_void_p)] + \
               [(n, C.c_int) for n in ("q_cols", "kv_cols", "dh", "KVH", "S")]


# (heads, KV heads, columns of a head, K): 9 and 24 column tiles, 300 (more than 256: two per wave up to 64 rows), odd K tiles
@pytest.mark.parametrize("H,KVH,dh,K", [(1, 1, 64, 72), (4, 1, 64, 256), (8, 2, 128, 200), (25, 25, 64, 1600)])
@pytest.mark.parametrize("rows", [1, 16, 17, 33, 49, 64, 65, 80, 129, 700])
def test_projection_appends_as_the_append_launch(H, KVH, dh, K, rows):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(rows * 31 + H)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    N, B, seq = (H + 2 * KVH) * dh, 9, 96
    X, W, bias = _operand(rnd(-(-rows // 16) * 16, K)), _operand(rnd(N, K)), rnd(N)
    at = torch.randperm(B * seq, generator=g, device="cuda")[:rows]
    at = torch.sort(at).values                                 # ascending rows and slots, runs of any length, no slot twice
    b, slot = (at // seq).int().contiguous(), (at % seq).int().contiguous()
    n = torch.tensor([rows], dtype=torch.int32, device="cuda")
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    res = []
    for fused in (False, True):
        y = torch.full((rows, N), float("nan"), device="cuda")
        k, v = (torch.full((B, KVH, seq, dh), -1, dtype=torch.int16, device="cuda") for _ in range(2))
        if fused:
            kv = _Kv(k.data_ptr(), v.data_ptr(), b.data_ptr(), slot.data_ptr(), H * dh, KVH * dh, dh, KVH, seq)
            _lib()["_ZN8sprinter15launch_gemm_qkvEPKvS1_mPKiiiPKfPfRKNS_6KvDestEiP12ihipStream_t"](
                _ptr(W), _ptr(X), C.c_size_t(X.numel()), _ptr(n), N, K, _ptr(bias), _ptr(y), C.byref(kv), rows, stream)
        else:
            _lib()["_ZN8sprinter11launch_gemmEiiPKvS1_S1_mPKiiiPKfPfiPviiP12ihipStream_t"](
                1, 0, _ptr(W), _ptr(None), _ptr(X), C.c_size_t(X.numel()), _ptr(n), N, K, _ptr(bias), _ptr(y), N, _ptr(None), N, rows, stream)
            d = _Dims(0, 1, H * dh, H, KVH, dh, 64, 64, seq, N, 1e-5, 1e4)
            r = _Rows(*(t.data_ptr() for t in (n, b, b, slot, slot)))
            _lib()["_ZN8sprinter16launch_attentionEiRKNS_9ModelDimsEPKfS4_RKNS_7RowDescEPvS8_miiS8_iPfP12ihipStream_tii"](
                1, C.byref(d), _ptr(y), _ptr(y), C.byref(r), _ptr(k), _ptr(v), C.c_size_t(0), seq, seq, _ptr(None), rows, _ptr(None), stream, 1, 0)
        torch.cuda.synchronize()
        res.append([t.cpu().numpy() for t in (y[:, :H * dh], k, v)])
    for name, a, c in zip(("queries", "keys", "values"), *res):
        assert np.array_equal(a, c), name
    assert not np.isnan(res[0][0]).any() and (res[0][1] != -1).any()
