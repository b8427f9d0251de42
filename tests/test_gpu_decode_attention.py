"""Decode attention by itself: rows that end anywhere in a wave's blocks, over caches that hold NaN from the row's own slot on."""
import ctypes as C
import pytest
from test_gpu_prefill_attention import _Dims, _Pass, _Rows, _lib

pytestmark = pytest.mark.gpu


# the last key's place in a block, in a step of the waves and in the number of steps (odd and even); one workgroup per row and several
@pytest.mark.parametrize("dh,H,KVH", [(128, 4, 4), (128, 8, 2), (64, 4, 4), (64, 8, 1)])
@pytest.mark.parametrize("slots", [(0, 1, 31, 32, 63, 96, 127, 128, 129, 160, 255, 256, 257, 383, 384, 400), (5,), (511, 900)])
def test_rows_of_every_length_in_blocks(dh, H, KVH, slots):
    import torch
    p = _Pass(dh, H, KVH, [(b, s, 1) for b, s in enumerate(slots)], True, dh + H + len(slots))
    at = torch.arange(p.B, device="cuda"), slice(None), p.slot.long()
    p.v[at] = p.y[:, (H + KVH) * dh:].view(-1, KVH, dh).bfloat16()
    appended, full = p.vt.clone(), lambda v: v.view(p.B, KVH, p.seq // 32, 4, 8, dh // 16, 16).permute(0, 1, 2, 5, 3, 6, 4).contiguous()
    appended.copy_(full(p.v))
    p.k[at] = float("nan")
    before = p.v.clone()
    before[at] = float("nan")
    vt = full(before)
    out = torch.full((-(-p.E // 16), H * dh // 32, 4, 16, 8), float("nan"), dtype=torch.float16, device="cuda")
    split = torch.zeros(1 << 20, device="cuda")
    d = _Dims(1, 1, H * dh, H, KVH, dh, 64, 64, p.seq, p.dqkv, 1e-5, 1e4)
    r = _Rows(*(t.data_ptr() for t in (p.n, p.b, p.b, p.slot, p.slot)))
    ptr = lambda t: C.c_void_p(t.data_ptr())
    _lib()["_ZN8sprinter16launch_attentionEiRKNS_9ModelDimsEPKfS4_RKNS_7RowDescEPvS8_miiS8_iPfP12ihipStream_tii"](
        1, C.byref(d), ptr(p.y), ptr(p.rope), C.byref(r), ptr(p.k), ptr(vt), C.c_size_t(0), max(slots) + 1, p.seq, ptr(out), p.E, ptr(split),
        C.c_void_p(torch.cuda.current_stream().cuda_stream), 0, 0)
    torch.cuda.synchronize()
    assert torch.equal(vt.view(torch.int16), appended.view(torch.int16))       # the new value and nothing else
    key = p.y[:, H * dh:(H + KVH) * dh].view(-1, KVH, dh).double()
    c, s = (p.rope[:, None, :, i].double() for i in (0, 1))
    lo, hi = key[..., :dh // 2], key[..., dh // 2:]
    key = torch.cat([lo * c - hi * s, hi * c + lo * s], -1)
    big = torch.maximum(lo.abs(), hi.abs()).repeat(1, 1, 2)
    assert ((p.k[at].double() - key).abs() <= key.abs() * 2.0 ** -8 + big * 2.0 ** -22).all()   # bfloat16 of two float32 products
    rows = out.permute(0, 3, 1, 2, 4).reshape(-1, H, dh)
    want, bound = p.reference()
    assert rows[p.E:].isnan().all() and ((rows[:p.E].double() - want).abs() <= bound).all()
