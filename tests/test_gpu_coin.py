"""The p/q coin and the residual draw with a token's vocabulary cut into slices, launched by themselves, against the oracle."""
import ctypes as C
import numpy as np
import pytest
from oracle import sprinter as osp
from test_gpu_products import _lib, _ptr

pytestmark = pytest.mark.gpu

SEED, MAX_LOGIT = 77, 16.0
# Error of ln p(x) - ln q(x) in float32: four quantities of the logits' size, each rounded a few times (2^-24 of its size), and two
# sums of exponentials (3 roundings per exponential, 40 additions one after the other at most: 8 of a thread per block, 5 blocks).
DELTA = 4 * 3 * MAX_LOGIT * 2.0 ** -24 + 2 * 43 * 2.0 ** -24


class SdArgs(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("dl", "tl", "n_rows", "t_b", "t_pos", "t_last", "draft_tok")] + \
               [("V", C.c_int), ("inv_temperature", C.c_float), ("seed_lo", C.c_uint), ("seed_hi", C.c_uint),
                ("committed", C.c_void_p), ("coin_kept", C.c_void_p)]


def inputs(n, V):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n + V)
    lq = torch.randn(n, V, device="cuda", generator=g) * 2
    lp = lq + torch.randn(n, V, device="cuda", generator=g) * 1.5
    x = torch.multinomial(torch.softmax(lq, -1), 1, generator=g).flatten().int()
    return lq.clamp(-MAX_LOGIT, MAX_LOGIT), lp.clamp(-MAX_LOGIT, MAX_LOGIT), x


def correct(lq, lp, x, last, room):
    """committed tokens and the count of kept ones; room: bytes of scratch per token"""
    import torch
    n, V = lq.shape
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    rows, b, pos, kept, out = i32([n]), i32(range(n)), i32([3 * i + 2 for i in range(n)]), i32([0]), i32([-7] * n)
    work = torch.full((n * room,), 0xAA, dtype=torch.uint8, device="cuda")
    a = SdArgs(lq.data_ptr(), lp.data_ptr(), rows.data_ptr(), b.data_ptr(), pos.data_ptr(), last.data_ptr(), x.data_ptr(), V, 1.0,
               SEED, 0, out.data_ptr(), kept.data_ptr())
    for _ in range(2):                                         # (the second finds the first one's scratch)
        kept.zero_()
        _lib()["_ZN8sprinter17launch_sd_correctERKNS_6SdArgsEiPvmP12ihipStream_t"](
            C.byref(a), n, _ptr(work), C.c_size_t(work.numel()), C.c_void_p(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
    return out.cpu().numpy(), int(kept.item())


# a word, a block of 2048 less and more than full, several slices; the scratch of narrow rows: one slice, slices of several blocks
@pytest.mark.parametrize("n,V,room", [(5, 1, 192), (33, 255, 192), (40, 2048, 192), (40, 2049, 28), (24, 8191, 60), (80, 50257, 4096),
                                      (6, 50257, 192), (3, 128256, 4096), (4, 133000, 4096)])
def test_coin_and_residual_of_a_sliced_vocabulary(n, V, room):
    import torch
    lq, lp, x = inputs(n, V)
    last = torch.ones(n, dtype=torch.int32, device="cuda")
    if n > 4: last[n // 2] = 0                                 # an entry that commits nothing
    if V > 1:
        lp[0, : min(V // 2, 2048)] = -float("inf")             # a slice without weight
        x[0] = V - 1
        lp[1, V // 2] = float("nan")                           # a row that is no distribution keeps the drafted token
    got, kept = correct(lq, lp, x, last, room)
    q, p, xs, exact = lq.cpu().numpy(), lp.cpu().numpy(), x.cpu().numpy(), 0
    want_kept = 0
    for i in range(n):
        if not last[i]:
            assert got[i] == -7
            continue
        want_kept += int(got[i] == xs[i])                      # (a residual draw is never x: p(x) < q(x) there)
        if V > 1 and i == 1:
            assert got[i] == xs[i]
            continue
        r = osp.sd_correction(q[i], p[i], int(xs[i]), 1.0, SEED, i, 3 * i + 3, always_draw=True)
        if got[i] == r["tok"]:
            exact += 1
        elif r["kept"] != (got[i] == xs[i]):
            assert abs(np.log(r["coin"]) - r["log_ratio"]) <= DELTA, i
        else:
            assert got[i] == r["runner_up"] and r["margin"] <= DELTA * r["band"] + 2.0 ** -19, i   # (noise: two logarithms)
    assert kept == want_kept
    assert exact >= 0.9 * (n - 2)
