"""Prefill attention by itself: every entry's output of both kernels against float64 attention over the same cache."""
import ctypes as C
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


class _Dims(C.Structure):
    _fields_ = [(n, C.c_int) for n in "arch n_layer d H KVH dh ff V max_pos dqkv".split()] + [("eps", C.c_float), ("theta", C.c_float)]


class _Rows(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in "n_rows b tok pos slot".split()]


def _lib():
    from paper_2502_04557_amd import binding
    return binding.load_library()


def _shared(dh, H, KVH, entries, ctx, run_len):
    return bool(_lib()["_ZN8sprinter11attn_sharedEiiiiii"](dh, H, KVH, entries, ctx, run_len) & 1)


class _Pass:
    """One pass over runs (batch row, first position, positions); every cache slot beyond a row's last position is NaN."""

    def __init__(self, dh, H, KVH, runs, rope, seed):
        import torch
        g = torch.Generator(device="cuda").manual_seed(seed)
        rnd = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
        self.a, self.runs = (dh, H, KVH, rope), runs
        self.E = sum(n for _, _, n in runs)
        self.B, self.seq = max(b for b, _, _ in runs) + 1, -(-max(s + n for _, s, n in runs) // 32) * 32
        ints = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
        self.b = ints([b for b, _, n in runs for _ in range(n)])
        self.slot = ints([s + i for _, s, n in runs for i in range(n)])
        self.n = ints([self.E])
        self.dqkv = (H + 2 * KVH) * dh
        self.y = rnd(self.E, self.dqkv)
        angle = rnd(self.E, dh // 2) * 10
        self.rope = torch.stack([angle.cos(), angle.sin()], -1).contiguous()
        self.k = rnd(self.B, KVH, self.seq, dh).bfloat16()
        self.v = rnd(self.B, KVH, self.seq, dh).bfloat16()
        last = {b: s + n for b, s, n in runs}
        for b in range(self.B):
            self.k[b, :, last.get(b, 0):] = float("nan")
            self.v[b, :, last.get(b, 0):] = float("nan")
        # value tiles: [block of 32 keys][16 columns][8 keys][column][key]
        self.vt = self.v.view(self.B, KVH, self.seq // 32, 4, 8, dh // 16, 16).permute(0, 1, 2, 5, 3, 6, 4).contiguous()

    def run(self, ctx, run_len, launched=None):
        """Outputs [entries, H, dh]; launched: rows the launch is sized for (at least the entries)."""
        import torch
        dh, H, KVH, rope = self.a
        E = launched or self.E
        out = torch.full((-(-E // 16), H * dh // 32, 4, 16, 8), float("nan"), dtype=torch.float16, device="cuda")
        d = _Dims(1 if rope else 0, 1, H * dh, H, KVH, dh, 64, 64, self.seq, self.dqkv, 1e-5, 1e4)
        r = _Rows(*(t.data_ptr() for t in (self.n, self.b, self.b, self.slot, self.slot)))
        p = lambda t: C.c_void_p(t.data_ptr())
        _lib()["_ZN8sprinter16launch_attentionEiRKNS_9ModelDimsEPKfS4_RKNS_7RowDescEPvS8_miiS8_iPfP12ihipStream_tii"](
            1, C.byref(d), p(self.y), p(self.rope), C.byref(r), p(self.k), p(self.vt), C.c_size_t(0), ctx, self.seq, p(out), E, C.c_void_p(0),
            C.c_void_p(torch.cuda.current_stream().cuda_stream), 3, run_len)
        torch.cuda.synchronize()
        rows = out.permute(0, 3, 1, 2, 4).reshape(-1, H, dh)
        assert rows[self.E:].isnan().all()                     # nothing behind the last entry is written
        return rows[:self.E]

    def reference(self, drop=None):
        """(attention, bound of the kernels' error) in float64; drop: keys that are left out."""
        import torch
        dh, H, KVH, rope = self.a
        q = self.y[:, :H * dh].view(self.E, H, dh).double()
        if rope:
            c, s = (self.rope[:, None, :, i].double() for i in (0, 1))
            lo, hi = q[..., :dh // 2], q[..., dh // 2:]
            q = torch.cat([lo * c - hi * s, hi * c + lo * s], -1)
        q = q / dh ** 0.5
        outs, bounds, at = [], [], 0
        for b, s0, n in self.runs:
            keys = s0 + n
            k, v = (t[b, :, :keys].double().repeat_interleave(H // KVH, 0) for t in (self.k, self.v))
            qr = q[at:at + n].transpose(0, 1)
            hidden = torch.arange(keys, device="cuda")[None] > s0 + torch.arange(n, device="cuda")[:, None]
            if drop is not None:
                hidden = hidden | ((torch.arange(keys, device="cuda") >= drop[0]) & (torch.arange(keys, device="cuda") < drop[1]))[None]
                hidden[:, 0] = False
            w = torch.softmax((qr @ k.transpose(1, 2)).masked_fill(hidden, float("-inf")), -1)
            outs.append((w @ v).transpose(0, 1))
            # queries and weights as two bfloat16 each (2^-17 of the value), products added in float32 (2^-16 of their absolute sum, for
            # all roundings together); a score off by e changes the result by 2 e of the weighted absolute values at most
            e = (qr.abs() @ k.abs().transpose(1, 2)).amax(-1, keepdim=True) * 2.0 ** -16
            bounds.append(((2 * e + 2.0 ** -16) * (w @ v.abs())).transpose(0, 1))
            at += n
        o = torch.cat(outs)
        return o, torch.cat(bounds) + torch.clamp(o.abs() * 2.0 ** -11, min=2.0 ** -25)


def _mixed(longest, total):
    """One long run, then runs of 1 - 40 positions that begin and end anywhere in a window of 16, 32 or 64 entries, some of them not at
    position 0 (the rest of a row that an earlier pass began), single ones among them; the last window is not full."""
    r = np.random.default_rng(longest)
    runs, left = [(0, 0, longest)], total - longest
    while left > 0:
        n = int(min(left, r.choice([1, 1, 2, 7, 15, 16, 17, 33, 40])))
        runs.append((len(runs), int(r.choice([0, 0, 5, 31, 64])), n))
        left -= n
    return runs


@pytest.mark.parametrize("rope", [True, False])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("H, KVH", [(64, 32), (64, 16), (64, 8)])
@pytest.mark.parametrize("runs", [[(0, 0, 517)], _mixed(150, 503), _mixed(1, 510), [(0, 96, 300), (1, 0, 33), (2, 700, 200)]])
def test_shared_by_four_waves(dh, H, KVH, runs, rope):
    """2, 4 and 8 heads per KV head: four waves take 64, 32 and 16 entries of one or several runs, some of them none of a run's; contexts from
    one block of 32 keys to more than the ring holds.  Every output within the bound and the same bits as from one wave by itself."""
    import torch
    p = _Pass(dh, H, KVH, runs, rope, seed=H // KVH + dh)
    assert _shared(dh, H, KVH, p.E, 4096, 64) and not _shared(dh, H, KVH, p.E, 4096, 1)
    got, (want, bound) = p.run(4096, 64), p.reference()
    worst = float(((got.double() - want).abs() / bound).max())
    print(dh, H, KVH, len(runs), "runs", p.E, "entries, worst share of the bound", round(worst, 3), flush=True)
    assert worst <= 1
    assert torch.equal(got, p.run(4096, 1))
    assert torch.equal(got, p.run(4096, 64, launched=p.E + 70))   # (a launch for more entries than there are)
    # the bound tells a missing block of keys, and one missing key
    for drop in ((32, 64), (3, 4)):
        if max(s + n for _, s, n in runs) > drop[1]:
            off = (p.reference(drop)[0] - want).abs() / bound
            assert float(off.max()) > 4


@pytest.mark.parametrize("rope", [True, False])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("H, KVH", [(4, 4), (8, 4), (8, 1)])
@pytest.mark.parametrize("runs", [[(0, 0, 1)], [(0, 0, 100)], _mixed(70, 231), [(0, 60, 40), (1, 0, 5), (2, 333, 64)]])
def test_one_wave_by_itself(dh, H, KVH, runs, rope):
    """One head over 32 entries or two heads of a KV head over 16: the queries requested once for all runs of the window."""
    p = _Pass(dh, H, KVH, runs, rope, seed=H + dh)
    assert not _shared(dh, H, KVH, p.E, 4096, 64)
    got, (want, bound) = p.run(4096, 64), p.reference()
    worst = float(((got.double() - want).abs() / bound).max())
    print(dh, H, KVH, len(runs), "runs", p.E, "entries, worst share of the bound", round(worst, 3), flush=True)
    assert worst <= 1
