"""Float32 attention by itself against float64: contexts that end anywhere in the steps of the four waves and of their 16 streams of keys,
and values at which a maximum per stream is not one per row."""
import ctypes as C
import numpy as np
import pytest
from test_gpu_prefill_attention import _Dims, _Rows, _lib

pytestmark = pytest.mark.gpu


class _Step:
    """One entry per batch row, entry i at slots[i].  The caches are NaN from each row's own slot on."""

    def __init__(self, dh, H, KVH, slots, rope, seed):
        import torch
        g = torch.Generator(device="cuda").manual_seed(seed)
        rnd = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
        ints = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
        self.dh, self.H, self.KVH, self.rope, self.slots, n = dh, H, KVH, rope, slots, len(slots)
        self.n, self.slot, self.dqkv, self.seq = ints([n]), ints(slots), (H + 2 * KVH) * dh, max(slots) + 3
        self.b = ints([(5 * i + 2) % n if n % 5 else i for i in range(n)])           # (a row's place in the list is not its place in the caches)
        self.y = rnd(n, self.dqkv)
        angle = rnd(n, dh // 2) * 10
        self.cs = torch.stack([angle.cos(), angle.sin()], -1).contiguous()
        self.k, self.v = rnd(n, KVH, self.seq, dh), rnd(n, KVH, self.seq, dh)
        for b, s in zip(self.b.tolist(), slots):
            self.k[b, :, s:], self.v[b, :, s:] = float("nan"), float("nan")

    def new(self):
        """(queries, keys, values) of the entries in float64, rotated, and the absolute sums behind queries and keys."""
        import torch
        dh, H, KVH = self.dh, self.H, self.KVH
        q, k, v = (t.double().view(len(self.slots), -1, dh) for t in self.y.split([H * dh, KVH * dh, KVH * dh], 1))
        if not self.rope:
            return q, k, v, q.abs(), k.abs()
        c, s = (self.cs[:, None, :, i].double() for i in (0, 1))
        halves = lambda t: (t[..., :dh // 2], t[..., dh // 2:])
        turn = lambda lo, hi: torch.cat([lo * c - hi * s, hi * c + lo * s], -1)
        size = lambda lo, hi: torch.cat([lo * c.abs() + hi * s.abs(), hi * c.abs() + lo * s.abs()], -1)
        return turn(*halves(q)), turn(*halves(k)), v, size(*halves(q.abs())), size(*halves(k.abs()))

    def run(self, phase=0):
        """Outputs [rows, H, dh]; phase 0 appends and attends, 1 only appends, 2 only attends."""
        import torch
        n, dh, H = len(self.slots), self.dh, self.H
        out = torch.full((n, H, dh), float("nan"), device="cuda")
        d = _Dims(int(self.rope), 1, H * dh, H, self.KVH, dh, 64, 64, self.seq, self.dqkv, 1e-5, 1e4)
        r = _Rows(*(t.data_ptr() for t in (self.n, self.b, self.b, self.slot, self.slot)))
        p = lambda t: C.c_void_p(t.data_ptr())
        _lib()["_ZN8sprinter16launch_attentionEiRKNS_9ModelDimsEPKfS4_RKNS_7RowDescEPvS8_miiS8_iPfP12ihipStream_tii"](
            0, C.byref(d), p(self.y), p(self.cs), C.byref(r), p(self.k), p(self.v), C.c_size_t(0), max(self.slots) + 1, self.seq, p(out), n, C.c_void_p(0),
            C.c_void_p(torch.cuda.current_stream().cuda_stream), phase, 0)
        torch.cuda.synchronize()
        return out

    def reference(self, drop=None):
        """(attention, bound of the kernel's error) in float64; drop: a key that is left out."""
        import torch
        G, outs, bounds = self.H // self.KVH, [], []
        q, kn, vn, qa, ka = self.new()
        for i, (b, s) in enumerate(zip(self.b.tolist(), self.slots)):
            per_head = lambda t: t.repeat_interleave(G, 0)
            k, v = (per_head(torch.cat([c[b, :, :s].double(), own[i, :, None]], 1)) for c, own in ((self.k, kn), (self.v, vn)))
            size = per_head(torch.cat([self.k[b, :, :s].double().abs(), ka[i, :, None]], 1))
            score = (q[i, :, None] * k).sum(-1) / self.dh ** 0.5
            if drop is not None and 0 <= drop < s:
                score[:, drop] = float("-inf")
            w = torch.softmax(score, -1)
            seen = torch.isfinite(score)
            # A score is 8 products per lane at most and 4 levels of a tree over rotated (3 roundings each), scaled operands: 24 roundings of
            # the absolute sum; its distance from a maximum, two exponentials (each of an argument of up to twice the sum) 8 more.  Weights and
            # values are added key by key in 16 streams, then over the streams, and divided: s / 16 + 40 roundings of the weighted absolute values.
            e = torch.where(seen, (qa[i, :, None] * size).sum(-1) / self.dh ** 0.5, 0.).amax(-1, keepdim=True) * 32 * 2.0 ** -24
            o = torch.where(w[..., None] > 0, w[..., None] * v, 0.).sum(1)
            outs.append(o)
            bounds.append((2 * e + (s / 16 + 40) * 2.0 ** -24) * torch.where(w[..., None] > 0, w[..., None] * v.abs(), 0.).sum(1))
        return torch.stack(outs), torch.stack(bounds)


# a step of the four waves is 128 keys: one step, its last key, the next one's first, several; scores that rise (every step has a new
# maximum), fall, or neither
SLOTS = (0, 1, 3, 31, 32, 33, 96, 127, 128, 129, 160, 255, 256, 257, 511, 512, 777)


@pytest.mark.parametrize("rope", [True, False])
@pytest.mark.parametrize("dh,H,KVH", [(64, 3, 3), (64, 4, 2), (64, 8, 2), (64, 16, 2), (128, 2, 2), (128, 4, 2), (128, 4, 1), (128, 8, 1)])
@pytest.mark.parametrize("rise", [0., 0.2, -0.2])
def test_rows_of_every_length(dh, H, KVH, rise, rope):
    import torch
    p = _Step(dh, H, KVH, SLOTS, rope, dh + H)
    q, kn, vn, _, ka = p.new()
    for i, (b, s) in enumerate(zip(p.b.tolist(), p.slots)):
        along = q[i, ::H // KVH].float()
        p.k[b, :, :s] += (along / along.norm(dim=-1, keepdim=True))[:, None] * (torch.arange(s, device="cuda") * rise)[None, :, None]
    (want, bound), before, at = p.reference(), (p.k.clone(), p.v.clone()), (p.b.long(), slice(None), p.slot.long())
    got = p.run()
    worst = float(((got.double() - want).abs() / bound).max())
    print(dh, H, KVH, rise, rope, "worst share of the bound", round(worst, 3), flush=True)
    assert worst <= 1
    if rise == 0:
        off = ((p.reference(drop=20)[0] - want).abs() / bound).amax((1, 2))
        assert (off[torch.tensor(SLOTS, device="cuda") > 20] > 4).all()      # (the bound tells a missing key in every row)
    # appended: the new key and value of every row, and nothing else
    assert ((p.k[at].double() - kn).abs() <= ka * 3 * 2.0 ** -24).all() and torch.equal(p.v[at], vn.float())
    for c, old in zip((p.k, p.v), before):
        old[at] = c[at]
        assert torch.equal(c.view(torch.int32), old.view(torch.int32))
    # the same in two launches, as passes take it whose entries share a row's caches
    after = p.k.clone(), p.v.clone()
    p.k[at], p.v[at] = float("nan"), float("nan")
    assert p.run(1).isnan().all()
    for c, whole in zip((p.k, p.v), after):
        assert torch.equal(c.view(torch.int32), whole.view(torch.int32))
    assert torch.equal(p.run(2), got)


# the limits are the errors of an attention with one maximum per row and a tree over the weights, measured on these inputs and rounded up
@pytest.mark.parametrize("dh,lo,hi,limit", [(64, 16, 60, 1.25e-7), (64, 60, 130, 1.37e-7), (64, 130, 300, 1.52e-7), (128, 60, 130, 1.46e-7), (128, 130, 300, 1.68e-7)])
def test_error_is_no_larger_than_with_one_maximum_per_row(dh, lo, hi, limit):
    errors = []
    for seed in range(24):
        p = _Step(dh, 8, 8, tuple(np.random.default_rng(seed).integers(lo, hi, 16).tolist()), True, seed)
        want, got = p.reference()[0], p.run().double()
        errors.append(float((got - want).norm() / want.norm()))
    print(dh, lo, hi, "error", np.mean(errors), flush=True)
    assert np.mean(errors) <= limit


# the keys that score -inf: all of one stream, all of a wave's first blocks, the row's first 128 (the first step of every wave), its own
@pytest.mark.parametrize("dh,H,KVH", [(64, 4, 4), (128, 8, 2), (64, 8, 1)])
@pytest.mark.parametrize("gone", [lambda j, s: j % 4 == 1, lambda j, s: j // 32 % 4 == 1, lambda j, s: j < 128, lambda j, s: j == s], ids=["stream", "wave", "step", "own"])
def test_keys_that_score_minus_infinity_have_no_weight(dh, H, KVH, gone):
    import torch
    p = _Step(dh, H, KVH, (130, 200, 300), False, dh + H)
    p.y[:, :H * dh].view(-1, H, dh)[..., 0].abs_().add_(0.1)              # every query's first column is positive
    for i, (b, s) in enumerate(zip(p.b.tolist(), p.slots)):
        at = torch.tensor([gone(j, s) for j in range(s)], device="cuda")
        p.k[b, :, :s, 0] = torch.where(at, float("-inf"), p.k[b, :, :s, 0])
        if gone(s, s):
            p.y[i, H * dh:(H + KVH) * dh].view(KVH, dh)[:, 0] = float("-inf")
    want, bound = p.reference()
    assert want.isfinite().all()
    assert ((p.run().double() - want).abs() <= bound).all()


# the row's own key in the place of 0 - 31 others of its block, in each wave's
@pytest.mark.parametrize("dh,H,KVH", [(64, 4, 4), (128, 8, 2), (64, 8, 1)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_value_that_is_not_finite_reaches_its_column_alone(dh, H, KVH, value):
    import torch
    p = _Step(dh, H, KVH, (0, 1, 5, 31, 32, 70, 127, 128, 200), False, dh + H)
    own = p.y[:, (H + KVH) * dh:].view(-1, KVH, dh)
    own[..., 3], own[..., dh - 1] = 0.5, 0.5
    want, bound = p.reference()
    own[..., 3], own[..., dh - 1] = value, -value
    got = p.run().double()
    assert ((got - want).abs() <= bound)[..., [c for c in range(dh) if c not in (3, dh - 1)]].all()
    for c, x in ((3, value), (dh - 1, -value)):
        assert (got[..., c] == x).all() if x == x else got[..., c].isnan().all()
