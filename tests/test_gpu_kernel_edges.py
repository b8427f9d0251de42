"""Kernel variants at the edges of the sizes their launchers choose them for: row counts around a row tile and a pass,
widths that leave a half-filled last k tile or column tile, K shares, small and ragged vocabularies.  Logits, hidden states,
scores and tokens of every step against the oracle replayed on the GPU's history, with the tolerances of parity_util."""
import numpy as np
import pytest
import workloads as W

pytestmark = pytest.mark.gpu


def _check(draft, target, B, dtype, *, ver_hidden=24, prompt_len=5, prompt_len_min=2, n_gen=3, tau=0.5, max_seq=48, seed=7, whole_prompt=False, chunk_rows=0, full_row=False):
    """Decode steps of one configuration; returns the rejected rows per step.  full_row: the last prompt has the full length."""
    from parity_util import Pair, compare_replay, close_enough, eps_of
    cfg = W.SprinterCfg(draft, target, ver_hidden, dtype, B, max_seq, tau=tau, seed=seed, name="edges", batch=B, prompt_len=prompt_len,
                        prompt_len_min=prompt_len_min, n_gen=n_gen, prompt_dist="uniform", weight_seed=500 + seed, prompt_seed=600 + seed, chunk_rows=chunk_rows)
    p = Pair(cfg, ver_scale=8.0)
    if full_row:
        p.prompts, p.plen = np.pad(p.prompts, ((0, 0), (0, prompt_len - p.prompts.shape[1]))), p.plen.copy()
        p.plen[-1] = prompt_len
        p.prompts[-1] = np.random.default_rng(seed).integers(0, draft.vocab, prompt_len)
    eps = eps_of(cfg)
    outs, _ = p.gpu_steps(n_gen)
    g = {k: np.stack([o[k2] for o in outs], axis=1) for k, k2 in
         (("tok", "committed_tok"), ("accept", "accept"), ("score", "score"), ("draft_tok", "draft_tok"))}
    rec = p.oracle(n_gen, forced=dict(tok=g["tok"], accept=g["accept"]), keep_logits=True, whole_prompt_prefill=whole_prompt)
    print(B, dtype, compare_replay(cfg, g, rec), flush=True)
    for s, o in enumerate(outs):
        R = int(o["n_rej"][0])
        assert list(o["rej_idx"][:R]) == list(np.flatnonzero(o["accept"] == 0))
        assert close_enough(o["draft_logits"], rec["draft_logits"][s], eps).all()
        assert close_enough(o["draft_hidden"], rec["draft_hidden"][s], eps).all()
        if R:
            assert close_enough(o["target_logits"][:R], rec["target_logits"][s], eps).all()
            assert close_enough(o["target_hidden"][:R], rec["target_hidden"][s], eps).all()
    p.close()
    return [int(o["n_rej"][0]) for o in outs]


def _gpt(L, d, ff, V):
    return W.ModelCfg(W.ARCH_GPT, L, d, d // 64, d // 64, ff, V, 48)


def _llama(L, d, H, KVH, ff, V):
    return W.ModelCfg(W.ARCH_LLAMA, L, d, H, KVH, ff, V, 48, 1e-5, 10000.0)


@pytest.mark.parametrize("B", [1, 16, 17, 33])
@pytest.mark.parametrize("ff", [72, 1096])
def test_float32_matrix_kernels(B, ff):
    """Float32 matrix kernels: one and two row tiles, a second pass over the rows; K = 64 (fewer groups of 16 k than waves), 72
    (half a group at the end), 192, 512 and 1096 (two K shares); both FFN kinds; a vocabulary with a ragged last column tile."""
    _check(_gpt(1, 64, ff, 331), _llama(1, 512, 8, 4, ff, 331), B, W.DT_F32)
    _check(_llama(1, 192, 3, 3, ff, 35), _gpt(1, 256, ff, 35), B, W.DT_F32)


@pytest.mark.parametrize("dtype", [W.DT_F32, W.DT_BF16])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 5])
def test_norm_inside_the_product(B, dtype):
    """One to five rows: the norm folded into QKV / FFN-up, with both norms, gate + up and GELU and 257 - 265 column tiles (at 2048
    columns in pairs), a last one that is not full; deep enough that a layer reads the statistics of the one before.  tau > 1: the target
    sees the same rows.  (The ends of the row counts: test_norm_inside_the_product_at_its_limits.)"""
    _check(_gpt(2, 128, 200, 83), _llama(3, 512, 4, 2, 4104, 83), B, dtype, tau=1.5)
    _check(_llama(3, 640, 10, 5, 136, 83), _gpt(2, 2048 if B == 2 else 1024, 4232, 83), B, dtype, tau=1.5)


@pytest.mark.parametrize("dtype", [W.DT_F32, W.DT_BF16])
@pytest.mark.parametrize("B", [5, 8, 9, 12, 13, 16, 17])
def test_norm_inside_the_product_of_narrow_models(B, dtype):
    """Up to 512 columns the norm is folded in up to 16 rows, eight groups of threads with one or two rows each: the first and last row
    counts of each, one row beyond, rows of 128 to 512 columns (a group's threads from a quarter to all in use), heads of 128
    with rotary factors for 16 rows, 257 column tiles and more."""
    _check(_gpt(2, 128, 200, 83), _llama(3, 512, 4, 2, 4104, 83), B, dtype, tau=1.5)
    _check(_llama(2, 320, 5, 5, 136, 83), _gpt(2, 448, 4232, 83), B, dtype, tau=1.5)


@pytest.mark.parametrize("dtype", [W.DT_F32, W.DT_BF16])
@pytest.mark.parametrize("B", [4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("gpt_is_wide", [False, True])
def test_norm_inside_the_product_at_its_limits(B, dtype, gpt_is_wide):
    """Both sides of the last row counts with the norm inside: 1024 columns 8 in float32 and 16 in bf16, 2048 columns 4 and 8, each once with LayerNorm and
    GELU, once with RMSNorm, gate + up and rotary factors.  tau > 1: the target sees the same rows."""
    takes = lambda d: bool(_host("_ZN8sprinter15gemm_takes_normEiii", dtype, d, B) & 0xFF)
    f32 = dtype == W.DT_F32
    assert takes(1024) == (B <= (8 if f32 else 16)) and takes(2048) == (B <= (4 if f32 else 8))
    if gpt_is_wide:
        _check(_llama(2, 1024, 16, 4, 264, 83), _gpt(2, 2048, 520, 83), B, dtype, tau=1.5)
    else:
        _check(_gpt(2, 1024, 264, 83), _llama(2, 2048, 16, 4, 520, 83), B, dtype, tau=1.5)


@pytest.mark.parametrize("B, prompt_len", [(7, 20), (9, 59), (8, 114)])
def test_tiles_of_many_rows(B, prompt_len):
    """Prefill passes of 133, 522 and 904 rows (none a multiple of a tile): the 32- and 64-row tiles with K shares, at 904 rows also the
    256-row tile (FFN-up of the target) and the 128-row tile (its FFN-down); a last k tile that is a quarter full and an odd number of
    k tiles (FFN-down, K = 3080 and 5128), column tiles beyond the last one, GELU and SwiGLU.  The prefilled caches carry every
    position, so the first steps' logits depend on all of them.  (Every tile: test_every_tile_with_every_epilogue.)"""
    draft = W.ModelCfg(W.ARCH_GPT, 2, 768, 12, 12, 3080, 331, 128)
    target = W.ModelCfg(W.ARCH_LLAMA, 2, 1024, 16, 16, 5128, 331, 128, 1e-5, 10000.0)
    _check(draft, target, B, W.DT_BF16, prompt_len=prompt_len, prompt_len_min=0, n_gen=2, tau=1.5, max_seq=128, whole_prompt=True)


@pytest.mark.parametrize("chunk_rows", [0, 64])
@pytest.mark.parametrize("group", [1, 2, 8])
def test_prefill_attention_runs(group, chunk_rows):
    """Prompts of 1 - 40 tokens: runs that begin and end anywhere in a block of 8 cached slots, of 16 or 32 entries and of 32
    keys, one or many in a block, whole in one pass or split over passes of 64 entries; 1, 2 and 8 query heads per KV head, head
    dimensions 64 and 128, with and without rotary positions.  (Two layers: the first one's attention is what the second one caches.)"""
    draft = W.ModelCfg(W.ARCH_LLAMA, 2, 512, 8, 8 // group, 136, 83, 48, 1e-5, 10000.0)
    target = _llama(2, 1024, 8, 8 // group, 136, 83) if group > 1 else _gpt(2, 128, 136, 83)
    _check(draft, target, 13, W.DT_BF16, prompt_len=41, prompt_len_min=1, tau=1.5, whole_prompt=True, chunk_rows=chunk_rows, seed=21 + group)


@pytest.mark.parametrize("chunk_rows", [0, 2112])
@pytest.mark.parametrize("group, B, longest", [(2, 6, 770), (4, 11, 390), (8, 20, 200)])
def test_prefill_attention_shared_by_waves(group, B, longest, chunk_rows):
    """Ragged prompts whose longest one has the first length that the rule shares, 16 heads of 128: whole in one pass, or in two of which the
    second goes back to one wave (the kernels give the same bits).  Two layers: the first one's attention is what the second one caches."""
    draft = W.ModelCfg(W.ARCH_GPT, 1, 128, 2, 2, 136, 83, 1088)
    target = W.ModelCfg(W.ARCH_LLAMA, 2, 2048, 16, 16 // group, 136, 83, 1088, 1e-5, 10000.0)
    seed = 41 + group
    cfg = W.SprinterCfg(draft, target, 24, W.DT_BF16, B, 1088, seed=seed, name="rule", batch=B, prompt_len=longest, prompt_len_min=longest // 4,
                        prompt_dist="uniform", prompt_seed=600 + seed)
    plen = W.make_prompts(cfg)[1]
    plen[-1] = longest                                       # (full_row)
    E = int(plen.sum()) - B
    shared = lambda entries: bool(_host("_ZN8sprinter11attn_sharedEiiiiii", 128, 16, 16 // group, entries, int(plen.max()), E // B) & 1)
    assert shared(min(E, chunk_rows or E)) and (not chunk_rows or not shared(E - chunk_rows)), (E, plen)
    _check(draft, target, B, W.DT_BF16, prompt_len=longest, prompt_len_min=longest // 4, tau=1.5, n_gen=2, max_seq=-(-(longest + 4) // 32) * 32,
           whole_prompt=True, chunk_rows=chunk_rows, seed=seed, full_row=True)


@pytest.mark.parametrize("B", [17, 40, 65, 80])
def test_small_tiles(B):
    """17 - 80 rows of one step, all rejected: the 32- and 64-row tiles with K shares down to three k tiles each, a row count
    just beyond a tile and beyond two, a half-filled last k tile, the wide gate + up product (FFN 5128: 161 workgroups of 32
    columns) next to the K-split kernel for the narrow ones."""
    _check(_gpt(1, 192, 712, 83), _llama(1, 512, 8, 2, 5128, 83), B, W.DT_BF16, tau=1.5, prompt_len=3, n_gen=2)


@pytest.mark.parametrize("group", [1, 2, 8])
def test_short_runs_share_a_pass(group):
    """Full-prefix work lists: runs of 1 to 40 entries that begin and end anywhere in a group of 16 / G positions (the first
    pass over a prompt-free cache is long, later ones follow the rejections), contexts beyond one block of keys per wave."""
    from parity_util import Pair, compare_replay
    draft = W.ModelCfg(W.ARCH_GPT, 1, 128, 2, 2, 136, 83, 160)
    target = W.ModelCfg(W.ARCH_LLAMA, 2, 1024, 8, 8 // group, 136, 83, 160, 1e-5, 10000.0)
    cfg = W.SprinterCfg(draft, target, 24, W.DT_BF16, 5, 160, tau=0.5, seed=31 + group, name="runs", batch=5, prompt_len=110,
                        prompt_len_min=3, n_gen=24, prompt_dist="uniform", weight_seed=531, prompt_seed=631, target_ctx_mode=W.CTX_FULL_PREFIX)
    p = Pair(cfg, ver_scale=8.0)
    g, _ = p.gpu_generate(cfg.n_gen)
    rec = p.oracle(cfg.n_gen, forced=dict(tok=g["tok"], accept=g["accept"]))
    rep = compare_replay(cfg, g, rec)
    print(group, rep, flush=True)
    assert 0 < rep["reject_rate"] < 1
    p.close()


@pytest.mark.parametrize("B", [1, 3])
def test_keys_shared_by_several_workgroups(B):
    """Few rows with contexts long enough that 8 workgroups share a row's keys, in one step each: one or two query heads per KV
    head, head dimension 128 (from 800 positions) and 64 (from 1600), the new key in the last block of another workgroup's."""
    draft = W.ModelCfg(W.ARCH_LLAMA, 1, 256, 4, 4, 136, 83, 1700, 1e-5, 10000.0)
    target = W.ModelCfg(W.ARCH_LLAMA, 1, 1024, 8, 8 if B == 3 else 4, 136, 83, 1700, 1e-5, 10000.0)
    _check(draft, target, B, W.DT_BF16, prompt_len=1630, prompt_len_min=810, tau=1.5, n_gen=3, max_seq=1664, whole_prompt=True)


@pytest.mark.parametrize("group", [1, 4])
def test_non_finite_token_leaves_earlier_window_entries_alone(group):
    """A drafted token whose target embedding is not a number spoils the target's view of the positions from its own on, and
    nothing before: up to that point the round (coins, residual draws) is that of a target with a finite embedding, although
    earlier entries of the window share one pass over the row's keys and values with the later ones."""
    from dataclasses import replace
    from parity_util import Pair
    X, gamma, B = 3, 4, 40
    draft = _llama(1, 128, 2, 2, 136, 11)
    target = _llama(2, 512, 4, 4 // group, 136, 11)
    cfg = W.SprinterCfg(draft, target, 24, W.DT_BF16, B, 48, temperature=0.15, seed=51, name="nan", batch=B, prompt_len=30,
                        prompt_len_min=3, prompt_dist="uniform", weight_seed=551, prompt_seed=651, sd_gamma=gamma)
    rounds = []
    for value in (0.0, np.nan):
        dw, tw, vw = W.make_weights(cfg)
        tw["tok_emb"][X] = value
        p = Pair(cfg, weights=(dw, tw, vw))
        p.prompts[p.prompts == X] = X + 1
        p.gpu.prefill(p.prompts, p.plen)
        rounds.append({k: v.cpu().numpy() for k, v in p.gpu.sd_generate(gamma, 1).items()})
        p.close()
    clean, nan = rounds
    assert np.array_equal(clean["draft"], nan["draft"])
    decided_before = 0
    for b in range(B):
        at = np.flatnonzero(clean["draft"][b, 0] == X)
        first = int(at[0]) if len(at) else gamma               # entries 0 .. first of the window have not seen X
        n = int(clean["n_acc"][b, 0])
        if n <= first:
            assert int(nan["n_acc"][b, 0]) == n and np.array_equal(nan["tok"][b], clean["tok"][b]), (b, first, n)
            decided_before += first < gamma
        else:
            assert int(nan["n_acc"][b, 0]) > first
    print(group, "rows with X in the window that were decided before it:", decided_before, flush=True)
    assert decided_before >= 2


@pytest.mark.parametrize("B, lo, hi", [(300, 1, 4), (16, 6, 9), (96, 9, 9), (1, 2, 2)])
def test_prefill_of_short_prompts(B, lo, hi):
    """Few cached positions per row, which the attention of short runs takes (up to 7 in the mean, or below 2 in large batches), and
    8 of them, which is the first mean the kernel for long runs gets; rows without any among them."""
    draft = W.ModelCfg(W.ARCH_LLAMA, 2, 256, 4, 2, 136, 83, 48, 1e-5, 10000.0)
    target = _llama(2, 512, 4, 1, 136, 83)
    _check(draft, target, B, W.DT_BF16, prompt_len=hi, prompt_len_min=lo, tau=1.5, n_gen=2, whole_prompt=True, seed=61)


EPI_F32, EPI_GELU, EPI_SWIGLU, EPI_PART = 0, 2, 3, 4


def _host(name, *args):
    """An internal host function of the library (a launcher's rule), by its mangled name."""
    from paper_2502_04557_amd import binding
    return binding.load_library()[name](*args)


def _takes_tile(epi, N, rows):
    return bool(_host("_ZN8sprinter15gemm_takes_tileEiii", epi, N, rows) & 1)


def _tiles(m, rows):
    """What the launcher picks for the four products of a layer at `rows` rows: the tile (0: 256 x 256, 1: 128 x 128, 2: 64 x 128, 3: 64 x 64,
    4: 32 x 64) and, of partial products, the K shares.  A few rows of a fused pass are not meant."""
    up = EPI_GELU if m.arch == W.ARCH_GPT else EPI_SWIGLU
    pick = lambda *a: divmod(_host("_ZN8sprinter16gemm_tile_choiceEiiiii", *a), 16)
    return dict(qkv=pick(EPI_F32, rows, m.d_qkv, m.d_model, 1)[0], o=pick(EPI_PART, rows, m.d_model, m.d_model, 8),
                up=pick(up, rows, m.d_ff, m.d_model, 1)[0], down=pick(EPI_PART, rows, m.d_model, m.d_ff, 8))


def _g(d, ff):
    return W.ModelCfg(W.ARCH_GPT, 2, d, d // 64, d // 64, ff, 83, 320)


def _l(dh, H, KVH, ff):
    return W.ModelCfg(W.ARCH_LLAMA, 2, dh * H, H, KVH, ff, 83, 320, 1e-5, 10000.0)


@pytest.mark.parametrize("B, P, draft, target, draft_tiles, target_tiles", [
    (8, 258, _g(256, 712), _l(128, 16, 8, 72), dict(qkv=2, o=(3, 1), up=2, down=(2, 3)), dict(qkv=0, o=(0, 2), up=4, down=(3, 1))),
    (8, 258, _g(192, 8200), _l(64, 8, 1, 136), dict(qkv=2, o=(4, 1), up=1, down=(1, 7)), dict(qkv=2, o=(2, 1), up=3, down=(2, 1))),
    (8, 162, _g(128, 264), _l(128, 16, 2, 72), dict(up=4), dict(qkv=1, o=(1, 1))),
    (3, 258, _g(768, 3080), _l(64, 12, 12, 5128), dict(), dict(o=(2, 3), up=0, down=(2, 6))),
    (7, 148, _l(64, 8, 4, 72), _g(768, 8200), dict(), dict(qkv=2, o=(3, 1), up=0, down=(1, 4))),
    (9, 59, _g(128, 136), _l(64, 8, 4, 72), dict(), dict(qkv=3, o=(3, 3), up=4, down=(4, 1))),
    (6, 12, _l(64, 2, 1, 8200), _l(128, 12, 12, 8200), dict(up=2, down=(4, 8)), dict(up=1, o=(4, 3), down=(3, 5))),
    (5, 8, _g(128, 8200), _l(64, 2, 2, 136), dict(up=3, down=(4, 8)), dict()),
])
def test_every_tile_with_every_epilogue(B, P, draft, target, draft_tiles, target_tiles):
    """Prefill passes of 35 - 2056 rows that are picked for each of the five tiles with each epilogue (float32, GELU, gate + up, partial
    products in one and in several shares), a few rows beyond a tile's multiple, with odd and even numbers of k tiles, a last one that is
    not full, and column tiles beyond the last one."""
    rows = B * (P - 1)
    for m, want in ((draft, draft_tiles), (target, target_tiles)):
        got = _tiles(m, rows)
        assert want == {k: got[k] for k in want}, got
        if rows <= 64 and "up" in want:
            assert _takes_tile(EPI_GELU if m.arch == W.ARCH_GPT else EPI_SWIGLU, m.d_ff, rows)
    _check(draft, target, B, W.DT_BF16, prompt_len=P, prompt_len_min=0, n_gen=2, tau=1.5, max_seq=-(-(P + 4) // 32) * 32, whole_prompt=True, seed=71)


@pytest.mark.parametrize("target", [_l(64, 33, 33, 776), _g(2176, 776)])
def test_large_tile_adds_itself(target):
    """4080 rows of O-proj and FFN-down on the 256 x 256 tile in one K share, which adds the product (GPT: and the bias) to the residual rows:
    255 row tiles (the last tile of 256 rows is not full), column tiles beyond the last one, odd and even numbers of k tiles (25, 66, 68)."""
    rows = 16 * 255
    got = _tiles(target, rows)
    assert got["o"] == got["down"] == (0, 1), got
    _check(_g(128, 136), target, 16, W.DT_BF16, prompt_len=256, prompt_len_min=0, n_gen=2, tau=1.5, max_seq=288, whole_prompt=True, seed=75)


@pytest.mark.parametrize("target", [_l(64, 32, 32, 3064), _g(2048, 5896)])
def test_last_round_in_halves(target):
    """4080 rows of products whose 16 x 24 tiles of 256 x 256 fill the compute units once and half of them again: the rest goes out in halves
    (QKV with and without bias, gate + up) or, of the eight waves of GELU, in a second round; a last column tile that is not full (3064, 5896)."""
    rows = 16 * 255
    got = _tiles(target, rows)
    for k, cols in (("qkv", target.d_qkv), ("up", target.d_ff * (2 if target.arch == W.ARCH_LLAMA else 1))):
        assert got[k] == 0 and 0 < 16 * -(-cols // 256) - 256 <= 128, (k, got)
    _check(_g(128, 136), target, 16, W.DT_BF16, prompt_len=256, prompt_len_min=0, n_gen=2, tau=1.5, max_seq=288, whole_prompt=True, seed=76)


@pytest.mark.parametrize("B", [17, 33, 64])
@pytest.mark.parametrize("gelu, gate_up", [(4096, 4096), (4104, 4104), (8192, 72), (8200, 72)])
def test_either_side_of_the_wide_product_rules(B, gelu, gate_up):
    """17 - 64 rows, 2 - 4 row tiles: FFN-up on the K-split kernel with one column tile per wave (256 tiles) and with two (257 and 512), and
    just beyond on the LDS tiles; gate + up likewise (256 and 257 tiles)."""
    assert [_takes_tile(EPI_GELU, n, B) for n in (4096, 4104, 8192, 8200)] == [False, False, False, True]
    assert [_takes_tile(EPI_SWIGLU, n, B) for n in (4096, 4104)] == [False, True]
    _check(_gpt(1, 128, gelu, 83), _llama(1, 192, 3, 3, gate_up, 83), B, W.DT_BF16, tau=1.5, prompt_len=3, n_gen=2, seed=81)


@pytest.mark.parametrize("H, KVH, B, longest, split", [(8, 8, 16, 1100, 2), (8, 8, 10, 1300, 3), (8, 4, 16, 1150, 4), (8, 8, 6, 1400, 5),
                                                       (16, 2, 21, 1600, 6), (8, 4, 9, 1850, 7), (8, 1, 3, 2100, 8)])
def test_keys_shared_in_several_steps(H, KVH, B, longest, split):
    """Every split of a row's keys over 2 - 8 workgroups, the longest rows in more than one step per workgroup; 1 - 8 query heads per KV
    head; shorter rows leave some workgroups without keys."""
    dh = 64 if split == 6 else 128
    for ctx in (longest, longest + 2):
        assert _host("_ZN8sprinter10attn_splitEiiii", dh, KVH, B, ctx) == split
    assert longest > 256 * split                             # (8 waves of 32 keys per workgroup and step)
    draft = W.ModelCfg(W.ARCH_LLAMA, 1, 128, 2, 2, 72, 83, 2200, 1e-5, 10000.0)
    target = W.ModelCfg(W.ARCH_LLAMA, 1, dh * H, H, KVH, 72, 83, 2200, 1e-5, 10000.0)
    _check(draft, target, B, W.DT_BF16, prompt_len=longest, prompt_len_min=40, tau=1.5, n_gen=2, max_seq=-(-(longest + 4) // 32) * 32,
           whole_prompt=True, seed=90 + split)
