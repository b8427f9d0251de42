"""CPU-only checks of the boundary: the shared library loads, exports every
symbol the header declares, and validates configurations without a GPU."""
import ctypes as C
import os
import re
import pytest
import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2502_04557_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build_library(verbose=False)
    return binding.load_library()


def test_exports_every_declared_symbol(lib):
    hdr = open(os.path.join(ROOT, "include", "sprinter.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(sprinter_[a-z_]+)\s*\(", hdr))
    assert {"sprinter_load_weights", "sprinter_prefill", "sprinter_step", "sprinter_generate"} <= declared
    from paper_2502_04557_amd import binding
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name


@pytest.mark.parametrize("dh, H, KVH, lens, shared", [
    # measured: one wave / four waves sharing, us
    (128, 32, 8, [511] * 8, True),                 # 73.4 / 65.7
    (128, 32, 8, [999] * 4, True),                 # 110 / 89
    (128, 16, 8, [1499] * 3, True),                # 101 / 80
    (128, 16, 8, [999] * 4, True),                 # 73 / 65
    (64, 32, 8, [1999] * 2, True),                 # (four of 1500 - 2000: 97 / 88)
    (128, 16, 2, [299], False),                    # 16.8 / 18.3: too few waves
    (128, 16, 2, [255] * 2, False),                # 14.4 / 16.1
    (64, 8, 1, [999] * 2, False),                  # 30.8 / 33.1
    (64, 8, 1, [511] * 4, False),                  # 17.7 / 18.8
    (64, 32, 8, [767] * 6, False),                 # 57 / 62: short keys
    (64, 12, 6, [1030] + [10] * 100, False),       # 32 / 41: one long prompt among short ones
    (128, 16, 8, [1030] + [10] * 100, False),      # 51 / 58
    (128, 16, 8, [1030] + [9] * 300, False),       # 60 / 70
    (128, 16, 8, [199] * 20, False),               # 28 / 30
    (128, 32, 32, [999] * 4, False),               # no grouped queries
])
def test_shared_prefill_attention_only_where_it_is_ahead(lib, dh, H, KVH, lens, shared):
    """Which attention kernel a prefill pass takes, at measured points on either side (lens: cached positions per row, one pass)."""
    rule = lib["_ZN8sprinter11attn_sharedEiiiiii"]
    assert bool(rule(dh, H, KVH, sum(lens), max(lens) + 1, sum(lens) // len(lens)) & 1) == shared


def test_struct_layout_matches_header():
    from paper_2502_04557_amd import binding
    assert C.sizeof(binding.ModelCfgC) == 40
    assert C.sizeof(binding.CfgC) == 2 * 40 + 5 * 4 + 2 * 4 + 8 + 4 * 4 + 4   # incl. 4 bytes padding before seed
    assert binding.CfgC.seed.offset % 8 == 0
    assert C.sizeof(binding.StepOutC) == 10 * 8 and C.sizeof(binding.StatsC) == 32


def _ws(lib, cfg):
    from paper_2502_04557_amd import binding
    c = binding.cfg_to_c(cfg)
    n = C.c_size_t(0)
    rc = lib.sprinter_workspace_bytes(C.byref(c), C.byref(n))
    return rc, n.value, lib.sprinter_last_error(None).decode()


def test_workspace_sizes_cover_kv_caches(lib):
    for name in W.CONFIG_NAMES:
        cfg = W.config(name)
        rc, n, _ = _ws(lib, cfg)
        assert rc == 0
        es = 4 if cfg.dtype == W.DT_F32 else 2
        kv = sum(2 * m.n_layer * cfg.max_batch * m.n_kv_head * cfg.max_seq * m.d_head * es
                 for m in (cfg.draft, cfg.target))
        assert n > kv and n < kv + 40e9


def test_config_validation(lib):
    from dataclasses import replace
    base = W.mini_config("gpt", W.DT_BF16)
    cases = [
        (replace(base, draft=replace(base.draft, d_model=200)), "not divisible"),
        (replace(base, draft=replace(base.draft, n_head=2)), "head dimension"),           # 96
        (replace(base, target=replace(base.target, vocab=999)), "vocabular"),
        (replace(base, max_batch=0), "max_batch"),
        (replace(base, max_batch=2000), "max_batch"),
        (replace(base, max_seq=4096), "max_pos"),
        (replace(base, dtype=7), "dtype"),
        (replace(base, target_ctx_mode=2), "target_ctx_mode"),
        (replace(base, reject_mode=2), "reject_mode"),
        (replace(base, sd_gamma=17), "sd_gamma"),
        (replace(base, sd_gamma=-1), "sd_gamma"),
        (replace(base, chunk_rows=100), "chunk_rows"),
        (replace(base, chunk_rows=8192), "chunk_rows"),
        (replace(base, reject_mode=1, temperature=0.0), "temperature"),
        (replace(base, temperature=-1.0), "temperature"),
        (replace(base, draft=replace(base.draft, arch=5)), "arch"),
        (replace(base, draft=replace(base.draft, d_ff=643)), "multiples of 8"),
    ]
    for cfg, word in cases:
        rc, _, msg = _ws(lib, cfg)
        assert rc == -2 and word in msg, (rc, msg, word)
    from paper_2502_04557_amd import binding
    c = binding.cfg_to_c(base)
    c.ver_d_in = 100
    n = C.c_size_t(0)
    assert lib.sprinter_workspace_bytes(C.byref(c), C.byref(n)) == -2
    assert lib.sprinter_workspace_bytes(None, C.byref(n)) == -1
    # no GPU work is needed to refuse a NULL context
    assert lib.sprinter_step(None, None) == -1
    assert lib.sprinter_generate(None, 4, None, None, None, None) == -1
    assert lib.sprinter_prefill(None, None, None, 1, 1) == -1
    assert lib.sprinter_sd_generate(None, 2, 1, None, 0, None, None, None) == -1


def test_create_static_rejects_what_does_not_fit(lib):
    """The size check of sprinter_create_static comes before any device call, so it can be forced here."""
    from paper_2502_04557_amd import binding
    hdr = open(os.path.join(ROOT, "include", "sprinter.h")).read()
    limit = int(re.search(r"SPRINTER_STATIC_WORKSPACE_BYTES \(\(size_t\)(\d+) << 20\)", hdr).group(1)) << 20
    cfg = W.config("c2")
    rc, need, _ = _ws(lib, cfg)
    assert rc == 0 and need > limit
    ctx = C.c_void_p(None)
    c = binding.cfg_to_c(cfg)
    rc = lib.sprinter_create_static(C.byref(c), None, C.byref(ctx))
    msg = lib.sprinter_last_error(None).decode()
    assert rc == -3 and not ctx.value
    assert str(need) in msg and str(limit) in msg
    assert lib.sprinter_create_static(None, None, C.byref(ctx)) == -1
    assert lib.sprinter_create_static(C.byref(c), None, None) == -1


@pytest.mark.parametrize("dtype", [W.DT_F32, W.DT_BF16])
@pytest.mark.parametrize("kind", ["gpt", "llama"])
def test_workspace_grows_with_max_seq_by_the_caches_alone(lib, kind, dtype):
    """A longer max_seq costs the KV caches and the token history of its positions and nothing else: 256-byte alignment of the
    one buffer that is no multiple of it is all the slack there is."""
    from dataclasses import replace
    base = W.mini_config(kind, dtype, max_batch=4)
    base = replace(base, draft=replace(base.draft, max_pos=4096), target=replace(base.target, max_pos=4096))
    es = 4 if dtype == W.DT_F32 else 2
    per_pos = 4 * base.max_batch + sum(2 * m.n_layer * base.max_batch * m.n_kv_head * m.d_head * es for m in (base.draft, base.target))
    short, long = (_ws(lib, replace(base, max_seq=s)) for s in (64, 1024))
    assert short[0] == 0 and long[0] == 0
    assert abs((long[1] - short[1]) - (1024 - 64) * per_pos) <= 256


def test_long_caches_of_a_small_pair_fit_the_static_workspace(lib):
    """60000 positions of a one-layer pair with one KV head of 64 columns: 2 x 15 MB of caches."""
    m = W.ModelCfg(W.ARCH_LLAMA, 1, 256, 4, 1, 512, 1000, 60000, 1e-5, 10000.0)
    rc, need, _ = _ws(lib, W.SprinterCfg(m, m, 32, W.DT_BF16, 1, 60000, chunk_rows=64))
    assert rc == 0 and need <= 40 << 20


@pytest.mark.parametrize("dh,G,longest", [(64, 1, 15936), (64, 2, 7808), (64, 4, 3744), (64, 8, 1712), (128, 1, 15488), (128, 2, 7424), (128, 4, 3392), (128, 8, 1376)])
def test_longest_context_of_float32_mode(lib, dh, G, longest):
    """The lengths that float32 mode takes, as the header gives them; bf16 mode has no such limit."""
    m = W.ModelCfg(W.ARCH_LLAMA, 1, 8 * dh, 8, 8 // G, 512, 1000, 16384, 1e-5, 10000.0)
    for dtype, seq, rc in ((W.DT_F32, longest, 0), (W.DT_F32, longest + 1, -2), (W.DT_BF16, longest + 1, 0)):
        got, _, msg = _ws(lib, W.SprinterCfg(m, m, 32, dtype, 1, seq, chunk_rows=64))
        assert got == rc and (rc == 0 or f"up to {longest} " in msg), (dtype, seq, msg)
