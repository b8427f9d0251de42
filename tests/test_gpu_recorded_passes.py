"""Passes that come again and again, through 12 layers: a context on the caller's workspace and one on the library's static workspace must
give the same tokens, flags and scores, bit for bit, over repeated calls with eager work in between (a step that exports logits, a new
prefill with another batch, new weights, contexts that grow past the length at which the attention's launches change); and none of it
takes device memory, as recording such passes in graphs did (2 MB each)."""
from dataclasses import replace
import numpy as np
import pytest
import workloads as W

pytestmark = pytest.mark.gpu


def _cfg(dtype, **over):
    base = W.mini_config("linear", dtype)                 # (GPT draft of 2 heads, LLaMA target with grouped queries; fits the static workspace)
    deep = lambda m: replace(m, n_layer=12, max_pos=560)
    return replace(base, draft=deep(base.draft), target=deep(base.target), max_seq=560, max_batch=3, batch=3, prompt_len=500, prompt_len_min=480,
                   chunk_rows=64 if dtype == W.DT_BF16 else 0, **over)


def _widen(vw):
    # spread the verifier's scores so that both branches (and the target pass, with any number of rows) occur
    return {k: (v * 40 if k.endswith(("w1", "w2")) else v) for k, v in vw.items()}


def _run(cfg, static):
    from paper_2502_04557_amd import binding
    s, outs = binding.Sprinter(cfg, "cuda:0", static_workspace=static), []
    keep = lambda o: outs.append({k: v.cpu().numpy() for k, v in o.items()})
    try:
        for seed in (0, 1):                               # other weights the second time
            dw, tw, vw = W.make_weights(replace(cfg, weight_seed=77 + seed))
            for which, w in zip((binding.DRAFT, binding.TARGET, binding.VERIFIER), (dw, tw, _widen(vw))):
                s.load_weights(which, w)
            prompts, plen = W.make_prompts(cfg)
            for rows in (3, 2):
                s.prefill(prompts[:rows], plen[:rows])
                if cfg.sd_gamma:
                    for _ in range(3):
                        keep(s.sd_generate(cfg.sd_gamma, 4))
                else:
                    keep(s.generate(24))                  # (the rows pass 512 cached positions on the way)
                    keep(s.step(debug=cfg.target_ctx_mode == 0))
                    keep(s.generate(12))
                    keep(s.step())
    finally:
        s.close()
    return outs


@pytest.mark.parametrize("dtype", [W.DT_BF16, W.DT_F32])
@pytest.mark.parametrize("over", [dict(), dict(target_ctx_mode=W.CTX_FULL_PREFIX, reject_mode=W.REJECT_SD), dict(sd_gamma=2)], ids=["steps", "full_prefix", "rounds"])
def test_recorded_passes_match_launches(dtype, over):
    cfg = _cfg(dtype, **over)
    ref, got = _run(cfg, static=True), _run(cfg, static=False)
    assert len(ref) == len(got)
    for i, (a, b) in enumerate(zip(ref, got)):
        assert a.keys() == b.keys()
        for k in a:
            assert np.array_equal(a[k], b[k]), (i, k)
    if not cfg.sd_gamma:
        acc = np.concatenate([o["accept"].ravel() for o in got])
        assert 0 < acc.mean() < 1


def test_generate_takes_no_device_memory():
    """The workspace is all the device memory a context uses, however often the same pass comes."""
    import torch
    from paper_2502_04557_amd import binding
    cfg = _cfg(W.DT_BF16)
    _run(cfg, static=True)                                # (kernels are loaded at their first launch)
    dw, tw, vw = W.make_weights(cfg)
    prompts, plen = W.make_prompts(cfg)
    s = binding.Sprinter(cfg, "cuda:0")
    try:
        for which, w in zip((binding.DRAFT, binding.TARGET, binding.VERIFIER), (dw, tw, _widen(vw))):
            s.load_weights(which, w)
        s.prefill(prompts, plen)
        s.generate(1)
        left = lambda: (torch.cuda.synchronize(), torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved())[1]   # (what torch holds does not count)
        before = left()
        for _ in range(36):
            s.generate(1)
        assert left() >= before
    finally:
        s.close()
