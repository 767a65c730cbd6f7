"""The many-row prompt pass (bf16 storage, prompts of more than two nine-row passes)
against the oracle: first token, then draft and target logits of steps that read
every key, value and drafter-history row the pass wrote.

Sizes are those at which it can go wrong: prompts that end inside, at and just past a
16-position part, the context's last position, one to many slots (three and two
operand planes, one or two parts per attention block, several passes), 64- and
128-column product tiles, k-splits of one, two and four, frame counts that end
inside a 32-frame step.  Tolerances are the repository's: both sides keep their
caches in bf16 and compute in fp32, and the bar is above the differences seen (at most
8e-3) and below those of one wrong token of the prompt (target logits 20 bars and more,
among 230 tokens five; the drafter's a third of that).
"""
import numpy as np
import pytest
import torch

from wf_fixtures import MICRO, make_weights, make_memory, make_prefix
from oracle import OracleOpts, Session

pytestmark = pytest.mark.gpu

TOL_MICRO, TOL = 1e-3, 2e-2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(cfg, lens, tol, std=0.02, check=None, steps=2):
    from lockstep import Lockstep
    W = make_weights(cfg, std=std)
    prompts = [make_prefix(cfg, i, n) for i, n in enumerate(lens)]
    ls = Lockstep(cfg, W, prompts, [cfg.n_ctx] * len(lens), tol, check=check,
                  opts=OracleOpts(dtype=np.float32, kv_bf16=True))
    for _ in range(steps):
        ls.step()
    print(f"{cfg.name} x{len(lens)}: max |dlogit| draft {ls.max_dlogit:.2e} target {ls.max_tlogit:.2e}, "
          f"near ties {ls.near_ties}")
    return ls


@pytest.mark.parametrize("lens", [[19], [31], [32], [33], [64 - 9], [19, 48, 5], [32, 1, 33, 17, 55]])
def test_part_edges(lens):
    cfg = MICRO.with_(name="micro-bf16-pre", dtype="bf16", n_vocab=501, n_frames=45)
    _run(cfg, lens, TOL_MICRO).close()


@pytest.mark.parametrize("n_frames,flags", [(31, {}), (33, {"draft_history": False}), (300, {"draft_pos": "abs"}),
                                            (300, {"draft_audio": False})])
def test_frames_and_variants(n_frames, flags):
    cfg = MICRO.with_(name="micro-bf16-pre", dtype="bf16", n_vocab=501, n_frames=n_frames, **flags)
    _run(cfg, [40, 23], TOL_MICRO).close()


def test_prompt_fills_the_context():
    """A prompt of n_ctx - 1 tokens leaves one position: its step verifies the anchor."""
    cfg = MICRO.with_(name="micro-bf16-pre", dtype="bf16", n_vocab=501)
    for lens in ([63], [63, 64]):
        ls = _run(cfg, lens, TOL_MICRO, steps=1)
        assert ls.eng.state()[:len(lens), 4].cpu().tolist() == [1] * len(lens)
        ls.close()


@pytest.mark.parametrize("d_model,batch,lens", [(512, 12, (50, 64)), (512, 20, (40, 64)), (768, 40, (33, 64))])
def test_many_slots(d_model, batch, lens):
    """One and two parts per attention block, groups that end inside a slot, several
    passes (40 slots of up to four parts: 2560 rows in two)."""
    cfg = MICRO.with_(name=f"w{d_model}-pre", dtype="bf16", n_layer=2, d_model=d_model, n_head=d_model // 64,
                      d_ff=4 * d_model, n_vocab=501, taps=(0, 1), n_ctx=64, n_frames=70)
    ls_ = [lens[0] + (7 * i) % (lens[1] - lens[0] - 8) for i in range(batch)]
    _run(cfg, ls_, TOL, std=0.05, check=[0, 1, batch // 2, batch - 1], steps=1).close()


@pytest.mark.parametrize("length", [150, 230, 430])
def test_width_1280_tiles(length):
    """One slot at width 1280: 64 x 64 and 64 x 128 tiles of the three-plane products,
    k-splits of one, two and four."""
    cfg = MICRO.with_(name="w1280-pre", dtype="bf16", n_layer=2, d_model=1280, n_head=20, d_ff=5120, n_vocab=501,
                      taps=(0, 1), n_ctx=448, n_frames=130)
    _run(cfg, [length], TOL, steps=1).close()


def test_refill_leaves_other_slots():
    """A slot prefilled again in a running batch: its neighbours' caches stay theirs."""
    cfg = MICRO.with_(name="micro-bf16-pre", dtype="bf16", n_vocab=501)
    ls = _run(cfg, [30, 41, 25], TOL_MICRO)
    prompt = make_prefix(cfg, 9, 37)
    ls.eng.prefill(1, torch.from_numpy(prompt[None].copy()).cuda(), [37], [cfg.n_ctx])
    ls.sess[1] = Session(ls.T, ls.D, make_memory(cfg, 1), prompt, cfg.n_ctx)
    for _ in range(2):
        ls.step()
    ls.close()


@pytest.mark.parametrize("lens", [[9], [40], [40, 23]])
def test_profile_names_the_prompt_pass(lens):
    """A profiled prompt call times every product, attention and LayerNorm launch, in the
    nine-row passes (9 tokens) as in the many-row one."""
    cfg = MICRO.with_(name="micro-bf16-pre", dtype="bf16", n_vocab=501)
    ls = _run(cfg, lens, TOL_MICRO, steps=0)
    prompt = np.stack([np.resize(make_prefix(cfg, i, n), max(lens)) for i, n in enumerate(lens)])
    ls.eng.profile(True)
    ls.eng.prefill(0, torch.from_numpy(prompt).cuda(), lens, [cfg.n_ctx] * len(lens))
    prof = ls.eng.profile_summary()
    ls.eng.profile(False)
    ls.close()
    L, D = cfg.n_layer, cfg.n_draft_layer
    want = {"gemv_qkv": L, "attn_self": L, "gemv_q2": L, "attn_cross": L, "gemv_fc1": L, "gemv_fc2": L, "gemv_hproj": 1,
            "gemv_hist_kv": D, "head": 1}
    if lens != [9]:
        want |= {"gemv_o": 2 * L, "reduce_ln": 3 * L + 1, "layernorm": 1 + D - 1}
    for role, n in want.items():
        assert prof.get(role, {}).get("launches", 0) >= n and prof[role]["exec_ms"] > 0, (role, prof.get(role))
        if lens != [9] and role not in ("layernorm", "attn_cross"):
            assert prof[role]["launches"] == n, (role, prof[role])


@pytest.mark.parametrize("batch,without", [(1, 8176896), (3, 9789696)])
def test_workspace_without_the_prompt_pass(batch, without, monkeypatch):
    """A workspace that lacks only the many-row pass's buffers (its size before there was
    one) is accepted and runs prompts nine positions per pass; one byte less is not."""
    import ctypes
    from paper_2609_32869_amd import WfError, binding, load_library
    lib = load_library()

    class Library:
        size = without

        def __getattr__(self, name):
            return getattr(lib, name)

        def wf_workspace_bytes(self, cfg, out):
            assert lib.wf_workspace_bytes(cfg, out) == 0
            out._obj.value = min(out._obj.value, self.size)
            return 0

    cfg = MICRO.with_(dtype="bf16")
    full = ctypes.c_size_t()
    ccfg = binding.make_config(cfg, batch)
    assert lib.wf_workspace_bytes(ctypes.byref(ccfg), ctypes.byref(full)) == 0 and full.value > without
    small = Library()
    monkeypatch.setattr(binding, "load_library", lambda: small)
    ls = _run(cfg, [40, 23, 31][:batch], TOL_MICRO)
    ls.close()
    small.size = without - 1
    with pytest.raises(WfError, match="workspace too small"):
        binding.WhisperFlash(cfg, batch, [torch.zeros(1, device="cuda")] * len(make_weights(cfg).order))
