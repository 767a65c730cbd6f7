"""Parity of the HIP path (called through the C ABI) with the oracle.

Bar: token ids and accepted lengths identical wherever the oracle's top-2
margin exceeds the logit tolerance; logits within max |delta| <= 2e-2 for bf16
storage (bf16 caches against fp32 oracle arithmetic on the same bf16
weights) and <= 1e-3 for fp32 storage.
"""
import numpy as np
import pytest
import torch

from wf_fixtures import MICRO, TINY, LARGE_V3, make_weights, make_memory, make_prefix, make_prefix_lengths, plant_drafts
from oracle import OracleOpts, Target, plain_greedy

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-3
TOL_BF16 = 2e-2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _planted(ls, refs, rng):
    K = ls.cfg.block_k
    ov = np.zeros((ls.n, K), np.int32)
    for i, s in enumerate(ls.sess):
        cont = (list(refs[i]) + [0] * (K + 1))[s.emitted:s.emitted + K]
        ov[i] = plant_drafts(cont, int(rng.integers(0, K + 1)), ls.cfg.n_vocab, rng)
    return ov


def test_micro_lockstep_natural_and_planted():
    from lockstep import Lockstep
    cfg = MICRO
    W = make_weights(cfg)
    prompts = [make_prefix(cfg, 0, 5), make_prefix(cfg, 1, 13), make_prefix(cfg, 2, 27)]
    max_new = [30, 12, 40]
    ls = Lockstep(cfg, W, prompts, max_new, TOL_F32)
    for _ in range(3):
        ls.step()
    T = Target(cfg, W.values, OracleOpts())
    refs = [plain_greedy(T, make_memory(cfg, i), prompts[i], max_new[i]) for i in range(3)]
    rng = np.random.default_rng(0)
    for _ in range(12):
        ls.step(override=_planted(ls, refs, rng))
    # the whole transcript equals plain greedy decoding
    for i, s in enumerate(ls.sess):
        if ls.live[i]:
            assert s.out == refs[i][:len(s.out)]
    assert max(ls.accepted) > 0
    ls.close()


def test_micro_k_max_and_budget_edges():
    from lockstep import Lockstep
    cfg = MICRO
    W = make_weights(cfg)
    # prompt ending near the context limit: budget caps k at n_ctx - L - 1
    prompts = [make_prefix(cfg, 3, cfg.n_ctx - 6), make_prefix(cfg, 4, 1)]
    ls = Lockstep(cfg, W, prompts, [100, 3], TOL_F32)
    T = Target(cfg, W.values, OracleOpts())
    refs = [plain_greedy(T, make_memory(cfg, i), prompts[i], m) for i, m in enumerate([100, 3])]
    rng = np.random.default_rng(1)
    for k_max in (0, 3, 8, 8, 8, 8):
        ls.step(k_max=k_max, override=_planted(ls, refs, rng))
    for i, s in enumerate(ls.sess):
        assert s.done
    ls.close()


def test_tiny_greedy_64_tokens_equal_plain_greedy():
    """Tiny Whisper-shaped decoder, fp32 weights, prefix 32, 64 greedy tokens."""
    from lockstep import Lockstep
    cfg = TINY
    W = make_weights(cfg)
    prompt = make_prefix(cfg, 0, 32)
    ls = Lockstep(cfg, W, [prompt], [64], TOL_F32)
    T = Target(cfg, W.values, OracleOpts())
    ref = plain_greedy(T, make_memory(cfg, 0), prompt, 64)
    rng = np.random.default_rng(2)
    n = 0
    while not ls.sess[0].done and n < 70:
        ov = _planted(ls, [ref], rng) if n % 2 else None
        ls.step(override=ov)
        n += 1
    assert ls.live[0], ls.near_ties
    assert ls.sess[0].out == ref
    ls.close()


# bf16 storage at micro scale with a ragged vocabulary (501: a partial last column
# tile of the head) and a ragged frame count (45: a partial last key octet).
MICRO_BF16 = MICRO.with_(name="micro-bf16", dtype="bf16", n_vocab=501, n_frames=45)
TOL_MICRO_BF16 = 2e-3


def _run_planted(ls, refs, rng, steps, natural_every=3):
    for n in range(steps):
        ls.step(override=None if n % natural_every == 0 else _planted(ls, refs, rng))


def test_micro_bf16_b1_split_operands():
    """Batch 1, bf16: operands split into three bf16 terms (fp32-exact products)."""
    from lockstep import Lockstep
    cfg = MICRO_BF16
    W = make_weights(cfg)
    prompts = [make_prefix(cfg, 0, 11)]
    ls = Lockstep(cfg, W, prompts, [48], TOL_MICRO_BF16)
    opts = OracleOpts(dtype=np.float32, kv_bf16=True)
    T = Target(cfg, W.values, opts)
    refs = [plain_greedy(T, make_memory(cfg, 0), prompts[0], 48)]
    _run_planted(ls, refs, np.random.default_rng(5), 12)
    print(f"micro-bf16 b1: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, near ties {ls.near_ties}")
    assert ls.steps == 12
    ls.close()


@pytest.mark.parametrize("d_model,batch", [(512, 1), (768, 1), (512, 3), (768, 3)])
def test_bf16_other_widths(d_model, batch):
    """bf16 at Whisper base and small widths (8 and 12 heads), 2003-token
    vocabulary (a ragged last head tile) and 700 frames.  One slot: the folded
    LayerNorm over 64 or 96 eight-column items per row, output-product column
    groups of 64 or 96, sixteen k-splits of the second MLP product (one k-step
    per wave), a 32-column head, five 128-frame chunks and a ragged 60; every
    block is tapped, so each block's tap reaches the drafter through the next
    block's query product and the last block's through the reduction kernel.
    Three slots: two-plane operands over one 64-row block, the k-split residual
    products, a 512-frame chunk and a ragged 188 merged.  Weights at std 0.05,
    under which the greedy continuation varies (35-49 distinct tokens of 60)
    rather than repeating one token."""
    from lockstep import Lockstep
    cfg = MICRO.with_(name=f"w{d_model}-bf16", dtype="bf16", n_layer=3, d_model=d_model, n_head=d_model // 64,
                      d_ff=4 * d_model, n_vocab=2003, taps=(0, 1, 2), n_ctx=128, n_frames=700)
    W = make_weights(cfg, std=0.05)
    lens, max_new = [23, 7, 40][:batch], [60, 20, 45][:batch]
    prompts = [make_prefix(cfg, i, n) for i, n in enumerate(lens)]
    ls = Lockstep(cfg, W, prompts, max_new, TOL_BF16)
    T = Target(cfg, W.values, OracleOpts(dtype=np.float32, kv_bf16=True))
    refs = [plain_greedy(T, make_memory(cfg, i), prompts[i], max_new[i]) for i in range(batch)]
    _run_planted(ls, refs, np.random.default_rng(9), 12)
    print(f"{cfg.name} b{batch}: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, "
          f"near ties {ls.near_ties}")
    assert ls.steps == 12
    assert max(ls.accepted) > 0
    ls.close()


def test_micro_bf16_b1_offset_residual():
    """Batch 1, bf16, with a residual stream whose mean (about 4, from a shifted
    output bias of the first block) is tens of times its spread.  At batch 1 a
    LayerNorm feeding a product is applied after it, r((x*g)W^T - m gW^T) + bW^T,
    and the two terms nearly cancel for such rows; the logits must still agree
    with the fp32 oracle to the bf16 tolerance (LayerNorm itself is shift
    invariant, so the oracle's rows are well conditioned)."""
    from lockstep import Lockstep
    from wf_fixtures.gen import _round_inplace
    cfg = MICRO_BF16
    W = make_weights(cfg)
    b = W.values["t0.attn.o.b"]
    b += 4.0
    _round_inplace(b.reshape(-1))
    prompts = [make_prefix(cfg, 0, 11)]
    ls = Lockstep(cfg, W, prompts, [40], TOL_MICRO_BF16)
    opts = OracleOpts(dtype=np.float32, kv_bf16=True)
    T = Target(cfg, W.values, opts)
    refs = [plain_greedy(T, make_memory(cfg, 0), prompts[0], 40)]
    _run_planted(ls, refs, np.random.default_rng(6), 8)
    print(f"micro-bf16 b1 offset: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, near ties {ls.near_ties}")
    assert ls.steps == 8
    ls.close()


def test_micro_bf16_b3_two_plane_operands():
    """Batch 3, bf16: each operand value as two bf16 planes (hi + lo), products
    accurate to fp32 rounding; compared with the plain fp32 oracle."""
    from lockstep import Lockstep
    cfg = MICRO_BF16
    W = make_weights(cfg)
    prompts = [make_prefix(cfg, 0, 4), make_prefix(cfg, 1, 20), make_prefix(cfg, 2, 9)]
    max_new = [40, 9, 30]
    opts = OracleOpts(dtype=np.float32, kv_bf16=True)
    ls = Lockstep(cfg, W, prompts, max_new, TOL_MICRO_BF16, opts=opts)
    T = Target(cfg, W.values, opts)
    refs = [plain_greedy(T, make_memory(cfg, i), prompts[i], max_new[i]) for i in range(3)]
    _run_planted(ls, refs, np.random.default_rng(6), 10)
    print(f"micro-bf16 b3: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, near ties {ls.near_ties}")
    ls.close()


@pytest.mark.timeout(900)
def test_micro_bf16_b64_wide_tiles():
    """64 slots (576 rows, nine 64-row blocks), bf16, d 1024 (16 heads), FFN 2560:
    the q|k|v (3072 columns, k/v appended to the paged cache), first MLP (2560
    columns, GELU into the next operand) and drafter q|k|v products on 64 x 64 tiles
    whose waves split k (operand rows read from 16x32 fragment order), the row blocks
    in one part or two over the XCDs; ragged prompts, planted drafts on six followed
    slots."""
    from lockstep import Lockstep
    cfg = MICRO_BF16.with_(name="micro-wide", d_model=1024, n_head=16, d_ff=2560)
    W = make_weights(cfg)
    n = 64
    lens = [int(x) for x in make_prefix_lengths(n, 1, 40, seed=301)]
    prompts = [make_prefix(cfg, s, lens[s]) for s in range(n)]
    check = [0, 9, 31, 32, 50, 63]
    opts = OracleOpts(dtype=np.float32, kv_bf16=True)
    ls = Lockstep(cfg, W, prompts, [30] * n, TOL_MICRO_BF16, opts=opts, check=check)
    refs = {i: plain_greedy(ls.T, make_memory(cfg, i), prompts[i], 30) for i in check}
    rng = np.random.default_rng(7)
    for _ in range(5):
        ls.step(override=_planted_subset(ls, refs, rng))
    print(f"micro-wide b64: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, "
          f"accepted {ls.accepted}, near ties {ls.near_ties}")
    assert ls.steps == 5 and max(ls.accepted) > 0
    ls.close()


@pytest.mark.timeout(900)
@pytest.mark.parametrize("frames", [300, 900, 1300])
def test_micro_bf16_b64_cross_attention_by_pair(frames):
    """64 slots x 16 heads (1024 (head, slot) pairs): the bf16 cross-attention runs
    one block per pair over the 128-frame chunks (the next chunk's keys and values
    loaded during the current one, rows folded into running maxima and sums);
    300 / 900 / 1300 frames take 3 / 8 / 11 chunks (odd and even counts of the
    two alternating register sets).  The last chunk is ragged: at 900 frames
    (896..1023) only its first wave holds frames and the other three are masked
    whole, at 300 and 1300 (256..383, 1280..1407) the second wave ends inside
    its frames.  Planted drafts on six followed slots."""
    from lockstep import Lockstep
    cfg = MICRO_BF16.with_(name=f"micro-wide-{frames}f", d_model=1024, n_head=16, d_ff=2560, n_frames=frames)
    W = make_weights(cfg)
    n = 64
    lens = [int(x) for x in make_prefix_lengths(n, 1, 40, seed=303)]
    prompts = [make_prefix(cfg, s, lens[s]) for s in range(n)]
    check = [0, 13, 31, 32, 47, 63]
    opts = OracleOpts(dtype=np.float32, kv_bf16=True)
    ls = Lockstep(cfg, W, prompts, [30] * n, TOL_MICRO_BF16, opts=opts, check=check)
    refs = {i: plain_greedy(ls.T, make_memory(cfg, i), prompts[i], 30) for i in check}
    rng = np.random.default_rng(9)
    for _ in range(4):
        ls.step(override=_planted_subset(ls, refs, rng))
    print(f"micro-wide {frames}f b64: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, "
          f"accepted {ls.accepted}, near ties {ls.near_ties}")
    assert ls.steps == 4 and max(ls.accepted) > 0
    ls.close()


@pytest.mark.timeout(900)
def test_micro_bf16_b96_width1280_all_slots():
    """96 slots (864 rows) at width 1280 (20 heads), FFN 5120, two blocks: the
    1280-column products take 280 tile blocks (unsplit), and W'_o and W_2 append
    blocks that read the next product's weights (W_1, the next block's q|k|v) ahead.  Every slot is compared with the oracle,
    so a tile block lost to the appended ones would show in some slot's logits."""
    from lockstep import Lockstep
    cfg = MICRO_BF16.with_(name="micro-1280", d_model=1280, n_head=20, d_ff=5120)
    W = make_weights(cfg)
    n = 96
    lens = [int(x) for x in make_prefix_lengths(n, 1, 40, seed=302)]
    prompts = [make_prefix(cfg, s, lens[s]) for s in range(n)]
    opts = OracleOpts(dtype=np.float32, kv_bf16=True)
    ls = Lockstep(cfg, W, prompts, [30] * n, TOL_MICRO_BF16, opts=opts)
    for _ in range(3):
        ls.step()
    print(f"micro-1280 b96: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, "
          f"near ties {ls.near_ties}")
    assert ls.steps == 3 and sum(ls.live) >= n - 4
    ls.close()


def test_bf16_b96_width768_all_slots():
    """96 slots at width 768 (12 heads), FFN 3072, 700 frames, two blocks: the
    products of 36, 12 and 48 column blocks in four parts over the XCDs, the row blocks in two,
    the read-ahead blocks carry those widths, and the cross-attention runs one
    block per (head, slot) over six 128-frame chunks, the last one ragged (60
    frames).  Every slot is compared with the oracle."""
    from lockstep import Lockstep
    cfg = MICRO.with_(name="w768-bf16", dtype="bf16", d_model=768, n_head=12, d_ff=3072, n_vocab=2003,
                      n_ctx=128, n_frames=700)
    W = make_weights(cfg, std=0.05)
    n = 96
    lens = [int(x) for x in make_prefix_lengths(n, 1, 40, seed=303)]
    prompts = [make_prefix(cfg, s, lens[s]) for s in range(n)]
    ls = Lockstep(cfg, W, prompts, [30] * n, TOL_BF16)
    for _ in range(3):
        ls.step()
    print(f"w768 b96: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, near ties {ls.near_ties}")
    assert ls.steps == 3 and sum(ls.live) >= n - 4
    ls.close()


@pytest.mark.timeout(900)
# Several slots over many frames: bf16 cross-attention splits the frames into
# chunks of 256 (997 = 3 x 256 + 229: the last chunk ends inside a 16-frame
# score tile and inside an 8-frame value group, read from the zero padding of
# the transposed values) whose partial softmax sums a second kernel merges.
def test_micro_bf16_b3_chunked_cross_attention():
    from lockstep import Lockstep
    cfg = MICRO_BF16.with_(name="micro-bf16-997f", n_frames=997)
    W = make_weights(cfg)
    prompts = [make_prefix(cfg, 0, 6), make_prefix(cfg, 1, 17), make_prefix(cfg, 2, 30)]
    max_new = [24, 24, 24]
    opts = OracleOpts(dtype=np.float32, kv_bf16=True)
    ls = Lockstep(cfg, W, prompts, max_new, TOL_MICRO_BF16, opts=opts)
    T = Target(cfg, W.values, opts)
    refs = [plain_greedy(T, make_memory(cfg, i), prompts[i], max_new[i]) for i in range(3)]
    _run_planted(ls, refs, np.random.default_rng(7), 6)
    print(f"micro-bf16 997 frames b3: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, near ties {ls.near_ties}")
    assert ls.steps == 6
    ls.close()


@pytest.mark.timeout(900)
def test_micro_bf16_b1_chunked_cross_attention():
    """One slot, bf16, 300 frames: chunks of 128, 128 and a ragged 44 merged,
    the three-term operand split written by the merge kernel."""
    from lockstep import Lockstep
    cfg = MICRO_BF16.with_(name="micro-bf16-300f", n_frames=300)
    W = make_weights(cfg)
    prompts = [make_prefix(cfg, 0, 13)]
    ls = Lockstep(cfg, W, prompts, [40], TOL_MICRO_BF16)
    opts = OracleOpts(dtype=np.float32, kv_bf16=True)
    T = Target(cfg, W.values, opts)
    refs = [plain_greedy(T, make_memory(cfg, 0), prompts[0], 40)]
    _run_planted(ls, refs, np.random.default_rng(9), 8)
    print(f"micro-bf16 300 frames b1: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, near ties {ls.near_ties}")
    assert ls.steps == 8
    ls.close()


def test_tiny_b2_chunked_cross_attention():
    """fp32, two slots over 1500 frames: 19 chunks of 80 frames and a ragged 60."""
    from lockstep import Lockstep
    cfg = TINY
    W = make_weights(cfg)
    prompts = [make_prefix(cfg, 0, 9), make_prefix(cfg, 1, 25)]
    ls = Lockstep(cfg, W, prompts, [20, 20], TOL_F32)
    T = Target(cfg, W.values, OracleOpts())
    refs = [plain_greedy(T, make_memory(cfg, i), prompts[i], 20) for i in range(2)]
    _run_planted(ls, refs, np.random.default_rng(8), 5)
    print(f"tiny b2: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, near ties {ls.near_ties}")
    for i, s in enumerate(ls.sess):
        if ls.live[i]:
            assert s.out == refs[i][:len(s.out)]
    ls.close()


def test_large_v3_bf16_lockstep_b1():
    """Whisper-large-v3 shapes, bf16 weights/caches, one slot, prefix in [20, 200]."""
    from lockstep import Lockstep
    cfg = LARGE_V3
    W = make_weights(cfg)
    L = int(make_prefix_lengths(1, 20, 200)[0])
    prompt = make_prefix(cfg, 0, L)
    ls = Lockstep(cfg, W, [prompt], [448], TOL_BF16)
    for _ in range(2):
        ls.step()
    # planted acceptance using the GPU's own argmax continuation is checked
    # through the oracle inside the step comparison
    print(f"large-v3: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, near ties {ls.near_ties}")
    ls.close()


def test_large_v3_bf16_lockstep_b1_long_prefix():
    """One slot with a 430-token prefix and the random drafter's own proposals: two
    steps verify nine rows each from positions 430 and 431 (rows up to 439 carry
    keys of 14 32-key waves of the fused causal self-attention, and pages to the
    slot's 28th); the last context position is reached by
    test_large_v3_b1_verify_reaches_last_context_position."""
    from lockstep import Lockstep
    cfg = LARGE_V3
    W = make_weights(cfg)
    prompt = make_prefix(cfg, 0, 430)
    ls = Lockstep(cfg, W, [prompt], [448], TOL_BF16)
    for _ in range(2):
        ls.step()
    print(f"large-v3 long prefix: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}, "
          f"near ties {ls.near_ties}")
    ls.close()


# ---------------------------------------------------------------- large batches (sampled slots)
# At batch >= 2 operands are two bf16 planes (products accurate to fp32
# rounding), compared with the plain fp32 oracle; the oracle follows a sample of
# the slots, which are independent by construction (no per-row dependence on
# the batch).
LARGE_BATCH_OPTS = dict(dtype=np.float32, kv_bf16=True, exact=False)


def _planted_subset(ls, refs, rng):
    """Planted drafts for the checked slots (oracle greedy continuation with index r
    replaced); the other slots keep random tokens."""
    K = ls.cfg.block_k
    ov = rng.integers(0, ls.cfg.n_vocab, size=(ls.n, K)).astype(np.int32)
    for i, s in enumerate(ls.sess):
        if s is None or i not in refs:
            continue
        cont = (list(refs[i]) + [0] * (K + 1))[s.emitted:s.emitted + K]
        ov[i] = plant_drafts(cont, int(rng.integers(0, K + 1)), ls.cfg.n_vocab, rng)
    return ov


@pytest.mark.timeout(1200)
def test_large_v3_b16_ragged_planted():
    """16 slots, prefixes uniform in [4, 440] over 16-token pages, first-rejection
    index uniform in 0..8; the oracle follows the shortest, the longest and two
    other slots (the longest exercises the context-limited budget)."""
    from lockstep import Lockstep
    cfg = LARGE_V3
    W = make_weights(cfg)
    n = 16
    lens = [int(x) for x in make_prefix_lengths(n, 4, 440, seed=300)]
    prompts = [make_prefix(cfg, s, lens[s]) for s in range(n)]
    check = sorted({int(np.argmin(lens)), int(np.argmax(lens)), 3, 9})
    opts = OracleOpts(**LARGE_BATCH_OPTS)
    ls = Lockstep(cfg, W, prompts, [cfg.n_ctx] * n, TOL_BF16, opts=opts, check=check)
    print(f"b16: lens {lens}, checked {check}", flush=True)
    refs = {i: plain_greedy(ls.T, make_memory(cfg, i), prompts[i], 24) for i in check}
    rng = np.random.default_rng(4)
    for step in range(4):
        ls.step(override=_planted_subset(ls, refs, rng))
        print(f"b16 step {step}: accepted so far {ls.accepted}, max dlogit draft {ls.max_dlogit:.2e} "
              f"target {ls.max_tlogit:.2e}, near ties {ls.near_ties}", flush=True)
    assert max(ls.accepted) > 0
    ls.close()


@pytest.mark.timeout(1500)
def test_large_v3_b96_sampled_slots():
    """96 slots (864 verify rows per step), prefixes uniform in [4, 440], one
    acoustic memory per slot; the oracle follows three slots."""
    from lockstep import Lockstep
    cfg = LARGE_V3
    W = make_weights(cfg)
    n = 96
    lens = [int(x) for x in make_prefix_lengths(n, 4, 440, seed=300)]
    prompts = [make_prefix(cfg, s, lens[s]) for s in range(n)]
    check = [0, 47, 95]
    opts = OracleOpts(**LARGE_BATCH_OPTS)
    ls = Lockstep(cfg, W, prompts, [cfg.n_ctx] * n, TOL_BF16, opts=opts, check=check)
    print(f"b96: checked slots {check} with prefixes {[lens[i] for i in check]}", flush=True)
    for step in range(2):
        ls.step()
        print(f"b96 step {step}: max dlogit draft {ls.max_dlogit:.2e} target {ls.max_tlogit:.2e}, "
              f"near ties {ls.near_ties}", flush=True)
    assert ls.steps == 2
    ls.close()
