"""The Whisper audio encoder on the HIP path (through the C ABI) against the oracle.

  * the log-mel frontend (fp64 on both sides) agrees to 1e-5;
  * the acoustic memory agrees with the oracle computed with the same bf16
    rounding of every product input (encoder_check.py), at micro and large-v3 shapes;
  * end to end: waveform -> GPU encoder -> wf_encode_memory_set -> prefill ->
    draft + verify steps, against the oracle decoding from its own encoder
    output (logits within the decoder's bf16 tolerance, tokens identical
    wherever the margin exceeds it).
"""
import numpy as np
import pytest
import torch

from encoder_check import encode_and_compare, rel
from wf_fixtures import (MICRO, MICRO_ENC, LARGE_V3_ENC, make_encoder_weights, make_audio, make_weights,
                         make_prefix)
from oracle import OracleOpts
from oracle.encoder import Encoder, log_mel
from oracle.numerics import bf16

pytestmark = pytest.mark.gpu

ENC_OPTS = OracleOpts(dtype=np.float32, gemm_bf16=True, exact=False)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _encoder(ecfg):
    from paper_2609_32869_amd import WhisperEncoder
    W = make_encoder_weights(ecfg)
    return WhisperEncoder.from_host(ecfg, [W.values[n] for n, _ in W.order]), W


def test_logmel_frontend():
    ecfg = MICRO_ENC
    enc, _ = _encoder(ecfg)
    for slot in range(2):
        x = make_audio(ecfg, slot)
        got = enc.logmel(torch.from_numpy(x).cuda()).cpu().numpy()
        want = log_mel(x, ecfg.n_mels)
        print(f"log-mel slot {slot}: max |d| {np.abs(got - want).max():.2e}")
        np.testing.assert_allclose(got, want, rtol=0, atol=1e-5)
    enc.close()


def test_micro_encoder_matches_oracle():
    encode_and_compare(MICRO_ENC, 2)


@pytest.mark.timeout(900)
def test_large_v3_encoder_matches_oracle():
    encode_and_compare(LARGE_V3_ENC, 1, std=0.02)


def test_scores_of_minus_infinity():
    """Keys whose scores are -inf have no weight, also where they fill the first tile of 64, and
    the greatest of the others, 1.3e38, all of it: sound in the first third of the signal makes
    hidden channel 0 large there, W_k multiplies it past fp32's range, and queries are 1 in
    that dimension."""
    ecfg = MICRO_ENC.with_(name="enc-inf", n_ctx=210, d_model=64, n_head=1, n_layer=1, d_ff=64)
    W = make_encoder_weights(ecfg, std=0.05)
    V = W.values
    x = make_audio(ecfg, 0)
    x[75 * 2 * ecfg.hop:] = 0
    level = log_mel(x, ecfg.n_mels).sum(0)                     # per frame; two frames per position
    for name in ("conv1.w", "conv1.b", "conv2.w", "conv2.b", "e0.attn.q.w", "e0.attn.q.b", "e0.attn.k.w"):
        V[name][:] = 0
    V["conv1.w"][0, :, 1] = 1
    V["conv1.b"][0] = bf16(np.float32(-(level[:140].min() + level[160:].max()) / 2))
    V["conv2.w"][0, 0, 1] = 1
    V["e0.attn_ln.g"][:], V["e0.attn_ln.b"][:] = 1, 0
    V["e0.attn.q.b"][0] = 1
    V["e0.attn.k.w"][0, 0] = bf16(np.float32(-6e37))
    with np.errstate(over="ignore", invalid="ignore"):
        E = Encoder(ecfg, V, ENC_OPTS)
        want = bf16(E.encode(x))
    from paper_2609_32869_amd import WhisperEncoder
    enc = WhisperEncoder.from_host(ecfg, [V[n] for n, _ in W.order])
    got = enc.run(torch.from_numpy(x[None]).cuda()).float().cpu().numpy()[0]
    enc.close()
    assert np.isfinite(want).all()
    print(f"scores of -inf: {rel(got, want):.2e}")
    assert rel(got, want) <= 1e-2


def test_waveform_to_tokens_micro():
    """Waveform -> GPU encoder -> decoder steps, against the oracle decoding from its
    own encoder output (the decoder's acoustic memory is the only coupling)."""
    from lockstep import Lockstep
    ecfg, cfg = MICRO_ENC, MICRO.with_(name="micro-bf16-audio", dtype="bf16", n_vocab=501)
    assert cfg.n_frames == ecfg.n_ctx and cfg.d_model == ecfg.d_model
    enc, EW = _encoder(ecfg)
    audio = np.stack([make_audio(ecfg, s) for s in range(2)])
    mem_gpu = enc.run(torch.from_numpy(audio).cuda())
    E = Encoder(ecfg, EW.values, ENC_OPTS)
    mems = [bf16(E.encode(audio[s])).astype(np.float32) for s in range(2)]
    W = make_weights(cfg)
    prompts = [make_prefix(cfg, 0, 6), make_prefix(cfg, 1, 11)]
    ls = Lockstep(cfg, W, prompts, [30, 30], 2e-2, opts=OracleOpts(dtype=np.float32, kv_bf16=True), mems=mems)
    ls.eng.encode_memory_set(0, mem_gpu)          # the GPU decoder reads the GPU encoder's memory
    ls.eng.prefill(0, torch.from_numpy(np.stack([np.pad(p, (0, 11 - len(p))) for p in prompts]).astype(np.int32)).cuda(),
                   [len(p) for p in prompts], [30, 30])
    for _ in range(4):
        ls.step()
    print(f"waveform->tokens: max |dlogit| draft {ls.max_dlogit:.2e} target {ls.max_tlogit:.2e}, near ties {ls.near_ties}")
    ls.close()
    enc.close()
