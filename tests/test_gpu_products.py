"""The matrix products (bf16 storage) at sizes that end inside a tile, through the calls
that reach them: the request-time ones on 256 x 128 tiles, a step's on 64 x 64.

Both sides round to bf16 at the same points and accumulate in fp32, so a difference
is a rounding that falls the other way: the acoustic memory's bar stands in
encoder_check.py, the logits' bar is the decoder's.
"""
import numpy as np
import pytest
import torch

from encoder_check import encode_and_compare
from wf_fixtures import (MICRO, MICRO_ENC, make_encoder_weights, make_audio, make_memory, make_weights,
                         make_prefix)
from oracle import OracleOpts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_wide_mlp_product():
    """First MLP product of 16384 columns over 300 rows (44 in the second row tile)."""
    encode_and_compare(MICRO_ENC.with_(name="enc-wide", n_ctx=300, d_model=256, n_head=4, n_layer=1, d_ff=16384), 1)


@pytest.mark.parametrize("n", [4, 5])
def test_requests_share_a_pass(n):
    """Requests that go through the layers together (four at most: five in 3 + 2), 50
    positions each with 14 rows between them."""
    encode_and_compare(MICRO_ENC.with_(name="enc-batch", n_ctx=50), n)


# Four requests (n_ctx positions, width, MLP width) and the row tiles that their products take.
# Requests stand up(n_ctx, 64) rows apart, no multiple of 128, so tiles of 128 and 256 rows
# hold the end of one request and the start of the next.
BATCHED = [(804, 704, 2112, {"qkv": 128, "o": 64, "w1": 128, "w2": 64, "conv1": 256, "conv2": 64}),
           (932, 1088, 128, {"qkv": 256, "o": 256, "w1": 64, "w2": 256, "conv1": 256, "conv2": 256}),
           (1028, 1088, 128, {"qkv": 256, "o": 256, "w1": 64, "w2": 256, "conv1": 256, "conv2": 128})]


@pytest.mark.parametrize("n_ctx,d_model,d_ff", [c[:3] for c in BATCHED])
def test_row_tiles_over_two_requests(n_ctx, d_model, d_ff):
    """Four requests' products on tiles of 128 and 256 rows (test_split_cpu.py holds the tile rule
    to these): q | k with the transposed values, residual rows, the strided convolution."""
    encode_and_compare(MICRO_ENC.with_(name="enc-span", n_ctx=n_ctx, d_model=d_model, n_head=d_model // 64, n_layer=1,
                                       d_ff=d_ff), 4)


@pytest.mark.parametrize("n_ctx,size", [(48, 1114880), (50, 1125888), (50, 1600000)])
def test_encoder_workspace_for_fewer_requests(n_ctx, size, monkeypatch):
    """Three requests in a workspace for one (its size before requests shared a pass; one byte
    less is refused) and for two."""
    from paper_2609_32869_amd import WfError, WhisperEncoder, binding, load_library
    lib = load_library()

    class Library:
        bytes = size

        def __getattr__(self, name):
            return getattr(lib, name)

        def wf_encoder_workspace_bytes(self, cfg, out):
            assert lib.wf_encoder_workspace_bytes(cfg, out) == 0 and out._obj.value > self.bytes
            out._obj.value = self.bytes
            return 0

    ecfg = MICRO_ENC.with_(name="enc-small", n_ctx=n_ctx)
    small = Library()
    monkeypatch.setattr(binding, "load_library", lambda: small)
    encode_and_compare(ecfg, 3)
    if size < 1200000:
        small.bytes = size - 1
        with pytest.raises(WfError, match="workspace too small"):
            WhisperEncoder(ecfg, [torch.zeros(1, device="cuda")] * len(make_encoder_weights(ecfg).order))


@pytest.mark.parametrize("n_frames", [300, 256])
def test_acoustic_keys_and_values_of_many_blocks(n_frames):
    """Twelve blocks' keys and transposed values in one launch: rows that end inside a
    tile and at its edge, zero padding of the values up to 512 frames."""
    from lockstep import Lockstep
    cfg = MICRO.with_(name="xkv-wide", dtype="bf16", n_layer=12, d_model=512, n_head=8, d_ff=512, n_vocab=501,
                      taps=(0, 5, 11), n_frames=n_frames)
    W = make_weights(cfg)
    ls = Lockstep(cfg, W, [make_prefix(cfg, 0, 7)], [20], 2e-2, opts=OracleOpts(dtype=np.float32, kv_bf16=True))
    for _ in range(2):
        ls.step()
    print(f"frames {n_frames}: max |dlogit| draft {ls.max_dlogit:.2e} target {ls.max_tlogit:.2e}")
    ls.close()


@pytest.mark.parametrize("batch,d_ff", [(7, 352), (8, 96), (15, 160)])
def test_step_products_at_tile_edges(batch, d_ff):
    """Several slots' products on 64 x 64 tiles whose waves split k: 63, 72 and 135 rows,
    MLP widths that end inside a column tile, k-splits of one 32-wide step (two of the
    four waves have nothing to multiply) and widths too ragged to split."""
    from lockstep import Lockstep
    cfg = MICRO.with_(name="step-edges", dtype="bf16", n_vocab=501, n_frames=45, d_ff=d_ff)
    W = make_weights(cfg)
    ls = Lockstep(cfg, W, [make_prefix(cfg, i, 3 + i) for i in range(batch)], [20] * batch, 2e-3,
                  opts=OracleOpts(dtype=np.float32, kv_bf16=True))
    for _ in range(3):
        ls.step()
    print(f"b{batch} d_ff {d_ff}: max |dlogit| draft {ls.max_dlogit:.3e} target {ls.max_tlogit:.3e}", flush=True)
    assert ls.steps == 3
    ls.close()


@pytest.mark.parametrize("n_fft", [6, 162, 250, 254, 506, 512])
def test_frontend_window_lengths(n_fft):
    """The two-stage transform at 2 x 3, 9 x 18, 10 x 25, 2 x 127, 22 x 23 and 16 x 32: an odd
    first factor, the longest second one and the longest window, against numpy's rfft (fp64
    on both sides; the bar is the stored fp32 log10 value's)."""
    from oracle.encoder import log_mel
    from paper_2609_32869_amd import WhisperEncoder
    ecfg = MICRO_ENC.with_(name="enc-fft", n_fft=n_fft)
    W = make_encoder_weights(ecfg)
    enc = WhisperEncoder.from_host(ecfg, [W.values[k] for k, _ in W.order])
    x = make_audio(ecfg, 0)
    got = enc.logmel(torch.from_numpy(x).cuda()).cpu().numpy()
    enc.close()
    want = log_mel(x, ecfg.n_mels, n_fft)
    np.testing.assert_allclose(got, want[:, :got.shape[1]], rtol=0, atol=1e-5)


@pytest.mark.parametrize("n_frames,offset", [(65, 0), (64, 1)])
def test_fp32_acoustic_keys_and_values(n_frames, offset):
    """fp32 storage: the keys and values of every block and slot in one launch, a last tile of
    one frame, and an acoustic memory that is not 16-byte aligned."""
    from lockstep import Lockstep
    cfg = MICRO.with_(name="xkv-f32", n_frames=n_frames)
    W = make_weights(cfg)
    ls = Lockstep(cfg, W, [make_prefix(cfg, i, 7 + i) for i in range(3)], [20] * 3, 1e-3,
                  opts=OracleOpts(dtype=np.float32))
    if offset:  # the same memory again from an address 4 bytes past a multiple of 16
        mem = torch.from_numpy(np.stack([make_memory(cfg, i) for i in range(3)]).astype(np.float32))
        shifted = torch.empty(mem.numel() + 4, device="cuda")[offset:offset + mem.numel()].view(mem.shape)
        shifted.copy_(mem)
        ls.eng.encode_memory_set(0, shifted)
    for _ in range(3):
        ls.step()
    assert ls.steps == 3
    ls.close()


@pytest.mark.parametrize("d_ff", [32, 96, 352])
def test_fp32_second_mlp_product_split(d_ff):
    """fp32 storage: k-splits of one step (two splits), an empty last split, and splits that
    do not divide the k-steps."""
    from lockstep import Lockstep
    cfg = MICRO.with_(name="fc2-f32", d_ff=d_ff)
    W = make_weights(cfg)
    ls = Lockstep(cfg, W, [make_prefix(cfg, i, 7 + i) for i in range(2)], [20] * 2, 1e-3,
                  opts=OracleOpts(dtype=np.float32))
    for _ in range(3):
        ls.step()
    assert ls.steps == 3
    ls.close()
