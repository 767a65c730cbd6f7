"""The calls a program makes of this library, as cases to time.

Three kinds of pass, over the model shapes the repository names:

  step     one draft + verify + accept step of a batch, the call a decoding loop
           repeats for every emitted block of tokens;
  request  what precedes the loop for new requests: (optionally) the acoustic
           keys and values of their audio, the prompt's prefill, the first step;
  encode   waveforms to acoustic memory; logmel: the feature frontend alone.

The weights are random, drawn as the tests and the benchmark draw them (N(0, 0.02),
LayerNorm gains around 1), and so are memories, prompts and planted drafts.  A
planted draft keeps the rows that a step verifies the same whatever rounding does
to the drafter's own argmax (random weights never agree with themselves); the
drafter still runs, and its logits are returned.  The first anchor is forced with
the suppression mask, as a Whisper program forces its first timestamp token: one
rounding of a near tie would change every row after it.

Every pass returns logits.  The emitted tokens are thresholds of these logits.
"""
import math

import torch

from paper_2609_32869_amd import WhisperEncoder, WhisperFlash

K = 8           # mask positions of a draft block
ROWS = K + 1    # rows that a step verifies per slot


class Shape:
    """Attributes that the binding reads."""

    def __init__(self, **kw):
        self.__dict__.update(kw)


def decoder(model):
    """Decoder shapes: the four widths that the tests and the benchmark run."""
    layers, d, ff, vocab, taps, dtype = {
        "large": (32, 1280, 5120, 51866, (1, 8, 15, 22, 29), "bf16"),
        "small": (12, 768, 3072, 51865, (1, 4, 7, 10), "bf16"),
        "base": (6, 512, 2048, 51865, (0, 2, 4), "bf16"),
        "tiny": (4, 384, 1536, 51865, (0, 1, 2, 3), "f32"),
    }[model]
    return Shape(n_layer=layers, d_model=d, n_head=d // 64, d_ff=ff, n_vocab=vocab, taps=taps, dtype=dtype,
                 n_ctx=448, n_frames=1500, n_draft_layer=2, block_k=K, eos_id=50257, draft_flags=0)


def encoder(model):
    layers, d, ff, mels = {"large": (32, 1280, 5120, 128), "small": (12, 768, 3072, 80), "base": (6, 512, 2048, 80)}[model]
    return Shape(n_mels=mels, n_ctx=1500, d_model=d, n_head=d // 64, n_layer=layers, d_ff=ff, n_fft=400, hop=160,
                 sample_rate=16000)


def listed():
    step = {"kind": "step", "k_max": K, "temperature": 0.0, "graph": True}
    req = {"kind": "request", "slots": 1, "batch": 1, "memory": True}
    return [
        # the correctness workload: a small fp32 decoder, batch 1, 32-token prompt
        dict(step, name="step_tiny_b1", model="tiny", batch=1, lo=32, hi=32),
        # interactive decoding of one recording (prompts U[20, 200], their mean)
        dict(step, name="step_b1", model="large", batch=1, lo=110, hi=110),
        # sampled decoding at temperature 0.7 with the rejection rule, eight recordings
        dict(step, name="step_b8_sampled", model="large", batch=8, lo=20, hi=200, temperature=0.7),
        # batch transcription: ragged contexts, 16 and 96 recordings
        dict(step, name="step_b16", model="large", batch=16, lo=4, hi=439),
        dict(step, name="step_b96", model="large", batch=96, lo=4, hi=439),
        # a small fp32 decoder's requests from acoustic memory to their first tokens
        dict(req, name="request_tiny_b3", model="tiny", slots=3, batch=3, lo=4, hi=37),
        # one recording from acoustic memory to its first tokens, the plain four-token prompt
        dict(req, name="request_b1", model="large", lo=4, hi=4),
        # the next window of one recording: 223 tokens of earlier text and the task tokens
        dict(req, name="prefill_b1", model="large", lo=227, hi=227, memory=False),
        # a batch engine in which two recordings replace finished ones
        dict(req, name="refill_2_of_16", model="large", slots=16, batch=2, lo=4, hi=227),
        # a whole batch of prompts, ragged up to the context's end
        dict(req, name="prefill_b16", model="large", slots=16, batch=16, lo=4, hi=439, memory=False),
        # the audio encoder: one 30 s window, and the windows of four recordings
        {"name": "encode_b1", "kind": "encode", "model": "large", "batch": 1},
        {"name": "encode_b4", "kind": "encode", "model": "large", "batch": 4},
    ]


def log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo - 0.49), math.log(hi + 0.49)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "request", "request", "encode"])
    if kind == "encode":
        if rng.random() < 0.2:
            return {"kind": "logmel", "model": rng.choice(["large", "small"]), "batch": 1}
        return {"kind": "encode", "model": rng.choice(["large", "large", "small", "base"]), "batch": rng.randint(1, 4)}
    model = rng.choice(["large", "large", "large", "small", "base", "tiny"])
    lo = log_int(rng, 1, 224)
    if kind == "step":
        batch = log_int(rng, 1, 16 if model == "tiny" else 96)
        return {"kind": "step", "model": model, "batch": batch, "lo": lo, "hi": lo if batch == 1 else rng.randint(lo, 439),
                "k_max": rng.choice([K, K, K, 4, 0]), "temperature": rng.choice([0.0, 0.0, 0.7, 1.0]),
                "graph": rng.random() < 0.7}
    slots = log_int(rng, 1, 16)
    batch = rng.randint(1, min(slots, 4 if model == "tiny" else 16))
    return {"kind": "request", "model": model, "slots": slots, "batch": batch, "lo": lo,
            "hi": lo if batch == 1 else rng.randint(lo, 300), "memory": rng.random() < 0.6}


# ---------------------------------------------------------------- inputs

def block_tensors(d, f):
    ln, mat = [("g", (d,)), ("", (d,))], (d, d)
    return (ln + [("w", mat), ("", (d,)), ("w", mat), ("w", mat), ("", (d,)), ("w", mat), ("", (d,))]
            + ln + [("w", mat), ("", (d,)), ("w", mat), ("w", mat), ("", (d,)), ("w", mat), ("", (d,))]
            + ln + [("w", (f, d)), ("", (f,)), ("w", (d, f)), ("", (d,))])


BLOCK = ["ln1g", "ln1b", "qw", "qb", "kw", "vw", "vb", "ow", "ob", "ln2g", "ln2b", "q2w", "q2b", "k2w", "v2w", "v2b",
         "o2w", "o2b", "ln3g", "ln3b", "f1w", "f1b", "f2w", "f2b"]
ENC_BLOCK = ["ln1g", "ln1b", "qw", "qb", "kw", "vw", "vb", "ow", "ob", "ln3g", "ln3b", "f1w", "f1b", "f2w", "f2b"]


def decoder_tensors(s):
    d, f = s.d_model, s.d_ff
    norm = [("g", (d,)), ("", (d,))]
    t = [("w", (s.n_vocab, d)), ("w", (s.n_ctx, d))]
    t += block_tensors(d, f) * s.n_layer + norm
    t += [("w", (d, len(s.taps) * d)), ("", (d,)), ("", (d,))] + block_tensors(d, f) * s.n_draft_layer + norm
    return t


def encoder_tensors(s):
    d, f, mat = s.d_model, s.d_ff, (s.d_model, s.d_model)
    ln = [("g", (d,)), ("", (d,))]
    blk = (ln + [("w", mat), ("", (d,)), ("w", mat), ("w", mat), ("", (d,)), ("w", mat), ("", (d,))]
           + ln + [("w", (f, d)), ("", (f,)), ("w", (d, f)), ("", (d,))])
    return [("w", (d, s.n_mels, 3)), ("", (d,)), ("w", (d, d, 3)), ("", (d,))] + blk * s.n_layer + ln


def draw_weights(tensors, dtype, gen):
    flat = torch.empty(sum(math.prod(shape) for _, shape in tensors), dtype=dtype, device="cuda")
    step = 1 << 27
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, device="cuda", generator=gen).mul_(0.02)
    out, at = [], 0
    for kind, shape in tensors:
        v = flat[at:at + math.prod(shape)].view(shape)
        if kind == "g":
            v += 1.0
        out.append(v)
        at += v.numel()
    return out


def inputs(case, seed):
    """Everything a pass reads, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * seed + 17)
    if case["kind"] in ("encode", "logmel"):
        s = encoder(case["model"])
        x = Shape(shape=s, weights=draw_weights(encoder_tensors(s), torch.bfloat16, gen))
        # voiced sound: three harmonic tones with slow envelopes, and a little noise
        n = 2 * s.n_ctx * s.hop
        t = torch.arange(n, device="cuda", dtype=torch.float64) / s.sample_rate
        audio = 0.005 * torch.randn((case["batch"], n), device="cuda", generator=gen)
        for b in range(case["batch"]):
            r = torch.rand((3, 4), device="cuda", generator=gen, dtype=torch.float64)
            for k in range(3):
                f0 = 90.0 + 210.0 * r[k, 0]
                env = 0.5 + 0.5 * torch.sin(2 * math.pi * (0.5 + 2.5 * r[k, 1]) * t + 2 * math.pi * r[k, 2])
                for h in range(1, 6):
                    audio[b] += ((0.05 / h) * env * torch.sin(2 * math.pi * f0 * h * t + 2 * math.pi * r[k, 3])).float()
        x.audio = audio
        return x
    s = decoder(case["model"])
    dtype = torch.bfloat16 if s.dtype == "bf16" else torch.float32
    x = Shape(shape=s, weights=draw_weights(decoder_tensors(s), dtype, gen))
    n = case["batch"]
    x.memory = torch.empty((n, s.n_frames, s.d_model), dtype=dtype, device="cuda")
    for i in range(n):
        x.memory[i] = torch.randn((s.n_frames, s.d_model), device="cuda", generator=gen)
    # prompt lengths evenly over [lo, hi], in the seed's order
    lens = lengths(case)
    order = torch.randperm(n, generator=torch.Generator().manual_seed(seed)).tolist()
    x.lens = [lens[i] for i in order]
    ids = lambda *shape: torch.randint(0, 50257, shape, device="cuda", generator=gen, dtype=torch.int32)  # noqa: E731
    x.prompt = ids(n, max(x.lens))
    x.drafts = ids(n, K)
    x.anchor = 50365 if s.n_vocab > 50365 else s.n_vocab - 1
    return x


def lengths(case):
    n, lo, hi = case["batch"], case["lo"], case["hi"]
    return [hi if n == 1 else lo + round(i * (hi - lo) / (n - 1)) for i in range(n)]


# ---------------------------------------------------------------- passes

_stream = None


def stream():
    """The stream of the decoding loop (a captured step needs one of its own)."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def start_slots(st):
    """Prompts of the batch's slots into the engine; the first token is the forced one."""
    eng, x = st.eng, st.x
    eng.set_sampling(0.0, suppress=st.mask)
    eng.prefill(st.slot0, x.prompt, x.lens, [448] * len(x.lens), stream=stream())
    eng.set_sampling(st.case["temperature"] if "temperature" in st.case else 0.0, seed=500)


def prepare(case, seed):
    x = inputs(case, seed)
    st = Shape(case=case, x=x)
    if case["kind"] in ("encode", "logmel"):
        st.eng = WhisperEncoder(x.shape, x.weights)
    else:
        n = case["batch"]
        slots = case.get("slots", n)
        st.slot0 = (slots - n) // 2
        st.eng = WhisperFlash(x.shape, slots, x.weights)
        st.eng.set_debug(True)  # keep the logits
        st.mask = torch.ones(x.shape.n_vocab, dtype=torch.uint8, device="cuda")
        st.mask[x.anchor] = 0
        ints = lambda *shape: torch.zeros(shape, dtype=torch.int32, device="cuda")  # noqa: E731
        st.outs = (ints(n, ROWS), ints(n), ints(n), ints(n))
        torch.cuda.synchronize()
        if case["kind"] == "step" or not case["memory"]:
            st.eng.encode_memory_set(st.slot0, x.memory, stream=stream())
        if case["kind"] == "step":
            start_slots(st)
            torch.cuda.synchronize()
            st.saved = st.eng.state().clone()
    torch.cuda.synchronize()
    x.weights = None  # the engine has its own copy
    return st


def run(st):
    case, x, eng = st.case, st.x, st.eng
    with torch.cuda.stream(stream()):
        if case["kind"] == "logmel":
            return eng.logmel(x.audio[0])
        if case["kind"] == "encode":
            return eng.run(x.audio)
        n, k_max, graph = case["batch"], K, False
        if case["kind"] == "step":
            k_max, graph = case["k_max"], case["graph"]
            eng.state().copy_(st.saved)  # each pass is the same step of the loop: 64 bytes per slot
        else:
            if case["memory"]:
                eng.encode_memory_set(st.slot0, x.memory)
            start_slots(st)
        eng.step(st.slot0, n, k_max, draft_override=x.drafts, outs=st.outs, use_graph=graph)
        at = slice(st.slot0, st.slot0 + n)
        out = {"target": eng.target_logits()[at, :k_max + 1]}
        if k_max > 0:  # plain decoding drafts nothing
            out["draft"] = eng.draft_logits()[at, 1:]
        return out


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    if case["kind"] in ("encode", "logmel"):
        s, n = encoder(case["model"]), case["batch"]
        t, d, f = s.n_ctx, s.d_model, s.d_ff
        audio, mel = 4 * 2 * t * s.hop * n, 2 * t * s.n_mels * n
        dft = 2.5 * 512 * 9 * 2 * t * n  # a fast transform of every frame
        if case["kind"] == "logmel":
            return {"bytes": audio + 4 * mel, "flops": dft}
        params = 3 * d * s.n_mels + 3 * d * d + s.n_layer * (4 * d * d + 2 * d * f)
        flops = 2 * t * n * (2 * 3 * d * s.n_mels + 3 * d * d + s.n_layer * (4 * d * d + 2 * d * f + 2 * t * d))
        return {"bytes": 2 * params + audio + 2 * t * d * n, "flops": flops + dft}
    s, n = decoder(case["model"]), case["batch"]
    e = 2 if s.dtype == "bf16" else 4
    d, f, L, D, V, T = s.d_model, s.d_ff, s.n_layer, s.n_draft_layer, s.n_vocab, s.n_frames
    block = 6 * d * d + 2 * d * f         # weights that every row passes (without the acoustic k and v products)
    hist = len(s.taps) * d * d + 2 * d * d * D
    lens = lengths(case)
    k_max = case.get("k_max", K)
    drafting = k_max > 0
    rows = n * (k_max + 1)
    # the step: weights once, each slot's acoustic and text keys and values once, logits out
    weights = L * block + V * d + hist + (D * block if drafting else 0)
    xkv = 2 * T * d * n * (L + (D if drafting else 0))
    skv = sum(2 * p * d for p in lens) * (L + (D if drafting else 0))
    out = 4 * V * (rows + (n * K if drafting else 0))
    step_bytes = e * (weights + xkv + skv) + out
    att = 4 * d * sum(p + ROWS / 2 + T for p in lens)
    step_flops = 2 * rows * (L * block + V * d + hist) + (k_max + 1) * L * att
    if drafting:
        step_flops += 2 * n * ROWS * (D * block + V * d) + ROWS * D * att
    if case["kind"] == "step":
        return {"bytes": step_bytes, "flops": step_flops}
    # prompts: weights and acoustic memory once more (one pass over them all), text keys and values written
    p = sum(lens)
    flops = step_flops + 2 * p * (L * block + hist) + 2 * n * V * d + sum(4 * d * q * (q / 2 + T) for q in lens) * L
    nbytes = step_bytes + e * (L * block + V * d + hist + 2 * T * d * n * L) + e * 2 * p * d * (L + D)
    if case["memory"]:
        flops += 2 * n * T * 2 * d * d * (L + D)
        nbytes += e * (2 * d * d * (L + D) + n * T * d + 2 * T * d * n * (L + D))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the distance from the 64-bit result that the library showed."""
    if case["kind"] == "logmel":
        return {"rel": 5e-7, "max": 5e-6}  # fp64 inside, one rounding to fp32
    if case["kind"] == "encode":
        return {"rel": 1.5e-2, "max": 0.2}  # bf16 product inputs and output: 3.8e-3
    if case["model"] == "tiny":
        return {"rel": 4e-6, "max": 4e-5}  # fp32 throughout: 4.5e-7, two of them apart, longer sums
    # fp32 arithmetic over key / value caches rounded to bf16: up to 7e-4 (a rounding
    # that falls the other way travels on), largest single logits 3.5e-3
    return {"rel": 4e-3, "max": 2e-2}


# ---------------------------------------------------------------- the same in 64 bits

def norm(x, g, b):
    m = x.mean(-1, keepdim=True)
    v = ((x - m) ** 2).mean(-1, keepdim=True)
    return (x - m) / torch.sqrt(v + 1e-5) * g + b


def gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def heads(x, h):
    return x.reshape(x.shape[0], h, -1).transpose(0, 1).contiguous()


def attend(q, k, v, h, seen=None):
    s = torch.matmul(heads(q, h), heads(k, h).transpose(1, 2).contiguous()) / 8.0
    if seen is not None:
        s = s.masked_fill(~seen, -math.inf)
    return torch.matmul(torch.softmax(s, -1), heads(v, h)).transpose(0, 1).reshape(q.shape[0], -1)


def rotate(x, pos, h):
    # rotate-half pairs (i, i + 32) of each head; the angle is an fp32 product
    om = torch.tensor([10000.0 ** (-2.0 * i / 64.0) for i in range(32)], dtype=torch.float64).float().cuda()
    th = (pos.float()[:, None] * om[None, :]).double()
    c, s = torch.cos(th)[:, None], torch.sin(th)[:, None]
    y = x.reshape(x.shape[0], h, 64)
    a, b = y[..., :32], y[..., 32:]
    return torch.cat([a * c - b * s, b * c + a * s], -1).reshape(x.shape)


def exact(case, seed):
    x = inputs(case, seed)
    return exact_audio(case, x) if case["kind"] in ("encode", "logmel") else exact_text(case, x)


def exact_text(case, x):
    s, n = x.shape, case["batch"]
    h, d = s.n_head, s.d_model
    stored = (lambda t: t.bfloat16().double()) if s.dtype == "bf16" else (lambda t: t)  # the caches' type
    W = iter(x.weights)
    emb, pos_emb = next(W).double(), next(W).double()
    blocks = [dict(zip(BLOCK, [next(W) for _ in BLOCK])) for _ in range(s.n_layer)]
    fg, fb = next(W).double(), next(W).double()
    hw, hb, mask = next(W).double(), next(W).double(), next(W).double()
    dblocks = [dict(zip(BLOCK, [next(W) for _ in BLOCK])) for _ in range(s.n_draft_layer)]
    dg, db = next(W).double(), next(W).double()
    k_max = case.get("k_max", K)
    # rows of all slots, one after the other: prompt, anchor, verified drafts
    cut, toks, pos = [0], [], []
    for i, p in enumerate(x.lens):
        t = torch.cat([x.prompt[i, :p], torch.tensor([x.anchor], device="cuda", dtype=torch.int32), x.drafts[i, :k_max]])
        toks.append(t.long())
        pos.append(torch.arange(len(t), device="cuda"))
        cut.append(cut[-1] + len(t))
    hrow = emb[torch.cat(toks)] + pos_emb[torch.cat(pos)]
    each = [slice(cut[i], cut[i + 1]) for i in range(n)]

    def tail(b, r, part):
        """Cross-attention and MLP of block b on rows r; part: each slot's rows."""
        q = norm(r, b["ln2g"], b["ln2b"]) @ b["q2w"].T + b["q2b"]
        o = torch.empty_like(q)
        for i, at in enumerate(part):
            m = x.memory[i].double()
            o[at] = attend(q[at], stored(m @ b["k2w"].T), stored(m @ b["v2w"].T + b["v2b"]), h)
        r = r + o @ b["o2w"].T + b["o2b"]
        return r + gelu(norm(r, b["ln3g"], b["ln3b"]) @ b["f1w"].T + b["f1b"]) @ b["f2w"].T + b["f2b"]

    taps = []
    for l, b in enumerate(blocks):
        b = {k: v.double() for k, v in b.items()}
        a = norm(hrow, b["ln1g"], b["ln1b"])
        q, k, v = a @ b["qw"].T + b["qb"], stored(a @ b["kw"].T), stored(a @ b["vw"].T + b["vb"])
        o = torch.empty_like(q)
        for at in each:
            m = at.stop - at.start
            o[at] = attend(q[at], k[at], v[at], h, torch.ones((m, m), dtype=torch.bool, device="cuda").tril())
        hrow = tail(b, hrow + o @ b["ow"].T + b["ob"], each)
        if l in s.taps:
            taps.append(hrow)
    last = torch.cat([hrow[at.stop - k_max - 1:at.stop] for at in each])
    out = {"target": (norm(last, fg, fb) @ emb.T).reshape(n, k_max + 1, -1)}
    if k_max == 0:
        return out
    hist = torch.cat(taps, 1) @ hw.T + hb
    r = torch.cat([emb[x.anchor][None], mask.repeat(K, 1)]).repeat(n, 1)
    part = [slice(i * ROWS, (i + 1) * ROWS) for i in range(n)]
    for b in dblocks:
        b = {k: v.double() for k, v in b.items()}
        a, ah = norm(r, b["ln1g"], b["ln1b"]), norm(hist, b["ln1g"], b["ln1b"])
        o = torch.empty_like(r)
        for i, (at, p) in enumerate(zip(part, x.lens)):
            rows, at_h = torch.arange(p, p + ROWS, device="cuda"), slice(cut[i], cut[i] + p)
            kh = stored(rotate(ah[at_h] @ b["kw"].T, torch.arange(p, device="cuda"), h))
            vh = stored(ah[at_h] @ b["vw"].T + b["vb"])
            kb, vb = rotate(a[at] @ b["kw"].T, rows, h), a[at] @ b["vw"].T + b["vb"]
            o[at] = attend(rotate(a[at] @ b["qw"].T + b["qb"], rows, h), torch.cat([kh, kb]), torch.cat([vh, vb]), h)
        r = tail(b, r + o @ b["ow"].T + b["ob"], part)
    out["draft"] = (norm(r, dg, db) @ emb.T).reshape(n, ROWS, -1)[:, 1:]
    return out


def mel_filters(s):
    to_mel = lambda f: f * 3.0 / 200.0 if f < 1000.0 else 15.0 + 27.0 * math.log(f / 1000.0) / math.log(6.4)  # noqa: E731
    to_hz = lambda m: m * 200.0 / 3.0 if m < 15.0 else 1000.0 * 6.4 ** ((m - 15.0) / 27.0)  # noqa: E731
    top = to_mel(s.sample_rate / 2)
    edge = [to_hz(top * i / (s.n_mels + 1)) for i in range(s.n_mels + 2)]
    hz = torch.arange(s.n_fft // 2 + 1, dtype=torch.float64, device="cuda") * s.sample_rate / s.n_fft
    rows = []
    for lo, c, hi in zip(edge, edge[1:], edge[2:]):
        rows.append(torch.clamp(torch.minimum((hz - lo) / (c - lo), (hi - hz) / (hi - c)), min=0.0) * 2.0 / (hi - lo))
    return torch.stack(rows)


def exact_logmel(s, audio):
    half = s.n_fft // 2
    a = audio.double()
    a = torch.cat([a[1:half + 1].flip(0), a, a[-half - 1:-1].flip(0)])
    frames = a.unfold(0, s.n_fft, s.hop)[:-1]
    i = torch.arange(s.n_fft, dtype=torch.float64, device="cuda")
    frames = frames * (0.5 - 0.5 * torch.cos(2 * math.pi * i / s.n_fft))
    k = torch.arange(half + 1, dtype=torch.float64, device="cuda")
    ang = 2 * math.pi * torch.remainder(i[:, None] * k[None, :], s.n_fft) / s.n_fft
    power = (frames @ torch.cos(ang)) ** 2 + (frames @ torch.sin(ang)) ** 2
    lg = torch.log10(torch.clamp(mel_filters(s) @ power.T, min=1e-10))
    return (torch.maximum(lg, lg.max() - 8.0) + 4.0) / 4.0


def exact_audio(case, x):
    s = x.shape
    if case["kind"] == "logmel":
        return exact_logmel(s, x.audio[0])
    h, d = s.n_head, s.d_model
    out = []
    for a in x.audio:
        W = iter(x.weights)
        c1, b1, c2, b2 = (next(W).double() for _ in range(4))
        r = exact_logmel(s, a).T

        def conv(r, w, b, stride):
            z = torch.zeros_like(r[:1])
            r = torch.cat([z, r, z])
            t = torch.arange(0, r.shape[0] - 2, stride, device="cuda")
            return gelu(sum(r[t + j] @ w[:, :, j].T for j in range(3)) + b)

        r = conv(conv(r, c1, b1, 1), c2, b2, 2)
        inv = torch.exp(-math.log(10000.0) / (d // 2 - 1) * torch.arange(d // 2, dtype=torch.float64, device="cuda"))
        ang = torch.arange(s.n_ctx, dtype=torch.float64, device="cuda")[:, None] * inv[None, :]
        r = r + torch.cat([torch.sin(ang), torch.cos(ang)], 1)
        for _ in range(s.n_layer):
            b = {k: next(W).double() for k in ENC_BLOCK}
            y = norm(r, b["ln1g"], b["ln1b"])
            o = attend(y @ b["qw"].T + b["qb"], y @ b["kw"].T, y @ b["vw"].T + b["vb"], h)
            r = r + o @ b["ow"].T + b["ob"]
            r = r + gelu(norm(r, b["ln3g"], b["ln3b"]) @ b["f1w"].T + b["f1b"]) @ b["f2w"].T + b["f2b"]
        out.append(norm(r, next(W).double(), next(W).double()))
    return torch.stack(out)
