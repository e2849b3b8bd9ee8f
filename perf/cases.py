"""Timing cases of the framework: the calls a streaming-recognition program makes, at the sizes it makes them.

A program keeps one encoder, one decoder side and one front end per model for as long as it runs and calls them once
per processing round, with whatever audio its streams hold at that moment.  So the handles (weights, workspaces sized for
the largest round) are made once per model and kept here, and a case is what changes from round to round: how many
streams, how long their buffers are, how many prompt tokens they carry.

kinds   encode    log-mel buffers in device memory -> encoder states
        logmel    raw 16 kHz audio -> packed log-mel (hush word appended at the raw level)
        decode    encoder states -> cross-attention K/V of every layer, then the prompt prefill
        pipeline  audio -> log-mel -> encoder -> cross K/V -> prefill, one round as a whole
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2412_11272_amd import binding as wf
from paper_2412_11272_amd import synth

MODELS = ["tiny", "base", "small", "medium", "large-v3"]
MAX_STREAMS = 64
MAX_SECONDS = 30.0
MIN_SECONDS = 0.5
MAX_TOTAL_FRAMES = 100_000          # capacity of every handle: 64 streams of 15 s on average
MAX_PROMPT = 224
SPF = synth.SAMPLES_PER_FRAME


def _case(name, kind, model, streams, lo_s, hi_s, *, lengths=0, hush=True, mel_bf16=False, out_bf16=False, prompt_lo=0, prompt_hi=0):
    return {"name": name, "kind": kind, "model": model, "streams": streams, "lo_s": lo_s, "hi_s": hi_s, "lengths": lengths, "hush": hush,
            "mel_bf16": mel_bf16, "out_bf16": out_bf16, "prompt_lo": prompt_lo, "prompt_hi": prompt_hi}


def listed():
    return [
        # one speaker, the smallest model, one second of new audio: the call whose latency a user sees first
        _case("encode-tiny-1x1s", "encode", "tiny", 1, 1.0, 1.0),
        # one speaker, a few seconds in the buffer (odd frame count: an odd last token window)
        _case("encode-base-1x4s", "encode", "base", 1, 4.37, 4.37),
        # one speaker on the most accurate model: 8 s of buffered audio
        _case("encode-large-1x8s", "encode", "large-v3", 1, 8.0, 8.0, out_bf16=True),
        # a small server: 16 ragged streams
        _case("encode-small-16", "encode", "small", 16, 1.0, 10.0, lengths=3),
        # eight equal buffers after trimming to 6 s, the usual state between two trims
        _case("encode-medium-8x6s", "encode", "medium", 8, 6.0, 6.0, out_bf16=True),
        # the padded way of using such a model: 30 s windows, no hush segment
        _case("encode-medium-8x30s", "encode", "medium", 8, 30.0, 30.0, hush=False),
        # the heavy ragged batch of a loaded server: 64 streams from 1 to 30 s; half-precision features and states
        _case("encode-large-64", "encode", "large-v3", 64, 1.0, 30.0, lengths=5, mel_bf16=True, out_bf16=True),
        # features of one short buffer, and of a whole loaded round
        _case("logmel-1x4s", "logmel", "base", 1, 4.37, 4.37),
        _case("logmel-64", "logmel", "large-v3", 64, 1.0, 30.0, lengths=5),
        # what follows the encoder for one speaker, and for the loaded server (about 100 prompt tokens per stream)
        _case("decode-base-1", "decode", "base", 1, 4.37, 4.37, prompt_lo=100, prompt_hi=100),
        _case("decode-large-64", "decode", "large-v3", 64, 1.0, 30.0, lengths=5, prompt_lo=90, prompt_hi=110),
        # one whole round from audio to the first logits, four ragged streams on the middle model
        _case("pipeline-small-4", "pipeline", "small", 4, 2.0, 15.0, lengths=7, prompt_lo=20, prompt_hi=120),
    ]


def draw(rng: random.Random):
    """One more case of the same ranges: any model, 1 .. 64 streams and 0.5 .. 30 s of audio (both spread over their
    logarithm), any mix of types; no more work than the largest listed case."""
    largest = max(work(c)["flops"] for c in listed())

    def log_uniform(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    while True:
        kind = rng.choice(["encode", "encode", "encode", "logmel", "decode", "pipeline"])
        a, b = log_uniform(MIN_SECONDS, MAX_SECONDS), log_uniform(MIN_SECONDS, MAX_SECONDS)
        p = int(round(log_uniform(8, MAX_PROMPT)))
        hush = kind == "pipeline" or rng.random() < 0.8
        c = _case("", kind, rng.choice(MODELS), int(round(log_uniform(1, MAX_STREAMS))), round(min(a, b), 2), round(max(a, b), 2),
                  lengths=rng.randrange(1, 1 << 30), hush=hush, mel_bf16=rng.random() < 0.5, out_bf16=rng.random() < 0.5)
        if kind in ("decode", "pipeline"):
            c["prompt_lo"], c["prompt_hi"] = max(1, p // 2), p
        del c["name"]
        if work(c)["flops"] <= largest and sum(_frames(c)) + 50 * c["streams"] <= MAX_TOTAL_FRAMES:
            return c


# ---- sizes of a case --------------------------------------------------------------------------------------------
def _frames(case):
    """Payload frames of every stream (10 ms each), log-uniform in the case's range."""
    r = np.random.default_rng(case["lengths"])
    lo, hi = case["lo_s"], case["hi_s"]
    return [max(1, int(round(100 * lo * (hi / lo) ** u))) for u in r.random(case["streams"])]


def _hush_frames(case):
    return synth.HUSH_FRAMES if case["hush"] else 0


def _tokens(case):
    return [(t + _hush_frames(case) + 1) // 2 for t in _frames(case)]


def _prompts(case):
    r = np.random.default_rng(case["lengths"] + 1)
    return [int(v) for v in r.integers(case["prompt_lo"], case["prompt_hi"] + 1, size=case["streams"])]


# ---- what a program keeps: one handle per model -------------------------------------------------------------------
_kept = {}


def _keep(key, make):
    if key not in _kept:
        _kept[key] = make()
    return _kept[key]


def _normal(gen, *shape):
    return (torch.randn(shape, generator=gen, device="cuda") * synth.WEIGHT_STD).cpu().numpy()


def _mel_values(gen, *shape):
    x = torch.randn(shape, generator=gen, device="cuda") * synth.MEL_STD + synth.MEL_MEAN
    return x.clamp_(-1.0, 1.0)


def _generator(*seeds):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(np.random.SeedSequence([int(s) for s in seeds]).generate_state(1, np.uint64)[0] >> 1))
    return g


def _encoder(model, hush_frames):
    def make():
        s = synth.SHAPES[model]
        g = _generator(1, MODELS.index(model))
        d, f = s.d_model, s.d_mlp
        one, zero = np.ones(d, np.float32), np.zeros(d, np.float32)
        w = {"conv1_w": _normal(g, d, s.n_mels, 3), "conv1_b": _normal(g, d), "conv2_w": _normal(g, d, d, 3), "conv2_b": _normal(g, d),
             "lnf_g": one, "lnf_b": zero, "layers": []}
        for _ in range(s.n_layers):
            w["layers"].append({"ln1_g": one, "ln1_b": zero, "wq": _normal(g, d, d), "bq": _normal(g, d), "wk": _normal(g, d, d), "bk": None,
                                "wv": _normal(g, d, d), "bv": _normal(g, d), "wo": _normal(g, d, d), "bo": _normal(g, d), "ln2_g": one,
                                "ln2_b": zero, "w1": _normal(g, f, d), "b1": _normal(g, f), "w2": _normal(g, d, f), "b2": _normal(g, d)})
        hush = _mel_values(g, hush_frames, s.n_mels).cpu().numpy() if hush_frames else None
        cfg = wf.make_config(s, hush_frames, MAX_STREAMS, MAX_TOTAL_FRAMES, int(100 * MAX_SECONDS) + synth.HUSH_FRAMES)
        return wf.Encoder(cfg, w, hush)

    return _keep(("encoder", model, hush_frames), make)


def _decoder(model):
    def make():
        s = synth.DEC_SHAPES[model]
        g = _generator(2, MODELS.index(model))
        d, f = s.d_model, s.d_mlp
        one, zero = np.ones(d, np.float32), np.zeros(d, np.float32)
        w = {"tok_emb": _normal(g, s.n_vocab, d), "pos_emb": _normal(g, s.n_ctx, d), "lnf_g": one, "lnf_b": zero, "layers": []}
        for _ in range(s.n_layers):
            lw = {k: one for k in ("ln1_g", "lnx_g", "ln2_g")}
            lw.update({k: zero for k in ("ln1_b", "lnx_b", "ln2_b")})
            lw.update({k: _normal(g, d, d) for k in ("wq", "wk", "wv", "wo", "xwq", "xwk", "xwv", "xwo")})
            lw.update({k: _normal(g, d) for k in ("bq", "bv", "bo", "xbq", "xbv", "xbo", "b2")})
            lw.update({"w1": _normal(g, f, d), "b1": _normal(g, f), "w2": _normal(g, d, f)})
            w["layers"].append(lw)
        return wf.Decoder(s, w, MAX_STREAMS, MAX_TOTAL_FRAMES // 2 + MAX_STREAMS, MAX_STREAMS * MAX_PROMPT)

    return _keep(("decoder", model), make)


def _audio(gen, n):
    """Four tones with slow envelopes over white noise, clipped to [-1, 1]."""
    t = torch.arange(n, device="cuda", dtype=torch.float32) / synth.SAMPLE_RATE
    x = 0.02 * torch.randn(n, generator=gen, device="cuda")
    u = torch.rand(4, 5, generator=gen, device="cuda")
    for k in range(4):
        f, a, e = 80 + 3720 * u[k, 0], 0.05 + 0.2 * u[k, 1], 0.3 + 2.7 * u[k, 2]
        env = 0.5 * (1 + torch.sin(2 * math.pi * (e * t + u[k, 3])))
        x += a * env * torch.sin(2 * math.pi * (torch.remainder(f * t, 1.0) + u[k, 4]))
    return x.clamp_(-1.0, 1.0)


def _frontend(model, hush):
    def make():
        word = _audio(_generator(3, MODELS.index(model)), synth.HUSH_SAMPLES).cpu().numpy() if hush else None
        return wf.Frontend(synth.SHAPES[model].n_mels, word, MAX_STREAMS, MAX_TOTAL_FRAMES * SPF)

    return _keep(("frontend", model, hush), make)


# ---- one call ----------------------------------------------------------------------------------------------------
def prepare(case, seed):
    kind, model = case["kind"], case["model"]
    s = synth.SHAPES[model]
    g = _generator(4, seed)
    frames = _frames(case)
    offsets = np.concatenate([[0], np.cumsum(frames)[:-1]])
    st = {"kind": kind, "out_dtype": torch.bfloat16 if case["out_bf16"] else torch.float32,
          "mel_dtype": torch.bfloat16 if case["mel_bf16"] else torch.float32}
    if kind == "encode":
        st["encoder"] = _encoder(model, _hush_frames(case))
        mel = _mel_values(g, sum(frames), s.n_mels)
        if not case["hush"]:              # the padded window: what a 6 s buffer leaves empty is silence
            for o, t in zip(offsets, frames):
                if t > 2400:
                    mel[int(o) + 600:int(o) + t] = synth.PAD_VALUE
        st.update(mel=mel.to(st["mel_dtype"]), offsets=offsets.astype(np.int32), frames=np.asarray(frames, np.int32))
    if kind in ("logmel", "pipeline"):
        st["frontend"] = _frontend(model, case["hush"])
        st.update(audio=_audio(g, sum(frames) * SPF), sample_offsets=(offsets * SPF).astype(np.int64),
                  samples=np.asarray([t * SPF for t in frames], np.int32))
    if kind == "pipeline":
        st["encoder"] = _encoder(model, 0)            # the hush word is already in the audio
        st["features"] = np.asarray([t + _hush_frames(case) for t in frames], np.int32)
    if kind in ("decode", "pipeline"):
        st["decoder"] = _decoder(model)
        ds = synth.DEC_SHAPES[model]
        tokens, prompts = _tokens(case), _prompts(case)
        st["prompts"] = [torch.randint(ds.n_vocab, (p,), generator=g, device="cuda").cpu().numpy().astype(np.int32) for p in prompts]
        st["cross_kv"] = torch.empty((ds.n_layers, sum(tokens), 2 * ds.d_model), device="cuda", dtype=torch.bfloat16)
        if kind == "decode":
            st["enc"] = torch.randn((sum(tokens), s.d_model), generator=g, device="cuda").to(torch.bfloat16)
            st["cu"] = np.concatenate([[0], np.cumsum(tokens)]).astype(np.int32)
    return st


def run(st):
    kind = st["kind"]
    if kind == "encode":
        return st["encoder"].encode(st["mel"], st["offsets"], st["frames"], out_dtype=st["out_dtype"])
    if kind == "logmel":
        return st["frontend"].logmel(st["audio"], st["sample_offsets"], st["samples"], out_dtype=st["mel_dtype"])
    if kind == "decode":
        enc, cu = st["enc"], st["cu"]
    else:
        mel, cu_frames = st["frontend"].logmel(st["audio"], st["sample_offsets"], st["samples"], out_dtype=st["mel_dtype"])
        enc, cu = st["encoder"].encode(mel, cu_frames[:-1], st["features"], out_dtype=torch.bfloat16)
    kv = st["decoder"].cross_kv(enc, out=st["cross_kv"])
    r = st["decoder"].prefill(st["prompts"], cu, kv, hidden_dtype=st["out_dtype"], want_logits=True, want_self_kv=True)
    return {"states": enc, "cross_kv": kv, "hidden": r["hidden"], "logits": r["logits"], "self_kv": r["self_kv"]}


# ---- what a call cannot do without --------------------------------------------------------------------------------
def work(case):
    kind, model = case["kind"], case["model"]
    s, ds = synth.SHAPES[model], synth.DEC_SHAPES[model]
    d, f, N, C = s.d_model, s.d_mlp, s.n_layers, s.n_mels
    h = _hush_frames(case)
    frames = [t + h for t in _frames(case)]
    tokens = [(t + 1) // 2 for t in frames]
    F, M = sum(frames), sum(tokens)
    mel_size, out_size = (2 if case["mel_bf16"] else 4), (2 if case["out_bf16"] else 4)
    bytes_, flops = 0.0, 0.0
    if kind in ("logmel", "pipeline"):
        # a real transform of 400 points (2.5 n log2 n), power, two filters under each bin, log and scaling
        flops += F * (2.5 * 400 * math.log2(400) + 3 * 201 + 4 * 201 + 4 * C)
        bytes_ += sum(_frames(case)) * SPF * 4 + (F * C * mel_size if kind == "logmel" else 0)
    if kind in ("encode", "pipeline"):
        flops += 2.0 * F * 3 * C * d + 2.0 * M * 3 * d * d + N * (2.0 * M * d * (4 * d + 2 * f) + 4.0 * d * sum(t * t for t in tokens))
        bytes_ += 2.0 * (3 * C * d + 3 * d * d + N * (4 * d * d + 2 * d * f))          # weights
        bytes_ += sum(_frames(case)) * C * mel_size if kind == "encode" else 0
        bytes_ += M * d * (out_size if kind == "encode" else 2)
    if kind in ("decode", "pipeline"):
        prompts = _prompts(case)
        P, B, V = sum(prompts), case["streams"], ds.n_vocab
        flops += N * (2.0 * M * d * 2 * d + 2.0 * P * d * (6 * d + 2 * f)) + 2.0 * B * d * V
        flops += N * (sum(2.0 * p * (p + 1) * d for p in prompts) + sum(4.0 * p * t * d for p, t in zip(prompts, tokens)))
        bytes_ += 2.0 * N * (8 * d * d + 2 * d * f) + 2.0 * V * d                       # weights and the embedding
        bytes_ += (2.0 * M * d if kind == "decode" else 0) + 2.0 * 2 * N * M * 2 * d    # states in; cross K/V out, and in again
        bytes_ += 2.0 * N * P * 2 * d + P * d * out_size + 4.0 * B * V
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """About four times what another order of the sums shows: every stream encoded or prefilled alone (other tile sizes)
    against the batch gives 2.9e-3 .. 4.1e-3 and at most 0.023 on the encoder states, 4.9e-3 .. 5.6e-3 and at most 0.033 on
    the decoder side; the log-mel in fp32 is 2.4e-7 and at most 8.3e-5 (a nearly empty filter) from the same in fp64 over
    six seeds, and in bf16 a value next to a rounding boundary moves by one unit in the last place (2^-7 at most)."""
    if case["kind"] == "logmel":
        return {"rel": 1e-3, "max": 1e-2} if case["mel_bf16"] else {"rel": 1e-6, "max": 3.5e-4}
    return {"rel": 1.2e-2, "max": 0.1} if case["kind"] == "encode" else {"rel": 1.5e-2, "max": 0.13}
