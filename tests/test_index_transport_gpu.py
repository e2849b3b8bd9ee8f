"""The index arrays of a call travel in the arguments of its first kernel up to 960 ints (stream table of the front end: up to 64
streams) and by a copy beyond: calls on both sides of each limit against the oracles, and a short call after a long one."""
import numpy as np
import pytest

from oracle import decoder_oracle as D
from oracle import encoder_oracle as O
from oracle import frontend_oracle as F
from paper_2412_11272_amd import binding as wf
from paper_2412_11272_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
PREC = [pytest.param(wf.WF_PRECISION_F32, H.F32_TOL, id="f32"), pytest.param(wf.WF_PRECISION_BF16, H.BF16_TOL, id="bf16")]


@pytest.mark.parametrize("precision,tol", PREC)
def test_encoder_stream_counts(precision, tol):
    """4 (B + 1) prefix sums and offsets + 2 ints per work item (one per stream here): 958 ints at B = 159, 964 at B = 160."""
    import torch
    wl, w, hush, _ = H.inputs("unit", True)
    r = np.random.default_rng(5)
    mels = [r.standard_normal((int(t), wl.shape.n_mels)).astype(np.float32).clip(-1, 1) for t in r.integers(1, 40, 161)]
    enc = wf.Encoder(wf.make_config(wl.shape, len(hush), 161, 161 * (40 + len(hush)), 40 + len(hush), precision=precision), w, hush)
    try:
        for B in (160, 159, 161, 1):
            flat, offs, nf = wf.pack_mels(mels[:B])
            out, cu = enc.encode(torch.from_numpy(flat).cuda(), offs, nf)
            assert bool(wf.encode_route(enc.cfg, nf) & wf.WF_ROUTE_INLINE_INDEX) == (B < 160)
            ref, cu_ref = O.encode_batch(w, wl.shape.n_heads, mels[:B], hush)
            assert cu.tolist() == cu_ref.tolist()
            assert H.rel_err(out.cpu().numpy(), ref) <= tol, B
    finally:
        enc.close()


@pytest.mark.parametrize("precision,tol", PREC)
def test_prefill_prompt_lengths(precision, tol):
    """2 ints per prompt token, 3 (B + 1), 2 per work item: 960 ints for prompts of 156, 152 and 160 tokens, 962 with one token more."""
    import torch
    shape = synth.DEC_SHAPES["unit"]
    w = synth.make_decoder_weights(shape, 7, affine_random=True)
    dec = wf.Decoder(shape, w, 3, 60, 480, precision)
    try:
        for lens in ([157, 152, 160], [156, 152, 160], [3, 1, 2]):
            enc = synth.make_enc_states(60, shape.d_model, 8)
            prompts = synth.make_prompts(lens, shape.n_vocab, 9)
            cu = np.array([0, 20, 21, 60], np.int32)
            kv = dec.cross_kv(torch.from_numpy(enc).cuda().to(dec.act_dtype))
            got = dec.prefill(prompts, cu, kv, hidden_dtype=torch.float32)
            ref_h, ref_l, _ = D.prefill_batch(w, shape.n_heads, prompts, enc, cu)
            assert H.rel_err(got["hidden"].cpu().numpy(), ref_h) <= tol, lens
            assert H.rel_err(got["logits"].cpu().numpy(), ref_l) <= tol, lens
    finally:
        dec.close()


@pytest.mark.parametrize("frames", [1, 90], ids=["small-blocks", "large-blocks"])
def test_frontend_stream_counts(frames):
    import torch
    lens = [201 + 160 * (frames + i % 5) + i for i in range(65)]
    hush = synth.make_hush_audio(3)
    audios = [synth.make_audio(n, 40 + i) for i, n in enumerate(lens)]
    fe = wf.Frontend(80, hush, 65, sum(lens) + 65 * len(hush))
    try:
        for B in (65, 64, 63, 2):
            offs = np.concatenate([[0], np.cumsum(lens[:B])[:-1]])
            out, cu = fe.logmel(torch.from_numpy(np.concatenate(audios[:B])).cuda(), offs, lens[:B])
            ref, cu_ref = F.log_mel_batch(audios[:B], hush, 80)
            assert cu.tolist() == cu_ref.tolist()
            # fp32 transform against fp64: 1e-7 of the loudest bin on one 8 decades down is 4e-4 in log10, 1e-4 after the / 4
            assert np.abs(out.cpu().numpy() - ref).max() <= 1e-4, B
    finally:
        fe.close()


def test_lengths_in_a_column():
    """Stream lengths as a [B, 1] array, as they come from an array of records."""
    import torch
    audio = torch.from_numpy(synth.make_audio(4000, 3)).cuda()
    fe = wf.Frontend(80, None, 2, 4000)
    try:
        lens = np.array([[1600], [2400]], np.int32)
        got, cu = fe.logmel(audio, np.array([[0], [1600]]), lens)
        ref, cu_ref = fe.logmel(audio, [0, 1600], [1600, 2400])
        assert cu.tolist() == cu_ref.tolist() and torch.equal(got, ref)
    finally:
        fe.close()
