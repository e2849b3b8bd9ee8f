"""End-to-end parity of wf_encode_batch against the CPU oracle on seeded workloads, plus the edge
cases of the ragged path.  Metric and tolerances: max|gpu - oracle| / max|oracle| <= 2e-2 under bf16
MFMA with fp32 accumulation, <= 1e-4 on the fp32 debug path."""
import numpy as np
import pytest

from oracle import encoder_oracle as O
from paper_2412_11272_amd import binding as wf
from paper_2412_11272_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _check(name, precision, affine=False, **kw):
    ref, cu_ref = H.oracle_batch(name, affine)
    got, cu = H.gpu_encode(name, precision, affine, **kw)
    assert cu.tolist() == cu_ref.tolist()
    assert got.shape == ref.shape and np.all(np.isfinite(got))
    err = H.rel_err(got, ref)
    rows = H.per_stream_report(got, ref, cu)
    worst = max(r[2] for r in rows)
    print(f"\n[{name} precision={precision}] global rel err {err:.3e}, worst per-stream {worst:.3e}")
    return err, worst


def test_stem_alone_at_large_tile_batch_size():
    """No transformer block, ~53 k tokens: both convolutions take the 256 x 256 direct-load kernel (gathered
    3-tap windows, taps masked at every stream boundary, GELU + position epilogue); whole output against the
    oracle."""
    err, worst = _check("stem-wide", wf.WF_PRECISION_BF16, affine=True)
    assert err <= 2e-2 and worst <= 2e-2, (err, worst)


@pytest.mark.parametrize("name,affine", [("unit", True), ("unit-sharp", True), ("tiny-ragged", False), ("tiny-sharp", True),
                                         ("cfg1", False), ("cfg2-2s", False), ("cfg2-4s", False), ("cfg2-8s", False),
                                         ("cfg3", False)])
def test_fp32_debug_path(name, affine):
    err, worst = _check(name, wf.WF_PRECISION_F32, affine)
    assert err <= H.F32_TOL and worst <= 2 * H.F32_TOL


@pytest.mark.parametrize("name,affine", [("unit", True), ("unit-sharp", True), ("tiny-ragged", False), ("tiny-sharp", True),
                                         ("cfg1", False), ("cfg2-2s", False), ("cfg2-4s", False), ("cfg2-8s", False),
                                         ("cfg3", False)])
def test_bf16_path(name, affine):
    err, worst = _check(name, wf.WF_PRECISION_BF16, affine)
    assert err <= H.BF16_TOL and worst <= 2 * H.BF16_TOL


def test_bf16_input_and_output_dtypes():
    import torch
    err, _ = _check("tiny-ragged", wf.WF_PRECISION_BF16, mel_dtype=torch.bfloat16, out_dtype=torch.bfloat16)
    assert err <= H.BF16_TOL
    err, _ = _check("unit", wf.WF_PRECISION_F32, True, out_dtype=torch.bfloat16)
    assert err <= 6e-3        # fp32 arithmetic, one final bf16 rounding


def test_final_rows_are_normalised():
    got, _ = H.gpu_encode("tiny-ragged", wf.WF_PRECISION_BF16)
    np.testing.assert_allclose(got.mean(axis=1), 0, atol=1e-4)
    v = got.var(axis=1)
    assert np.all(v > 0.9) and np.all(v < 1.0 + 1e-4)


def test_run_to_run_bitwise_determinism():
    a, _ = H.gpu_encode("tiny-ragged", wf.WF_PRECISION_BF16)
    b, _ = H.gpu_encode("tiny-ragged", wf.WF_PRECISION_BF16)
    assert np.array_equal(a, b)


def test_ragged_equals_per_stream_and_padded_layout_and_reuse():
    """Each stream alone == its rows in the packed batch; a padded mel layout (offsets i*T_max) gives the
    same result as the packed layout; one encoder object serves successive batches of different size."""
    import torch
    wl, w, hush, mels = H.inputs("tiny-ragged")
    ref, cu_ref = H.oracle_batch("tiny-ragged")
    enc = wf.encoder_for_workload(wl, w, hush, wf.WF_PRECISION_BF16)
    try:
        flat, offs, nf = wf.pack_mels(mels)
        full, cu = enc.encode(torch.from_numpy(flat).cuda(), offs, nf)
        full = full.cpu().numpy()
        tmax = max(nf)
        padded = np.full((len(mels) * tmax, wl.shape.n_mels), 9.0, np.float32)     # garbage between streams
        for i, m in enumerate(mels):
            padded[i * tmax:i * tmax + len(m)] = m
        out_p, cu_p = enc.encode(torch.from_numpy(padded).cuda(), [i * tmax for i in range(len(mels))], nf)
        assert cu_p.tolist() == cu.tolist() and np.array_equal(out_p.cpu().numpy(), full)
        for i in (3, 0, 4):                                                        # smaller batches afterwards
            one, cu1 = enc.encode(torch.from_numpy(mels[i]).cuda(), [0], [len(mels[i])])
            one = one.cpu().numpy()
            assert cu1.tolist() == [0, cu[i + 1] - cu[i]]
            assert H.rel_err(one, ref[cu[i]:cu[i + 1]]) <= H.BF16_TOL
            # same arithmetic per row whatever the batch: GEMM rows and attention are independent of neighbours
            # (both batches are small enough for the small-batch kernels; a batch of more than about a thousand
            # tokens runs on other kernels, whose results differ from these at the level of bf16 rounding)
            np.testing.assert_allclose(one, full[cu[i]:cu[i + 1]], atol=1e-5)
        order = [5, 2, 0, 1, 4, 3]
        flat2, offs2, nf2 = wf.pack_mels([mels[i] for i in order])
        out2, cu2 = enc.encode(torch.from_numpy(flat2).cuda(), offs2, nf2)
        out2 = out2.cpu().numpy()
        for pos, i in enumerate(order):
            np.testing.assert_allclose(out2[cu2[pos]:cu2[pos + 1]], full[cu[i]:cu[i + 1]], atol=1e-5)
    finally:
        enc.close()


def test_hush_disabled_equals_caller_appended_hush():
    import torch
    wl, w, hush, mels = H.inputs("unit", True)
    got, cu = H.gpu_encode("unit", wf.WF_PRECISION_F32, True)
    cfg = wf.make_config(wl.shape, 0, len(mels), sum(len(m) + len(hush) for m in mels), max(len(m) for m in mels) + len(hush),
                         wf.WF_PRECISION_F32)
    enc = wf.Encoder(cfg, w, None)
    try:
        flat, offs, nf = wf.pack_mels([np.concatenate([m, hush]) for m in mels])
        out, cu2 = enc.encode(torch.from_numpy(flat).cuda(), offs, nf)
        assert cu2.tolist() == cu.tolist()
        assert np.array_equal(out.cpu().numpy(), got)
    finally:
        enc.close()


def test_capacity_and_argument_errors_on_a_live_encoder():
    import torch
    wl, w, hush, mels = H.inputs("unit", True)
    enc = wf.encoder_for_workload(wl, w, hush, wf.WF_PRECISION_BF16)
    try:
        flat, offs, nf = wf.pack_mels(mels)
        mel = torch.from_numpy(flat).cuda()
        with pytest.raises(wf.WfError) as e:
            enc.encode(mel, offs, nf, out=torch.empty((10, wl.shape.d_model), device="cuda"))
        assert e.value.code == wf.WF_E_CAPACITY and "out_capacity" in str(e.value)
        with pytest.raises(wf.WfError) as e:
            enc.encode(mel, list(offs) + [0], list(nf) + [5])
        assert e.value.code == wf.WF_E_CAPACITY
        with pytest.raises(wf.WfError) as e:
            enc.encode(mel, [0], [max(nf) + 1])
        assert e.value.code == wf.WF_E_CAPACITY
        with pytest.raises(wf.WfError) as e:
            enc.encode(mel, [-1], [5])
        assert e.value.code == wf.WF_E_INVALID_ARG
        out, _ = enc.encode(mel, offs, nf)                   # still usable after rejected calls
        torch.cuda.synchronize()
        ref, _ = H.oracle_batch("unit", True)
        assert H.rel_err(out.cpu().numpy(), ref) <= H.BF16_TOL
    finally:
        enc.close()


def test_maximum_length_stream_and_single_frame_stream():
    """30 s + hush = 1525 tokens (the longest stream any configuration produces) next to a 1-frame stream."""
    import torch
    shape = synth.SHAPES["tiny"]
    wl = synth.Workload("edge-max", shape, [3000, 1, 2], seed_index=9)
    w, hush, mels = synth.materialize(wl)
    ref, cu_ref = O.encode_batch(w, shape.n_heads, mels, hush)
    enc = wf.encoder_for_workload(wl, w, hush, wf.WF_PRECISION_BF16)
    try:
        flat, offs, nf = wf.pack_mels(mels)
        out, cu = enc.encode(torch.from_numpy(flat).cuda(), offs, nf)
        assert cu.tolist() == [0, 1525, 1551, 1577] == cu_ref.tolist()
        assert H.rel_err(out.cpu().numpy(), ref) <= H.BF16_TOL
    finally:
        enc.close()


def test_kernel_stats_cover_every_launch():
    import torch
    wl, w, hush, mels = H.inputs("tiny-ragged")
    enc = wf.encoder_for_workload(wl, w, hush, wf.WF_PRECISION_BF16)
    try:
        flat, offs, nf = wf.pack_mels(mels)
        mel = torch.from_numpy(flat).cuda()
        enc.set_profiling(True)
        enc.encode(mel, offs, nf)
        st = {s["name"]: s for s in enc.kernel_stats()}
        n = wl.shape.n_layers
        assert st["gemm_qkv"]["launches"] == n and st["attention"]["launches"] == n
        # a batch this small (868 tokens) normalises inside the QKV and fc1 kernels: no LayerNorm launches in the blocks
        assert st["layernorm"]["launches"] == 0
        assert st["prep_pack_hush"]["launches"] == 1 and st["layernorm_final"]["launches"] == 1
        assert sum(s["launches"] for s in st.values()) == 4 + 5 * n
        assert all(s["total_ms"] > 0 for s in st.values() if s["launches"])
        enc.set_profiling(False)
        enc.encode(mel, offs, nf)
        assert sum(s["launches"] for s in enc.kernel_stats()) == 0
    finally:
        enc.close()

def test_many_short_streams():
    """400 streams of 1..40 frames (rows of the work list, index arrays and prefix sums far outnumber the
    tiles): both precisions against the oracle."""
    import torch
    shape = synth.SHAPES["unit"]
    rng = np.random.default_rng(400)
    nf = [int(x) for x in rng.integers(1, 41, size=400)]
    wl = synth.Workload("many-short", shape, nf, hush_frames=5, seed_index=11)
    w, hush, mels = synth.materialize(wl)
    ref, cu_ref = O.encode_batch(w, shape.n_heads, mels, hush)
    for precision, tol in ((wf.WF_PRECISION_BF16, 2e-2), (wf.WF_PRECISION_F32, 1e-4)):
        enc = wf.encoder_for_workload(wl, w, hush, precision)
        flat, offs, n = wf.pack_mels(mels)
        out, cu = enc.encode(torch.from_numpy(flat).cuda(), offs, n)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy()
        enc.close()
        assert cu.tolist() == cu_ref.tolist()
        assert H.rel_err(got, ref) <= tol


# Residual products of few rows on a wide model leave partial sums to the LayerNorm behind them: two to four parts, parts of
# unequal depth, tiles of 32 to 128 rows with a ragged last one, one product of a block cut and the other not.
@pytest.mark.parametrize("d,heads,frames,hush", [(1280, 20, [150], 0), (1280, 20, [800], 50), (1280, 20, [600, 601, 1], 50), (1024, 16, [799], 50),
                                                 (768, 12, [301, 300], 25), (768, 12, [2049], 0), (640, 10, [65], 0)])
def test_cut_residual_products(d, heads, frames, hush):
    import torch
    wl = synth.Workload("wide", synth.Shape(80, d, 2, heads, 4 * d), frames, hush_frames=hush, seed_index=11)
    w, h, mels = synth.materialize(wl, affine_random=True)
    ref, cu_ref = O.encode_batch(w, heads, mels, h if hush else None)
    enc = wf.encoder_for_workload(wl, w, h, wf.WF_PRECISION_BF16)
    try:
        flat, offs, nf = wf.pack_mels(mels)
        mel = torch.from_numpy(flat).cuda()
        out, cu = enc.encode(mel, offs, nf)
        got = out.float().cpu().numpy()
        again = enc.encode(mel, offs, nf)[0].float().cpu().numpy()
    finally:
        enc.close()
    assert cu.tolist() == cu_ref.tolist() and np.array_equal(got, again)
    assert np.all(np.isfinite(got)) and H.rel_err(got, ref) <= H.BF16_TOL


# Batches whose lanes have sizes on the other side of a kernel choice than the batch as a whole: the attention form (twice), the
# small-batch products, a second MLP product whose reduction is cut, 192 x 256 tiles (on one lane only)
@pytest.mark.parametrize("d,heads,d_mlp,tokens", [(384, 6, 1536, [1408, 1280, 1525, 1525, 1525, 1000]), (384, 6, 1536, [1280, 1300, 1525, 1525, 1525, 1040]),
                                                  (384, 6, 1536, [500, 8000]), (128, 2, 4096, [1500] * 6), (1280, 20, 2816, [1500] * 5 + [1300])])
def test_lanes_do_not_change_a_bit(d, heads, d_mlp, tokens):
    import torch
    wl = synth.Workload("lanes", synth.Shape(80, d, 2, heads, d_mlp), [2 * t for t in tokens], hush_frames=0, seed_index=4)
    w, _, mels = synth.materialize(wl, affine_random=True)
    enc = wf.encoder_for_workload(wl, w, None, wf.WF_PRECISION_BF16)
    try:
        flat, offs, nf = wf.pack_mels(mels)
        mel = torch.from_numpy(flat).cuda()
        outs = []
        for lanes in (1, 2, 3, 4):
            enc.set_lanes(lanes)
            outs.append(enc.encode(mel, offs, nf)[0])
        for out in outs[1:]:
            assert torch.equal(out, outs[0])
    finally:
        enc.close()


def test_packed_features_beyond_4_gib():
    """The packed log-mel matrix is the only one that may be wider than the widest activation (2 x 80 bins against 128) and so
    pass 4 GiB in a configuration that is accepted: 9400 streams of 30 s that all read the same frames give the same rows."""
    import torch
    shape = synth.Shape(80, 128, 1, 2, 128)
    B, T = 9400, 3000
    w = synth.make_weights(shape, 71)
    mel = synth.make_mels(shape, [T], 72)[0]
    assert B * T * shape.n_mels * 2 > 1 << 32
    enc = wf.Encoder(wf.make_config(shape, 0, B, B * T, T, wf.WF_PRECISION_BF16), w, None)
    try:
        out, cu = enc.encode(torch.from_numpy(mel).cuda(), [0] * B, [T] * B, out_dtype=torch.bfloat16)
        rows = out.view(B, T // 2, 128)
        assert cu[-1] == B * (T // 2) and torch.isfinite(rows[0]).all()
        assert torch.equal(rows[1:], rows[:1].expand(B - 1, -1, -1))
        one, _ = enc.encode(torch.from_numpy(mel).cuda(), [0], [T])
        assert H.rel_err(one.float().cpu().numpy(), rows[0].double().cpu().numpy()) <= H.BF16_TOL
    finally:
        enc.close()
