"""Cross-attention keys and values of all layers from one launch: every kernel the grouped product can run on (few rows, one tile
per CU, 128 x 128 and large tiles), a cache with more rows than the batch, one layer, and rows behind the batch left alone."""
import numpy as np
import pytest

from paper_2412_11272_amd import binding as wf
from paper_2412_11272_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [pytest.param(wf.WF_PRECISION_F32, 1e-5, id="f32"), pytest.param(wf.WF_PRECISION_BF16, H.BF16_TOL, id="bf16")])
@pytest.mark.parametrize("d,layers,M", [(128, 1, 5), (256, 3, 1), (256, 3, 33), (384, 4, 300), (256, 5, 1500), (640, 2, 777), (256, 4, 9000), (384, 7, 12001)])
def test_every_layer(d, layers, M, precision, tol):
    import torch
    shape = synth.DecoderShape(d, layers, d // 64, 2 * d, 300, 32)
    w = synth.make_decoder_weights(shape, 5 + d, affine_random=True)
    enc = synth.make_enc_states(M, d, 6)
    dec = wf.Decoder(shape, w, 1, M, 8, precision)
    try:
        x = torch.from_numpy(enc).cuda().to(dec.act_dtype)
        out = torch.full((layers, M + 3, 2 * d), 7.0, device="cuda", dtype=dec.act_dtype)
        got = dec.cross_kv(x, out=out)
        torch.cuda.synchronize()
        assert got.shape == (layers, M + 3, 2 * d) and bool((got[:, M:] == 7.0).all())
        rounded = x.double()
        for l, lw in enumerate(w["layers"]):
            m = np.concatenate([lw["xwk"], lw["xwv"]])
            m = torch.from_numpy(m).cuda().to(dec.act_dtype).double()
            ref = rounded @ m.T + torch.from_numpy(np.concatenate([np.zeros(d), lw["xbv"]])).cuda()
            # the same rounded operands on both sides: fp32 sums, and the rounding of a bf16 result
            assert float((got[l, :M].double() - ref).abs().max() / ref.abs().max()) <= tol, l
    finally:
        dec.close()


def test_more_layers_than_one_launch_reaches():
    """32-bit offsets reach 127 layers of d = 2048: 129 take two launches, the second of which starts within every array."""
    import torch
    d, layers, M = 2048, 129, 3
    shape = synth.DecoderShape(d, layers, d // 64, 128, 128, 8)
    assert (((1 << 31) - 1) // (4 * d * d)) == 127
    one = synth.make_decoder_weights(synth.DecoderShape(d, 3, d // 64, 128, 128, 8), 9, affine_random=True)
    w = dict(one, layers=[dict(one["layers"][l % 3], xbv=one["layers"][l % 3]["xbv"] + np.float32(0.25 * l)) for l in range(layers)])
    dec = wf.Decoder(shape, w, 1, M, 8, wf.WF_PRECISION_BF16)
    try:
        x = torch.from_numpy(synth.make_enc_states(M, d, 6)).cuda().to(dec.act_dtype)
        got = dec.cross_kv(x)
        for l, lw in enumerate(w["layers"]):
            m = torch.from_numpy(np.concatenate([lw["xwk"], lw["xwv"]])).cuda().to(dec.act_dtype).double()
            ref = x.double() @ m.T + torch.from_numpy(np.concatenate([np.zeros(d), lw["xbv"]])).cuda()
            assert float((got[l, :M].double() - ref).abs().max() / ref.abs().max()) <= H.BF16_TOL, l
    finally:
        dec.close()
