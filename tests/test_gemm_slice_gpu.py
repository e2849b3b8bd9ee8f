"""The product whose reduction is shared by the eight waves of a workgroup: every tile, remainders of rows and columns of tiles,
reductions of fewer K steps than waves and with every remainder of waves, whole encoders whose products it runs (row-major and
panel operands, both convolutions), against the fp64 oracle."""
import numpy as np
import pytest

from oracle import encoder_oracle as O
from paper_2412_11272_amd import binding as wf
from paper_2412_11272_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


# 16 x 16, 16 x 32, 32 x 32, 64 x 32 and 64 x 64 tiles (by the estimate of pick_slice), one row and rows off the tile's edge
SLICED = [(75, 384, 1536), (33, 256, 448), (15, 128, 576), (100, 1280, 1280), (244, 512, 2048), (150, 512, 512), (250, 512, 1088), (425, 512, 1984),
          (925, 384, 1536), (700, 384, 1024), (1020, 1024, 512), (64, 2304, 768), (1, 384, 384), (17, 384, 5056), (1024, 512, 448), (1023, 1024, 448),
          (600, 1536, 448), (33, 128, 512)]
# in the model's residual updates only: with bf16 results the pipelined kernel takes them
SLICED_RESIDUAL = [(100, 1280, 5120), (17, 640, 5056), (1023, 384, 384)]
# beside them: short reductions on four waves, one tile too many
OTHERS = [(1, 384, 64), (1024, 512, 192), (1023, 384, 128), (1024, 1024, 64), (700, 1536, 384), (130, 1152, 384), (1024, 256, 320)]


def _sliced(M, N, K, epi):
    return wf.gemm_kernel_choice(M, N, K, epi)[0] == 0 and wf.gemm_small_choice(M, N, K, epi)[0] == 8


def test_shapes_reach_every_tile():
    assert all(_sliced(*s, epi) for s in SLICED for epi in (0, 1, 2))
    assert all(_sliced(*s, 2) for s in SLICED_RESIDUAL) and not any(_sliced(*s, epi) for s in SLICED_RESIDUAL for epi in (0, 1))
    assert not any(_sliced(*s, epi) for s in OTHERS for epi in (0, 1))
    tiles = [wf.gemm_small_choice(*s, 0)[1:] for s in SLICED]
    assert set(tiles) == {(16, 16), (16, 32), (32, 32), (64, 32), (64, 64)}
    ragged = {t for (M, _, _), t in zip(SLICED, tiles) if M % t[0]}
    assert ragged == set(tiles)                    # each of them with a last row tile that is not full
    assert {-(-K // 64) % 8 for _, _, K in SLICED} >= {0, 1, 6, 7}      # waves with one K step less, and with none


@pytest.mark.parametrize("M,N,K", SLICED + SLICED_RESIDUAL + OTHERS)
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_product(M, N, K, epi):
    import torch
    g = torch.Generator().manual_seed(M + N + K + epi)
    a = torch.randn(M, K, generator=g).bfloat16()
    w = (0.05 * torch.randn(N, K, generator=g)).bfloat16()
    b, x = torch.randn(N, generator=g), torch.randn(M, N, generator=g)
    out = x.cuda() if epi == 2 else torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    wf.op_linear(wf.WF_PRECISION_BF16, a.cuda(), w.cuda(), b.cuda(), out, epi)
    ref = a.double() @ w.double().T + b.double()
    ref = O.gelu(ref.numpy()) if epi == 1 else (ref + x if epi == 2 else ref).numpy()
    got = out.double().cpu().numpy()
    # exact products of bf16 values, fp32 sums of up to 5120 of them (2e-5), or the rounding of the result to bf16 (2^-9, GELU 4.7e-4)
    assert np.abs(got - ref).max() <= (2e-5 if epi == 2 else 5e-3) * np.abs(ref).max()


# (d, heads, n_mels, frames): few enough tokens for every product of a wide block, for some of them, for none; a first convolution
# whose taps straddle K steps (80 bins) and one whose do not (128); streams of one frame
@pytest.mark.parametrize("d,heads,mels,frames", [(1280, 20, 128, [30]), (1280, 20, 128, [126, 1]), (768, 12, 80, [99, 1, 2]), (1024, 16, 80, [255]),
                                                 (768, 12, 80, [600, 401]), (640, 10, 128, [1281]), (512, 8, 80, [1, 437, 3]), (384, 6, 80, [2046])])
def test_encoder(d, heads, mels, frames):
    import torch
    wl = synth.Workload("slice", synth.Shape(mels, d, 2, heads, 4 * d), frames, hush_frames=0, seed_index=12)
    w, _, mel = synth.materialize(wl, affine_random=True)
    ref, cu_ref = O.encode_batch(w, heads, mel, None)
    enc = wf.encoder_for_workload(wl, w, None, wf.WF_PRECISION_BF16)
    try:
        flat, offs, nf = wf.pack_mels(mel)
        x = torch.from_numpy(flat).cuda()
        out, cu = enc.encode(x, offs, nf)
        again = enc.encode(x, offs, nf)[0]
    finally:
        enc.close()
    assert cu.tolist() == cu_ref.tolist() and torch.equal(out, again)
    assert H.rel_err(out.cpu().numpy(), ref) <= H.BF16_TOL
