"""LayerNorm fused into a product of short rows: every row tile (16, 32, 48, 64) with remainders, one and several rounds of tiles per
workgroup, depths known when compiled (384, 512) and others, against the fp64 oracle."""
import numpy as np
import pytest

from oracle import encoder_oracle as O
from paper_2412_11272_amd import binding as wf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 384, 384), (75, 1152, 384), (500, 1536, 384), (701, 1536, 384), (1024, 1536, 384), (100, 1536, 512), (244, 1536, 512),
                                   (425, 1536, 512), (430, 2048, 512), (601, 2048, 512), (1020, 1536, 512), (1023, 2048, 512), (1, 512, 512),
                                   (47, 128, 64), (333, 1024, 320), (415, 1536, 448), (500, 2048, 448), (64, 256, 128)])
@pytest.mark.parametrize("epi", [0, 1])
def test_ln_product(M, N, K, epi):
    import torch
    r = np.random.default_rng(M + N + K + epi)
    x = (r.standard_normal((M, K)) * 2 + r.standard_normal((M, 1)) * 3).astype(np.float32)
    g, s = (1 + 0.3 * r.standard_normal(K)).astype(np.float32), (0.2 * r.standard_normal(K)).astype(np.float32)
    w = torch.from_numpy((0.05 * r.standard_normal((N, K))).astype(np.float32)).bfloat16()
    b = r.standard_normal(N).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    wf.op_ln_linear(dev(x), dev(g), dev(s), w.cuda(), dev(b), out, epi)
    u = torch.from_numpy(O.layer_norm(x.astype(np.float64), g, s)).float().bfloat16().double().numpy()
    ref = u @ w.double().numpy().T + b
    ref = O.gelu(ref) if epi else ref
    got = out.double().cpu().numpy()
    # the operand is rounded to bf16 on both sides (a value next to a boundary may round the other way: 2^-8 of one of K terms), the
    # result once more (2^-9)
    assert np.abs(got - ref).max() <= 6e-3 * np.abs(ref).max()


def test_weights_of_more_than_4_gib():
    """Short rows against 4 194 432 columns: byte offsets of the weights pass 2^32."""
    import torch
    M, N, K = 2, (1 << 22) + 128, 512
    assert N * K * 2 > 1 << 32
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(M, K, generator=gen, device="cuda")
    w = torch.randn(N, K, generator=gen, device="cuda", dtype=torch.bfloat16)
    b = torch.randn(N, generator=gen, device="cuda")
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    wf.op_ln_linear(x, torch.ones(K, device="cuda"), torch.zeros(K, device="cuda"), w, b, out, 0)
    u = torch.nn.functional.layer_norm(x.double(), (K,)).float().bfloat16().float()
    for n in range(0, N, 1 << 20):
        ref = u @ w[n:n + (1 << 20)].float().T + b[n:n + (1 << 20)]
        # operands rounded on both sides, fp32 sums, the result rounded to bf16 (2^-9)
        assert float((out[:, n:n + (1 << 20)].float() - ref).abs().max() / ref.abs().max()) <= 6e-3, n
