"""A product of more tiles than the multiplications that replace the divisions of the tile order are exact for (65 536)."""
import pytest

from paper_2412_11272_amd import binding as wf

pytestmark = pytest.mark.gpu


def test_more_than_65536_tiles():
    import torch
    M, N, K = 128 * 65600 + 5, 128, 64
    assert wf.gemm_kernel_choice(M, N, K, 0) == (2, 128, 128)
    g = torch.Generator(device="cuda").manual_seed(1)
    a = torch.randn(M, K, generator=g, device="cuda", dtype=torch.bfloat16)
    w = (0.05 * torch.randn(N, K, generator=g, device="cuda")).bfloat16()
    b = torch.randn(N, generator=g, device="cuda")
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    wf.op_linear(wf.WF_PRECISION_BF16, a, w, b, out, 0)
    for r0 in range(0, M, 1 << 20):
        ref = a[r0:r0 + (1 << 20)].float() @ w.float().T + b
        # fp32 sums of 64 products on both sides, one result rounded to bf16 (2^-9)
        assert float((out[r0:r0 + (1 << 20)].float() - ref).abs().max() / ref.abs().max()) <= 5e-3, r0
