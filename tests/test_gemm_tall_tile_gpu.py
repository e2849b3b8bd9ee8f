"""Products whose large tiles end in a poorly filled round run on 192 x 256 tiles: both sides of the rule, ragged last rows, one and two
rounds of the chip, against float64; the same bits as the large tiles; an operand of more than 2 GiB."""
import pytest

from paper_2412_11272_amd import binding as wf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,tall", [(2600, 4096, 1024, True), (3072, 4096, 768, True), (3073, 4096, 768, False), (2561, 4096, 832, True), (2560, 4096, 704, False),
                                        (6420, 3840, 1280, True), (6401, 3840, 768, True), (6145, 3840, 768, False), (6000, 4096, 1024, False)])
@pytest.mark.parametrize("epi", [0, 1])
def test_product(M, N, K, tall, epi):
    import torch
    if M > 6144 and epi == 1 and K < 1280:         # two rounds of the chip with GELU: deeper reductions only
        tall = False
    assert (wf.gemm_kernel_choice(M, N, K, epi) == (1, 192, 256)) == tall
    g = torch.Generator(device="cuda").manual_seed(M + N + K + epi)
    a = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    w = (0.05 * torch.randn(N, K, generator=g, device="cuda")).bfloat16()
    b = torch.randn(N, generator=g, device="cuda")
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    wf.op_linear(wf.WF_PRECISION_BF16, a, w, b, out, epi)
    ref = a.double() @ w.double().T + b.double()
    if epi:
        ref = torch.nn.functional.gelu(ref)
    # exact products of bf16 values, fp32 sums, the result rounded to bf16 (2^-9; GELU 4.7e-4 before it)
    assert float((out.double() - ref).abs().max() / ref.abs().max()) <= 5e-3


@pytest.mark.parametrize("M,N,K", [(2600, 4096, 1024), (2561, 4096, 832), (6420, 3840, 1280), (8800, 2816, 1280)])
@pytest.mark.parametrize("epi", [0, 1])
def test_same_bits_as_the_large_tiles(M, N, K, epi):
    """A batch takes this tile on one lane and not on several, where it has to give the same rows."""
    import torch
    rows = 12001
    assert wf.gemm_kernel_choice(M, N, K, epi) == (1, 192, 256) and wf.gemm_kernel_choice(rows, N, K, epi)[0] == 2
    g = torch.Generator(device="cuda").manual_seed(M + N + epi)
    a = torch.randn(rows, K, generator=g, device="cuda").bfloat16()
    w = (0.05 * torch.randn(N, K, generator=g, device="cuda")).bfloat16()
    b = torch.randn(N, generator=g, device="cuda")
    full = torch.empty((rows, N), dtype=torch.bfloat16, device="cuda")
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    wf.op_linear(wf.WF_PRECISION_BF16, a, w, b, full, epi)
    wf.op_linear(wf.WF_PRECISION_BF16, a[:M], w, b, out, epi)
    assert torch.equal(out, full[:M])


def test_operand_beyond_2_gib():
    import torch
    M, N, K = 49001, 256, 22016
    assert wf.gemm_kernel_choice(M, N, K, 0) == (1, 192, 256) and M * K * 2 > 1 << 31
    g = torch.Generator(device="cuda").manual_seed(5)
    a = torch.randn(M, K, generator=g, device="cuda", dtype=torch.bfloat16)
    w = (0.05 * torch.randn(N, K, generator=g, device="cuda")).bfloat16()
    b = torch.randn(N, generator=g, device="cuda")
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    wf.op_linear(wf.WF_PRECISION_BF16, a, w, b, out, 0)
    assert bool(torch.isfinite(out).all())
    for rows in (slice(0, 200), slice(M // 2, M // 2 + 200), slice(M - 200, M)):
        ref = a[rows].double() @ w.double().T + b.double()
        # fp32 sums of 22016 products (1e-4), the result rounded to bf16 (2^-9)
        assert float((out[rows].double() - ref).abs().max() / ref.abs().max()) <= 5e-3
