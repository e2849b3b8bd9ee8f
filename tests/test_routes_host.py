"""Which way a batch takes through the encoder and a product through the small-batch kernels, from the code that decides it (CPU only)."""
import pytest

from paper_2412_11272_amd import binding as wf


def _cfg(n_mels, streams, frames, d=128):
    return wf.WfConfig(n_mels=n_mels, d_model=d, n_layers=0, n_heads=d // 64, d_mlp=128, hush_frames=0, max_streams=streams,
                       max_total_frames=streams * frames, max_frames_per_stream=frames, precision=0, ln_eps=1e-5)


@pytest.mark.parametrize("streams,inline", [(1, True), (159, True), (160, False)])
def test_index_arrays_of_many_streams_go_by_copy(streams, inline):
    """4 (B + 1) prefix sums and offsets + 2 ints per work item, 960 ints in the arguments."""
    flags = wf.encode_route(_cfg(80, streams, 200), [200] * streams)
    assert bool(flags & wf.WF_ROUTE_INLINE_INDEX) == inline


@pytest.mark.parametrize("frames,inline", [(16000, True), (16400, False)])
def test_index_arrays_of_huge_features_go_by_copy(frames, inline):
    """The form that takes the index arrays in its arguments counts its threads in 32 bits: 2^31 of them and more (here 2 streams of
    65 536 features of eight values a frame) go by the other form, not to an error."""
    cfg = _cfg(8 * 65536, 2, frames)
    assert wf.config_check(cfg) == wf.WF_OK
    assert bool(wf.encode_route(cfg, [frames, frames]) & wf.WF_ROUTE_INLINE_INDEX) == inline


@pytest.mark.parametrize("n_mels,frames,d,sliced", [(80, 300, 384, True), (128, 300, 1280, True), (128, 3000, 1280, False), (80, 20000, 384, False),
                                                    (1 << 20, 2000, 128, True), (1 << 20, 2046, 128, True), (1 << 20, 2048, 128, False),
                                                    (1 << 21, 1100, 128, False)])
def test_sliced_first_convolution_reaches_its_windows(n_mels, frames, d, sliced):
    """It addresses the packed features with 32-bit byte offsets: 4 GiB of them and more (2048 frames of 2^20 values) go to a kernel
    that does not, however few the rows."""
    cfg = _cfg(n_mels, 1, frames, d)
    assert wf.config_check(cfg) == wf.WF_OK
    assert bool(wf.encode_route(cfg, [frames]) & wf.WF_ROUTE_SLICED_CONV1) == sliced


def test_a_refused_batch_has_no_route():
    with pytest.raises(wf.WfError):
        wf.encode_route(_cfg(80, 2, 100), [101, 5])


@pytest.mark.parametrize("M,N,K,epi,waves", [(16, 128, 64, 0, 4), (1024, 384, 64, 2, 4), (500, 768, 256, 0, 4), (130, 1536, 320, 2, 4), (1300, 128, 192, 2, 4),
                                             (130, 1152, 384, 0, 4), (300, 1536, 384, 1, 4), (75, 1152, 384, 0, 8), (650, 1152, 384, 0, 8),
                                             (300, 384, 384, 2, 8), (800, 384, 384, 2, 8), (500, 1536, 448, 0, 8), (75, 384, 1536, 2, 8)])
def test_short_reductions_stay_on_four_waves(M, N, K, epi, waves):
    """Eight waves share long reductions; short ones (by measurement up to 320 values, and wide products of 384) lose by it."""
    assert wf.gemm_kernel_choice(M, N, K, epi)[0] == 0
    assert wf.gemm_small_choice(M, N, K, epi)[0] == waves


@pytest.mark.parametrize("M,N,K,epi", [(1, 128, (1 << 24) + 64, 2), (16, 256, 1 << 23, 2), (1024, 128, (1 << 21) + 128, 2)])
def test_operands_beyond_32_bit_offsets_stay_on_pointers(M, N, K, epi):
    """Weights or activations of 4 GiB: the four-wave kernel, whatever the depth."""
    assert max(N, M) * K * 2 >= 1 << 32
    assert wf.gemm_small_choice(M, N, K, epi)[0] == 4
    assert wf.gemm_small_choice(M, N, K // 256 * 64, epi)[0] == 8


@pytest.mark.parametrize("M,N,K,epi,tall", [(8768, 2816, 768, 1, False), (6464, 3840, 1024, 1, False), (8768, 2816, 1280, 1, True), (6464, 3840, 1280, 0, True),
                                            (8768, 2816, 768, 0, True), (3072, 4096, 768, 1, True)])
def test_two_rounds_of_tall_tiles_with_gelu_need_a_deep_reduction(M, N, K, epi, tall):
    assert (wf.gemm_kernel_choice(M, N, K, epi) == (1, 192, 256)) == tall
