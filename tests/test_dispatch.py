"""Which kernel a GEMM of given sizes goes to (rpo_gemm_plan: the library's own choice, made on the host)."""
import pytest

from paper_2601_19404_amd import binding as rpo


@pytest.fixture(autouse=True)
def default_path():
    rpo.rpo_set_kernel_path(0)


# measured us of the tiles and of the waves: below, the faster one by 10 % or more
@pytest.mark.parametrize("M,N,K,waves", [
    (64, 64, 1024, True), (64, 4096, 16, False), (64, 4096, 128, True), (1000, 1024, 128, False), (1000, 1024, 512, True),
    (150, 4096, 32, False), (1100, 512, 32, False), (16000, 64, 64, False), (16000, 64, 2048, True), (2000, 2048, 512, False)])
def test_generic_fp32_goes_to_the_faster_kernel(M, N, K, waves):
    for epilogue in (0, 1, 2):
        assert rpo.rpo_gemm_plan(M, N, K, rpo.RPO_F32, epilogue)["waves"] == waves
    if N % 2 == 0:
        assert rpo.rpo_gemm_plan(M, N, K, rpo.RPO_F32, 3)["waves"]


@pytest.mark.parametrize("M,N,K,waves", [   # K no multiple of 8: not on the matrix cores
    (64, 64, 1020, True), (150, 4096, 30, False), (150, 4096, 2044, False), (1000, 1024, 2044, False), (1000, 512, 1020, True),
    (1000, 512, 2044, False), (64, 8192, 2044, False), (2500, 128, 510, True), (200, 1000, 2044, True), (16000, 64, 510, False)])
def test_generic_bf16_goes_to_the_faster_kernel(M, N, K, waves):
    plan = rpo.rpo_gemm_plan(M, N, K, rpo.RPO_BF16, 0)
    assert plan["kernel"] == "gemm_generic" and plan["waves"] == waves


@pytest.mark.parametrize("M,N,K,turn_mb,weights_pass", [
    (8, 2048, 1536, 0, False), (8, 4096, 4096, 0, False), (8, 5120, 20480, 0, False), (24, 37888, 3584, 0, False),
    (64, 50000, 3584, 0, True),                                                                # a matrix by itself
    (8, 2048, 1536, 183, False), (8, 151936, 1536, 183, False), (64, 2048, 1536, 246, True), (100, 2048, 1536, 2600, True)])
def test_weights_that_the_caches_hold_carry_no_hint(M, N, K, turn_mb, weights_pass):
    """Weights that come round again before the caches have lost them (a matrix used over and over, a small model) are
    asked for as usual: with the non-temporal hint a decode step of a model of 90 MB took 1.1 times as long."""
    assert rpo.rpo_gemm_plan(M, N, K, rpo.RPO_BF16, 0, 0, turn_mb << 20)["weights_pass"] == weights_pass


@pytest.mark.parametrize("M,N,K,kernel,splits", [
    (900, 5120, 17408, "gemm256x192", 3), (1024, 5120, 17408, "gemm256x192", 3), (1280, 3584, 18944, "gemm256x192", 3),
    (900, 1536, 8960, "gemm256x192", 8), (700, 1536, 8960, "gemm128", 3), (2500, 1536, 8960, "gemm128", 1),
    (1920, 3584, 18944, "gemm128", 1), (648, 3584, 18944, "gemm128", 1), (1024, 4096, 4096, "gemm128", 1), (4200, 5120, 17408, "gemm256x192", 1)])
def test_deep_chunks_split_k_over_wide_tiles_where_that_is_cheaper(M, N, K, kernel, splits):
    """1024 x 5120 x 17408 took 304 us on 128x128 tiles, two of them on some CUs, against 247 in three K ranges."""
    for epilogue in (0, 2):
        plan = rpo.rpo_gemm_plan(M, N, K, rpo.RPO_BF16, epilogue, 96 << 20)
        assert (plan["kernel"], plan["splits"]) == (kernel, splits)
