"""rpo_gemm_nt_noalloc (the entry point that allocates nothing: K-split partial sums in the
library's own fixed device array) against rpo_gemm_nt with a caller-provided workspace: the same
kernels and the same split, so the results are identical bit for bit.  Two calls in a row, the
second on a smaller problem (the array keeps the first call's partial sums), then the size limit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _operands(M, N, K, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    a = torch.randn(M, K, device="cuda", generator=g).to(torch.bfloat16)
    w = (torch.randn(N, K, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    return a, w


def test_noalloc_gemm_matches_workspace_gemm_twice_second_call_smaller():
    from paper_2601_19404_amd import binding as rpo
    rpo.lib()
    rpo.rpo_set_kernel_path(0)
    ws = torch.empty(96 << 20, dtype=torch.uint8, device="cuda")
    # set-up: the first call on a device looks up the array's address, which makes the runtime load
    # the code object that holds it (its 16 MiB are taken then, once, until the process ends)
    a0, w0 = _operands(64, 256, 1024, seed=1)
    rpo.rpo_gemm_nt_noalloc(a0, w0, torch.zeros(64, 256, device="cuda"), 1)
    # skinny problems with a deep K: split along K, partial sums in the scratch (the last three on tiles of 64 rows and
    # in the few-row kernel; 40 x 2048 x 2048 is not split any more)
    for (M, N, K, epi) in ((512, 1536, 8960, 2), (200, 1536, 8960, 2), (96, 768, 4096, 1), (40, 2048, 2048, 3),
                           (40, 2048, 8192, 3), (40, 1536, 8960, 2), (8, 512, 4096, 2)):
        a, w = _operands(M, N, K, seed=M + N)
        n_out = N // 2 if epi == 3 else N
        dt = torch.bfloat16 if epi in (0, 3) else torch.float32
        base = torch.randn(M, n_out, device="cuda").to(dt)
        ref, got = base.clone(), base.clone()
        torch.cuda.synchronize()
        free_before = torch.cuda.mem_get_info()[0]            # device-wide free memory (hipMemGetInfo)
        rpo.rpo_gemm_nt_noalloc(a, w, got, epi)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] >= free_before     # the call took no device memory
        rpo.rpo_gemm_nt(a, w, ref, epi, ws)
        torch.cuda.synchronize()
        assert torch.equal(ref, got), f"M={M} N={N} K={K} epilogue={epi}"
        # and against plain fp32 arithmetic, so that both being wrong together would show
        exact = a.float() @ w.float().t()
        if epi == 3:
            exact = torch.nn.functional.silu(exact[:, :n_out]) * exact[:, n_out:]
        elif epi == 2:
            exact = base.float() + exact
        np.testing.assert_allclose(got.float().cpu().numpy(), exact.cpu().numpy(), atol=0.15, rtol=2e-2)


def test_noalloc_gate_up_beyond_the_scratch_on_unsplit_tiles():
    from paper_2601_19404_amd import binding as rpo
    rpo.lib()
    rpo.rpo_set_kernel_path(0)
    # 24 tiles of 256 x 256 in seven K splits would need 40 MB: 256 x 160 tiles without a split, as without a workspace
    a, w = _operands(700, 2048, 3584, seed=6)
    got, ref = (torch.zeros(700, 1024, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    rpo.rpo_gemm_nt_noalloc(a, w, got, 3)
    rpo.rpo_gemm_nt(a, w, ref, 3, None)
    torch.cuda.synchronize()
    assert torch.equal(ref, got)
    exact = a.float() @ w.float().t()
    exact = torch.nn.functional.silu(exact[:, :1024]) * exact[:, 1024:]
    assert (got.float() - exact).norm() / exact.norm() < 4e-3     # half a last place of bf16


@pytest.mark.parametrize("M,N,K,epi", [(772, 3072, 8192, 2), (846, 3072, 8192, 0), (640, 3584, 4160, 2)])
def test_noalloc_chunk_beyond_the_scratch_on_narrow_tiles(M, N, K, epi):
    """The cheapest K split of the first two takes four ranges of wide tiles, 38 MB and more: the tiles that do with what the
    array holds take them, as rpo_gemm_nt does with 16 MiB."""
    from paper_2601_19404_amd import binding as rpo
    rpo.lib()
    rpo.rpo_set_kernel_path(0)
    free = rpo.rpo_gemm_plan(M, N, K, rpo.RPO_BF16, epi, 1 << 30)
    assert (free["splits"] * M * N * 4 > 16 << 20) == (K == 8192)
    a, w = _operands(M, N, K, seed=7)
    got, ref = (torch.zeros(M, N, device="cuda", dtype=torch.float32 if epi == 2 else torch.bfloat16) for _ in range(2))
    rpo.rpo_gemm_nt_noalloc(a, w, got, epi)
    rpo.rpo_gemm_nt(a, w, ref, epi, torch.empty(16 << 20, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(ref, got)
    exact = a.float() @ w.float().t()
    assert (got.float() - exact).norm() / exact.norm() < (1e-4 if epi == 2 else 4e-3)     # fp32 sums; half a last place of bf16


def test_noalloc_gemm_rejects_what_the_scratch_cannot_hold():
    from paper_2601_19404_amd import binding as rpo
    rpo.lib()
    rpo.rpo_set_kernel_path(0)
    # gate/up-shaped, 128 rows, F = 4160, K = 3584: 65 tiles of 128 x 128, four K splits of
    # 128 x 8320 fp32 partial sums = 17.0 MB, just above the 16 MiB the array holds
    a, w = _operands(128, 8320, 3584, seed=5)
    c = torch.zeros(128, 4160, device="cuda", dtype=torch.bfloat16)
    with pytest.raises(rpo.RpoError) as e:
        rpo.rpo_gemm_nt_noalloc(a, w, c, 3)
    assert e.value.code == rpo.RPO_ENOMEM and "scratch" in str(e.value)
    torch.cuda.synchronize()
    assert float(c.float().abs().max()) == 0.0    # nothing was enqueued
