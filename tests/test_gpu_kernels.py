"""GPU parity of the stand-alone entry points: GEMM, decode attention, sampler, advantages.
Every call goes through the C ABI (paper_2601_19404_amd.binding)."""
import numpy as np
import pytest
import torch

from oracle import advantages as oadv
from oracle import sampler as osampler
from oracle import transformer as T
from paper_2601_19404_amd import synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rpo():
    from paper_2601_19404_amd import binding
    binding.lib()
    yield binding
    binding.rpo_set_kernel_path(0)


def _gemm_case(rpo, M, N, K, dtype, epi, path, seed=0, pad=0, ws_mb=0):
    g = torch.Generator().manual_seed(seed)
    a = torch.randn(M, K + pad, generator=g).to(dtype)[:, :K]
    w = (torch.randn(N, K + pad, generator=g) * 0.1).to(dtype)[:, :K]
    c0 = torch.randn(M, N + pad, generator=g)
    ref = T.lm_head({"lm_head": w.float().numpy()}, a.float().numpy())      # fp64 A @ W^T
    ad, wd = a.cuda(), w.cuda()
    # keep the padded strides on the device too
    ad = torch.empty(M, K + pad, dtype=dtype, device="cuda")[:, :K].copy_(a)
    wd = torch.empty(N, K + pad, dtype=dtype, device="cuda")[:, :K].copy_(w)
    if epi == 0:
        cd = torch.zeros(M, N + pad, dtype=dtype, device="cuda")[:, :N]
    else:
        cd = torch.empty(M, N + pad, dtype=torch.float32, device="cuda")[:, :N].copy_(c0[:, :N])
    ws = torch.empty(ws_mb << 20, dtype=torch.uint8, device="cuda") if ws_mb else None
    rpo.rpo_set_kernel_path(path)
    rpo.rpo_gemm_nt(ad, wd, cd, epi, ws)
    torch.cuda.synchronize()
    got = cd.float().cpu().numpy().astype(np.float64)
    if epi == 2:
        ref = ref + c0[:, :N].numpy().astype(np.float64)
    scale = np.sqrt(K) * 0.1
    if epi == 0 and dtype == torch.bfloat16:
        tol = 2.0 ** -8 * np.abs(ref) + 1e-5 * scale        # one bf16 rounding of the result
    else:
        tol = 1e-6 * np.abs(ref) + 2e-5 * scale             # fp32 accumulation
    err = np.abs(got - ref)
    assert np.all(err <= tol), f"max err {err.max()} at {np.unravel_index(err.argmax(), err.shape)}"


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("shape", [(1, 7, 8), (64, 64, 64), (130, 200, 136), (33, 515, 72), (300, 129, 1024)])
def test_gemm_mfma_bf16(rpo, shape, epi):
    _gemm_case(rpo, *shape, torch.bfloat16, epi, path=0)


@pytest.mark.parametrize("ws_mb", [0, 64])
@pytest.mark.parametrize("shape", [(512, 2048, 1536), (64, 4096, 1536), (200, 1536, 8960), (1000, 640, 1536), (2100, 1536, 512),
                                   (504, 1536, 8960), (8, 1536, 8960)])
def test_gemm_mfma_bf16_model_shapes(rpo, shape, ws_mb):
    """Every tile shape (256x256, 256x128, 128x128, 64x128), with and without K splitting."""
    for epi in (0, 1, 2):
        _gemm_case(rpo, *shape, torch.bfloat16, epi, path=0, seed=3, ws_mb=ws_mb)


@pytest.mark.parametrize("M", [1, 8, 9, 16, 17, 31, 33, 64])
@pytest.mark.parametrize("N,K", [(5, 64), (200, 192), (1536, 1536), (4100, 320), (80, 8960), (16390, 128)])
def test_gemm_skinny_row_and_column_edges(rpo, M, N, K):
    """The few-row kernel: edges of its 8-row loads and 16 / 64-column blocks, fewer K slabs than waves, slabs that
    do not divide among the waves or the K ranges, padded strides, with and without a K-split workspace."""
    for epi in (0, 1, 2):
        for ws_mb, pad in ((0, 0), (64, 8)):
            _gemm_case(rpo, M, N, K, torch.bfloat16, epi, path=0, seed=7, ws_mb=ws_mb, pad=pad)


@pytest.mark.parametrize("M", [5, 16, 30, 50])
@pytest.mark.parametrize("N", [4096, 4104, 8192, 8204, 12288, 12300, 16400, 24580])
def test_gemm_skinny_blocks_per_workgroup(rpo, M, N):
    """One to four 16-column weight blocks per workgroup: the widest of each choice, and one that ends inside a block."""
    for epi in (0, 1, 2):
        _gemm_case(rpo, M, N, 320, torch.bfloat16, epi, path=0, seed=13, pad=8 if N % 8 else 0)


@pytest.mark.parametrize("M,N,K,epi,few", [
    (64, 768, 8192, 0, False), (64, 768, 8192, 3, False), (1, 1536, 8192, 3, True), (24, 2048, 8192, 3, False),
    (33, 512, 4160, 1, False), (17, 512, 6208, 0, False), (64, 3584, 18944, 2, False), (48, 16384, 1024, 0, False),
    (64, 512, 4096, 0, True), (32, 512, 6144, 0, True), (16, 512, 8192, 1, True), (64, 1536, 8960, 2, True),
    (64, 10240, 2048, 0, True), (20, 32768, 256, 1, True), (40, 32768, 4096, 1, False)])
def test_gemm_few_rows_takes_the_faster_kernel(rpo, M, N, K, epi, few):
    """Up to 64 rows: a deep K that the tiles split over the CUs, and the widths where their rows fill better, stay
    with the tiles (64 x 768 x 8192 gate/up: 15 us against 42 when all of it went to the few-row kernel)."""
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a = torch.randn(M, K, device="cuda", generator=g).to(torch.bfloat16)
    w = (torch.randn(N, K, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    n_out = N // 2 if epi == 3 else N
    c = torch.zeros(M, n_out, device="cuda", dtype=torch.bfloat16 if epi in (0, 3) else torch.float32)
    ws = torch.empty(32 << 20, dtype=torch.uint8, device="cuda")
    rpo.rpo_set_kernel_path(0)
    rpo.rpo_profile_start(rpo.KERNEL_IDS["gemm_skinny"], 1)
    rpo.rpo_gemm_nt(a, w, c, epi, ws)
    assert rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm_skinny"])[0] == (1 if few else 0)
    exact = a.float() @ w.float().t()
    if epi == 3:
        exact = torch.nn.functional.silu(exact[:, :n_out]) * exact[:, n_out:]
    # bf16 results: half a last place; the fp32 sums of both sides: a few 2^-24 sqrt(K) of the terms' size
    err = (c.float() - exact).norm() / exact.norm()
    assert err < (4e-3 if epi in (0, 3) else 1e-4)


@pytest.mark.parametrize("M", [65, 128, 129, 250, 512])
@pytest.mark.parametrize("N,K", [(5, 64), (200, 192), (1540, 1536), (2048, 320), (2052, 3584), (4100, 128)])
def test_gemm_skinny_row_groups(rpo, M, N, K):
    """The same kernel in groups of 64 rows: a last group of one row, blocks of 16 / 32 / 64 columns and a column count
    that ends inside one, column blocks that do not divide among the XCDs; past one round of workgroups the tiles."""
    for epi, pad in ((0, 0), (2, 8)):
        _gemm_case(rpo, M, N, K, torch.bfloat16, epi, path=0, seed=11, pad=pad)


@pytest.mark.parametrize("M,N,K,epi,groups", [
    (400, 1100, 512, 2, False), (400, 1100, 1024, 2, True), (512, 2048, 1536, 0, True), (448, 2048, 512, 0, True), (448, 2064, 512, 0, False),
    (96, 8192, 1536, 2, False), (96, 8192, 2048, 2, True), (96, 8192, 1536, 0, True), (96, 4608, 192, 0, False)])
def test_gemm_row_groups_fit_one_round_of_every_xcd(rpo, M, N, K, epi, groups):
    """The eight XCDs take the column blocks in turn, with all their row groups: 32 workgroups each, not 256 in all."""
    rpo.rpo_set_kernel_path(0)
    rpo.rpo_profile_start(rpo.KERNEL_IDS["gemm_skinny"], 1)
    _gemm_case(rpo, M, N, K, torch.bfloat16, epi, path=0, seed=17)
    assert rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm_skinny"])[0] == (1 if groups else 0)


@pytest.mark.parametrize("path", [17, 19, 20, 21, 22, 27])
@pytest.mark.parametrize("shape", [(300, 520, 1536), (77, 1536, 4480)])
def test_gemm_mfma_bf16_every_tile_shape(rpo, shape, path):
    """Each tile shape forced in turn (16 + kernel id), with and without a K-split workspace."""
    for epi in (0, 1, 2):
        for ws_mb in (0, 64):
            _gemm_case(rpo, *shape, torch.bfloat16, epi, path=path, seed=5, ws_mb=ws_mb)


@pytest.mark.parametrize("path,ws_mb", [(0, 0), (0, 64), (1, 0), (27, 0), (30, 0)])
@pytest.mark.parametrize("M,F,K", [(512, 8960, 1536), (40, 1024, 768), (700, 256, 2048), (130, 96, 1024),
                                   (1, 32, 64), (512, 8960, 64), (8, 8960, 192), (17, 416, 128), (64, 18944, 576), (33, 2592, 448),
                                   (300, 18944, 3584), (264, 8032, 512), (100, 18944, 512), (200, 18944, 512),
                                   (192, 8960, 320), (129, 8992, 256), (72, 18944, 256), (128, 18944, 192),
                                   (1000, 8960, 192), (1100, 8960, 192), (2600, 8960, 192), (2600, 8960, 256),
                                   (9, 2048, 192), (30, 2080, 192), (64, 4128, 192), (8, 6176, 192), (50, 8224, 192),
                                   (16, 10272, 192), (33, 12288, 192), (7, 12320, 192), (40, 16416, 192), (64, 20512, 192)])
def test_gemm_swiglu(rpo, M, F, K, path, ws_mb):
    """Fused gate/up projection: C = silu(A Wg^T) * (A Wu^T), W = [gate rows; up rows].  Path 27 forces
    the 256x192 tile and path 30 the 128x160 one (gate / up rows interleaved in blocks of 16), which path 0 picks for
    decode batches (192 x 8960, 129 x 8992, 72 x 18944 and 128 x 18944: the latter; two rounds: 1000 x 8960 256x160, 1100 x 8960 256x192;
    2600 x 8960: 1232 tiles of 256x160, which resident workgroups walk)."""
    g = torch.Generator().manual_seed(M + F)
    a = torch.randn(M, K, generator=g).to(torch.bfloat16)
    w = (torch.randn(2 * F, K, generator=g) * 0.05).to(torch.bfloat16)
    gu = T.lm_head({"lm_head": w.float().numpy()}, a.float().numpy())
    ref = T.silu(gu[:, :F]) * gu[:, F:]
    c = torch.zeros(M, F, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(ws_mb << 20, dtype=torch.uint8, device="cuda") if ws_mb else None
    rpo.rpo_set_kernel_path(path)
    rpo.rpo_gemm_nt(a.cuda(), w.cuda(), c, 3, ws)
    torch.cuda.synchronize()
    got = c.float().cpu().numpy().astype(np.float64)
    err = np.abs(got - ref)
    tol = 2.0 ** -8 * np.abs(ref) + 3e-5 * np.sqrt(K)
    assert np.all(err <= tol), f"max err {err.max()}"


@pytest.mark.parametrize("shape", [(8200, 8256, 128), (8200, 8256, 192), (16500, 4000, 256), (8192, 6144, 192)])
def test_gemm_resident_workgroups_walk_many_tiles(rpo, shape):
    """1000+ tiles: the launch keeps one resident workgroup per CU that walks its share of the tiles
    (256x256 and, for the narrow N, 256x192 tiles; ragged last row and column tiles), with the minimum
    of two K slabs and with an odd slab count (the LDS stage a tile starts in alternates)."""
    for epi in (0, 1, 2):
        _gemm_case(rpo, *shape, torch.bfloat16, epi, path=0, seed=11)


@pytest.mark.parametrize("M,F,K", [(8200, 4128, 192), (8192, 4096, 128), (512, 8960, 192), (512, 8960, 256), (384, 8960, 1536)])
def test_gemm_swiglu_resident_and_three_stage_tiles(rpo, M, F, K):
    """Fused gate/up on the resident-workgroup launch (many tiles) and on the three-stage 256x160 decode
    tile with as few K slabs as it has stages."""
    g = torch.Generator().manual_seed(M + F + K)
    a = torch.randn(M, K, generator=g).to(torch.bfloat16)
    w = (torch.randn(2 * F, K, generator=g) * 0.05).to(torch.bfloat16)
    gu = T.lm_head({"lm_head": w.float().numpy()}, a.float().numpy())
    ref = T.silu(gu[:, :F]) * gu[:, F:]
    c = torch.zeros(M, F, dtype=torch.bfloat16, device="cuda")
    rpo.rpo_set_kernel_path(0)
    rpo.rpo_gemm_nt(a.cuda(), w.cuda(), c, 3, None)
    torch.cuda.synchronize()
    got = c.float().cpu().numpy().astype(np.float64)
    err = np.abs(got - ref)
    tol = 2.0 ** -8 * np.abs(ref) + 3e-5 * np.sqrt(K)
    assert np.all(err <= tol), f"max err {err.max()}"


@pytest.mark.parametrize("cpad", [8, 4, 1])
@pytest.mark.parametrize("M,N,K,epi,path", [
    (257, 528, 192, 0, 17), (300, 1003, 128, 0, 17), (140, 400, 256, 0, 27), (700, 1056, 192, 2, 17), (129, 520, 192, 1, 27),
    (600, 2112, 192, 3, 17), (600, 2112, 192, 3, 27), (600, 2112, 192, 3, 29), (200, 2112, 256, 3, 30), (90, 37888, 256, 3, 0),
    (200, 2112, 192, 3, 19), (257, 530, 192, 0, 19)])
def test_gemm_wide_tiles_column_ends_and_row_strides(rpo, M, N, K, epi, path, cpad):
    """The 16-byte stores of two neighbouring 16-column blocks and what stands in for them: columns that end inside
    a block, inside a pair of blocks or between them, row strides that are no multiple of 16 or of 8 bytes."""
    g = torch.Generator().manual_seed(K + N)
    a = torch.randn(M, K, generator=g).bfloat16()
    w = (torch.randn(N, K, generator=g) * 0.1).bfloat16()
    n_out = N // 2 if epi == 3 else N
    c0 = torch.randn(M, n_out + cpad, generator=g).to(torch.float32 if epi in (1, 2) else torch.bfloat16)
    c = c0.cuda()
    rpo.rpo_set_kernel_path(path)
    rpo.rpo_gemm_nt(a.cuda(), w.cuda(), c[:, :n_out], epi, None)
    torch.cuda.synchronize()
    ref = a.double() @ w.double().t()
    scale = K ** 0.5 * 0.1
    tol = 1e-6 * ref.abs() + 2e-5 * scale                       # fp32 accumulation
    if epi == 2:
        ref = ref + c0[:, :n_out].double()
    if epi == 3:                                                # |silu'| <= 1.1: the error of either factor times the other
        gate, up = ref[:, :n_out], ref[:, n_out:]
        ref = torch.nn.functional.silu(gate) * up
        tol = 4e-5 * scale * (1 + gate.abs() + up.abs())
    if epi in (0, 3):
        tol = tol + 2.0 ** -8 * ref.abs()                       # one bf16 rounding of the result
    got = c.cpu()
    assert bool(((got[:, :n_out].double() - ref).abs() <= tol).all())
    assert torch.equal(got[:, n_out:], c0[:, n_out:])           # nothing beyond the last column


def test_gemm_mfma_bf16_padded_strides(rpo):
    _gemm_case(rpo, 70, 90, 128, torch.bfloat16, 1, path=0, pad=8)
    _gemm_case(rpo, 70, 90, 128, torch.bfloat16, 2, path=0, pad=8)


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", [(1, 5, 3), (65, 130, 77), (128, 128, 256)])
def test_gemm_generic(rpo, shape, dtype, epi):
    _gemm_case(rpo, *shape, dtype, epi, path=1)
    if dtype == torch.float32:
        _gemm_case(rpo, *shape, dtype, epi, path=0)       # fp32 always takes the generic kernel


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K", [(1, 2, 1), (8, 20, 600), (9, 14, 64), (70, 66, 65), (33, 258, 257), (1030, 1040, 70)])
def test_gemm_generic_waves_and_tiles(rpo, M, N, K, epi):
    """fp32: eight rows and four weight rows per wave (their edges, K around the 64 lanes and the 256 values asked for
    at once), 64x64 tiles where there are more than 256 of them (the last shape; SwiGLU stays with the waves)."""
    if epi < 3:
        return _gemm_case(rpo, M, N, K, torch.float32, epi, path=0)
    g = torch.Generator().manual_seed(M + N)
    a, w = torch.randn(M, K, generator=g), torch.randn(N, K, generator=g) * 0.1
    c = torch.zeros(M, N // 2, device="cuda")
    rpo.rpo_set_kernel_path(0)
    rpo.rpo_gemm_nt(a.cuda(), w.cuda(), c, 3, None)
    gu = a.double() @ w.double().t()
    gate, up = gu[:, :N // 2], gu[:, N // 2:]
    err = (c.cpu().double() - torch.nn.functional.silu(gate) * up).abs()
    # 2e-5 sqrt(K) 0.1 on either factor (|silu'| <= 1.1), a few fp32 roundings of the product
    assert bool((err <= 4e-6 * K ** 0.5 * (1 + gate.abs() + up.abs()) + 1e-6 * (gate * up).abs()).all())


def test_gemm_rejects_bad_arguments(rpo):
    a = torch.zeros(4, 8, device="cuda")
    with pytest.raises(ValueError):
        rpo.rpo_gemm_nt(a, torch.zeros(4, 9, device="cuda"), torch.zeros(4, 4, device="cuda"), 1)
    with pytest.raises(rpo.RpoError) as e:
        rpo.rpo_gemm_nt(a, a, torch.zeros(4, 4, device="cuda"), 7)
    assert e.value.code == rpo.RPO_EINVAL


# ---------------------------------------------------------------------------
@pytest.mark.parametrize("vocab,rows,temperature", [(512, 8, 1.0), (151936, 6, 1.0), (152064, 3, 0.7),
                                                    (1000, 5, 0.7), (3, 4, 1.0), (257, 4, 2.5),
                                                    (2100, 1100, 1.0)])   # > 1024 rows: four waves per row
def test_sampler_bit_exact(rpo, vocab, rows, temperature):
    rng = np.random.default_rng(vocab)
    z = (rng.normal(size=(rows, vocab)) * 0.8).astype(np.float32)
    z[0, vocab // 2] = 6.0                                   # a peaked row
    if rows > 1:
        z[1] = -3.0e38                                       # all weight on one token
        z[1, vocab - 1] = 0.0
    zd = torch.from_numpy(z).cuda()
    seq = np.arange(100, 100 + rows).astype(np.uint64)
    seqd = torch.from_numpy(seq.astype(np.int64)).cuda()
    for step in (0, 1, 77):
        tok = torch.empty(rows, dtype=torch.int32, device="cuda")
        lp = torch.empty(rows, dtype=torch.float32, device="cuda")
        rpo.rpo_sample(zd, rows, vocab, vocab, None, rows, temperature, 12345678901234, seqd, step, tok, lp)
        torch.cuda.synchronize()
        otok, olp = osampler.sample(z, temperature, 12345678901234, seq, step)
        np.testing.assert_array_equal(tok.cpu().numpy(), otok)
        np.testing.assert_allclose(lp.cpu().numpy(), olp, atol=1e-4)
        # the same draw when the caller hands over the row maxima
        tok2 = torch.empty(rows, dtype=torch.int32, device="cuda")
        rpo.rpo_sample(zd, rows, vocab, vocab, None, rows, temperature, 12345678901234, seqd, step, tok2,
                       row_max_dev=zd.max(dim=1).values.contiguous())
        torch.cuda.synchronize()
        np.testing.assert_array_equal(tok2.cpu().numpy(), otok)
    assert tok.cpu().numpy()[1] == vocab - 1 if rows > 1 else True


@pytest.mark.parametrize("vocab,rows,with_max", [
    (151936, 512, True), (151936, 768, False),    # logits that no cache holds: 16 waves per row, with and without the maxima
    (131077, 600, True), (131077, 800, False),    # the same with rows that are not 16-byte aligned
    (65540, 1100, True), (98304, 1100, False),    # four waves per row
    (2100, 300, True), (1003, 1030, True)])       # as many rows of a small vocabulary
def test_sampler_bit_exact_many_rows(rpo, vocab, rows, with_max):
    g = torch.Generator(device="cuda").manual_seed(rows)
    zd = torch.randn(rows, vocab, device="cuda", generator=g) * 1.5
    seq = np.arange(7, 7 + rows).astype(np.uint64)
    tok = torch.empty(rows, dtype=torch.int32, device="cuda")
    lp = torch.empty(rows, dtype=torch.float32, device="cuda")
    rpo.rpo_sample(zd, rows, vocab, vocab, None, rows, 0.9, 99, torch.from_numpy(seq.astype(np.int64)).cuda(), 6, tok, lp,
                   row_max_dev=zd.max(dim=1).values.contiguous() if with_max else None)
    pick = np.unique(np.linspace(0, rows - 1, 24).astype(np.int64))
    otok, olp = osampler.sample(zd[torch.from_numpy(pick).cuda()].cpu().numpy(), 0.9, 99, seq[pick], 6)
    np.testing.assert_array_equal(tok.cpu().numpy()[pick], otok)
    np.testing.assert_allclose(lp.cpu().numpy()[pick], olp, atol=1e-4)


@pytest.mark.parametrize("vocab", [1, 255, 1024, 1025, 4096, 4097, 262144])   # segments of 1024, four per lane
def test_sampler_segments_and_tiny_weights(rpo, vocab):
    """Flat rows spread the draws over every segment; the lower half of the rows lies around the smallest weights
    (2^-40 of the maximum, and below: none) with every other token masked out."""
    rng = np.random.default_rng(vocab)
    rows = 96
    z = (rng.normal(size=(rows, vocab)) * 0.2).astype(np.float32)
    low = rng.uniform(-43.0, -36.0, size=(rows // 2, vocab)) / 1.4426950408889634
    z[rows // 2:] = np.where(rng.random((rows // 2, vocab)) < 0.5, low, -np.inf).astype(np.float32)
    z[rows // 2:, -1] = 0.0
    seq = np.arange(rows).astype(np.uint64)
    tok = torch.empty(rows, dtype=torch.int32, device="cuda")
    lp = torch.empty(rows, dtype=torch.float32, device="cuda")
    rpo.rpo_sample(torch.from_numpy(z).cuda(), rows, vocab, vocab, None, rows, 1.0, 5,
                   torch.from_numpy(seq.astype(np.int64)).cuda(), 2, tok, lp)
    torch.cuda.synchronize()
    otok, olp = osampler.sample(z, 1.0, 5, seq, 2)
    np.testing.assert_array_equal(tok.cpu().numpy(), otok)
    np.testing.assert_allclose(lp.cpu().numpy(), olp, atol=1e-4)


def test_sampler_row_map_stride_and_distribution(rpo):
    rng = np.random.default_rng(5)
    vocab, stride = 40, 64
    zpad = np.zeros((2, stride), np.float32)
    zpad[:, :vocab] = rng.normal(size=(2, vocab)).astype(np.float32) * 1.5
    zpad[:, vocab:] = 50.0                                   # padding must never be read
    n = 20000
    row_map = (np.arange(n) % 2).astype(np.int32)
    seq = np.arange(n).astype(np.uint64)
    tok = torch.empty(n, dtype=torch.int32, device="cuda")
    rpo.rpo_sample(torch.from_numpy(zpad).cuda(), 2, vocab, stride, torch.from_numpy(row_map).cuda(), n,
                   1.0, 9, torch.from_numpy(seq.astype(np.int64)).cuda(), 4, tok, None)
    torch.cuda.synchronize()
    got = tok.cpu().numpy()
    otok, _ = osampler.sample(zpad[:, :vocab], 1.0, 9, seq[:500], 4, row_map=row_map[:500])
    np.testing.assert_array_equal(got[:500], otok)
    assert got.max() < vocab
    for r in range(2):                                       # chi-square against the fp64 softmax
        p = np.exp(zpad[r, :vocab].astype(np.float64))
        p /= p.sum()
        cnt = np.bincount(got[row_map == r], minlength=vocab)
        chi2 = float(((cnt - cnt.sum() * p) ** 2 / (cnt.sum() * p)).sum())
        assert chi2 < 90.0                                   # 39 dof, p ~ 1e-5


def test_sampler_rejects_bad_arguments(rpo):
    z = torch.zeros(2, 8, device="cuda")
    s = torch.zeros(2, dtype=torch.int64, device="cuda")
    t = torch.zeros(2, dtype=torch.int32, device="cuda")
    for kw in (dict(temperature=0.0), dict(temperature=-1.0), dict(row_stride=4)):
        args = dict(temperature=1.0, row_stride=8)
        args.update(kw)
        with pytest.raises((rpo.RpoError, ValueError)):
            rpo.rpo_sample(z, 2, 8, args["row_stride"], None, 2, args["temperature"], 1, s, 0, t, None)
    rpo.rpo_sample(z, 2, 8, 8, None, 0, 1.0, 1, s, 0, t, None)      # zero rows: a no-op


# ---------------------------------------------------------------------------
def test_advantages_bit_exact(rpo):
    rng = np.random.default_rng(0)
    cases = [(rng.random((64, 8)) < 0.5).astype(np.float32), (rng.random((32, 8)) < 0.3).astype(np.float32),
             rng.normal(size=(100, 6)).astype(np.float32), np.ones((3, 4), np.float32),
             rng.normal(size=(5, 1)).astype(np.float32), rng.normal(size=(7, 16)).astype(np.float32) * 1e3]
    for r in cases:
        ng, g = r.shape
        for ddof, eps in ((0, 0.0), (1, 0.0), (0, 1e-4)):
            if ddof >= g:
                continue
            out = torch.empty(ng, g, dtype=torch.float32, device="cuda")
            rpo.grpo_advantages(torch.from_numpy(r).cuda(), ng, g, ddof, eps, out)
            torch.cuda.synchronize()
            ref = oadv.grpo_advantages(r, ddof, eps)
            np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    with pytest.raises(rpo.RpoError):
        rpo.grpo_advantages(torch.zeros(2, 2, device="cuda"), 2, 2, 2, 0.0, torch.zeros(2, 2, device="cuda"))
    with pytest.raises(rpo.RpoError):
        rpo.grpo_advantages(torch.zeros(2, 1, device="cuda"), 2, 1, 1, 0.0, torch.zeros(2, 1, device="cuda"))


def test_reward_shaping_then_advantages(rpo):
    """Eq. 11 on the GPU against the oracle (fp64 exp from two libraries: 1e-6), then Eq. 7 on the
    shaped rewards (bit-exact given the same inputs)."""
    from oracle import reward_shaping as ors
    rng = np.random.default_rng(4)
    ng, g = 37, 8
    r = (rng.random((ng, g)) < 0.6).astype(np.float32)
    ln = rng.integers(50, 4096, size=(ng, g)).astype(np.int32)
    out = torch.empty(ng, g, dtype=torch.float32, device="cuda")
    for alpha, lo, hi in ((0.01, 0.5, 1.0), (0.002, 0.1, 0.9)):
        rpo.rpo_shape_rewards(torch.from_numpy(r).cuda(), torch.from_numpy(ln).cuda(), ng, g, alpha, lo, hi, out)
        torch.cuda.synchronize()
        ref = ors.shape_rewards(r, ln, alpha, lo, hi)
        got = out.cpu().numpy()
        np.testing.assert_allclose(got, ref, atol=1e-6)
        assert np.all(got[r == 0] == 0)
        adv = torch.empty(ng, g, dtype=torch.float32, device="cuda")
        rpo.grpo_advantages(out, ng, g, 0, 0.0, adv)
        np.testing.assert_array_equal(adv.cpu().numpy(), oadv.grpo_advantages(got))
    with pytest.raises(rpo.RpoError):
        rpo.rpo_shape_rewards(out, torch.zeros(ng, g, dtype=torch.int32, device="cuda"), ng, g, 0.0, 0.5, 1.0, out)


def test_objective_forward(rpo):
    """Eq. 5-7 forward on the GPU against the oracle (fp64 on both sides: 1e-6 after the fp32 store)."""
    from oracle import objective as oo
    rng = np.random.default_rng(8)
    ng, g = 9, 6
    lens = rng.integers(0, 40, size=ng * g)
    lens[3] = 0
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = int(cu[-1])
    lp_old = (-rng.random(n) * 8).astype(np.float32)
    lp_new = (lp_old + rng.normal(size=n) * 0.3).astype(np.float32)
    lp_ref = (lp_old + rng.normal(size=n) * 0.2).astype(np.float32)
    adv = rng.normal(size=ng * g).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    for beta, ref in ((0.0, None), (0.04, lp_ref)):
        tok = torch.empty(n, dtype=torch.float32, device="cuda")
        j = torch.empty(ng, dtype=torch.float32, device="cuda")
        rpo.rpo_objective_forward(dev(lp_new), dev(lp_old), None if ref is None else dev(ref), dev(cu), dev(adv),
                                  ng, g, 0.2, beta, tok, j)
        torch.cuda.synchronize()
        tok_ref, j_ref = oo.group_objective(lp_new, lp_old, ref, cu, adv, g, 0.2, beta)
        np.testing.assert_allclose(tok.cpu().numpy(), tok_ref, rtol=1e-6, atol=1e-7)
        np.testing.assert_allclose(j.cpu().numpy(), j_ref, rtol=1e-6, atol=1e-7)
    with pytest.raises(rpo.RpoError):
        rpo.rpo_objective_forward(dev(lp_new), dev(lp_old), None, dev(cu), dev(adv), ng, g, 0.2, 0.1,
                                  None, torch.empty(ng, device="cuda"))


# ---------------------------------------------------------------------------
def test_profile_sampling_and_peak_probe(rpo):
    """Kernel timing brackets every n-th launch only; the peak probes return plausible rates."""
    a = torch.randn(300, 1536, device="cuda").to(torch.bfloat16)
    w = torch.randn(520, 1536, device="cuda").to(torch.bfloat16)
    c = torch.zeros(300, 520, device="cuda")
    rpo.rpo_set_kernel_path(17)                       # every launch below is kernel id 1
    for every, expect in ((1, 10), (4, 3)):
        rpo.rpo_profile_start(rpo.KERNEL_IDS["gemm256"], every)
        for _ in range(10):
            rpo.rpo_gemm_nt(a, w, c, 1, None)
        n, ms, flops, nbytes = rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm256"])
        assert n == expect and ms > 0.0
        assert flops == pytest.approx(expect * 2.0 * 300 * 520 * 1536)
    # two kernels timed at once: the SwiGLU instantiation of the same tile has an id of its own
    act = torch.zeros(300, 256, device="cuda", dtype=torch.bfloat16)
    rpo.rpo_profile_start(rpo.KERNEL_IDS["gemm256"], 1)
    rpo.rpo_profile_start(rpo.KERNEL_IDS["gemm256_swiglu"], 1)
    rpo.rpo_gemm_nt(a, w, c, 1, None)
    rpo.rpo_gemm_nt(a, w[:512], act, 3, None)
    rpo.rpo_gemm_nt(a, w[:512], act, 3, None)
    assert rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm256"])[0] == 1
    assert rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm256_swiglu"])[0] == 2
    rpo.rpo_set_kernel_path(0)
    with pytest.raises(rpo.RpoError):
        rpo.rpo_profile_start(rpo.KERNEL_IDS["gemm256"], 0)
    copy_gbps, mfma_tflops = rpo.rpo_probe_peaks(1 << 28)
    assert 500.0 < copy_gbps < 8000.0                 # below the published HBM peak
    assert 200.0 < mfma_tflops < 2500.0               # below the published bf16 MFMA peak


@pytest.mark.parametrize("M,N,K,split", [(520, 1024, 8192, True), (700, 2048, 3584, True), (2048, 2048, 3584, True),
                                         (2500, 2048, 3584, False), (2048, 2048, 1536, False), (1000, 17920, 1536, False),
                                         (2600, 17920, 256, False)])
def test_gate_up_of_few_tiles_splits_k(rpo, M, N, K, split):
    """Gate/up of 513 rows up: 256x256 tiles that split K over the CUs where those are too few, 256x160 ones (which
    cannot) where they fill their rounds better."""
    a = torch.randn(M, K, device="cuda").to(torch.bfloat16)
    w = (torch.randn(N, K, device="cuda") * 0.02).to(torch.bfloat16)
    c = torch.zeros(M, N // 2, device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(96 << 20, dtype=torch.uint8, device="cuda")
    rpo.rpo_set_kernel_path(0)
    for name in ("gemm256_swiglu", "gemm256x160"):
        rpo.rpo_profile_start(rpo.KERNEL_IDS[name], 1)
    rpo.rpo_gemm_nt(a, w, c, 3, ws)
    assert rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm256_swiglu"])[0] == (1 if split else 0)
    assert rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm256x160"])[0] == (0 if split else 1)
    exact = a.float() @ w.float().t()
    exact = torch.nn.functional.silu(exact[:, :N // 2]) * exact[:, N // 2:]
    assert (c.float() - exact).norm() / exact.norm() < 4e-3     # half a last place of bf16


def test_profile_sees_the_kernels_of_a_decode_step(rpo):
    """The few-row kernel (a K split with its reduction: one launch) and the 128x160 gate/up tile have ids of their own."""
    rpo.rpo_set_kernel_path(0)
    ws = torch.empty(32 << 20, dtype=torch.uint8, device="cuda")
    for name, shapes in (("gemm_skinny", ((8, 2048, 1536, 0), (40, 1536, 8960, 2), (200, 1536, 1536, 2))),
                         ("gemm128x160", ((192, 17920, 320, 3),))):
        for M, N, K, epi in shapes:
            a = torch.randn(M, K, device="cuda").to(torch.bfloat16)
            w = (torch.randn(N, K, device="cuda") * 0.05).to(torch.bfloat16)
            c = torch.zeros(M, N // 2 if epi == 3 else N, device="cuda",
                            dtype=torch.bfloat16 if epi in (0, 3) else torch.float32)
            rpo.rpo_profile_start(rpo.KERNEL_IDS[name], 1)
            rpo.rpo_gemm_nt(a, w, c, epi, ws)
            n, _, flops, _ = rpo.rpo_profile_stop(rpo.KERNEL_IDS[name])
            assert n == 1 and flops == pytest.approx(2.0 * M * N * K), f"{name} M={M} N={N} K={K}"


# ---------------------------------------------------------------------------
def _attn_decode_case(rpo, mcfg, prefix_lens, G, n_fill, suffix_views, check_groups, seed):
    """rpo_attn_decode (the shared-prefix decode attention of one layer, alone) against the plain
    softmax(q K^T / sqrt(dh)) V of the oracle.  The pages are filled by a real prefill + fork and
    n_fill decode steps on fixed tokens; the oracle builds the same keys / values (bf16 cache) with
    its own forward; the queries are random."""
    from paper_2601_19404_amd import rollout
    rng = np.random.default_rng(seed)
    w = synth.perturb_gains(synth.make_weights(mcfg, seed=seed))
    w_np = synth.weights_to_numpy(w)
    shape_q = util.oracle_shape(mcfg, storage="model")
    model = rpo.rpo_model_create(mcfg, util.to_device(w))
    ng = len(prefix_lens)
    B = ng * G
    prefixes = [rng.integers(0, mcfg.vocab, size=n).astype(np.int32) for n in prefix_lens]
    cu = np.concatenate([[0], np.cumsum(prefix_lens)]).astype(np.int32)
    batch = rpo.rpo_batch_create(model, ng, G, int(max(prefix_lens)), max(n_fill, 1), 64,
                                 max(int(sum(prefix_lens)), B, 1024))
    last = torch.empty(ng, mcfg.vocab, device="cuda")
    rpo.rpo_prefill_prefix(batch, torch.from_numpy(np.concatenate(prefixes)).cuda(), cu, last)
    rpo.rpo_kv_fork(batch)
    logits = torch.empty(B, mcfg.vocab, device="cuda")
    step_tok = lambda j: ((np.arange(B) * 7 + 13 * j) % mcfg.vocab).astype(np.int32)
    for j in range(n_fill):
        rpo.rpo_decode_step(batch, torch.from_numpy(step_tok(j)).cuda(), B, None, logits)
    width = mcfg.n_q_heads * mcfg.head_dim
    q = (torch.randn(B, width, generator=torch.Generator().manual_seed(seed)) * 1.5).to(torch.bfloat16)
    q_dev = q.cuda()
    q64 = q.float().numpy().astype(np.float64).reshape(B, mcfg.n_q_heads, mcfg.head_dim)
    worst = 0.0
    for n_suffix in suffix_views:
        out = torch.full((B, width), 7.0, dtype=torch.bfloat16, device="cuda")
        rpo.rpo_attn_decode(batch, 0, q_dev, B, n_suffix, None, out)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy().reshape(B, mcfg.n_q_heads, mcfg.head_dim)
        for g in check_groups:
            kv0, _ = T.prefill(shape_q, w_np, prefixes[g])
            for i in (0, G - 1):
                r = g * G + i
                kv = kv0.copy()
                for j in range(n_suffix):
                    T.decode_step(shape_q, w_np, int(step_tok(j)[r]), kv)
                ctx = prefix_lens[g] + n_suffix
                ref = T.attention_rows(shape_q, q64[r:r + 1], kv.k[0][:ctx], kv.v[0][:ctx], np.ones((1, ctx), bool))[0]
                err = np.abs(got[r] - ref).max() / np.abs(ref).max()
                worst = max(worst, float(err))
    print(f"decode attention alone vs oracle: max error {worst:.3e} of the output scale", flush=True)
    # bf16 output (2^-9), bf16 probabilities in the second product, bf16 K/V computed by two pipelines
    assert worst < 2e-2


def test_attn_decode_alone_small(rpo):
    mcfg = synth.ModelCfg("attn-1layer", 1, 768, 6, 1, 128, 256, 512, "bf16")
    _attn_decode_case(rpo, mcfg, prefix_lens=(300, 257, 640, 64, 130, 20), G=8, n_fill=70,
                      suffix_views=(0, 1, 37, 70), check_groups=(0, 2, 3, 5), seed=61)


@pytest.mark.parametrize("prefix_lens", [(300, 230), (600, 430), (1100, 950)])
def test_prefill_rotary_tiles(rpo, prefix_lens):
    """QKV projection of a prefill chunk on one-head tiles of 64 and 128 rows (the last rows of a tile missing, tiles
    across two sequences): keys and values through the attention over them, queries through the prefix logits."""
    mcfg = synth.ModelCfg("rotary-prefill", 1, 256, 12, 2, 128, 256, 512, "bf16")
    _attn_decode_case(rpo, mcfg, prefix_lens=prefix_lens, G=2, n_fill=1, suffix_views=(0,), check_groups=(0, 1), seed=81)
    rng = np.random.default_rng(82)
    w = synth.perturb_gains(synth.make_weights(mcfg, seed=82))
    model = rpo.rpo_model_create(mcfg, util.to_device(w))
    batch = rpo.rpo_batch_create(model, 2, 1, max(prefix_lens), 1, 64, sum(prefix_lens))
    prefixes = [rng.integers(0, mcfg.vocab, size=n).astype(np.int32) for n in prefix_lens]
    last = torch.empty(2, mcfg.vocab, device="cuda")
    rpo.rpo_profile_start(rpo.KERNEL_IDS["gemm32"], 1)
    rpo.rpo_prefill_prefix(batch, torch.from_numpy(np.concatenate(prefixes)).cuda(),
                           np.concatenate([[0], np.cumsum(prefix_lens)]).astype(np.int32), last)
    # up to 256 tiles of 128 rows and one head; beyond (the third case) wider tiles and a rotary kernel
    assert rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm32"])[0] == (1 if sum(prefix_lens) <= 2048 else 0)
    got = last.cpu().numpy()
    for g in range(2):
        _, ref = T.prefill(util.oracle_shape(mcfg, storage="bf16"), synth.weights_to_numpy(w), prefixes[g])
        ref = np.asarray(ref).reshape(-1, mcfg.vocab)[-1]
        # a single layer with the same bf16 roundings: six ulps of the logit scale at most
        assert np.abs(got[g] - ref).max() <= 6 * 2.0 ** -8 * np.abs(ref).max()


@pytest.mark.parametrize("M,N,K", [(4609, 3584, 5120), (5000, 3584, 6144), (11000, 1536, 8960), (11264, 1540, 8960),
                                   (4609, 3584, 8960), (4700, 3584, 18944)])
def test_gemm_whole_rounds_and_the_rest(rpo, M, N, K):
    """Accumulating projections whose last round of 256x256 tiles is mostly empty: the remaining rows (one, a few, more
    than a tile) in a launch of their own, at the right place of A and C."""
    g = torch.Generator(device="cuda").manual_seed(M)
    a = torch.randn(M, K + 8, generator=g, device="cuda").bfloat16()[:, :K]
    w = (torch.randn(N, K, generator=g, device="cuda") * 0.1).bfloat16()
    c0 = torch.randn(M, N + 4, generator=g, device="cuda")
    c = c0.clone()
    rpo.rpo_set_kernel_path(0)
    assert 0 < rpo.rpo_gemm_plan(M, N, K, rpo.RPO_BF16, 2, 96 << 20)["first_rows"] < M          # two launches
    rpo.rpo_gemm_nt(a, w, c[:, :N], 2, torch.empty(96 << 20, dtype=torch.uint8, device="cuda"))
    ref = a.double() @ w.double().t()
    assert bool(((c[:, :N].double() - c0[:, :N].double() - ref).abs() <= 2e-6 * ref.abs() + 2e-5 * K ** 0.5 * 0.1).all())
    assert torch.equal(c[:, N:], c0[:, N:])


def test_prefill_chunk_of_whole_rounds_and_the_rest(rpo):
    """The same inside a model, where the norm of all rows follows: a prefill in one chunk (4750 rows: the down
    projection in two launches) against chunks of one sequence, which are too small for it, and both against the oracle
    for the last sequence, whose last rows are the second launch's."""
    mcfg = synth.ModelCfg("whole-rounds", 2, 3584, 28, 4, 128, 5120, 512, "bf16")
    plan = [rpo.rpo_gemm_plan(rows, 3584, 5120, rpo.RPO_BF16, 2, 96 << 20)["first_rows"] for rows in (4750, 1193)]
    assert 0 < plan[0] < 4750 and plan[1] == 0
    lens = [1190, 1187, 1180, 1193]
    rng = np.random.default_rng(5)
    w = synth.perturb_gains(synth.make_weights(mcfg, seed=5, device="cuda"))
    model = rpo.rpo_model_create(mcfg, w)
    toks = torch.from_numpy(rng.integers(0, mcfg.vocab, size=sum(lens)).astype(np.int32)).cuda()
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    out = []
    for max_rows in (sum(lens), 1200):
        batch = rpo.rpo_batch_create(model, len(lens), 1, max(lens), 1, 64, max_rows)
        last = torch.empty(len(lens), mcfg.vocab, device="cuda")
        rpo.rpo_prefill_prefix(batch, toks, cu, last)
        out.append(last.cpu())
    # two bf16 pipelines of two layers: six ulps of the logit scale (measured elsewhere up to 5.5)
    assert float((out[0] - out[1]).abs().max()) <= 6 * 2.0 ** -8 * float(out[1].abs().max())
    ref = torch.from_numpy(T.prefill(util.oracle_shape(mcfg, storage="bf16"), synth.weights_to_numpy(w),
                                     toks[int(cu[3]):].cpu().numpy())[1])
    for o in out:
        assert float((o[3].double() - ref).abs().max()) <= 6 * 2.0 ** -8 * float(ref.abs().max())


@pytest.mark.parametrize("d_model,hq,hk,ffn", [(256, 2, 1, 320), (1536, 12, 2, 1024), (3584, 28, 4, 2080), (4096, 8, 2, 10304), (336, 2, 2, 256)])
def test_few_rows_take_the_norm_apart(rpo, d_model, hq, hk, ffn):
    """The RMSNorm between O and gate/up of up to 32 rows (sums of squares per 16 columns, a factor per row) against 40
    rows of the same batch, where it is a kernel of its own (and widths that keep it: 336 is no multiple of 64)."""
    mcfg = synth.ModelCfg("norm-apart", 2, d_model, hq, hk, 128, ffn, 512, "bf16")
    w = synth.perturb_gains(synth.make_weights(mcfg, seed=9))
    model = rpo.rpo_model_create(mcfg, util.to_device(w))
    rng = np.random.default_rng(d_model)
    toks = torch.from_numpy(rng.integers(0, 512, size=20 * 5).astype(np.int32)).cuda()
    step = torch.from_numpy(rng.integers(0, 512, size=40).astype(np.int32)).cuda()

    def logits(rows):
        batch = rpo.rpo_batch_create(model, 20, 2, 5, 2, 64, 512)
        rpo.rpo_prefill_prefix(batch, toks, (np.arange(21) * 5).astype(np.int32), torch.empty(20, 512, device="cuda"))
        rpo.rpo_kv_fork(batch)
        out = torch.zeros(40, 512, device="cuda")
        rpo.rpo_decode_step(batch, step, rows, None, out)
        return out.cpu()

    ref = logits(40)
    shape, w_np, seqs = util.oracle_shape(mcfg, storage="bf16"), synth.weights_to_numpy(w), toks.cpu().numpy().reshape(20, 5)
    exact = {}
    for r in (0, 6, 31):
        kv, _ = T.prefill(shape, w_np, seqs[r // 2])
        exact[r] = torch.from_numpy(T.decode_step(shape, w_np, int(step[r]), kv))
    for rows in (1, 7, 8, 9, 16, 17, 31, 32, 33):
        apart = all(rpo.rpo_gemm_plan(rows, *nk, rpo.RPO_BF16, epi, 96 << 20)["norm_apart"]
                    for epi, nk in ((2, (d_model, hq * 128)), (3, (2 * ffn, d_model))))
        assert apart == (rows <= 32 and d_model % 64 == 0 and d_model <= 4096), rows
        got = logits(rows)
        # two bf16 pipelines of two layers: six ulps of the logit scale
        assert float((got - ref)[:rows].abs().max()) <= 6 * 2.0 ** -8 * float(ref[:rows].abs().max()), rows
        for r, x in exact.items():
            if r < rows:
                assert float((got[r].double() - x).abs().max()) <= 6 * 2.0 ** -8 * float(x.abs().max()), (rows, r)


@pytest.mark.parametrize("rows", [66, 72, 128, 136, 256, 258])
@pytest.mark.parametrize("d_model,vocab", [(256, 1004), (128, 520)])
def test_lm_head_row_maxima_on_every_tile(rpo, rows, d_model, vocab):
    """Logits with their row maxima (128- and 256-row tiles, a vocabulary that ends inside a tile, two K slabs) against
    the plain logits of the same hidden rows, which another kernel computes."""
    mcfg = synth.ModelCfg("lm-rows", 1, d_model, 2, 1, 128, 256, vocab, "bf16")
    w = synth.perturb_gains(synth.make_weights(mcfg, seed=3))
    model = rpo.rpo_model_create(mcfg, util.to_device(w))
    rng = np.random.default_rng(rows)
    ng = 43
    toks = torch.from_numpy(rng.integers(0, vocab, size=ng * 5).astype(np.int32)).cuda()
    step = torch.from_numpy(rng.integers(0, vocab, size=ng * 6).astype(np.int32)).cuda()
    out = []
    for with_max in (True, False):
        batch = rpo.rpo_batch_create(model, ng, 6, 5, 2, 64, 512)
        rpo.rpo_prefill_prefix(batch, toks, (np.arange(ng + 1) * 5).astype(np.int32), torch.empty(ng, vocab, device="cuda"))
        rpo.rpo_kv_fork(batch)
        logits = torch.full((ng * 6, vocab), 3.0, device="cuda")
        row_max = torch.full((ng * 6,), -7.0, device="cuda")
        rpo.rpo_decode_step(batch, step, rows, None, logits, None, row_max if with_max else None)
        out.append((logits.cpu(), row_max.cpu()))
    a, b = out[0][0], out[1][0]
    assert torch.equal(out[0][1][:rows], a[:rows].max(dim=1).values)
    assert bool((out[0][1][rows:] == -7.0).all()) and bool((a[rows:] == 3.0).all())
    assert float((a - b)[:rows].abs().max()) <= 1e-5 * float(b[:rows].abs().max())      # fp32 sums in another order


@pytest.mark.parametrize("d_model,vocab,rows,tile", [
    (1536, 49156, 41, True), (1536, 49156, 64, True), (2112, 49156, 33, True), (1536, 49156, 40, False), (1536, 48896, 64, False),
    (2048, 49156, 64, False), (1472, 49156, 64, False), (1536, 49154, 64, False)])
def test_lm_head_of_few_rows_takes_the_faster_kernel(rpo, d_model, vocab, rows, tile):
    """33 to 64 rows: the 128x256 tile for a large vocabulary and a K that is neither small nor a multiple of 2048 (64 rows
    of 152064 x 3584: 306 us in the few-row kernel, 277 so)."""
    mcfg = synth.ModelCfg("lm-few", 1, d_model, 2, 1, 128, 256, vocab, "bf16")
    w = synth.make_weights(mcfg, seed=4, device="cuda")
    model = rpo.rpo_model_create(mcfg, w)
    rng = np.random.default_rng(rows)
    toks = torch.from_numpy(rng.integers(0, vocab, size=16 * 5).astype(np.int32)).cuda()
    step = torch.from_numpy(rng.integers(0, vocab, size=64).astype(np.int32)).cuda()
    rpo.rpo_set_kernel_path(0)
    out = []
    for with_max in (True, False):
        batch = rpo.rpo_batch_create(model, 16, 4, 5, 2, 64, 128)
        rpo.rpo_prefill_prefix(batch, toks, (np.arange(17) * 5).astype(np.int32), torch.empty(16, vocab, device="cuda"))
        rpo.rpo_kv_fork(batch)
        logits = torch.full((64, vocab), 3.0, device="cuda")
        row_max = torch.full((64,), -7.0, device="cuda")
        rpo.rpo_profile_start(rpo.KERNEL_IDS["gemm256"], 1)
        rpo.rpo_decode_step(batch, step, rows, None, logits, None, row_max if with_max else None)
        n = rpo.rpo_profile_stop(rpo.KERNEL_IDS["gemm256"])[0]
        assert n == (1 if with_max and tile else 0)
        out.append((logits.cpu(), row_max.cpu()))
    a, b = out[0][0], out[1][0]
    assert torch.equal(out[0][1][:rows], a[:rows].max(dim=1).values)
    assert bool((out[0][1][rows:] == -7.0).all()) and bool((a[rows:] == 3.0).all())
    assert float((a - b)[:rows].abs().max()) <= 1e-5 * float(b[:rows].abs().max())      # fp32 sums in another order
    if tile:
        shape, w_np = util.oracle_shape(mcfg, storage="bf16"), synth.weights_to_numpy(w)
        for r in (0, rows - 1):
            kv, _ = T.prefill(shape, w_np, toks.cpu().numpy().reshape(16, 5)[r // 4])
            x = torch.from_numpy(T.decode_step(shape, w_np, int(step[r]), kv))
            # one layer with the same bf16 roundings: six ulps of the logit scale
            assert float((a[r].double() - x).abs().max()) <= 6 * 2.0 ** -8 * float(x.abs().max())


@pytest.mark.parametrize("head_dim", [2, 10, 16, 24, 32, 48, 64, 80, 200, 256])
def test_attn_generic_head_dims(rpo, head_dim):
    """The vector-ALU attention: four, two and one group of lanes, up to four channels a lane, heads that are and are
    not read in 16-byte pieces; contexts that end inside and at the end of an octet and of 64 tokens."""
    mcfg = synth.ModelCfg("attn-generic", 1, 64, 4, 2, head_dim, 64, 256, "bf16")
    _attn_decode_case(rpo, mcfg, prefix_lens=(130, 64, 5), G=2, n_fill=3, suffix_views=(1, 3), check_groups=(0, 1, 2),
                      seed=70 + head_dim)


@pytest.mark.parametrize("prefix_lens", [(2100, 1200, 70), (1310, 700), (1180,)])
def test_attn_decode_alone_more_than_eight_prefix_pieces(rpo, prefix_lens):
    """A few groups with long prefixes: 16, 10 and 9 prefix pieces; the shorter groups leave some of theirs empty."""
    mcfg = synth.ModelCfg("attn-1layer-fine", 1, 256, 6, 1, 128, 256, 512, "bf16")
    _attn_decode_case(rpo, mcfg, prefix_lens=prefix_lens, G=8, n_fill=3, suffix_views=(3,),
                      check_groups=range(len(prefix_lens)), seed=63)


def test_attn_decode_alone_benchmark_shape(rpo):
    """The 1.5B benchmark's attention launch: 64 groups x 8 rollouts, 12 q / 2 kv heads, ~2000-token
    shared prefixes (31-32 shared pages per group, four prefix pieces per group and KV head), 150
    private tokens per rollout; two groups recomputed by the oracle."""
    mcfg = synth.ModelCfg("attn-1layer-c1", 1, 1536, 12, 2, 128, 256, 512, "bf16")
    wl = synth.make_workload(synth.C1)
    lens = tuple(int(synth.C1.prompt_len + synth.C1.traj_len - mk) for mk in wl.m)
    _attn_decode_case(rpo, mcfg, prefix_lens=lens, G=8, n_fill=150, suffix_views=(150,), check_groups=(0, 63),
                      seed=62)
