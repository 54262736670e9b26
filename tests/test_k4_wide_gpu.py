"""K4's wide tiles with loading waves: every layout, both tile heights, K of one slab up to more than the rings hold.

Operands are small integers, so the products are exact in fp32 in any order of the sum (|sum| <= 9 K < 2^24) and compared
for equality; what surrounds the operands is NaN and what surrounds C must stay as it was."""
import pytest
import torch

from paper_2605_28213_amd import gemm

pytestmark = pytest.mark.gpu
K4, ROW, COL = gemm.GEMM_K4_MFMA, gemm.GEMM_ROW_MAJOR, gemm.GEMM_COL_MAJOR
TYPES = {gemm.GEMM_BF16: torch.bfloat16, gemm.GEMM_F16: torch.float16}


def framed(rows, cols, pad, batch, dtype, gen):
    n = batch * rows * (cols + pad)
    flat = torch.full((n + 8,), float("nan"), device="cuda", dtype=dtype)
    start = 8 if (flat.data_ptr() + 2 * (n - pad)) % 4096 == 0 else 0       # (an odd last row that ends a page goes to another kernel)
    x = flat[start : start + n].view(batch, rows, cols + pad)
    x[:, :, :cols] = torch.randint(-3, 4, (batch, rows, cols), generator=gen, device="cuda").to(dtype)
    return x


def check(dt, M, N, K, la, lb, batch, pads, expect, biased, out32):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    td, pa, pb, pc = TYPES[dt], *pads
    A = framed(*((M, K) if la == ROW else (K, M)), pa, batch, td, gen)
    B = framed(*((K, N) if lb == ROW else (N, K)), pb, batch, td, gen)
    ot = torch.float32 if out32 else td
    C = torch.full((batch, M, N + pc), 7.0, device="cuda", dtype=ot)
    bias = torch.randint(-5, 6, (N,), generator=gen, device="cuda").float() if biased else None
    d = gemm.make_desc(M, N, K, dt, gemm.GEMM_F32 if out32 else dt, la, lb, lda=A.shape[2], ldb=B.shape[2], ldc=N + pc, batch=batch,
                       stride_a=A[0].numel(), stride_b=B[0].numel(), stride_c=C[0].numel(), bias=bias)
    q = gemm.gemm_query(K4, d, A, B, C)
    assert (q.threads, q.bm, q.bn) == ((512, expect, 128) if isinstance(expect, int) else expect), (q, M, N, K)
    assert gemm.gemm_run_ex(K4, d, A, B, C) == gemm.GEMM_OK
    torch.cuda.synchronize()
    for i in range(batch):
        a, b = A[i, :, : (K if la == ROW else M)].float(), B[i, :, : (N if lb == ROW else K)].float()
        ref = (a if la == ROW else a.t()) @ (b if lb == ROW else b.t())
        if biased:
            ref = ref + bias
        assert torch.equal(C[i, :, :N], ref.to(ot)), (M, N, K, la, lb, i)
    assert torch.equal(C[:, :, N:], torch.full_like(C[:, :, N:], 7.0))


@pytest.mark.parametrize("dt", list(TYPES))
@pytest.mark.parametrize("slabs", [1, 2, 3, 4, 5, 6, 9, 11])
def test_aligned_operands_in_every_length_of_the_rings(dt, slabs):
    """More than 128 tiles of 128; rows and columns end inside a tile (1 row and 1 column past it, or all but one)."""
    M, N = (1409, 1537) if slabs % 2 else (1535, 1407)
    check(dt, M, N, 64 * slabs, ROW, COL, 1, (0, 8, 0), 128, slabs == 3, slabs % 2 == 0)


@pytest.mark.parametrize("dt", list(TYPES))
@pytest.mark.parametrize("la,lb", [(ROW, ROW), (COL, ROW), (COL, COL), (ROW, COL)])
@pytest.mark.parametrize("K", [321, 384, 447, 640])
def test_any_layout_alignment_and_k_on_128_tiles(dt, la, lb, K):
    """K of 1, 63 and 64 elements in its last slab, rows aligned to an element; a batch whose C rows are odd."""
    check(dt, 1409, 1535, K, la, lb, 1, (1, 3, 1), 128, K == 447, False)
    check(dt, 127, 129, K, la, lb, 70, (8, 0, 0), 128, False, True)


@pytest.mark.parametrize("la,lb", [(ROW, ROW), (COL, ROW), (COL, COL), (ROW, COL)])
def test_any_layout_on_256_tiles(la, lb):
    """176 tiles of 256 x 128 (the fewest), rows and columns ending inside them; 24 slabs, one element in the last, and more."""
    check(gemm.GEMM_F16, 2561, 1921, 24 * 64 - 63, la, lb, 1, (1, 2, 3), 256, True, False)
    check(gemm.GEMM_BF16, 2815, 2047, 26 * 64 + 8, la, lb, 1, (0, 0, 1), 256, False, True)


@pytest.mark.parametrize("dt", list(TYPES))
@pytest.mark.parametrize("M,N,K,batch,pads", [(2561, 2817, 14 * 64 + 1, 1, (1, 3, 1)), (4000, 4063, 17 * 64 - 1, 1, (0, 0, 0)), (250, 200, 15 * 64, 129, (8, 0, 8)), (130, 258, 20 * 64 + 8, 127, (2, 2, 0))])
def test_row_major_operands_of_one_round_of_256_square_tiles(dt, M, N, K, batch, pads):
    """129 to 255 tiles: the persistent kernel with workgroups that have no tile; 15 slabs, one element in the last or missing."""
    check(dt, M, N, K, ROW, ROW, batch, pads, (256, 256, 256), M == 250, K % 2 == 0)


@pytest.mark.parametrize("dt", list(TYPES))
def test_aligned_operands_on_256_tiles(dt):
    check(dt, 2561, 1928, 16 * 64, ROW, COL, 1, (0, 0, 0), 256, False, False)
    check(dt, 200, 100, 18 * 64, ROW, COL, 177, (64, 0, 4), 256, True, True)


@pytest.mark.parametrize("dt,td", [(gemm.GEMM_BF16, torch.bfloat16), (gemm.GEMM_F16, torch.float16), (gemm.GEMM_FP8_E4M3, torch.float8_e4m3fn)])
@pytest.mark.parametrize("M,N,slabs", [(97, 98, 32), (128, 129, 51), (257, 300, 96), (128, 10000, 48)])
def test_k_ranges_with_a_rotated_walk(dt, td, M, N, slabs):
    """Split-K on wide tiles: ranges of 16 slabs and more, one tile and many, rows and columns ending inside a tile."""
    K = slabs * (128 if dt == gemm.GEMM_FP8_E4M3 else 64)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B = (torch.randint(-3, 4, (r, K), generator=gen, device="cuda").float() for r in (M, N))
    a8, b8 = A.to(td), B.to(td)
    C = torch.full((M, N + 3), 7.0, device="cuda")
    bias = torch.randint(-5, 6, (N,), generator=gen, device="cuda").float()
    d = gemm.make_desc(M, N, K, dt, gemm.GEMM_F32, ROW, COL, ldc=N + 3, bias=bias)
    need = gemm.gemm_query(K4, d, a8, b8, C).workspace_bytes
    assert need > 0
    ws = torch.full((need + 256,), 255, dtype=torch.uint8, device="cuda")
    d.workspace, d.workspace_bytes = ws.data_ptr(), need
    q = gemm.gemm_query(K4, d, a8, b8, C)
    assert q.threads == 512 and "+splitK(" in q.path and q.grid <= 256, q
    for _ in range(2):
        assert gemm.gemm_run_ex(K4, d, a8, b8, C) == gemm.GEMM_OK
        torch.cuda.synchronize()
        assert torch.equal(C[:, :N], A @ B.t() + bias) and bool((C[:, N:] == 7.0).all()) and bool((ws[need:] == 255).all())


@pytest.mark.parametrize("dt,td", [(gemm.GEMM_F16, torch.float16), (gemm.GEMM_FP8_E4M3, torch.float8_e4m3fn)])
@pytest.mark.parametrize("M,N,slabs,ranges", [(128, 22016, 72, 1), (97, 16380, 100, 2), (101, 10239, 161, 7), (128, 16513, 99, 3)])
def test_k_ranges_of_a_streamed_operand(dt, td, M, N, slabs, ranges):
    """A B of 192 MiB and more: one range, ranges that divide the slabs but not the factor, and more of them than one round; the
    scratch past the partial sums stays as it was.  (bf16's loop is fp16's.)"""
    K = slabs * (128 if dt == gemm.GEMM_FP8_E4M3 else 64)
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    A, B = (torch.randint(-3, 4, (r, K), generator=gen, device="cuda").to(td) for r in (M, N))
    C = torch.full((M, N + 3), 7.0, device="cuda")
    d = gemm.make_desc(M, N, K, dt, gemm.GEMM_F32, ROW, COL, ldc=N + 3)
    need = gemm.gemm_query(K4, d, A, B, C).workspace_bytes
    ws = torch.full((need + 256,), 255, dtype=torch.uint8, device="cuda")
    d.workspace, d.workspace_bytes = ws.data_ptr(), need
    q = gemm.gemm_query(K4, d, A, B, C)
    assert "(rotated)" in q.path and q.grid == ranges * -(-N // 128) and need >= ranges * M * N * 4, q
    assert gemm.gemm_run_ex(K4, d, A, B, C) == gemm.GEMM_OK
    torch.cuda.synchronize()
    assert torch.equal(C[:, :N], A.float() @ B.float().t()) and bool((C[:, N:] == 7.0).all()) and bool((ws[need:] == 255).all())


@pytest.mark.parametrize("M,N,slabs,batch", [(129, 300, 1, 3), (300, 257, 2, 2), (1000, 900, 3, 1), (97, 511, 5, 4), (500, 640, 6, 2), (1409, 1535, 7, 1), (200, 300, 9, 25), (130, 1030, 14, 13)])
def test_e4m3_alternates_its_register_slots(M, N, slabs, batch):
    """Odd and even numbers of slabs, fewer and more than the rings hold; a scale per problem (a power of two: exact)."""
    K = 128 * slabs
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B = (torch.randint(-3, 4, (batch, r, K), generator=gen, device="cuda").float() for r in (M, N))
    a8, b8 = A.to(torch.float8_e4m3fn), B.to(torch.float8_e4m3fn)
    scale = torch.tensor([2.0 ** (i % 3 - 1) for i in range(batch)], device="cuda")
    for out, td in ((gemm.GEMM_F32, torch.float32), (gemm.GEMM_BF16, torch.bfloat16)):
        C = torch.full((batch, M, N + 1), 7.0, device="cuda", dtype=td)
        d = gemm.make_desc(M, N, K, gemm.GEMM_FP8_E4M3, out, ROW, COL, ldc=N + 1, batch=batch, stride_a=M * K, stride_b=N * K, stride_c=M * (N + 1), scale_b=scale)
        q = gemm.gemm_query(K4, d, a8, b8, C)
        assert (q.threads, q.bm, q.bn) == (512, 128, 128), q
        assert gemm.gemm_run_ex(K4, d, a8, b8, C) == gemm.GEMM_OK
        torch.cuda.synchronize()
        for i in range(batch):
            assert torch.equal(C[i, :, :N], ((A[i] @ B[i].t()) * scale[i]).to(td)) and bool((C[i, :, N:] == 7.0).all()), i
