"""GPU tests of 16/8-bit products whose operands are k-contiguous and 16-byte aligned
while k is not a whole number of the kernel's stages (64 for the 16-bit formats, 128
for FP8): read where they are, with nothing past the last k taken in.

Small integers and powers of two: the results are exact and compared exactly.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FMT = {"fp16": (2, torch.float16, 64), "bf16": (3, torch.bfloat16, 64), "fp8_e4m3": (4, torch.float8_e4m3fn, 128)}


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    ctx = gpu_util.Ctx()
    yield gpu_util, ctx
    ctx.close()


def product(ctx, fmt, m, n, k, tA, tB, seed=0):
    """alpha = 2, beta = 1; NaN behind the last row of every stored column of A and B, which are padded to
    whole 16-byte vectors.  Returns the device result, the leading padding and the expected matrix."""
    from paper_2406_02701_amd import mpcr
    prec, td, _ = FMT[fmt]
    f8 = fmt == "fp8_e4m3"
    rng = np.random.default_rng([m, n, k, seed])

    def operand(rows, cols):
        x = rng.integers(-3, 4, (rows, cols)).astype(np.float64)
        ld = (rows + 15) // 16 * 16
        flat = np.full((cols, ld), np.nan)
        flat[:, :rows] = x.T
        sc = rng.integers(-2, 3, ((rows + 127) // 128, (cols + 127) // 128)).astype(np.int8)
        if f8:
            x = x * np.exp2(-np.repeat(np.repeat(sc, 128, 0), 128, 1)[:rows, :cols].astype(np.float64))
        return x, torch.from_numpy(flat).to(td).cuda(), ld, torch.from_numpy(np.ascontiguousarray(sc.T)).cuda()

    A, bA, lda, sA = operand(*((k, m) if tA else (m, k)))
    B, bB, ldb, sB = operand(*((n, k) if tB else (k, n)))
    C0 = rng.integers(-9, 10, (m, n)).astype(np.float64)
    C = torch.from_numpy(np.ascontiguousarray(C0.T)).float().cuda()
    ctx.check(mpcr.mpcr_gemm(ctx.ptr, prec, int(tA), int(tB), m, n, k, 2.0, bA.data_ptr(), lda,
                             sA.data_ptr() if f8 else None, bB.data_ptr(), ldb, sB.data_ptr() if f8 else None, 1.0,
                             C.data_ptr(), m, 1))
    return C.double().cpu().numpy().T, 2.0 * ((A.T if tA else A) @ (B.T if tB else B)) + C0


# a part of a stage alone, behind one and several whole stages: one element, whole and broken 16-byte vectors,
# all but one element; both operands in place, or one of them packed
@pytest.mark.parametrize("fmt", list(FMT))
@pytest.mark.parametrize("tA,tB", [(True, False), (False, False), (True, True)])
@pytest.mark.parametrize("whole", [0, 1, 3])
@pytest.mark.parametrize("m,n", [(1, 1), (130, 70), (17, 300)])
def test_partial_last_stage(g, fmt, tA, tB, whole, m, n):
    _, ctx = g
    st = FMT[fmt][2]
    for tail in (1, 7, 8, 15, 16, 17, st // 2, st // 2 + 1, st - 16, st - 1):
        got, want = product(ctx, fmt, m, n, whole * st + tail, tA, tB)
        assert np.array_equal(got, want), tail


# 256 x 256 blocks, ragged rows and columns; from k = 512 the 16-bit formats take whole stages only
@pytest.mark.parametrize("fmt", list(FMT))
@pytest.mark.parametrize("k", [40, 200, 523])
def test_partial_last_stage_large_blocks(g, fmt, k):
    _, ctx = g
    got, want = product(ctx, fmt, 3501, 3900, k, True, False)
    assert np.array_equal(got, want)


# the device memory in use does not grow by a copy of the operand (0.65 GB in 16-bit, 0.33 GB in FP8)
@pytest.mark.parametrize("fmt", list(FMT))
def test_no_copy_of_the_operand(g, fmt):
    gu, _ = g
    from paper_2406_02701_amd import mpcr
    prec, td, _ = FMT[fmt]
    m, n, k = 40000, 16, 8208
    A = torch.zeros((m, k), dtype=torch.uint8 if prec == 4 else td, device="cuda")
    B = torch.zeros((n, k), dtype=A.dtype, device="cuda")
    C = torch.full((n, m), 5.0, dtype=torch.float32, device="cuda")
    sA = torch.zeros(((m + 127) // 128, (k + 127) // 128), dtype=torch.int8, device="cuda")
    sc = sA.data_ptr() if prec == 4 else None
    ctx = gu.Ctx()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx.check(mpcr.mpcr_gemm(ctx.ptr, prec, 1, 0, m, n, k, 1.0, A.data_ptr(), k, sc, B.data_ptr(), k, sc, 0.0,
                             C.data_ptr(), m, 1))
    torch.cuda.synchronize()
    taken = free - torch.cuda.mem_get_info()[0]
    ctx.close()
    assert torch.count_nonzero(C) == 0
    assert taken < 1 << 26
