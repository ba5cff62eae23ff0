"""GPU tests of the kernels at the edges of their tiles, blocks and dispatch rules.

Factor: |L L^T - A| <= 8 n u max(diag A) element by element (the bound of a
blocked Cholesky whose triangular solves use inverted 32 x 32 blocks of a
well-conditioned factor), and the 1-based column of the first pivot that is not
positive.  Solves: the refined solution's forward error is at most the condition
number (below 1e3 here) times the backward error the refinement stops at (1e-13):
1e-10.  Matrix products: small integers and powers of two, exact in every format,
so the results are compared exactly.
"""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    ctx = gpu_util.Ctx()
    yield gpu_util, ctx
    ctx.close()


def spd(n, corr=0.9):
    """|i - j|-geometric correlation plus a nugget: condition number below 25."""
    i = np.arange(n)
    return corr ** np.abs(i[:, None] - i[None, :]) + np.eye(n)


def lower_map(nt, off, band=0):
    m = np.full((nt, nt), 255, np.uint8)
    for i in range(nt):
        for j in range(i + 1):
            m[i, j] = 0 if i - j <= band else off
    return m


def factor(gu, ctx, A, nb, m):
    from paper_2406_02701_amd import mpcr
    n = A.shape[0]
    dA, hm = gu.dev(A), gu.u8map(m)
    tm = mpcr.tilemap(n, nb, hm)
    f, info = ctypes.c_void_p(), ctypes.c_int64(-1)
    st = mpcr.mpcr_potrf_tiled(ctx.ptr, n, dA.data_ptr(), n, ctypes.byref(tm), ctypes.byref(f), ctypes.byref(info))
    return st, f, info.value


# one tile to many, ragged and whole; 640: panel solves beyond 512; 256 with 10 tiles and 512 with
# 4: on both sides of the direct update; 7 tiles of 512: beyond the single-stream order
@pytest.mark.parametrize("nb,n", [(128, 1), (128, 127), (128, 128), (128, 129), (128, 1000), (256, 257), (256, 1024),
                                  (256, 2500), (384, 1000), (512, 513), (512, 1536), (512, 2048), (512, 3500),
                                  (640, 1300)])
def test_factor_fp64(g, nb, n):
    gu, ctx = g
    from paper_2406_02701_amd import mpcr
    A = spd(n)
    st, f, info = factor(gu, ctx, A, nb, lower_map((n + nb - 1) // nb, 0))
    ctx.check(st)
    dL = gu.empty(n, n)
    ctx.check(mpcr.mpcr_factor_to_dense(ctx.ptr, f, dL.data_ptr(), n))
    L = np.tril(gu.host(dL, (n, n)))
    mpcr.mpcr_factor_destroy(f)
    assert info == 0
    assert np.max(np.abs(L @ L.T - A)) <= 8 * n * U * np.max(np.diag(A))


# first and last columns of the 16-wide panels, of the 128 blocks and of the tiles
@pytest.mark.parametrize("nb,n,bad", [(128, 128, 0), (128, 128, 15), (128, 128, 16), (128, 128, 127), (256, 700, 128),
                                      (256, 700, 255), (256, 700, 256), (256, 700, 699), (512, 600, 305)])
@pytest.mark.parametrize("pivot", [-1.0, 0.0, np.nan])
def test_failed_pivot(g, nb, n, bad, pivot):
    gu, ctx = g
    from paper_2406_02701_amd import mpcr
    A = spd(n)
    A[bad, :] = A[:, bad] = 0.0
    A[bad, bad] = pivot
    st, f, info = factor(gu, ctx, A, nb, lower_map((n + nb - 1) // nb, 0))
    if f:
        mpcr.mpcr_factor_destroy(f)
    assert st == mpcr.MPCR_ERR_NOT_SPD and info == bad + 1


# one right-hand side, a whole chunk, one more; one tile, odd and even numbers of tiles (pairs from
# the second solve of a call on), more than 16 tiles behind a step, more than 32 (no pairs); FP32 and
# 16/8-bit tiles off the diagonal
@pytest.mark.parametrize("nb,n,off", [(128, 100, 1), (128, 256, 1), (128, 384, 3), (256, 1000, 1), (256, 1200, 2),
                                      (128, 3000, 1), (128, 4400, 1), (512, 1100, 4)])
@pytest.mark.parametrize("nrhs", [1, 16, 17, 33])
def test_refined_solve(g, nb, n, off, nrhs):
    gu, ctx = g
    from paper_2406_02701_amd import mpcr
    A = spd(n)
    st, f, _ = factor(gu, ctx, A, nb, lower_map((n + nb - 1) // nb, off))
    ctx.check(st)
    B = np.random.default_rng(nrhs).standard_normal((n, nrhs))
    dA, dB, dX = gu.dev(A), gu.dev(B), gu.empty(n, nrhs)
    opts = mpcr.mpcr_refine_opts_t(1e-13, 50, 1, 0, 0, 0, 0, 0, 0.0, 0)
    diag = mpcr.mpcr_diag_t()
    ctx.check(mpcr.mpcr_potrs(ctx.ptr, f, nrhs, dB.data_ptr(), n, dX.data_ptr(), n, dA.data_ptr(), n,
                              ctypes.byref(opts), ctypes.byref(diag)))
    mpcr.mpcr_factor_destroy(f)
    X, ref = gu.host(dX, (n, nrhs)), np.linalg.solve(A, B)
    assert diag.converged and np.linalg.norm(X - ref) <= 1e-10 * np.linalg.norm(ref)


# a factor store that is factored again within one call: its pairs belong to the old factor
def test_pairs_follow_the_factor(g):
    gu, ctx = g
    from paper_2406_02701_amd import mpcr
    n, nb = 700, 128
    rng = np.random.default_rng(3)
    locs, z = gu.dev(rng.random((n, 2))), gu.dev(rng.standard_normal(n))
    hm = gu.u8map(lower_map((n + nb - 1) // nb, 1))
    tm = mpcr.tilemap(n, nb, hm)
    opts = mpcr.mpcr_refine_opts_t(1e-13, 50, 1, 0, 0, 0, 0, 0, 0.0, 0)

    def loglik(c, rg):
        out, d = np.empty(1), mpcr.mpcr_diag_t()
        th = gu.theta(1.0, rg, 0.5, 0.1)
        c.check(mpcr.mpcr_gauss_loglik(c.ptr, n, locs.data_ptr(), z.data_ptr(), 1, ctypes.byref(th), ctypes.byref(tm),
                                       1, ctypes.byref(opts), mpcr.f64p(out), ctypes.byref(d)))
        return out[0]

    again = [loglik(ctx, rg) for rg in (0.1, 0.02, 0.1)]
    for rg, v in zip((0.1, 0.02, 0.1), again):
        fresh = gu.Ctx()
        assert abs(loglik(fresh, rg) - v) <= 1e-12 * abs(v)
        fresh.close()


FMT = {"fp64": (0, torch.float64), "fp32": (1, torch.float32), "fp16": (2, torch.float16), "bf16": (3, torch.bfloat16),
       "fp8_e4m3": (4, torch.float8_e4m3fn)}


def gemm_exact(gu, ctx, fmt, m, n, k, tA, tB, beta, pad, shift):
    """Operands in columns `pad` elements longer than needed, `shift` elements into their buffers."""
    from paper_2406_02701_amd import mpcr
    prec, td = FMT[fmt]
    rng = np.random.default_rng(m + 7 * n + 31 * k)

    def operand(rows, cols):
        x = rng.integers(-3, 4, (rows, cols)).astype(np.float64)
        ld = rows + pad
        flat = np.full(shift + ld * max(cols, 1), 3.0)
        for c in range(cols):
            flat[shift + c * ld: shift + c * ld + rows] = x[:, c]
        buf = torch.from_numpy(flat).to(td).cuda()
        sc = rng.integers(-2, 3, ((rows + 127) // 128, (cols + 127) // 128)).astype(np.int8)
        if fmt == "fp8_e4m3":
            x = x * np.exp2(-np.repeat(np.repeat(sc, 128, 0), 128, 1)[:rows, :cols].astype(np.float64))
        return x, buf, ld, torch.from_numpy(np.ascontiguousarray(sc.T)).cuda()

    A, bA, lda, sA = operand(*((k, m) if tA else (m, k)))
    B, bB, ldb, sB = operand(*((n, k) if tB else (k, n)))
    ldc = m + pad
    C0 = rng.integers(-9, 10, (m, n)).astype(np.float64)
    cdt = torch.float64 if fmt == "fp64" else torch.float32
    flat = np.full(shift + ldc * n, 77.0)
    for c in range(n):
        flat[shift + c * ldc: shift + c * ldc + m] = C0[:, c]
    bC = torch.from_numpy(flat).to(cdt).cuda()
    f8 = fmt == "fp8_e4m3"
    ctx.check(mpcr.mpcr_gemm(ctx.ptr, prec, int(tA), int(tB), m, n, k, 2.0,
                             bA.data_ptr() + shift * bA.element_size(), lda, sA.data_ptr() if f8 else None,
                             bB.data_ptr() + shift * bB.element_size(), ldb, sB.data_ptr() if f8 else None, beta,
                             bC.data_ptr() + shift * bC.element_size(), ldc, 0 if fmt == "fp64" else 1))
    got = bC.double().cpu().numpy()
    want = flat.copy()
    R = 2.0 * ((A.T if tA else A) @ (B.T if tB else B)) + beta * C0
    for c in range(n):
        want[shift + c * ldc: shift + c * ldc + m] = R[:, c]
    assert np.array_equal(got, want)


# around the 16 x 16 tiles, the 64 and 128 blocks and the k chunks; columns that no 16-byte vector fits
@pytest.mark.parametrize("fmt", list(FMT))
@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (63, 65, 17), (64, 64, 16), (129, 127, 31), (130, 257, 128), (3, 300, 130),
                                   (301, 2, 64)])
@pytest.mark.parametrize("pad,shift", [(0, 0), (1, 1), (5, 3)])
def test_gemm_sizes_and_alignments(g, fmt, tA, tB, m, n, k, pad, shift):
    gemm_exact(*g, fmt, m, n, k, tA, tB, float((m + k) % 2), pad, shift)


# enough blocks for the 128 x 128 (FP32) and 256 x 256 (16/8-bit) kernels, with edges
@pytest.mark.parametrize("fmt", list(FMT))
@pytest.mark.parametrize("tA,tB", [(False, False), (True, True)])
def test_gemm_large_block_edges(g, fmt, tA, tB):
    gemm_exact(*g, fmt, 4093, 4090, 37, tA, tB, 0.0, 0, 0)


# the 256 x 256 blocks of the 16/8-bit kernels, ragged rows and columns: one to five stages of k, and the k from
# which a wave takes 128 x 128 (an even and an odd number of stages)
@pytest.mark.parametrize("fmt", ["fp16", "bf16", "fp8_e4m3"])
@pytest.mark.parametrize("k", [1, 65, 130, 256, 449, 512, 513])
def test_gemm_large_block_stages(g, fmt, k):
    gemm_exact(*g, fmt, 3501, 3900, k, True, k % 2 == 1, 1.0, 0, 0)
