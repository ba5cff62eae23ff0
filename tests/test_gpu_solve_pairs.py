"""GPU tests of the solve sweeps by pairs of tiles (from a later solve of a call on):
who writes where, and from which factorisation the pairs come.

Matrices: |i - j|-geometric correlation plus the unit matrix, condition number
below 25, so the forward error of a solve is at most 25 times its backward error.
"""
import ctypes
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    ctx = gpu_util.Ctx()
    yield gpu_util, ctx
    ctx.close()


def spd(n, corr=0.9):
    i = np.arange(n)
    return corr ** np.abs(i[:, None] - i[None, :]) + np.eye(n)


def lower_map(nt, off):
    m = np.full((nt, nt), 255, np.uint8)
    for i in range(nt):
        m[i, :i], m[i, i] = off, 0
    return m


def factor(gu, ctx, A, nb, off):
    from paper_2406_02701_amd import mpcr
    n = A.shape[0]
    dA, hm = gu.dev(A), gu.u8map(lower_map((n + nb - 1) // nb, off))
    tm = mpcr.tilemap(n, nb, hm)
    f, info = ctypes.c_void_p(), ctypes.c_int64(-1)
    ctx.check(mpcr.mpcr_potrf_tiled(ctx.ptr, n, dA.data_ptr(), n, ctypes.byref(tm), ctypes.byref(f), ctypes.byref(info)))
    return dA, f


def refined(gu, ctx, f, dA, n, dB, nrhs, max_iter):
    """max_iter steps of iterative refinement, 1 + max_iter solves (the tolerance cannot be met)."""
    from paper_2406_02701_amd import mpcr
    dX = gu.empty(n, nrhs)
    opts = mpcr.mpcr_refine_opts_t(1e-300, max_iter, 1, 0, 0, 0, 0, 0, 0.0, 0)
    st = mpcr.mpcr_potrs(ctx.ptr, f, nrhs, dB.data_ptr(), n, dX.data_ptr(), n, dA.data_ptr(), n, ctypes.byref(opts), None)
    assert st in (mpcr.MPCR_OK, mpcr.MPCR_ERR_NOT_CONVERGED)
    return gu.host(dX, (n, nrhs))


# two contexts on two streams and threads solve with one factor at the same time, each its own
# right-hand sides and number of solves: a call's results are those it gives alone
def test_one_factor_in_two_contexts(g):
    gu, ctx = g
    from paper_2406_02701_amd import mpcr
    n, nb, nrhs = 1000, 128, 3
    A = spd(n)
    dA, f = factor(gu, ctx, A, nb, 1)
    gen = np.random.default_rng(5)
    B = [gen.standard_normal((n, nrhs)) for _ in range(2)]
    dB = [gu.dev(b) for b in B]
    steps = (9, 6)
    alone = [refined(gu, ctx, f, dA, n, dB[i], nrhs, steps[i]) for i in range(2)]
    torch.cuda.synchronize()
    got = [[], []]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            c = gu.Ctx()
            for _ in range(5):
                got[i].append(refined(gu, c, f, dA, n, dB[i], nrhs, steps[i]))
            c.close()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    mpcr.mpcr_factor_destroy(f)
    for i in range(2):
        assert np.max(np.abs(A @ alone[i] - B[i])) <= 1e-12 * np.max(np.abs(B[i]))
        assert len(got[i]) == 5
        for x in got[i]:
            assert np.array_equal(x, alone[i])


# tiles of 256 and more, an even and an odd number of them, as many solves as lead to the pairs of each and
# two more: the last iterate's residual is that of a refined solve (an iterate x + M^-1 r is rounded to
# u |x|, and FP32 tiles leave M within 2^-20 of A: after two steps the error is below 1e-12)
@pytest.mark.parametrize("nb,n,solves", [(256, 512, 5), (256, 768, 4), (512, 1024, 11), (512, 1500, 8), (640, 1280, 15),
                                         (640, 1800, 11), (1024, 2048, 35), (1024, 3000, 24)])
@pytest.mark.parametrize("nrhs", [1, 17])
def test_large_tiles(g, nb, n, solves, nrhs):
    gu, ctx = g
    from paper_2406_02701_amd import mpcr
    A = spd(n)
    dA, f = factor(gu, ctx, A, nb, 1)
    B = np.random.default_rng(n).standard_normal((n, nrhs))
    X = refined(gu, ctx, f, dA, n, gu.dev(B), nrhs, solves - 1)
    mpcr.mpcr_factor_destroy(f)
    ref = np.linalg.solve(A, B)
    assert np.linalg.norm(X - ref) <= 1e-12 * np.linalg.norm(ref)


# one call that factors the same store again and solves in between: the Newton steps of the Laplace
# approximation, whose second and later solves must not use pairs of an earlier step's factor.  (With the
# second step's pairs kept, the last range's mode is off by 2e-3 to 3e-3 at these sizes; right, the two
# Newton iterations agree to 1e-8, the square root of the stopping rule's 1e-12 being their last step, which
# converges quadratically.)
@pytest.mark.parametrize("nb,n", [(128, 300), (128, 400), (256, 900)])
def test_pairs_of_a_store_factored_again(g, nb, n):
    gu, ctx = g
    from oracle import laplace
    from tests.test_gpu_laplace import inla_data, run
    locs, y = inla_data(n, 43)
    alphas = np.array([0.1, 0.5, 0.9])
    lp, _, its, mode = run(gu, ctx, locs, y, alphas, m=lower_map((n + nb - 1) // nb, 0), nb=nb)
    ref = [laplace.laplace_logpost(locs, y, 0.1, a, 0.5, 10.0) for a in alphas]
    assert its == [r["iters"] for r in ref] and min(its) >= 4
    np.testing.assert_allclose(mode, ref[-1]["mode"], rtol=0, atol=1e-8)
    np.testing.assert_allclose(lp, [r["lpost"] for r in ref], rtol=1e-9)
