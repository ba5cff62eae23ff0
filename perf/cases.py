"""Timed cases of the library: what its users call, at the sizes they call it.

Every case goes through the C interface of include/mpcr.h (the ctypes binding
paper_2406_02701_amd.mpcr), with inputs in HBM where the interface takes device
pointers.  The kinds:

  loglik  one mpcr_gauss_loglik call: the step that a likelihood evaluation, a
          maximum likelihood fit and the benchmark repeat
  serve   a burst of requests through the serving engine, submitted at once and
          polled until every one is answered
  solve   a dense SPD matrix: tile factor, log-determinant, refined solve
  inla    the Laplace posterior of the range over a grid
  mala    a Metropolis-adjusted Langevin chain
  gemm    one matrix product in one of the formats

`listed` has the sizes of the repository's workloads, tests and benchmark (or
generic ones between them), `draw` more of the same ranges.
"""
from __future__ import annotations

import ctypes as C
import math
import time

import numpy as np
import torch

from paper_2406_02701_amd import mpcr

FMT = {"fp64": 0, "fp32": 1, "fp16": 2, "bf16": 3, "fp8": 4}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest requests: one tile, nothing but launches and latency
        _loglik("loglik_fp64_n256", n=256, nb=256, nrhs=1, nu=0.5, range=0.1, nugget=1e-8),
        # the 1024-site FP64 workload (the paper's direct evaluation)
        _loglik("loglik_fp64_n1024", n=1024, nb=256, nrhs=1, nu=0.5, range=0.1, nugget=1e-8),
        # a large request of the serving range, ragged, with the serving engine's map and refinement
        _loglik("loglik_mixed_n7919", n=7919, nb=256, nrhs=1, nu=1.5, range=0.1, nugget=1e-6, band64=1, band32=4,
                far="bf16", guard=0.01),
        # an FP64 evaluation of replicated observations at a size between the workloads
        _loglik("loglik_fp64_n12000", n=12000, nb=512, nrhs=16, nu=1.5, range=0.05, nugget=1e-6),
        # the 32768-site mixed-precision workload of the benchmark (its headline map, PCG, stored residual)
        _loglik("loglik_mixed_n32768", n=32768, nb=512, nrhs=16, nu=1.5, range=0.05, nugget=1e-6, band64=2, band32=8,
                far="bf16", guard=0.03, residual=1),
        # the serving engine under a burst of its request mix (n log-uniform in 256 .. 8192)
        {"name": "serve_burst_24", "kind": "serve", "count": 24, "n_lo": 256, "n_hi": 8192, "nb": 256, "slots": 4},
        # a user's own dense covariance: factor, log-determinant and refined solve of 32 right-hand sides
        {"name": "solve_mixed_n4000", "kind": "solve", "n": 4000, "nb": 256, "nrhs": 32, "nu": 0.5, "range": 0.1,
         "nugget": 1e-2, "map": "mixed"},
        # the Laplace posterior of the range (the paper's INLA analogue), a few range values
        {"name": "inla_n1000", "kind": "inla", "n": 1000, "nrange": 5},
        # the paper's MALA sampler on a regular grid
        {"name": "mala_n1024", "kind": "mala", "m": 32, "iters": 20},
        # the GEMM workload of the benchmark in its fastest widely used format
        {"name": "gemm_bf16_8192", "kind": "gemm", "prec": "bf16", "m": 8192, "n": 8192, "k": 8192, "ta": False,
         "tb": False},
        # a ragged product in the block-scaled 8-bit format
        {"name": "gemm_fp8_ragged", "kind": "gemm", "prec": "fp8", "m": 3001, "n": 2999, "k": 4003, "ta": True,
         "tb": False},
        # the format R users have by default in single precision, a middle size with a transposed operand
        {"name": "gemm_fp32_3000", "kind": "gemm", "prec": "fp32", "m": 3000, "n": 3000, "k": 3000, "ta": False,
         "tb": True},
    ]


def _loglik(name, **kw):
    c = {"kind": "loglik", "sigma2": 1.0, "residual": 0, "guard": 0.0, "band64": 0, "band32": 0, "far": "fp64"}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["loglik", "loglik", "loglik", "serve", "solve", "inla", "mala", "gemm", "gemm", "gemm"])
    if kind == "loglik":
        n = _log_int(rng, 200, 14000)
        nb = 256 if n < 6000 else rng.choice([256, 512])
        c = _loglik(None, n=n, nb=nb, nrhs=rng.choice([1, 1, 2, 7, 16, 19]), nu=rng.choice([0.5, 1.5, 2.5]),
                    sigma2=round(rng.uniform(0.5, 2.0), 3), range=round(rng.uniform(0.02, 0.2), 3),
                    nugget=rng.choice([1e-6, 1e-5, 1e-4, 1e-3]))
        if rng.random() < 0.5 and n > 1000:
            c.update(band64=1, band32=4, far=rng.choice(["bf16", "fp16"]), guard=0.01, residual=rng.choice([0, 1]))
        return c
    if kind == "serve":
        return {"kind": "serve", "count": rng.randint(3, 24), "n_lo": 256, "n_hi": _log_int(rng, 1000, 8192),
                "nb": 256, "slots": rng.choice([2, 4])}
    if kind == "solve":
        return {"kind": "solve", "n": _log_int(rng, 500, 6000), "nb": rng.choice([128, 256]),
                "nrhs": rng.choice([1, 5, 16, 32, 40]), "nu": rng.choice([0.5, 1.5]),
                "range": round(rng.uniform(0.05, 0.2), 3), "nugget": rng.choice([1e-2, 1e-1]),
                "map": rng.choice(["mixed", "fp64"])}
    if kind == "inla":
        return {"kind": "inla", "n": _log_int(rng, 200, 2500), "nrange": rng.choice([3, 5])}
    if kind == "mala":
        return {"kind": "mala", "m": rng.randint(14, 45), "iters": rng.randint(5, 20)}
    prec = rng.choice(["fp64", "fp32", "fp16", "bf16", "fp8"])
    hi = {"fp64": 4000, "fp32": 4600, "fp16": 8192, "bf16": 8192, "fp8": 8192}[prec]
    dims = [_log_int(rng, 100, hi) for _ in range(3)]
    if rng.random() < 0.4:  # whole blocks
        dims = [max(256, (d + 128) // 256 * 256) for d in dims]
    return {"kind": "gemm", "prec": prec, "m": dims[0], "n": dims[1], "k": dims[2], "ta": rng.random() < 0.5,
            "tb": rng.random() < 0.5}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rng(seed, stream):
    return np.random.Generator(np.random.PCG64([seed, stream]))


def _dev(x):
    """Device copy of a numpy array, column-major if it has two dimensions."""
    return torch.from_numpy(np.ascontiguousarray(x.T if x.ndim == 2 else x)).cuda()


class _Ctx:
    """A library context on torch's current stream, destroyed with its owner."""

    def __init__(self):
        self.ptr = C.c_void_p()
        mpcr.check(mpcr.mpcr_ctx_create(torch.cuda.current_device(),
                                        C.c_void_p(torch.cuda.current_stream().cuda_stream), C.byref(self.ptr)))

    def check(self, st):
        mpcr.check(st, self.ptr)

    def __del__(self):
        if self.ptr:
            mpcr.mpcr_ctx_destroy(self.ptr)
            self.ptr = None


def _u8(a):
    return a.ctypes.data_as(C.POINTER(C.c_uint8))


def _banded(n, nb, dmax, precs):
    nt = -(-n // nb)
    out = np.zeros((nt, nt), np.uint8)
    mpcr.check(mpcr.mpcr_tilemap_banded(n, nb, (C.c_int * len(dmax))(*dmax), (C.c_int * len(precs))(*precs),
                                        len(dmax), _u8(out)))
    return out


def _guarded(n, nb, band, amax, guard):
    out = np.zeros_like(band)
    mpcr.check(mpcr.mpcr_tilemap_guarded(n, nb, _u8(band), mpcr.f64p(amax), guard, _u8(out)))
    return out


def _morton_sorted(ctx, locs):
    n = locs.shape[0]
    dl = _dev(locs)
    perm = torch.empty(n, dtype=torch.int64, device="cuda")
    ctx.check(mpcr.mpcr_morton_order(ctx.ptr, n, dl.data_ptr(), perm.data_ptr()))
    return locs[perm.cpu().numpy()]


def _matern(d, nu):
    e = torch.exp(-d)
    return e if nu == 0.5 else (1 + d) * e if nu == 1.5 else (1 + d + d * d / 3) * e


def _covariance(locs, sigma2, range_, nu, nugget):
    """The covariance matrix of the sites in FP64 (torch, on the GPU)."""
    p = torch.from_numpy(np.ascontiguousarray(locs)).cuda()
    S = torch.empty(p.shape[0], p.shape[0], dtype=torch.float64, device="cuda")
    for r in range(0, p.shape[0], 2048):
        q = p[r:r + 2048]
        d = torch.sqrt((q[:, None, 0] - p[None, :, 0]) ** 2 + (q[:, None, 1] - p[None, :, 1]) ** 2)
        S[r:r + 2048] = sigma2 * _matern(d / range_, nu)
    S.diagonal().add_(nugget)
    return S


def _loglik_inputs(c, seed):
    g = _rng(seed, 1)
    return g.random((c["n"], 2)), g.standard_normal((c["n"], c["nrhs"]))


def _requests(c, seed):
    g = _rng(seed, 2)
    out = []
    for _ in range(c["count"]):
        n = int(round(math.exp(g.uniform(math.log(c["n_lo"]), math.log(c["n_hi"])))))
        th = (float(g.uniform(0.5, 2.0)), float(g.uniform(0.02, 0.3)), float(g.choice([0.5, 1.5, 2.5])), 1e-6)
        out.append((g.random((n, 2)), g.standard_normal(n), th))
    return out


def _serve_sizes(c):
    """Sizes of a burst as its distribution gives them, for the work count."""
    q = (np.arange(c["count"]) + 0.5) / c["count"]
    return np.exp(math.log(c["n_lo"]) + q * math.log(c["n_hi"] / c["n_lo"]))


def _inla_inputs(c, seed):
    """The INLA section's recipe: sites on a line, latent field with variance
    0.1 and range 0.6, Bernoulli observations with logit slope 10."""
    n = c["n"]
    g = _rng(seed, 3)
    locs = np.zeros((n, 2))
    step = n / (n - 1)
    locs[:, 0] = np.arange(n) * step
    # the exponential field on a line is an AR(1) process
    rho = math.exp(-step / 0.6)
    e = g.standard_normal(n)
    x = np.empty(n)
    x[0] = math.sqrt(0.1) * e[0]
    for i in range(1, n):
        x[i] = rho * x[i - 1] + math.sqrt(0.1 * (1 - rho * rho)) * e[i]
    y = (g.random(n) < 1.0 / (1.0 + np.exp(-10.0 * x))).astype(np.float64)
    return locs, y, np.linspace(0.05, 0.95, c["nrange"])


def _mala_inputs(c, seed):
    m, n = c["m"], c["m"] ** 2
    g = _rng(seed, 4)
    t = np.arange(m) / (m - 1)
    locs = np.stack([np.tile(t, m), np.repeat(t, m)], axis=1)
    return locs, g.random(n), g.standard_normal((n, c["iters"])), g.random(c["iters"])


def _gemm_operand(rows, cols, prec, gen):
    """A rows x cols column-major U(-1, 1) operand in format `prec` (a (cols,
    rows) tensor), with the scale exponents of its 128 x 128 blocks for FP8."""
    x = torch.rand((cols, rows), dtype=torch.float64, device="cuda", generator=gen) * 2 - 1
    if prec == "fp64":
        return x, None
    if prec == "fp32":
        return x.float(), None
    if prec in ("fp16", "bf16"):
        return x.to(torch.float16 if prec == "fp16" else torch.bfloat16), None
    bc, br = -(-cols // 128), -(-rows // 128)
    pad = torch.zeros((bc * 128, br * 128), dtype=torch.float64, device="cuda")
    pad[:cols, :rows] = x
    amax = pad.view(bc, 128, br, 128).abs().amax(dim=(1, 3))
    s = torch.floor(torch.log2(448.0 / amax)).to(torch.int8)
    scaled = torch.ldexp(pad.view(bc, 128, br, 128), s.double()[:, None, :, None]).view(bc * 128, br * 128)
    return scaled[:cols, :rows].contiguous().to(torch.float8_e4m3fn), s.contiguous()


def _gemm_inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    m, n, k = c["m"], c["n"], c["k"]
    A = _gemm_operand(*((k, m) if c["ta"] else (m, k)), c["prec"], gen)
    B = _gemm_operand(*((n, k) if c["tb"] else (k, n)), c["prec"], gen)
    return A, B


# ---------------------------------------------------------------------------
# prepare / run
# ---------------------------------------------------------------------------
def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def _prepare_loglik(c, seed):
    ctx = _Ctx()
    locs, z = _loglik_inputs(c, seed)
    n, nb = c["n"], c["nb"]
    th = mpcr.mpcr_theta_t(c["sigma2"], c["range"], c["nu"], c["nugget"])
    if c["guard"] > 0:
        band = _banded(n, nb, [c["band64"], c["band32"], -1], [0, 1, FMT[c["far"]]])
        dls = _dev(_morton_sorted(ctx, locs))
        amax = np.zeros(band.shape)
        ctx.check(mpcr.mpcr_covariance_tile_amax(ctx.ptr, n, nb, dls.data_ptr(), C.byref(th), mpcr.f64p(amax)))
        hmap = _guarded(n, nb, band, amax, c["guard"] * c["nugget"])
        opts = mpcr.mpcr_refine_opts_t(1e-13, 100, 0, 20, c["residual"], 1, 0)
    else:
        hmap = _banded(n, nb, [-1], [0])
        opts = mpcr.mpcr_refine_opts_t(1e-9, 0, 0, 20, 0, 0, 0)
    return {"run": _run_loglik, "ctx": ctx, "n": n, "nrhs": c["nrhs"], "locs": _dev(locs), "z": _dev(z), "th": th,
            "hmap": hmap, "tm": mpcr.tilemap(n, nb, hmap), "opts": opts}


def _run_loglik(s):
    out = np.empty(s["nrhs"])
    diag = mpcr.mpcr_diag_t()
    s["ctx"].check(mpcr.mpcr_gauss_loglik(s["ctx"].ptr, s["n"], s["locs"].data_ptr(), s["z"].data_ptr(), s["nrhs"],
                                          C.byref(s["th"]), C.byref(s["tm"]), 1, C.byref(s["opts"]), mpcr.f64p(out),
                                          C.byref(diag)))
    return {"loglik": out, "logdet": float(diag.logdet), "quad0": float(diag.quad0)}


class _Server:
    def __init__(self, budget, slots, opts):
        self.ptr = C.c_void_p()
        mpcr.check(mpcr.mpcr_serve_create(torch.cuda.current_device(), budget, slots, C.byref(opts),
                                          C.byref(self.ptr)))

    def __del__(self):
        if self.ptr:
            mpcr.mpcr_serve_destroy(self.ptr)
            self.ptr = None


def _prepare_serve(c, seed):
    opts = mpcr.mpcr_serve_opts_t(c["nb"], 1, 4, mpcr.MPCR_BF16, 0.01,
                                  mpcr.mpcr_refine_opts_t(1e-13, 100, 0, 20, 0, 1), 1)
    reqs = [(z.size, np.asfortranarray(locs), np.ascontiguousarray(z), mpcr.mpcr_theta_t(*th))
            for locs, z, th in _requests(c, seed)]
    return {"run": _run_serve, "srv": _Server(8 << 30, c["slots"], opts), "reqs": reqs}


def _run_serve(s):
    srv, reqs = s["srv"].ptr, s["reqs"]
    for i, (n, locs, z, th) in enumerate(reqs):
        mpcr.check(mpcr.mpcr_serve_submit(srv, i, n, mpcr.f64p(locs), mpcr.f64p(z), C.byref(th)))
    out, logdet = np.empty(len(reqs)), np.empty(len(reqs))
    rid, ll, st, diag = C.c_uint64(), C.c_double(), C.c_int(), mpcr.mpcr_diag_t()
    left = len(reqs)
    while left:
        if mpcr.mpcr_serve_poll(srv, C.byref(rid), C.byref(ll), C.byref(diag), None, None, C.byref(st), None) == 1:
            mpcr.check(st.value)
            out[rid.value], logdet[rid.value] = ll.value, diag.logdet
            left -= 1
        else:
            time.sleep(0.0001)
    return {"loglik": out, "logdet": logdet}


def _prepare_solve(c, seed):
    ctx = _Ctx()
    n, nb = c["n"], c["nb"]
    g = _rng(seed, 5)
    S = _covariance(_morton_sorted(ctx, g.random((n, 2))), 1.0, c["range"], c["nu"], c["nugget"])
    B = torch.from_numpy(g.standard_normal((c["nrhs"], n))).cuda()
    if c["map"] == "mixed":
        band = _banded(n, nb, [1, 4, -1], [0, 1, 3])
        nt = band.shape[0]
        amax = np.zeros((nt, nt))
        for i in range(nt):
            for j in range(i + 1):
                amax[i, j] = S[i * nb:(i + 1) * nb, j * nb:(j + 1) * nb].abs().max().item()
        hmap = _guarded(n, nb, band, amax, 0.01 * c["nugget"])
    else:
        hmap = _banded(n, nb, [-1], [0])
    return {"run": _run_solve, "ctx": ctx, "n": n, "nrhs": c["nrhs"], "S": S, "B": B, "X": torch.empty_like(B),
            "hmap": hmap, "tm": mpcr.tilemap(n, nb, hmap), "opts": mpcr.mpcr_refine_opts_t(1e-14, 100, 0, 20, 0)}


def _run_solve(s):
    ctx, n = s["ctx"], s["n"]
    f, info, logdet = C.c_void_p(), C.c_int64(), C.c_double()
    ctx.check(mpcr.mpcr_potrf_tiled(ctx.ptr, n, s["S"].data_ptr(), n, C.byref(s["tm"]), C.byref(f), C.byref(info)))
    ctx.check(mpcr.mpcr_factor_logdet(ctx.ptr, f, C.byref(logdet)))
    ctx.check(mpcr.mpcr_potrs(ctx.ptr, f, s["nrhs"], s["B"].data_ptr(), n, s["X"].data_ptr(), n, s["S"].data_ptr(), n,
                              C.byref(s["opts"]), None))
    mpcr.mpcr_factor_destroy(f)
    return {"x": s["X"], "logdet": logdet.value}


def _prepare_inla(c, seed):
    locs, y, ranges = _inla_inputs(c, seed)
    return {"run": _run_inla, "ctx": _Ctx(), "n": c["n"], "locs": _dev(locs), "y": _dev(y), "ranges": ranges,
            "mode": torch.empty(c["n"], dtype=torch.float64, device="cuda")}


def _run_inla(s):
    nr = s["ranges"].size
    lpost, post, its = np.empty(nr), np.empty(nr), (C.c_int * nr)()
    s["ctx"].check(mpcr.mpcr_inla_posterior(s["ctx"].ptr, s["n"], s["locs"].data_ptr(), s["y"].data_ptr(), 0.1, 0.5,
                                            10.0, mpcr.f64p(s["ranges"]), nr, 1e-12, 100, None, mpcr.f64p(lpost),
                                            mpcr.f64p(post), its, s["mode"].data_ptr()))
    return {"lpost": lpost, "posterior": post, "mode": s["mode"], "newton": np.array(its[:], np.int64)}


def _prepare_mala(c, seed):
    locs, z0, eps, unif = _mala_inputs(c, seed)
    n, iters = z0.size, unif.size
    return {"run": _run_mala, "ctx": _Ctx(), "n": n, "iters": iters, "locs": _dev(locs), "z0": _dev(z0),
            "eps": _dev(eps), "unif": unif, "target": mpcr.mpcr_theta_t(1.0, 0.5, 0.5, 0.0),
            "precond": mpcr.mpcr_theta_t(1.0, 0.05, 0.5, 0.0),
            "z": torch.empty(n, dtype=torch.float64, device="cuda"),
            "trace": torch.empty((iters, n), dtype=torch.float64, device="cuda")}


def _run_mala(s):
    acc, lr = (C.c_int * s["iters"])(), np.empty(s["iters"])
    s["ctx"].check(mpcr.mpcr_mala_run(s["ctx"].ptr, s["n"], s["locs"].data_ptr(), C.byref(s["target"]),
                                      C.byref(s["precond"]), 0.01, s["z0"].data_ptr(), s["iters"],
                                      s["eps"].data_ptr(), mpcr.f64p(s["unif"]), None, s["z"].data_ptr(),
                                      s["trace"].data_ptr(), acc, mpcr.f64p(lr)))
    return {"z": s["z"], "trace": s["trace"], "log_ratio": lr, "accepted": np.array(acc[:], np.int64)}


def _prepare_gemm(c, seed):
    (A, sa), (B, sb) = _gemm_inputs(c, seed)
    out = torch.float64 if c["prec"] == "fp64" else torch.float32
    return {"run": _run_gemm, "ctx": _Ctx(), "prec": FMT[c["prec"]], "ta": int(c["ta"]), "tb": int(c["tb"]),
            "m": c["m"], "n": c["n"], "k": c["k"], "A": A, "sa": sa, "B": B, "sb": sb,
            "C": torch.empty((c["n"], c["m"]), dtype=out, device="cuda")}


def _run_gemm(s):
    s["ctx"].check(mpcr.mpcr_gemm(s["ctx"].ptr, s["prec"], s["ta"], s["tb"], s["m"], s["n"], s["k"], 1.0,
                                  s["A"].data_ptr(), s["A"].shape[1], None if s["sa"] is None else s["sa"].data_ptr(),
                                  s["B"].data_ptr(), s["B"].shape[1], None if s["sb"] is None else s["sb"].data_ptr(),
                                  0.0, s["C"].data_ptr(), s["m"], 0 if s["prec"] == 0 else 1))
    return s["C"]


# ---------------------------------------------------------------------------
# the work that a pass cannot do without
# ---------------------------------------------------------------------------
def work(c):
    k = c["kind"]
    if k == "loglik":
        # the covariance comes from the sites: only the factor (lower triangle, written and read by the solve) has to
        # go through memory, in FP64 as an upper bound of its formats
        n, r = c["n"], c["nrhs"]
        return {"bytes": 8.0 * n * n + 8.0 * n * (2 + r), "flops": n ** 3 / 3 + 2.0 * n * n * r}
    if k == "serve":
        n = _serve_sizes(c)
        return {"bytes": float(np.sum(8 * n * n)), "flops": float(np.sum(n ** 3 / 3 + 2 * n * n))}
    if k == "solve":
        n, r = c["n"], c["nrhs"]
        return {"bytes": 8.0 * n * n * 1.5 + 16.0 * n * r, "flops": n ** 3 / 3 + 4.0 * n * n * r}
    if k == "inla":  # about seven Newton steps per range value, each one factorisation and two products with Sigma
        n = c["n"]
        return {"bytes": 8.0 * n * n * 7 * c["nrange"], "flops": 7 * c["nrange"] * (n ** 3 / 3 + 8.0 * n * n)}
    if k == "mala":  # two factors; per iteration two full solves' worth of sweeps, a product with M and one with L
        n = float(c["m"] ** 2)
        return {"bytes": 16.0 * n * n + c["iters"] * 20.0 * n * n, "flops": 2 * n ** 3 / 3 + c["iters"] * 11 * n * n}
    es = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2, "fp8": 1}[c["prec"]]
    m, n, kk = c["m"], c["n"], c["k"]
    return {"bytes": float(es * (m * kk + kk * n) + (8 if es == 8 else 4) * m * n), "flops": 2.0 * m * n * kk}


# ---------------------------------------------------------------------------
# the same in 64 bits, from torch alone
# ---------------------------------------------------------------------------
def _cholesky(S):
    """Lower Cholesky factor of S, in place (left-looking over 1024-column
    blocks; the diagonal blocks on the host)."""
    n, b = S.shape[0], 1024
    for j in range(0, n, b):
        e = min(n, j + b)
        if j:
            S[j:, j:e] -= S[j:, :j] @ S[j:e, :j].t().contiguous()
        D = torch.linalg.cholesky(S[j:e, j:e].cpu())
        inv_t = torch.linalg.solve_triangular(D, torch.eye(e - j, dtype=D.dtype), upper=False).t().contiguous()
        S[j:e, j:e] = D.cuda()
        if e < n:
            S[e:, j:e] = S[e:, j:e] @ inv_t.cuda()
    return S


def _forward(L, B):
    """L^-1 B by 1024-row blocks."""
    W, b = B.clone(), 1024
    for j in range(0, L.shape[0], b):
        e = min(L.shape[0], j + b)
        if j:
            W[j:e] -= L[j:e, :j] @ W[:j]
        W[j:e] = torch.linalg.solve_triangular(L[j:e, j:e].cpu().tril(), W[j:e].cpu(), upper=False).cuda()
    return W


def _backward(L, B):
    """L^-T B by 1024-row blocks."""
    W, b, n = B.clone(), 1024, L.shape[0]
    for j in reversed(range(0, n, b)):
        e = min(n, j + b)
        if e < n:
            W[j:e] -= L[e:, j:e].t().contiguous() @ W[e:]
        W[j:e] = torch.linalg.solve_triangular(L[j:e, j:e].cpu().tril().t(), W[j:e].cpu(), upper=True).cuda()
    return W


def _exact_loglik(locs, z, sigma2, range_, nu, nugget):
    n = locs.shape[0]
    L = _cholesky(_covariance(locs, sigma2, range_, nu, nugget))
    logdet = 2.0 * torch.log(L.diagonal()).sum().item()
    W = _forward(L, torch.from_numpy(np.ascontiguousarray(z)).cuda())
    quad = (W * W).sum(dim=0).cpu().numpy()
    return -0.5 * n * math.log(2 * math.pi) - 0.5 * logdet - 0.5 * quad, logdet, quad


def exact(case, seed):
    c, k = case, case["kind"]
    if k == "loglik":
        locs, z = _loglik_inputs(c, seed)
        ll, logdet, quad = _exact_loglik(locs, z, c["sigma2"], c["range"], c["nu"], c["nugget"])
        return {"loglik": ll, "logdet": logdet, "quad0": float(quad[0])}
    if k == "serve":
        got = [_exact_loglik(locs, z[:, None], *th) for locs, z, th in _requests(c, seed)]
        return {"loglik": np.array([g[0][0] for g in got]), "logdet": np.array([g[1] for g in got])}
    if k == "solve":
        s = _prepare_solve(c, seed)
        L = _cholesky(s["S"].clone())
        X = _backward(L, _forward(L, s["B"].t().contiguous()))
        return {"x": X.t().contiguous(), "logdet": 2.0 * torch.log(L.diagonal()).sum().item()}
    if k == "inla":
        return _exact_inla(c, seed)
    if k == "mala":
        return _exact_mala(c, seed)
    (A, sa), (B, sb) = _gemm_inputs(c, seed)

    def wide(x, s):
        x = x.double()
        if s is None:
            return x
        e = s.double().repeat_interleave(128, 0)[:x.shape[0]].repeat_interleave(128, 1)[:, :x.shape[1]]
        return torch.ldexp(x, -e)

    a, b = wide(A, sa), wide(B, sb)  # (cols, rows) of the stored matrices, i.e. their transposes
    at = a if not c["ta"] else a.t().contiguous()   # op(A)^T, k x m
    bt = b if not c["tb"] else b.t().contiguous()   # op(B)^T, n x k
    return bt @ at


def _exact_inla(c, seed):
    locs, y, ranges = _inla_inputs(c, seed)
    n, beta = c["n"], 10.0
    y, eye = torch.from_numpy(y), torch.eye(c["n"], dtype=torch.float64)
    lpost, its = [], []
    d = torch.from_numpy(np.abs(locs[:, None, 0] - locs[None, :, 0]))
    for r in ranges:
        S = 0.1 * torch.exp(-d / r)
        x, it = torch.zeros(n, dtype=torch.float64), 0
        while True:
            it += 1
            p = torch.sigmoid(beta * x)
            w, g = beta ** 2 * p * (1 - p), beta * (y - p)
            sw = w.sqrt()
            L = torch.linalg.cholesky(eye + sw[:, None] * S * sw[None, :])
            b = w * x + g
            a = b - sw * torch.cholesky_solve((sw * (S @ b))[:, None], L)[:, 0]
            new = S @ a
            step = ((new - x) ** 2).mean().item()
            x = new
            if step < 1e-12:
                break
        p = torch.sigmoid(beta * x)
        sw = (beta ** 2 * p * (1 - p)).sqrt()
        L = torch.linalg.cholesky(eye + sw[:, None] * S * sw[None, :])
        lik = (beta * x * y - torch.nn.functional.softplus(beta * x, threshold=1e9)).sum().item()
        lpost.append(lik - 0.5 * (a @ x).item() - torch.log(L.diagonal()).sum().item())
        its.append(it)
    lpost = np.array(lpost)
    e = np.exp(lpost - lpost.mean())
    wt = np.array([1.0] + [4.0 if i % 2 else 2.0 for i in range(1, len(e) - 1)] + [1.0])
    return {"lpost": lpost, "posterior": e / (np.sum(wt * e) * (ranges[1] - ranges[0]) / 3.0), "mode": x,
            "newton": np.array(its, np.int64)}


def _exact_mala(c, seed):
    locs, z0, eps, unif = _mala_inputs(c, seed)
    h = 0.01
    p = torch.from_numpy(locs)
    d = torch.sqrt((p[:, None, 0] - p[None, :, 0]) ** 2 + (p[:, None, 1] - p[None, :, 1]) ** 2)
    M = torch.exp(-d / 0.05)
    Ls, Lm = torch.linalg.cholesky(torch.exp(-d / 0.5)), torch.linalg.cholesky(h * M)

    def at(x):
        g = torch.cholesky_solve(x[:, None], Ls)[:, 0]
        return x, g, x - 0.5 * h * (M @ g)

    def qf(v):
        w = torch.linalg.solve_triangular(Lm, v[:, None], upper=False)
        return -0.5 * (w * w).sum().item()

    cur = at(torch.from_numpy(z0))
    trace, acc, lr = [], [], []
    for t in range(unif.size):
        new = at(cur[2] + Lm @ torch.from_numpy(np.ascontiguousarray(eps[:, t])))
        r = (-0.5 * (new[0] @ new[1]).item() + 0.5 * (cur[0] @ cur[1]).item() + qf(cur[0] - new[2])
             - qf(new[0] - cur[2]))
        ok = unif[t] < math.exp(min(0.0, r))
        cur = new if ok else cur
        trace.append(cur[0])
        acc.append(int(ok))
        lr.append(r)
    return {"z": cur[0], "trace": torch.stack(trace), "log_ratio": np.array(lr), "accepted": np.array(acc, np.int64)}
