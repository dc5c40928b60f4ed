"""Edges of the products' work splits against the FP64 oracle: the units of 16
column groups of a WF product (four groups per wave), the chunks of 2048 points
of the spatial order, the tap slices of a 1-D line, and the control step in the
products' launch (residual history and the iteration a solve stops in).
Tolerances on potentials: 1e-11 relative in FP64, 1e-5 in FP32, those of
these paths' other tests; the residual history as there."""
import sys

import numpy as np
import pytest
import torch

from oracle import uot_oracle as O
from paper_1607_05816_amd import synth
from tests.helpers import pot_rel_err, rounded

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1607_05816_amd import uot as U  # noqa: E402

DEV = torch.device("cuda:0")
DTYPES = [pytest.param(torch.float64, 1e-11, id="f64"), pytest.param(torch.float32, 1e-5, id="f32")]


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def T(a, dtype):
    return torch.tensor(np.asarray(a), dtype=dtype, device=DEV)


def npd_of(dtype):
    return np.float64 if dtype == torch.float64 else np.float32


def clouds(seed, N, M, d, npd):
    cp = synth.uniform_clouds(np.random.default_rng(seed), N, M, d)
    return [rounded(a, npd) for a in (cp.x, cp.y, cp.p, cp.q, cp.dx, cp.dy)]


def check(info, u, v, ref, eps, tolr):
    assert info["iters"] == ref["iters"]
    assert pot_rel_err(u.cpu(), ref["u"], eps) < tolr
    assert pot_rel_err(v.cpu(), ref["v"], eps) < tolr


@pytest.mark.parametrize("dtype,tolr", DTYPES)
@pytest.mark.parametrize("N", [1, 65])
@pytest.mark.parametrize("M", [1, 16, 17, 65, 256, 257, 530, 1100])
def test_wf_units(dtype, tolr, N, M):
    """Every group within the cut: units of 1 to 16 groups, the last wave of a
    unit with no group, one or part of one; more than 32 groups: several mask words."""
    x, y, p, q, dx, dy = clouds(N + M, N, M, 2, npd_of(dtype))
    eps, cut = 0.05, 4.0
    F = U.KL(0.5)
    say("case wf units", dtype, N, M)
    prob = U.points_problem(*(T(a, dtype) for a in (x, y, p, q, dx, dy)), F, F, cost=U.WF(cut))
    u, v, info = U.solve(prob, eps, tol=0.0, max_iter=10)
    ref = O.solve(O.PointsGeom(x, y, "wf", cut), *(np.log(a) for a in (p, q, dx, dy)), O.KL(0.5), O.KL(0.5), eps,
                  tol=0.0, max_iter=10)
    check(info, u, v, ref, eps, tolr)


@pytest.mark.parametrize("N", [2047, 2048, 2049, 4097])
def test_spatial_order_chunks(N):
    """Clouds of up to three sort chunks, many points equal (coordinates on 16
    levels): a permutation that lost or repeated a point would leave its
    potential unset."""
    M, eps = 2050, 1e-2
    x, y, p, q, dx, dy = clouds(N, N, M, 2, np.float32)
    x, y = np.round(x * 16) / 16, np.round(y * 16) / 16
    F = U.KL(0.5)
    say("case spatial order", N)
    prob = U.points_problem(*(T(a, torch.float32) for a in (x, y, p, q, dx, dy)), F, F)
    u, v, info = U.solve(prob, eps, tol=0.0, max_iter=10, dense_kernel=U.DENSE_MF3)
    ref = O.solve(O.PointsGeom(x, y), *(np.log(a) for a in (p, q, dx, dy)), O.KL(0.5), O.KL(0.5), eps, tol=0.0,
                  max_iter=10)
    check(info, u, v, ref, eps, 1e-5)


@pytest.mark.parametrize("dtype,tolr", DTYPES)
@pytest.mark.parametrize("n", [511, 512, 513, 1000, 2049])
@pytest.mark.parametrize("cut", [0.3, 4.0])
def test_line_slices(dtype, tolr, n, cut):
    """A line's taps in slices, from one to eight of them, inside a band and whole."""
    pr = synth.hist1d(2, n=n)
    npd = npd_of(dtype)
    p, q = rounded(pr.p, npd), rounded(pr.q, npd)
    d = rounded(np.full(n, pr.h[0]), npd)
    eps = 1e-3
    F = U.KL(0.5)
    say("case line slices", dtype, n, cut)
    prob = U.grid_problem(pr.shape, pr.h, *(T(a, dtype) for a in (p, q, d, d)), F, F, cost=U.WF(cut))
    u, v, info = U.solve(prob, eps, tol=0.0, max_iter=10)
    ref = O.solve(O.GridGeom(pr.shape, pr.h, "wf", cut), *(np.log(a) for a in (p, q, d, d)), O.KL(0.5), O.KL(0.5), eps,
                  tol=0.0, max_iter=10)
    check(info, u, v, ref, eps, tolr)


@pytest.mark.parametrize("kind", ["direct", "tf", "mfma", "mfma_bf16x3", "wf", "line"])
def test_hosted_control(kind):
    """The control step beside the Y product's blocks: the residuals of every
    iteration over an eps schedule, and a stop inside a chunk of iterations (the skipped
    half-steps after it leave the result as it was)."""
    dtype = torch.float64 if kind in ("direct", "wf", "line") else torch.float32
    npd, F = npd_of(dtype), U.KL(0.5)
    kw = {}
    if kind == "line":
        pr = synth.hist1d(3, n=700)
        p, q = rounded(pr.p, npd), rounded(pr.q, npd)
        dx = dy = rounded(np.full(700, pr.h[0]), npd)
        g = O.GridGeom(pr.shape, pr.h, "wf", 4.0)
        prob = U.grid_problem(pr.shape, pr.h, *(T(a, dtype) for a in (p, q, dx, dy)), F, F, cost=U.WF(4.0))
    else:
        x, y, p, q, dx, dy = clouds(7, 900, 1100, 2, npd)
        g = O.PointsGeom(x, y, "wf", 4.0) if kind == "wf" else O.PointsGeom(x, y)
        prob = U.points_problem(*(T(a, dtype) for a in (x, y, p, q, dx, dy)), F, F,
                                cost=U.WF(4.0) if kind == "wf" else U.SQEUCLID)
        if kind != "wf":
            kw["dense_kernel"] = {"direct": U.DENSE_DIRECT, "tf": U.DENSE_TF, "mfma": U.DENSE_MF,
                                  "mfma_bf16x3": U.DENSE_MF3}[kind]
    say("case hosted control", kind)
    eps, tol = 1e-2, 1e-3
    sched = dict(tol=tol, max_iter=400, eps0=1e-1, iters_per_stage=5)
    u, v, info = U.solve(prob, eps, record=True, check_every=32, eps_stages=4, **sched, **kw)
    ref = O.solve(g, *(np.log(a) for a in (p, q, dx, dy)), O.KL(0.5), O.KL(0.5), eps, n_stages=4, **sched)
    assert info["converged"] and ref["converged"] and 20 < info["iters"] < 400 and info["iters"] % 32
    assert info["iters"] == ref["iters"]
    np.testing.assert_allclose(info["res_hist"].numpy()[1:], ref["res"][1:], rtol=1e-3, atol=1e-7)
    tolr = 1e-11 if dtype == torch.float64 else 1e-5
    assert pot_rel_err(u.cpu(), ref["u"], eps) < tolr
    assert pot_rel_err(v.cpu(), ref["v"], eps) < tolr
