"""Line passes (uot_grid_line.hip) at the edges of their tiles, segments and
blocks, against the FP64 oracle and against the direct passes (grid_kernel 1,
separate kernels).  Tolerances as in test_gpu_parity.py: potentials to 1e-11
(FP64) and 1e-5 (FP32) of max(|u|_inf, eps) after a fixed iteration count, from
the rounding of a half-step (a few 2^-53 / 2^-24) times 1 / (1 - z1 z2)."""
import numpy as np
import pytest
import torch

from oracle import uot_oracle as O
from tests.helpers import oracle_div, pot_rel_err, rounded

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1607_05816_amd import uot as U  # noqa: E402

DEV = torch.device("cuda:0")
TOL = {torch.float64: 1e-11, torch.float32: 1e-5}
DTYPES = [torch.float32, torch.float64]

# sizes around a tile (16 cells), a segment (8 .. 64 taps), a block (512, 1024,
# 4096 cells; 1, 2, .. lines), fewer lines than a block takes, one cell per
# axis; eps spans the segment lengths (c = h^2 log2(e) / eps from 1e-4 to 0.7)
CASES = [
    ((16, 16), 1e-2), ((17, 33), 5e-3), ((31, 15), 2e-2), ((64, 48), 1e-3), ((1, 40), 1e-2), ((40, 1), 1e-2),
    ((3, 260), 1e-2), ((513, 5), 2e-3), ((1025, 2), 1e-3), ((2, 4096), 1e-3), ((65, 127), 2e-3),
    ((1,), 1e-2), ((16,), 1e-2), ((255,), 1e-3), ((512,), 1e-3), ((513,), 1e-3), ((1024,), 1e-3), ((1025,), 1e-3),
    ((5, 20, 30), 1e-2), ((4, 32, 32), 2e-3), ((9, 64, 64), 1e-2), ((3, 65, 64), 1e-2), ((33, 1, 17), 1e-2),
]


def T(a, dtype):
    return torch.tensor(np.asarray(a), dtype=dtype, device=DEV)


def case(shape, dtype, nb=1):
    npd = np.float32 if dtype == torch.float32 else np.float64
    rng = np.random.default_rng(sum(shape) + nb)
    size = int(np.prod(shape))
    h = tuple(1.0 / max(n, 8) for n in shape)
    p = rounded(rng.uniform(0.2, 2.0, (nb, size)), npd)
    q = rounded(rng.uniform(0.2, 2.0, (nb, size)), npd)
    p[:, :: 7] = 0.0   # exact zeros: potentials of -inf on both sides
    d = rounded(np.full(size, float(np.prod(h))), npd)
    return h, p, q, d


def log(a):
    with np.errstate(divide="ignore"):
        return np.log(a)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape,eps", CASES)
def test_solve_matches_oracle_and_direct_passes(shape, eps, dtype):
    h, p, q, d = case(shape, dtype)
    print("case line", shape, eps, dtype, flush=True)
    F1, F2 = U.KL(0.1), U.TV(0.2)
    prob = U.grid_problem(shape, h, T(p[0], dtype), T(q[0], dtype), T(d, dtype), T(d, dtype), F1, F2)
    kw = dict(eps0=10 * eps, eps_stages=3, iters_per_stage=3, tol=0.0, max_iter=15)
    u, v, info = U.solve(prob, eps, record=True, **kw)
    ud, vd, infod = U.solve(prob, eps, record=True, grid_kernel=U.GRID_DIRECT, **kw)
    # (a single cell without mass has residual 0 and stops at the last stage)
    assert info["iters"] == infod["iters"] == (15 if np.any(p[0] > 0) else 10)
    assert pot_rel_err(u.cpu(), ud.cpu(), eps) < TOL[dtype]
    assert pot_rel_err(v.cpu(), vd.cpu(), eps) < TOL[dtype]
    # the first residuals (far from 0) to the FP32 merge of their partials
    np.testing.assert_allclose(info["res_hist"][:4], infod["res_hist"][:4], rtol=1e-4)
    ref = O.solve(O.GridGeom(shape, h), log(p[0]), np.log(q[0]), np.log(d), np.log(d), oracle_div(F1), oracle_div(F2),
                  eps, tol=0.0, max_iter=info["iters"], eps0=10 * eps, n_stages=3, iters_per_stage=3)
    assert pot_rel_err(u.cpu(), ref["u"], eps) < TOL[dtype]
    assert pot_rel_err(v.cpu(), ref["v"], eps) < TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES)
def test_line_loop_stops_and_resumes(dtype):
    """One block iterates a 1-D problem: the chunk length must not matter, a
    tolerance stops it at the iteration the direct passes stop at (both reduce
    the residual in FP32, so within a rounding of tol: 1), and a solve resumed
    from its v repeats it."""
    n, eps = 200, 1e-2
    h, p, q, d = case((n,), dtype)
    F = U.KL(0.5)
    print("case line loop", dtype, flush=True)
    prob = U.grid_problem((n,), h, T(p[0], dtype), T(q[0], dtype), T(d, dtype), T(d, dtype), F, F)
    kw = dict(eps0=0.5, eps_stages=3, iters_per_stage=7)
    a = U.solve(prob, eps, tol=0.0, max_iter=61, check_every=50, **kw)
    b = U.solve(prob, eps, tol=0.0, max_iter=61, check_every=2, use_graph=False, **kw)
    c = U.solve_async(prob, eps, tol=0.0, max_iter=61, check_every=16, **kw)
    info = c.result()
    assert a[2]["iters"] == b[2]["iters"] == info["iters"] == 61
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert torch.equal(a[0], c.u) and torch.equal(a[1], c.v)
    tol = 1e-4
    s = U.solve(prob, eps, tol=tol, max_iter=5000, **kw)[2]
    t = U.solve(prob, eps, tol=tol, max_iter=5000, grid_kernel=U.GRID_DIRECT, **kw)[2]
    assert s["converged"] and s["residual"] <= tol and abs(s["iters"] - t["iters"]) <= 1
    ua, va, _ = U.solve(prob, eps, tol=0.0, max_iter=30)
    _, vb, _ = U.solve(prob, eps, tol=0.0, max_iter=20)
    uc, vc, _ = U.solve(prob, eps, tol=0.0, max_iter=10, v0=vb)
    assert torch.equal(ua, uc) and torch.equal(va, vc)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape,nb", [((33, 21), 5), ((64, 64), 40), ((7, 12, 10), 3)])
def test_fields_match_single_solves(shape, nb, dtype):
    eps = 5e-3
    h, p, q, d = case(shape, dtype, nb)
    print("case line fields", shape, nb, dtype, flush=True)
    F = U.KL(0.2)
    kw = dict(eps0=5e-2, eps_stages=2, iters_per_stage=4, tol=0.0, max_iter=20)
    u, v, info = U.solve_fields(shape, h, T(p, dtype), T(q, dtype), T(d, dtype), T(d, dtype), F, F, eps, record=True,
                                **kw)
    worst = 0.0
    for k in range(nb):
        prob = U.grid_problem(shape, h, T(p[k], dtype), T(q[k], dtype), T(d, dtype), T(d, dtype), F, F)
        uk, vk, ik = U.solve(prob, eps, grid_kernel=U.GRID_DIRECT, **kw)
        assert pot_rel_err(u[k].cpu(), uk.cpu(), eps) < TOL[dtype]
        assert pot_rel_err(v[k].cpu(), vk.cpu(), eps) < TOL[dtype]
        worst = max(worst, ik["residual"])
    assert info["residual"] == pytest.approx(worst, rel=1e-3)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("F2", [U.KL(0.3), U.EQ(), U.TV(0.1), U.RG(0.7, 1.3)])
@pytest.mark.parametrize("shape,nb", [((33, 20), 3), ((16, 64), 12), ((5, 2048), 2), ((6, 1500), 3)])
def test_barycenter_matches_oracle(shape, nb, F2, dtype):
    eps = 5e-3
    h, p, _, d = case(shape, dtype, nb)
    npd = np.float32 if dtype == torch.float32 else np.float64
    p = rounded(p + 0.3, npd)
    alpha = np.arange(1, nb + 1) / (nb * (nb + 1) / 2)
    print("case line barycentre", shape, nb, F2, dtype, flush=True)
    F1 = U.KL(0.2)
    u, v, logh, info = U.barycenter(shape, h, T(p, dtype), alpha, T(d, dtype), T(d, dtype), F1, F2, eps, tol=0.0,
                                    max_iter=8)
    ref = O.barycenter(O.GridGeom(shape, h), np.log(p), alpha, np.log(d), np.log(d), oracle_div(F1), oracle_div(F2),
                       eps, tol=0.0, max_iter=8)
    assert pot_rel_err(u.cpu(), ref["u"], eps) < TOL[dtype]
    assert pot_rel_err(v.cpu(), ref["v"], eps) < TOL[dtype]
    assert np.max(np.abs(logh.cpu().numpy() - ref["logh"])) / np.max(np.abs(ref["logh"])) < 10 * TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("shape,eps", [((300,), 5e-3), ((37, 70), 5e-3), ((6, 24, 40), 1e-2), ((70, 37, 5), 5e-3)])
def test_half_step_matches_oracle(shape, eps, side, dtype):
    h, p, q, d = case(shape, dtype)
    print("case line half step", shape, side, dtype, flush=True)
    F = U.KL(0.5)
    rng = np.random.default_rng(3)
    size = int(np.prod(shape))
    npd = np.float32 if dtype == torch.float32 else np.float64
    pin, pold = (rounded(0.05 * rng.standard_normal(size), npd) for _ in range(2))
    prob = U.grid_problem(shape, h, T(p[0], dtype), T(q[0], dtype), T(d, dtype), T(d, dtype), F, F)
    new, S, r = U.half_step(prob, eps, side, T(pin, dtype), T(pold, dtype))
    new2, S2, r2 = U.half_step_noalloc(prob, eps, side, T(pin, dtype), T(pold, dtype))
    assert torch.equal(new, new2) and torch.equal(S, S2) and r == r2
    ref = O.GridGeom(shape, h).lse_x(pin / eps + np.log(d), eps)
    # S is a log-sum-exp: a few roundings of its terms' exponents
    tol = {torch.float64: 1e-12, torch.float32: 2e-6}[dtype]
    assert np.max(np.abs(S.cpu().numpy() - ref)) < tol * max(1.0, np.max(np.abs(ref)))
