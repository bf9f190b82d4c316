"""The FP64 dataflow factorisation in 16-column panels: sizes around a panel
and a block, and a pivot that fails at the first and last column of a panel."""
import numpy as np
import pytest
import torch

from gpu_util import rel_err, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [1, 15, 16, 17, 48, 63, 65, 127, 128, 129, 193])
@pytest.mark.parametrize("scale", [1.0, 1e-130, 1e130])
def test_solve_at_panel_edges(R, scale):
    from paper_2502_17683_amd import test_solve
    say(f"panels R={R} scale={scale}")
    rng = np.random.default_rng(R)
    A = rng.standard_normal((R, R + 5))
    V = (A @ A.T / R + 0.5 * np.eye(R)) * scale
    M = rng.standard_normal((37, R))
    F, failed = test_solve(to_dev(V), to_dev(M))
    assert not failed
    # R sums of up to R terms in the factor and in either substitution
    assert rel_err(F.cpu().numpy() * scale, np.linalg.solve(V / scale, M.T).T) <= 50 * R * np.linalg.cond(V) * 1.1e-16


@pytest.mark.parametrize("c", [0, 15, 16, 31, 48, 63, 64, 79, 99])
@pytest.mark.parametrize("value", [-1.0, 0.0, np.nan, np.inf])
def test_failed_pivot(c, value):
    from paper_2502_17683_amd import test_solve
    say(f"panels failed pivot c={c} value={value}")
    R = 100
    rng = np.random.default_rng(c)
    A = rng.standard_normal((R, R + 5))
    V = A @ A.T / R + 0.5 * np.eye(R)
    V[c, c] = value
    _, failed = test_solve(to_dev(V), torch.ones((3, R), dtype=torch.float64, device="cuda"))
    assert failed


@pytest.mark.parametrize("r_cp", [1, 63, 65, 129])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_normal_matrix_formed_by_the_factorisation(r_cp, precision):
    """One sweep with V formed inside the dataflow factorisation against one
    with V formed by its own launch (a plan that solves in panels of one
    block), and the sweep repeated on the same plan (ready flags clear)."""
    from paper_2502_17683_amd import CPD
    from synth import init_factors, make_thc
    say(f"normal matrix r_cp={r_cp} {precision}")
    n, r_thc = 33, 130
    X, Z = make_thc(n, r_thc, r_cp)
    init = [to_dev(f) for f in init_factors([n] * 4, r_cp, 7 + r_cp)]
    got = []
    for panel in (0, 1):
        plan = CPD(to_dev(X), to_dev(Z), r_cp, init, tol=0.0, fit_floor=0.0, solve_panel=panel, precision=precision)
        for _ in range(2):
            plan.set_factors(init, torch.ones(r_cp, dtype=torch.float64, device="cuda"))
            plan.sweep(1)
            F, lam = plan.factors()
            got.append([x.double() for x in F + [lam]])
        cond = plan.stats()["cond_est"]
        plan.close()
    u = 2.0 ** -24 if precision == "fp32" else 2.0 ** -53
    for a, b, c, _ in zip(*got):
        assert torch.equal(a, b)
        assert float((a - c).norm() / c.norm()) <= 200 * r_cp * max(cond, 1.0) * u
