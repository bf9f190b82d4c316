"""The solve of a sweep by its residual, whose bound does not grow with the
condition of the normal matrix."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, say, to_dev
from synth import init_factors, make_thc

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("r_cp", [1, 63, 65, 129, 193])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_solve_residual_of_a_sweep(r_cp, precision):
    """F3 V - M3 after a sweep, with V from the factors that the sweep left
    and M3 its MTTKRP: the normal matrix that the factorisation forms, the
    factorisation and both solves of one to four block columns."""
    from paper_2502_17683_amd import CPD
    say(f"residual r_cp={r_cp} {precision}")
    n, r_thc = 100, 300
    X, Z = make_thc(n, r_thc, r_cp)
    plan = CPD(to_dev(X), to_dev(Z), r_cp, [to_dev(f) for f in init_factors([n] * 4, r_cp, 40 + r_cp)], tol=0.0,
               fit_floor=0.0, precision=precision)
    plan.sweep(1)
    F, lam = ([x.cpu().numpy() for x in y] if isinstance(y, list) else y.cpu().numpy() for y in plan.factors())
    M = plan.mttkrp(3).cpu().numpy()
    plan.close()
    V = np.ones((r_cp, r_cp))
    for m in range(3):
        V *= F[m].T @ F[m]
    S = F[3] * lam
    L = np.linalg.cholesky(V)
    u = 2.0 ** -24 if precision == "fp32" else 2.0 ** -53
    # the factorisation and two substitutions of r_cp terms, whose diagonal
    # blocks are applied as explicit inverses (the condition of L), the
    # entries of V (three sums of n terms and their products), the rounding
    # of F3 and lambda
    k = 3 * (r_cp + 1) * np.linalg.cond(L) + 3 * (n + 2) + 4
    bound = k * u * np.linalg.norm(np.abs(L) @ np.abs(L).T, 2) * np.linalg.norm(S)
    # (four values swapped in one tile, or one Gram left out of it: 4.5e-3 and more at two to four block columns)
    assert bound <= 3e-3 * np.linalg.norm(M)
    assert np.linalg.norm(S @ V - M) <= bound


@pytest.mark.parametrize("R", [64, 100, 193])
@pytest.mark.parametrize("panel", [0, 1])
@pytest.mark.parametrize("fp32", [False, True])
def test_solve_reads_the_lower_triangle(R, panel, fp32):
    """Grams in 32-tiles leave the upper right quadrant of a diagonal block
    as it was: other values above the diagonal change nothing."""
    from paper_2502_17683_amd import test_solve
    say(f"lower triangle R={R} panel={panel} fp32={fp32}")
    rng = np.random.default_rng(R)
    dt = torch.float32 if fp32 else torch.float64
    A = rng.standard_normal((R, R + 5))
    V = A @ A.T / R + 0.5 * np.eye(R)
    M = to_dev(rng.standard_normal((37, R)), dt)
    F, failed = test_solve(to_dev(V, dt), M, panel=panel)
    G, other = test_solve(to_dev(np.tril(V) + np.triu(rng.standard_normal((R, R)), 1), dt), M, panel=panel)
    assert not failed and not other and torch.equal(F, G)
