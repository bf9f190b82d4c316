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
