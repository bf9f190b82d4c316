"""The direct-load GEMM tiles at their edges: every tile form, remainders of
rows, columns and K, operands that fall back to the staged form, and the
products of a plan that are split over K."""
import numpy as np
import pytest
import torch

from gpu_util import say, to_dev
from oracle import matfree

pytestmark = pytest.mark.gpu


# (M, N, K): 32-, 64- and 128-tiles, each whole, with remainders, and with K
# below, at and past a k-step
@pytest.mark.parametrize("M,N,K", [(32, 32, 32), (34, 98, 2), (36, 100, 36), (1024, 1024, 16), (1030, 1026, 44),
                                   (2048, 4096, 32), (2044, 4100, 20)])
@pytest.mark.parametrize("a_t,b_t", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("fp32", [False, True])
def test_tile_forms(M, N, K, a_t, b_t, fp32):
    from paper_2502_17683_amd import test_gemm
    say(f"tiles M={M} N={N} K={K} a_t={a_t} b_t={b_t} fp32={fp32}")
    rng = np.random.default_rng(M + N + K)
    A = rng.standard_normal((K, M) if a_t else (M, K))
    B = rng.standard_normal((N, K) if b_t else (K, N))
    dt = torch.float32 if fp32 else torch.float64
    Ad, Bd = to_dev(A, dt), to_dev(B, dt)
    C = test_gemm(Ad, Bd, None, a_t, b_t).cpu().numpy().astype(np.float64)
    opA, opB = (x.cpu().numpy().astype(np.float64) for x in (Ad.T if a_t else Ad, Bd.T if b_t else Bd))
    u = 2.0 ** -24 if fp32 else 2.0 ** -53
    # K products and sums, and as many again for the FP64 reference
    assert np.all(np.abs(C - opA @ opB) <= 2 * (K + 1) * u * (np.abs(opA) @ np.abs(opB)))


# the last: 260 tiles of 64, four of them past a whole number per compute
# unit; R_thc odd: the plan's padded copies of X and Z
@pytest.mark.parametrize("dims,r_thc,r_cp", [((20, 30, 25, 41), 260, 70), ((100, 90, 110, 100), 501, 400),
                                             ((41, 203, 41, 203), 977, 491), ((300, 281, 40, 290), 513, 3290)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_split_products_of_a_plan(dims, r_thc, r_cp, precision):
    """MTTKRP of every mode, element by element within the rounding bound of
    its chain of products, twice (the counters of the split tiles are back at
    zero)."""
    from paper_2502_17683_amd import CPD
    say(f"split plan dims={dims} r_thc={r_thc} r_cp={r_cp} {precision}")
    rng = np.random.default_rng(r_thc)
    X = [rng.standard_normal((n, r_thc)) / np.sqrt(r_thc) for n in dims]
    Z = rng.standard_normal((r_thc, r_thc)) / np.sqrt(r_thc)
    F = [rng.standard_normal((n, r_cp)) for n in dims]
    F = [f / np.linalg.norm(f, axis=0) for f in F]
    plan = CPD([to_dev(x) for x in X], to_dev(Z), r_cp, [to_dev(f) for f in F], precision=precision, tol=0.0)
    u = 2.0 ** -24 if precision == "fp32" else 2.0 ** -53
    k = 2.1 * (3 * max(dims) + 2 * r_thc + 16) * u
    for n in range(4):
        ref = matfree.mttkrp(X, Z, F, n)
        A = matfree.mttkrp([np.abs(x) for x in X], np.abs(Z), [np.abs(f) for f in F], n)
        first, second = plan.mttkrp(n), plan.mttkrp(n)
        assert torch.equal(first, second)
        assert np.all(np.abs(first.cpu().numpy() - ref) <= k * A)
    plan.close()


@pytest.mark.parametrize("rows", [1, 17, 16383, 16384, 16400])
def test_inference_row_tiles(rows):
    """BF16 inference gives a row the same bits whichever row tile it falls
    into (16 rows a workgroup below 16384 rows, 64 from there on)."""
    from paper_2502_17683_amd import WarmStartMLP
    from synth import mlp_init_params
    rng = np.random.default_rng(rows)
    net = WarmStartMLP(mlp_init_params(3))
    x = torch.as_tensor(rng.standard_normal((rows, 8)).astype(np.float32), device="cuda")
    out = net.infer_bf16(x)
    part = torch.cat([net.infer_bf16(x[a:a + 5000].contiguous()) for a in range(0, rows, 5000)])
    assert torch.equal(out, part) and bool(torch.isfinite(out).all())


@pytest.mark.parametrize("r_cp", [1, 64, 65, 640, 641])
def test_backward_solve_forms_of_a_plan(r_cp):
    """One FP64 sweep with the backward solve as one product (up to ten block
    columns) and in block pairs (a plan with panels as wide as the matrix
    keeps them): both within the solve's rounding of each other, the
    asynchronous sweep bit for bit the synchronised one."""
    from paper_2502_17683_amd import CPD
    from synth import init_factors, make_thc
    n, r_thc = 45, 260
    X, Z = make_thc(n, r_thc, r_cp)
    init = [to_dev(f) for f in init_factors([n] * 4, r_cp, 1000 + r_cp)]
    got = []
    for panel, sync in ((0, True), (0, False), (64, True)):
        plan = CPD(to_dev(X), to_dev(Z), r_cp, init, tol=0.0, fit_floor=0.0, solve_panel=panel)
        plan.sweep(1, sync=sync)
        F, lam = plan.factors()
        got.append(F + [lam])
        cond = plan.stats()["cond_est"]
        plan.close()
    for a, b, c in zip(*got):
        assert torch.equal(a, b)
        # four updates, each a solve with a normal matrix of this condition
        err = float((a - c).norm() / c.norm())
        assert err <= 200 * r_cp * max(cond, 1.0) * 2.0 ** -53, (err, cond)
