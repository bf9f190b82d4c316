"""Every direct-load tile form at its edges, whichever form the rule would
take."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _check(M, N, K, a_t, b_t, fp32):
    from paper_2502_17683_amd import test_gemm
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    dt = torch.float32 if fp32 else torch.float64
    A = to_dev(rng.standard_normal((K, M) if a_t else (M, K)), dt)
    B = to_dev(rng.standard_normal((N, K) if b_t else (K, N)), dt)
    C = test_gemm(A, B, None, a_t, b_t)
    opA, opB = (x.cpu().numpy().astype(np.float64) for x in (A.T if a_t else A, B.T if b_t else B))
    u = 2.0 ** -24 if fp32 else 2.0 ** -53
    # K products and sums, and as many again for the FP64 reference
    assert np.all(np.abs(C.cpu().numpy() - opA @ opB) <= 2 * (K + 1) * u * (np.abs(opA) @ np.abs(opB)))
    return C


# one tile with rows and columns missing on both sides, several with
# remainders of a few rows or columns and of nearly a tile; K below, at and
# past a k-step of every form
@pytest.mark.parametrize("M,N,K", [(4, 124, 44), (132, 260, 20), (252, 388, 16), (100, 36, 260), (380, 28, 64)])
@pytest.mark.parametrize("a_t,b_t", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("fp32", [False, True])
def test_forced_forms(M, N, K, a_t, b_t, fp32):
    from paper_2502_17683_amd import test_tile_force
    say(f"forced forms M={M} N={N} K={K} a_t={a_t} b_t={b_t} fp32={fp32}")
    got = []
    try:
        for bm in (32, 64, 128):
            test_tile_force(bm)
            got.append(_check(M, N, K, a_t, b_t, fp32))
    finally:
        test_tile_force(0)
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


# two full rounds of 128-tiles, the last row and column of tiles not whole
@pytest.mark.parametrize("a_t,b_t", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("fp32", [False, True])
def test_large_tiles_with_remainders(a_t, b_t, fp32):
    say(f"128-tiles a_t={a_t} b_t={b_t} fp32={fp32}")
    _check(2044, 4092, 20, a_t, b_t, fp32)
