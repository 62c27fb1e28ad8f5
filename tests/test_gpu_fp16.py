"""The coarsest correction of FP16 storage is rounded to FP32 and then to FP16."""
import numpy as np
import pytest

from oracle.dense import matrix

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    from paper_2012_11744_amd import solver
    return solver


@pytest.mark.parametrize("n,bc", [((10, 8, 7), (0, 1, 1)), ((9, 9, 9), (1, 1, 1)), ((4, 4, 4), (0, 0, 0))])
def test_coarsest_correction_is_rounded_twice(S, n, bc):
    """On grids that are their own coarsest level: every value of 400 cycles.  One
    rounding of the sum differs from two in some 1 of 2e4 values; the error of
    numpy's pseudo-inverse (1e-12) moves a value over an edge of FP32 and then of
    FP16 in 1 of some 1e9."""
    shape = n[::-1]
    rng = np.random.default_rng(21)
    beta = [10.0 ** rng.uniform(-1.0, 0.0, shape) for _ in range(3)]
    for m in range(3):
        if bc[m]:
            np.moveaxis(beta[m], 2 - m, 0)[0] = 0.0
    h = 0.5
    P = np.linalg.pinv(matrix(beta, bc, h), rcond=1e-12, hermitian=True)
    differ = 0
    with S.Solver([torch.from_numpy(b).cuda() for b in beta], h, bc, precision="fp16",
                  coarsest=1024) as sol:
        assert sol.levels == 1
        for _ in range(400):
            r = rng.uniform(-1.0, 1.0, shape).astype(np.float16).astype(np.float64)
            got = sol.vcycle(torch.from_numpy(r).cuda()).cpu().numpy().reshape(-1)
            want = (P @ r.reshape(-1)).astype(np.float32).astype(np.float16).astype(np.float64)
            differ += int((got != want).sum())
    print(n, bc, "values that differ:", differ, flush=True)
    assert differ == 0
