"""Operators and cycles on the forms of the V-cycle's kernels that the ordinary
grids do not reach, against the same cycle from the single-kernel entry points."""
import numpy as np
import pytest

from test_gpu_coarsest import dev, reference_vcycle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    from paper_2012_11744_amd import solver
    return solver


def around_solids(n, bc, seed):
    """Coefficients with closed links around a block that no coarse cell of any
    level lines up with, and a right-hand side on the other cells."""
    shape = (n[2], n[1], n[0])
    rng = np.random.default_rng(seed)
    beta = [10.0 ** rng.uniform(-1.0, 0.0, shape) for _ in range(3)]
    solid = np.zeros(shape, dtype=bool)
    solid[1:shape[0] // 2, 3:shape[1] // 2 + 1, 5:shape[2] // 2 + 3] = True
    for m in range(3):
        if bc[m]:
            np.moveaxis(beta[m], 2 - m, 0)[0] = 0.0
        beta[m][solid | np.roll(solid, 1, 2 - m)] = 0.0
    r = np.where(solid, 0.0, rng.uniform(-1.0, 1.0, shape))
    r[~solid] -= r[~solid].mean()
    return [dev(b) for b in beta], dev(r), torch.from_numpy(solid).cuda()


# (nx, ny, nz), sweeps: levels of the two-sweep pass below and above 16384 cells,
# two of them, a pass and a single sweep, and the tail alone
SOLIDS = [((24, 20, 28), 2), ((32, 24, 40), 2), ((64, 48, 32), 3), ((16, 16, 16), 2), ((24, 16, 8), 2)]


@pytest.mark.parametrize("n,nu", SOLIDS)
@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 0, 1)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_excluded_cells(S, n, nu, bc, precision):
    """A cell without an open link stays 0 in a V-cycle without a diagonal term,
    although the prolongation adds to it, and the other cells hold what the
    cycle of the single kernels gives (bounds as for the levels without solids)."""
    beta, r, solid = around_solids(n, bc, 8)
    h, omega = 0.125, 1.2
    want, amp = reference_vcycle(S, beta, bc, h, r, 4, omega, nu)
    with S.Solver(beta, h, bc, precision=precision, nu_pre=nu, nu_post=nu, omega=omega,
                  general=True) as sol:
        got = sol.vcycle(r)
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    bound = 600 * eps + amp * (2.0 ** -53 if precision == "fp64" else 2.0 ** -40)
    err = ((got - want).abs().max() / want.abs().max()).item()
    print(n, bc, precision, "err %.1e bound %.1e" % (err, bound), flush=True)
    assert got[solid].abs().max().item() == 0.0
    assert err <= bound
