"""Coarsest operators that cannot be inverted: what a solve and a V-cycle say."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    from paper_2012_11744_amd import solver
    return solver


def closed(n):
    return [torch.zeros(n[::-1], dtype=torch.float64, device="cuda") for _ in range(3)]


def active(beta):
    act = torch.zeros_like(beta[0], dtype=torch.bool)
    for m in range(3):
        act |= (beta[m] > 0) | (beta[m].roll(-1, 2 - m) > 0)
    return act


def fields(beta, seed):
    """A mean-free right-hand side and a first guess on the active cells."""
    act = active(beta)
    rng = np.random.default_rng(seed)
    b, p = (torch.from_numpy(rng.uniform(-1.0, 1.0, tuple(act.shape))).cuda() * act
            for _ in range(2))
    return torch.where(act, b - b.sum() / act.sum(), b), p


# Links inside one coarse cell only: (nx, ny, nz), walls, the coarsest level's
# form (one tile of 64 cells; 125 cells of two colours; 125 as one matrix)
INSIDE = [((8, 8, 8), (0, 0, 0)), ((10, 10, 10), (1, 1, 1)), ((10, 10, 10), (0, 0, 0))]


@pytest.mark.parametrize("n,bc", INSIDE)
@pytest.mark.parametrize("outer", ["pcg", "dc"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
def test_zero_coarsest_operator_is_refused(S, n, bc, outer, precision):
    beta = closed(n)
    beta[0][4, 4, 5] = 1.0                  # between cells 4 and 5 along x
    beta[1][2, 3, 2] = 2.0
    b, p = fields(beta, 1)
    with S.Solver(beta, 1.0, bc, precision=precision, outer=outer, general=True) as sol:
        assert sol.levels == 2
        for _ in range(2):                  # refused each time
            with pytest.raises(Exception, match="coarsest operator is zero"):
                sol.solve(b, p=p)
            with pytest.raises(Exception, match="coarsest operator is zero"):
                sol.vcycle(b)
        # links between coarse cells: accepted
        open_ = [torch.ones_like(t) for t in beta]
        sol.update_coeffs(open_)
        full = torch.randn_like(b)
        p = sol.solve(full, tol=1e-9)
        res = (full - full.mean() - sol.apply(p)).norm() / (full - full.mean()).norm()
        assert float(res) <= 1.01e-9


def two_sets(n, w1, w2):
    """Two disconnected pairs of cells: 0 and nx with a link w1, 2 nx and 3 nx
    with a link w2."""
    beta = closed(n)
    f = beta[1].reshape(-1)
    f[n[0]] = w1
    f[3 * n[0]] = w2
    return beta


# With h = 1 the elimination of these meets a pivot of exactly 0, in exact
# arithmetic and in the kernels' (w2 = 4 w1: the pivots are 2, 2, 4, 0; with two
# colours and w2 = 3 w1 the Schur complement is a constant 2 x 2 matrix): one
# tile, one matrix of 80 cells, 128 and 260 cells of two colours
PAIRS = [((4, 4, 4), (1, 1, 1), 4.0), ((4, 5, 4), (1, 0, 1), 4.0), ((4, 4, 8), (1, 1, 1), 3.0),
         ((4, 5, 13), (1, 1, 1), 3.0)]


@pytest.mark.parametrize("n,bc,w2", PAIRS)
@pytest.mark.parametrize("outer", ["pcg", "dc"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_rejected_operator_leaves_a_warm_start_alone(S, n, bc, w2, outer, precision):
    beta = two_sets(n, 1.0, w2)
    b, p0 = fields(beta, 2)
    with S.Solver(beta, 1.0, bc, precision=precision, outer=outer, general=True, warm_start=True,
                  coarsest=1024) as sol:
        for rhs in (b, torch.zeros_like(b), sol.apply(p0)):   # iterates, b = 0, p0 solves it
            p = p0.clone()
            with pytest.raises(Exception, match="not definite"):
                sol.solve(rhs, p=p)
            assert torch.equal(p, p0)
            with pytest.raises(Exception, match="not definite"):
                sol.vcycle(rhs)
        sol.update_coeffs([torch.ones_like(t) for t in beta])   # a good operator again
        p = sol.solve(b, tol=1e-9, p=p0.clone())
        assert float((b - b.mean() - sol.apply(p)).norm() / (b - b.mean()).norm()) <= 1.01e-9


@pytest.mark.parametrize("outer", ["pcg", "dc"])
def test_zero_operator_leaves_a_warm_start_alone(S, outer):
    beta = closed((8, 8, 8))
    beta[0][4, 4, 5] = 1.0
    b, p0 = fields(beta, 3)
    with S.Solver(beta, 1.0, (0, 0, 0), outer=outer, general=True, warm_start=True) as sol:
        p = p0.clone()
        with pytest.raises(Exception, match="coarsest operator is zero"):
            sol.solve(b, p=p)
        assert torch.equal(p, p0)
