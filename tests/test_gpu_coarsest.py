"""The coarsest level's solve on grids that are their own coarsest level: one
V-cycle there is e = A^+ r with the pseudo-inverse the device builds, compared
with the pseudo-inverse of the face-wise dense matrix in numpy.

Sizes: one elimination tile (64 cells) exactly, one cell into the second, odd
counts, and the largest level (1024 cells).  Bound: an inverse of an n x n
matrix of condition kappa formed in FP64 is off by at most about n eps kappa
of its largest value.
"""
import numpy as np
import pytest

from general_cases import rand_case
from oracle.dense import matrix_gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (nx, ny, nz): none of them is halved
SIZES = [(4, 4, 4), (5, 13, 4), (9, 9, 9), (7, 11, 13), (16, 16, 4)]


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    from paper_2012_11744_amd import solver
    return solver


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def check(S, beta, sigma, bc, h, general, precision="fp64"):
    shape = beta[0].shape
    A = matrix_gen(beta, sigma, bc, h)
    act = np.diag(A) < 0
    B = A[np.ix_(act, act)]
    ev = np.abs(np.linalg.eigvalsh(B))
    live = ev > ev.max() * 1e-12            # drops the constant mode of a singular operator
    kappa = ev.max() / ev[live].min()
    P = np.zeros_like(A)
    P[np.ix_(act, act)] = np.linalg.pinv(B, rcond=1e-12, hermitian=True)
    r = np.random.default_rng(3).uniform(-1.0, 1.0, shape)
    want = (P @ r.reshape(-1)).reshape(shape)
    with S.Solver([dev(b) for b in beta], h, bc, precision=precision, coarsest=1024,
                  sigma=None if sigma is None else dev(sigma), general=general) as sol:
        assert sol.levels == 1
        got = sol.vcycle(dev(r)).cpu().numpy()
        again = sol.vcycle(dev(r)).cpu().numpy()
    assert np.array_equal(got, again)
    err = np.abs(got - want).max() / np.abs(want).max()
    # FP32 storage of the right-hand side and the correction: eps 2^-24 each
    bound = A.shape[0] * 2.0 ** -52 * kappa + (0 if precision == "fp64" else 4 * 2.0 ** -24 * kappa)
    print(shape, bc, "n", A.shape[0], "kappa %.1e err %.1e bound %.1e" % (kappa, err, bound), flush=True)
    assert err <= bound


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 0, 1), (1, 1, 1)])
def test_pressure_operator(S, n, bc):
    shape = (n[2], n[1], n[0])
    rng = np.random.default_rng(1)
    beta = [10.0 ** rng.uniform(-1.0, 0.0, shape) for _ in range(3)]
    for m in range(3):
        if bc[m]:
            np.moveaxis(beta[m], 2 - m, 0)[0] = 0.0
    check(S, beta, None, bc, 0.125, False)
    check(S, beta, None, bc, 0.125, False, "fp32")


@pytest.mark.parametrize("n", SIZES)
def test_general_operator(S, n):
    """Closed links, a diagonal term, a cell held by it alone, an excluded cell."""
    shape = (n[2], n[1], n[0])
    bc = (1, 0, 1)
    beta, sigma = rand_case(shape, bc, 7)
    for m in range(3):
        if bc[m]:
            np.moveaxis(beta[m], 2 - m, 0)[0] = 0.0
    check(S, beta, sigma, bc, 0.5, True)


# (nx, ny, nz), walls: levels above one tile whose cells have two colours (every
# periodic extent even), with a half-size matrix of 40 cells, 62 (of 125), one
# tile exactly, 75 and 130
COLOURS = [((4, 4, 5), (0, 0, 1)), ((5, 5, 5), (1, 1, 1)), ((4, 4, 8), (0, 0, 0)),
           ((5, 5, 6), (1, 1, 0)), ((4, 5, 13), (0, 1, 1))]


@pytest.mark.parametrize("n,bc", COLOURS)
def test_two_colours(S, n, bc):
    shape = (n[2], n[1], n[0])
    rng = np.random.default_rng(5)
    beta = [10.0 ** rng.uniform(-1.0, 0.0, shape) for _ in range(3)]
    for m in range(3):
        if bc[m]:
            np.moveaxis(beta[m], 2 - m, 0)[0] = 0.0
    check(S, beta, rng.uniform(0.0, 3.0, shape) * (rng.random(shape) < 0.5), bc, 0.5, True)
    check(S, beta, None, bc, 0.125, False)
    # excluded cells of both colours under the singular operator
    hole = np.zeros(shape, dtype=bool)
    hole.reshape(-1)[[5, 6, 20]] = True
    for m in range(3):
        beta[m][hole | np.roll(hole, 1, 2 - m)] = 0.0
    check(S, beta, None, bc, 0.125, True)


# (nx, ny, nz): grids that are whole tails of the V-cycle: 16^3 smooths two
# levels; the others one, over a coarsest level of 64 (staged in LDS), 120, 240,
# 384 and 512 cells (the last three solved by a kernel of their own)
TAILS = [(16, 16, 16), (8, 8, 8), (10, 12, 8), (12, 10, 16), (24, 16, 8), (8, 8, 64)]


def reference_vcycle(S, beta, bc, h, r, nu, omega, nu_fine=None):
    """The same cycle (nu sweeps on levels of at most 4096 cells, nu_fine on
    larger ones) from the single-kernel entry points, whose parity with
    the oracle is tested on its own, and numpy's pseudo-inverse."""
    shape = beta[0].shape
    n = shape[::-1]
    if int(np.prod(shape)) <= 64 or min(shape) < 8 or any(v % 2 for v in shape):
        A = matrix_gen([b.cpu().numpy() for b in beta], None, bc, h)
        ev = np.abs(np.linalg.eigvalsh(A))
        kappa = ev.max() / ev[ev > ev.max() * 1e-12].min()
        P = np.linalg.pinv(A, rcond=1e-12, hermitian=True)
        return dev((P @ r.cpu().numpy().reshape(-1)).reshape(shape)), A.shape[0] * kappa
    e = torch.zeros_like(r)
    sweeps = nu if int(np.prod(shape)) <= 4096 else nu_fine
    S.k_smooth(shape, h, bc, beta, r, e, sweeps=sweeps, zero_init=True, omega=omega)
    half = tuple(v // 2 for v in shape)
    rH = torch.empty(half, dtype=torch.float64, device="cuda")
    S.k_resid_restrict(shape, h, bc, beta, e, r, rH)
    bH = tuple(torch.empty_like(rH) for _ in range(3))
    S.k_coarsen_beta(shape, h, bc, beta, bH)
    eH, amp = reference_vcycle(S, bH, bc, 2 * h, rH, nu, omega, nu_fine)
    S.k_prolong_add_weighted(shape, h, bc, eH, S.k_prolong_weights(shape, h, bc, beta), e)
    for _ in range(sweeps):
        out = torch.empty_like(e)
        S.k_smooth_fused(shape, h, bc, beta, r, e, out, first_colour=1, omega=omega)
        e = out
    return e, amp


@pytest.mark.parametrize("n", TAILS)
@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 0, 1), (0, 1, 0)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_tail_cycle(S, n, bc, precision):
    shape = (n[2], n[1], n[0])
    rng = np.random.default_rng(5)
    beta = [10.0 ** rng.uniform(-1.0, 0.0, shape) for _ in range(3)]
    for m in range(3):
        if bc[m]:
            np.moveaxis(beta[m], 2 - m, 0)[0] = 0.0
    r = rng.uniform(-1.0, 1.0, shape)
    beta, r = [dev(b) for b in beta], dev(r - r.mean())
    h, nu, omega = 0.125, 4, 1.2
    want, amp = reference_vcycle(S, beta, bc, h, r, nu, omega)
    with S.Solver(beta, h, bc, precision=precision, nu_coarse=nu, omega=omega) as sol:
        got = sol.vcycle(r)
        again = sol.vcycle(r)
    assert torch.equal(got, again)
    # rounding: a few eps of the largest value at each of some 40 half sweeps
    # and transfers, which the (contracting) rest of the cycle does not amplify,
    # and n eps kappa of the coarsest solve; FP32 storage in all but that solve
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    bound = 400 * eps + amp * (2.0 ** -53 if precision == "fp64" else 2.0 ** -40)
    err = ((got - want).abs().max() / want.abs().max()).item()
    print(n, bc, precision, "err %.1e bound %.1e" % (err, bound), flush=True)
    assert err <= bound


# Levels above the tail, smoothed by the two-sweep pass in every storage type:
# several tiles of 64 x 8 cells and chunks of planes, rows that end inside a
# tile, at its edge, and within the four cells that a tile owns beyond it
# (nx = 68: one tile with walls, two when periodic), three sweeps (a pass and
# a single sweep), sides of one tile.
FUSED = [((32, 32, 32), 2), ((24, 20, 28), 2), ((36, 20, 8), 2), ((64, 24, 16), 2), ((68, 36, 20), 2), ((132, 20, 24), 2),
         ((136, 16, 24), 3), ((72, 40, 48), 2)]


@pytest.mark.parametrize("n,nu", FUSED)
@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 1, 1), (1, 0, 0), (0, 1, 1)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_fused_levels(S, n, nu, bc, precision):
    shape = (n[2], n[1], n[0])
    rng = np.random.default_rng(6)
    beta = [10.0 ** rng.uniform(-1.0, 0.0, shape) for _ in range(3)]
    for m in range(3):
        if bc[m]:
            np.moveaxis(beta[m], 2 - m, 0)[0] = 0.0
    r = rng.uniform(-1.0, 1.0, shape)
    beta, r = [dev(b) for b in beta], dev(r - r.mean())
    h, omega = 0.125, 1.2
    want, amp = reference_vcycle(S, beta, bc, h, r, 4, omega, nu)
    with S.Solver(beta, h, bc, precision=precision, nu_pre=nu, nu_post=nu, omega=omega) as sol:
        got = sol.vcycle(r)
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24     # as test_tail_cycle
    bound = 600 * eps + amp * (2.0 ** -53 if precision == "fp64" else 2.0 ** -40)
    err = ((got - want).abs().max() / want.abs().max()).item()
    print(n, bc, precision, "err %.1e bound %.1e" % (err, bound), flush=True)
    assert err <= bound


@pytest.mark.parametrize("zero", [False, True])
def test_two_sweep_pass_beyond_2_gib(S, zero):
    """Arrays past the reach of a 32-bit byte offset: data that repeat every 40
    planes give what the 40 planes alone give, to the rounding of the four
    colour updates (which products are fused depends on a plane's place in the
    march): 4 eps of the largest value each."""
    nx, ny, per, rep = 1024, 1024, 40, 13                       # 2.18 GB an array
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    small = [torch.rand((per, ny, nx), generator=g, device="cuda") for _ in range(5)]
    big = [t.repeat(rep, 1, 1) for t in small]
    outs = []
    for a in (small, big):
        out = torch.empty_like(a[0])
        S.k_smooth2_fused_f32(tuple(out.shape), 0.1, (1, 0, 0), a[:3], a[3], a[4], out,
                              zero_init=zero, omega=1.2)
        outs.append(out)
    torch.cuda.synchronize()
    assert big[0].numel() * 4 > 2 ** 31
    diff = max((o - outs[0]).abs().max().item() for o in outs[1].view(rep, per, ny, nx))
    assert diff <= 4 * 4 * 2.0 ** -24 * outs[0].abs().max().item()


# (nx, ny, nz): one workgroup, odd sizes (a cell per thread), 2 x 2 cells, more
# partial sums than threads, and two grids of the direction pass that exchanges
# rows: one whose residual update leaves its sums to a kernel of their own, one
# whose last block along x has 8 lanes
SOLVES = [(4, 4, 4), (9, 11, 9), (24, 20, 28), (96, 80, 64), (256, 192, 128), (272, 176, 80)]


@pytest.mark.parametrize("n", SOLVES)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_solve_scalars(S, n, precision):
    """The step lengths and direction coefficients that the outer iteration's
    kernels form for themselves: the true residual meets the tolerance that the
    recurrence reports (its drift is a few eps per iteration), and a repeat
    gives the same bits."""
    shape = (n[2], n[1], n[0])
    g = torch.Generator().manual_seed(9)
    beta = [(10.0 ** -torch.rand(shape, generator=g, dtype=torch.float64)).cuda()
            for _ in range(3)]
    beta[2][0] = 0.0
    b = torch.rand(shape, generator=g, dtype=torch.float64).cuda()
    b -= b.mean()
    with S.Solver(beta, 1.0 / n[0], (0, 0, 1), precision=precision, coarsest=1024) as sol:
        p = sol.solve(b, tol=1e-9).clone()
        again = sol.solve(b, tol=1e-9)
        rel = float((b - sol.apply(p)).norm() / b.norm())
        # link coefficients formed from densities
        sol.update_density(0.1 + torch.rand(shape, generator=g, dtype=torch.float64).cuda())
        p2 = sol.solve(b, tol=1e-9)
        rel2 = float((b - sol.apply(p2)).norm() / b.norm())
    print(n, precision, "rel %.3e %.3e" % (rel, rel2), flush=True)
    assert torch.equal(p, again)
    assert max(rel, rel2) <= 1e-9 * (1 + 1e-3) + 1e-12


@pytest.mark.parametrize("n", [(192, 128, 128), (256, 160, 80)])
def test_projection_either_side_of_the_cache_size(S, n):
    """u = u* - dt beta grad p below and above the size from which the velocities
    are streamed: three roundings of values up to the larger term."""
    shape = (n[2], n[1], n[0])
    g = torch.Generator().manual_seed(4)
    beta, us = ([torch.rand(shape, generator=g, dtype=torch.float64).cuda() + 0.5
                 for _ in range(3)] for _ in range(2))
    beta[1][:, 0] = 0.0
    p = torch.rand(shape, generator=g, dtype=torch.float64).cuda()
    h, dt = 0.25, 0.125
    with S.Solver(beta, h, (0, 1, 0), precision="fp32") as sol:
        u = sol.project(us, p, dt)
    for m in range(3):
        want = us[m] - dt / h * beta[m] * (p - torch.roll(p, 1, 2 - m))
        if m == 1:
            want[:, 0] = 0.0
        assert float((u[m] - want).abs().max()) <= 4 * 2.0 ** -52 * 2.5
