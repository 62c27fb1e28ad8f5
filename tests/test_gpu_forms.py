"""Operators and cycles on the forms of the V-cycle's kernels that the ordinary
grids do not reach, against the same cycle from the single-kernel entry points."""
import numpy as np
import pytest

from oracle.dense import matrix_gen
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


# -- a reference cycle in FP64 torch, with diagonal term, excluded cells and W-cycles

def links(beta, bc):
    """Low and high link coefficients per axis, walls closed."""
    lo = [b.clone() for b in beta]
    for m in range(3):
        if bc[m]:
            lo[m].select(2 - m, 0).zero_()
    return lo, [b.roll(-1, 2 - m) for m, b in enumerate(lo)]


def neighbour_sum(lo, hi, e):
    return sum(lo[m] * e.roll(1, 2 - m) + hi[m] * e.roll(-1, 2 - m) for m in range(3))


class Cycle:
    """The V- or W-cycle of the library: nu red-black sweeps on each side (nu_tail on
    levels of at most 4096 cells), coefficients rounded to the storage type."""

    def __init__(self, S, beta, sigma, bc, h, nu, nu_tail, omega, kind, store):
        self.bc, self.omega, self.kind = bc, omega, kind
        rnd = lambda t: t.to(store).double()
        self.lev = []
        while True:
            shape = tuple(beta[0].shape)
            cells = int(np.prod(shape))
            L = dict(shape=shape, h2=h * h, tail=cells <= 4096, nu=nu_tail if cells <= 4096 else nu)
            L["lo"], L["hi"] = links([rnd(b) for b in beta], bc)
            sg = None if sigma is None else rnd(h * h * sigma)
            L["sg"] = torch.zeros_like(beta[0]) if sg is None else sg
            L["dg"] = sum(L["lo"]) + sum(L["hi"]) + L["sg"]
            z, y, x = torch.meshgrid(*(torch.arange(v, device="cuda") for v in shape), indexing="ij")
            L["colour"] = [(x + y + z) % 2 == c for c in (0, 1)]
            self.lev.append(L)
            if cells <= 64 or min(shape) < 8 or any(v % 2 for v in shape):
                L["pinv"] = self.invert([b.cpu().numpy() for b in beta],
                                        None if sigma is None else sigma.cpu().numpy(), h)
                return
            L["w"] = S.k_prolong_weights(shape, h, bc, beta)
            L["S"], L["h"] = S, h
            half = tuple(v // 2 for v in shape)
            bH = tuple(torch.empty(half, dtype=torch.float64, device="cuda") for _ in range(3))
            S.k_coarsen_beta(shape, h, bc, beta, bH)
            sigma = None if sigma is None else self.mean8(sigma)
            beta, h = bH, 2 * h

    def invert(self, beta, sigma, h):
        A = matrix_gen(beta, sigma, self.bc, h)
        ev = np.abs(np.linalg.eigvalsh(A))
        self.amp = A.shape[0] * ev.max() / ev[ev > ev.max() * 1e-12].min()
        return dev(np.linalg.pinv(A, rcond=1e-12, hermitian=True))

    @staticmethod
    def mean8(x):
        return torch.nn.functional.avg_pool3d(x[None, None], 2)[0, 0].contiguous()

    def sweeps(self, L, r, e, order):
        for _ in range(L["nu"]):
            for c in order:
                gs = (neighbour_sum(L["lo"], L["hi"], e) - L["h2"] * r) / L["dg"]
                new = torch.where(L["dg"] > 0, (1 - self.omega) * e + self.omega * gs, 0 * e)
                e = torch.where(L["colour"][c], new, e)
        return e

    def run(self, l, r, e=None, kind=None):
        L = self.lev[l]
        if "pinv" in L:
            return (L["pinv"] @ r.reshape(-1)).reshape(L["shape"])
        kind = "v" if L["tail"] else (kind or self.kind)
        e = self.sweeps(L, r, torch.zeros_like(r) if e is None else e, (0, 1))
        Ae = (neighbour_sum(L["lo"], L["hi"], e) - L["dg"] * e) / L["h2"]
        rH = self.mean8(r - Ae)
        eH = self.run(l + 1, rH, None, kind)
        if kind == "w":
            eH = self.run(l + 1, rH, eH, "w")
        e = e.clone()
        L["S"].k_prolong_add_weighted(L["shape"], L["h"], self.bc, eH, L["w"], e)
        return self.sweeps(L, r, e, (1, 0))


# (nx, ny, nz), cycle: tails of one smoothed level whose coarsest is solved by a kernel
# of its own (384 and 512 cells) or in the same launch (64, 120), of two; and a level
# above a split tail, which a W-cycle enters a second time with its correction
CYCLES = [((24, 16, 8), "v"), ((8, 8, 64), "v"), ((8, 8, 8), "v"), ((10, 12, 8), "v"), ((16, 16, 16), "v"),
          ((48, 32, 16), "v"), ((48, 32, 16), "w"), ((40, 48, 32), "w")]


@pytest.mark.parametrize("n,kind", CYCLES)
@pytest.mark.parametrize("term", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
def test_general_cycle(S, n, kind, term, precision):
    """One cycle around solids, with and without a diagonal term, at an h whose
    square is no power of two.  Bounds, relative to the largest value: as in
    test_excluded_cells for the arithmetic; FP16 storage rounds the correction
    to 2^-11 when it leaves a level and the right-hand side when it enters one, twice
    as often in a W-cycle."""
    bc, h, omega = (1, 0, 1), 1.0 / 13, 1.2
    beta, r, solid = around_solids(n, bc, 9)
    # coefficients and a right-hand side that FP16 holds
    beta = [(b * 256).round() / 256 for b in beta]
    r = (r * 256).round() / 256
    sigma = None
    if term:
        g = torch.Generator(device="cuda").manual_seed(3)
        sigma = torch.rand(r.shape, generator=g, device="cuda", dtype=torch.float64)
        sigma = torch.where(solid | (sigma < 0.5), torch.zeros_like(sigma), sigma * 20.0)
    else:
        r = torch.where(solid, r, r - r[~solid].mean()).half().double()
    store = {"fp64": torch.float64, "fp32": torch.float32, "fp16": torch.float16}[precision]
    cyc = Cycle(S, beta, sigma, bc, h, 2, 4, omega, kind, store)
    want = cyc.run(0, r)
    with S.Solver(beta, h, bc, precision=precision, omega=omega, cycle=kind, sigma=sigma,
                  general=True) as sol:
        got = sol.vcycle(r)
        again = sol.vcycle(r)
    assert torch.equal(got, again)
    if precision == "fp64":
        bound = 1200 * 2.0 ** -53 + cyc.amp * 2.0 ** -53
    else:
        bound = 1200 * 2.0 ** -24 + cyc.amp * 2.0 ** -40
    if precision == "fp16":
        above = sum(not L["tail"] for L in cyc.lev)
        bound += 2.0 ** -11 * (1 + (8 if kind == "v" else 16) * above)
    on = ~solid if precision == "fp16" else torch.ones_like(solid)
    err = ((got - want)[on].abs().max() / want.abs().max()).item()
    print(n, kind, term, precision, "err %.1e bound %.1e" % (err, bound), flush=True)
    assert err <= bound


# -- the direction pass that exchanges rows (above 3 * 2^20 cells; all sides are then
# multiples of 16): walls along x and y, several blocks along x, a last one of 8 lanes

@pytest.mark.parametrize("n,bc", [((272, 176, 80), (1, 1, 0)), ((256, 96, 144), (0, 1, 1))])
@pytest.mark.parametrize("form", ["sigma", "closed", "rho"])
@pytest.mark.parametrize("precision", ["fp32", "fp64", "fp16"])
def test_direction_pass_by_rows(S, n, bc, form, precision):
    """The true residual, by the operator's own kernel, meets the tolerance that the
    recurrence reports, and a repeat gives the same bits."""
    beta, b, solid = around_solids(n, bc, 11)
    h, kw = 1.0 / n[0], {}
    if form == "sigma":
        kw["sigma"] = torch.where(solid, 0.0, 60.0 + 50.0 * b)
    elif form == "rho":
        solid = torch.zeros_like(solid)
        beta = [torch.ones_like(t) for t in beta]
        b = b - b.mean()
    with S.Solver(beta, h, bc, precision=precision, general=form != "rho", **kw) as sol:
        if form == "rho":
            g = torch.Generator(device="cuda").manual_seed(5)
            sol.update_density(0.1 + torch.rand(b.shape, generator=g, device="cuda",
                                                dtype=torch.float64))
        p = sol.solve(b, tol=1e-9)
        iters = sol.last_stats["outer_iters"]
        again = sol.solve(b, tol=1e-9, p=torch.empty_like(b))
        r = torch.where(solid, torch.zeros_like(b), b - sol.apply(p))
        rel = float(r.norm() / b.norm())
    print(n, bc, form, precision, "iters", iters, "rel %.3e" % rel, flush=True)
    assert torch.equal(p, again)
    assert rel <= 1e-9 * (1 + 1e-3) + 1e-12
    assert float(p[solid].abs().sum()) == 0.0
    assert iters <= 12                       # a wrong direction costs iterations first
