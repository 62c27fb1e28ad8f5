"""Grids whose arrays outgrow a 32-bit byte offset, on data that repeat, so that
the small grid of one period gives every value."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    from paper_2012_11744_amd import solver
    return solver


def rand(shape, seed, dtype=torch.float32):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.rand(shape, generator=g, device="cuda", dtype=dtype)


@pytest.mark.parametrize("form", ["zero", "regular", "dot"])
def test_fewest_planes_beyond_2_gib(S, form):
    """Eight planes of 8192 x 8192 cells, periodic along z: the march reaches
    further than one wrap.  Bounds: the values of the small grid to the rounding
    of the four colour updates (4 eps of the largest value each); the sum's terms
    are products of those values with right-hand sides of at most 1."""
    n, rep = 256, 32
    small = [rand((8, n, n), 10 + i) for i in range(5)]
    outs, dots = [], []
    for r in (1, rep):
        a = [t.repeat(1, r, r) for t in small]
        out = torch.empty_like(a[0])
        assert (out.numel() * 4 > 2 ** 31 - 16) == (r == rep)
        if form == "dot":
            dots.append(S.k_smooth2_fused_dot_f32(tuple(out.shape), 0.1, (0, 0, 0), a[:3], a[3],
                                                  a[4], out, omega=1.2))
        else:
            S.k_smooth2_fused_f32(tuple(out.shape), 0.1, (0, 0, 0), a[:3], a[3], a[4], out,
                                  zero_init=form == "zero", omega=1.2)
        torch.cuda.synchronize()
        outs.append(out)
        del a
    tol = 4 * 4 * 2.0 ** -24 * outs[0].abs().max().item()
    for j in range(rep):
        for i in range(rep):
            part = outs[1][:, j * n:(j + 1) * n, i * n:(i + 1) * n]
            assert (part - outs[0]).abs().max().item() <= tol
    if dots:
        assert abs(dots[1] - rep * rep * dots[0]) <= outs[1].numel() * tol


@pytest.mark.parametrize("form", ["plain", "closed", "sigma"])
def test_fp64_level_of_2_gib(S, form):
    """FP64 cycles and solves on 1024 x 512 x 512 cells, whose finest level is read by
    one resource per plane (with the dot product; with closed links; with a
    diagonal term), on data that repeat after 512 cells along x: those of 512^3.
    Cycle: 600 roundings of the largest value as on the small levels, and n eps kappa
    of the coarsest solve (128 cells, kappa below 1e3); the solves' residuals
    then agree far beyond 1e-6."""
    per = 64
    tile = [0.1 + 0.9 * rand((per, per, per), 20 + m, torch.float64) for m in range(3)]
    r = rand((per, per, per), 30, torch.float64)
    solid = torch.zeros((per, per, per), dtype=torch.bool, device="cuda")
    if form != "plain":
        solid[9:30, 11:40, 5:33] = True
        for m in range(3):
            tile[m][solid | solid.roll(1, 2 - m)] = 0.0
    r = torch.where(solid, torch.zeros_like(r), r - r[~solid].mean())
    sg = 0.5 * torch.where(solid, torch.zeros_like(r), r + 1.0)
    got = []
    for cells in ((512, 512, 512), (512, 512, 1024)):
        rep = [c // per for c in cells]
        big = lambda t: t.repeat(*rep)
        kw = {"sigma": big(sg)} if form == "sigma" else {}
        # a right-hand side of all wave lengths of the 512^3 grid
        b = big(r)
        b[:256] *= 0.5
        act = ~big(solid)
        if form != "sigma":
            b = torch.where(act, b - b[act].mean(), torch.zeros_like(b))
        beta = [big(t) for t in tile]
        # as many sweeps in the tail as above it: the wider grid has a level fewer there
        with S.Solver(beta, 0.5, (0, 0, 0), precision="fp64", general=form != "plain", nu_coarse=2,
                      **kw) as sol:
            del beta
            assert sol.levels == 8
            e = sol.vcycle(b)[:, :, :512].clone()
            far = sol.vcycle(b)[:, :, -512:].clone()
            p = sol.solve(b, tol=1e-6)
            got.append((e, far, p[:, :, -512:].clone(), sol.last_stats))
        del b, act, p
    (e, _, p, st), (e2, far2, p2, st2) = got
    bound = (600 + 128 * 1e3) * 2.0 ** -53 * e.abs().max().item()
    assert (e - e2).abs().max().item() <= bound
    assert (e - far2).abs().max().item() <= bound
    assert st["outer_iters"] == st2["outer_iters"]
    assert abs(st["rel_res"] / st2["rel_res"] - 1) <= 1e-6
    assert (p - p2).abs().max().item() <= 1e-6 * p.abs().max().item()
