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
