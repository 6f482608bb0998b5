"""The one-workgroup call where the other tests do not reach it: four levels and
more (the general path: matrix, W-cycle visits, levels beyond three) against the
oracle's cycles, the second of two levels relaxed or taken as a matrix at the
line between them, and the single-precision instance of every form, by one
mixed-precision cycle against one in double precision."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import oracle as O  # noqa: E402
from paper_1104_1703_amd import gen  # noqa: E402


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


def problem(shape):
    p = gen.random_small_problem(shape, 9, active_frac=0.8, blur=1.0)
    return p, [torch.from_numpy(a).cuda() for a in (p.mask, p.rho, p.dirichlet)]


# (finest shape, min_coarse_dim, levels of the call)
GENERAL = [((32, 32, 32), 2, 4), ((32, 32, 32), 1, 5), ((32, 32, 64), 1, 4), ((96, 32, 32), 1, 4), ((64, 16, 16), 1, 4)]


@pytest.mark.parametrize("shape,min_dim,levels", GENERAL)
@pytest.mark.parametrize("opts", [dict(), dict(n_cycles=2), dict(n_pre=1, n_post=3, n_coarse_sweeps=5, n_cycles=3)],
                         ids=["v", "w", "3"])
def test_four_levels_match_oracle(mg, shape, min_dim, levels, opts):
    print("general", shape, min_dim, opts, flush=True)
    p, (mask, rho, b) = problem(shape)
    orc = O.Oracle(p.mask, p.h, min_coarse_dim=min_dim)
    oo = {"n_coarse" if k == "n_coarse_sweeps" else k: v for k, v in opts.items()}
    act = p.mask == 1
    with mg.Hierarchy(mask, p.h, min_coarse_dim=min_dim, **opts) as H:
        assert sum(np.prod(H.dims(q)) <= 4096 for q in range(H.nlevels())) >= levels
        for order in (1, 2):
            f = H.fold(rho, b)
            x, x_o = torch.zeros_like(f), np.zeros(shape)
            for _ in range(3):
                x = H.vcycle(x, f, order=order)
                x_o = orc.vcycle(x_o, p.rho, p.dirichlet, order=order, **oo)
                assert np.abs(x.cpu().numpy() - x_o)[act].max() <= 1e-11 * np.abs(x_o[act]).max()


# two levels, 125 and 216 cells in the deepest: a pass for every five cells and one more
@pytest.mark.parametrize("shape,sweeps", [((20, 20, 20), 25), ((20, 20, 20), 26), ((24, 24, 24), 43), ((24, 24, 24), 44)])
def test_line_of_the_matrix_matches_oracle(mg, shape, sweeps):
    print("line", shape, sweeps, flush=True)
    p, (mask, rho, b) = problem(shape)
    orc = O.Oracle(p.mask, p.h)
    act = p.mask == 1
    with mg.Hierarchy(mask, p.h, n_coarse_sweeps=sweeps) as H:
        for order in (1, 2):
            f = H.fold(rho, b)
            x, x_o = torch.zeros_like(f), np.zeros(shape)
            for _ in range(2):
                x = H.vcycle(x, f, order=order)
                x_o = orc.vcycle(x_o, p.rho, p.dirichlet, order=order, n_coarse=sweeps)
                assert np.abs(x.cpu().numpy() - x_o)[act].max() <= 1e-11 * np.abs(x_o[act]).max()


# (finest shape, min_coarse_dim): every form of the call
FORMS = [((16, 16, 16), 4), ((32, 32, 32), 4), ((10, 14, 26), 4), ((22, 26, 30), 4), ((20, 24, 56), 4), ((12, 16, 32), 3),
         ((34, 30, 38), 4), ((24, 24, 24), 4), ((32, 32, 32), 2), ((64, 16, 16), 1)]


@pytest.mark.parametrize("shape,min_dim", FORMS)
@pytest.mark.parametrize("bc_order", ["first", "second"])
@pytest.mark.parametrize("n_cycles", [1, 2])
def test_single_precision_call(mg, shape, min_dim, bc_order, n_cycles):
    print("fp32", shape, min_dim, bc_order, n_cycles, flush=True)
    p, (mask, rho, b) = problem(shape)
    got = {}
    for precision in ("fp64", "mixed"):
        with mg.Hierarchy(mask, p.h, precision=precision, min_coarse_dim=min_dim, bc_order=bc_order,
                          n_cycles=n_cycles, max_cycles=1) as H:
            got[precision] = H.solve(rho, None, b, tol=1e-14, check=False)[0]
            levels = H.nlevels()
    # One cycle from zero, all of it in single precision.  A relaxation rounds its
    # eight operations to 2^-24 each; on level l a residual's rounding weighs 4^l
    # times as much as on the finest (h^2), each of at most 32 passes adds it
    # once, and both colours do: 16 x 32 x 4^(levels - 1) x 2^-24 of the largest
    # value bounds the difference
    tol = 16 * 32 * 4.0 ** (levels - 1) * 2.0 ** -24
    assert tol < 0.02
    diff = (got["mixed"] - got["fp64"]).abs().max().item()
    assert 0 < diff <= tol * got["fp64"].abs().max().item()
