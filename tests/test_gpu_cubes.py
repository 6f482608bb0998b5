"""Levels of few work items run every pass over whole 8^3 cubes: bit for bit
the marches (which the item-depth options select), on boxes whose edges end
inside a cube, a tile or exactly on one, in both precisions and orders."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1104_1703_amd import gen  # noqa: E402


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


MARCH = dict(item_depth_fine=16, item_depth_l1=4, item_depth_coarse=2)


@pytest.mark.parametrize("shape", [(8, 12, 10), (12, 36, 20), (16, 16, 32), (24, 40, 68), (40, 72, 104)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("opts", [dict(), dict(bc_order="first", n_pre=1, n_post=2), dict(precision="mixed"),
                                  dict(n_cycles=2, fuse_restrict=0), dict(n_pre=3, n_post=1, precision="mixed")],
                         ids=lambda o: "-".join(f"{k}={v}" for k, v in o.items()) or "default")
def test_cubes_equal_marches(mg, shape, opts):
    print("cubes", shape, opts, flush=True)
    p = gen.random_small_problem(shape, 5, active_frac=0.75, blur=1.5)
    mask, rho, b = (torch.from_numpy(a).cuda() for a in (p.mask, p.rho, p.dirichlet))
    guess = torch.from_numpy(np.random.default_rng(3).standard_normal(shape)).cuda()
    with mg.Hierarchy(mask, p.h, max_cycles=12, **opts) as H, mg.Hierarchy(mask, p.h, max_cycles=12, **opts, **MARCH) as M:
        for phi0 in (None, guess):
            x, ix = H.solve(rho, None if phi0 is None else phi0.clone(), b, tol=1e-11, check=False)
            y, iy = M.solve(rho, None if phi0 is None else phi0.clone(), b, tol=1e-11, check=False)
            assert ix["status"] == iy["status"] and ix["cycles"] == iy["cycles"]
            assert ix["history"] == iy["history"]
            assert torch.equal(x, y)
        assert H.residual_norm(rho, x, b) == M.residual_norm(rho, x, b)
