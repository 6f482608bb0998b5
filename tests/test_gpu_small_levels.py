"""The one-workgroup call on small levels: every form it takes (one level
relaxed, two and three levels, the deepest level as a matrix or relaxed, odd and
thin boxes, boxes too large for registers) against the oracle's cycles."""
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


# (finest shape, levels the small call gets)
SHAPES = [
    (16, 16, 16),    # 8^3 + matrix of 4^3
    (32, 32, 32),    # 16^3 + 8^3 + matrix
    (10, 14, 26),    # one odd level 5 x 7 x 13, relaxed
    (22, 26, 30),    # one odd level of 2145 cells
    (26, 26, 26),    # 13^3
    (20, 24, 56),    # 10 x 12 x 28 + 5 x 6 x 14, relaxed in registers
    (12, 16, 32),    # 6 x 8 x 16 (768 cells), or + the matrix of 3 x 4 x 8 with edges down to 3
    (34, 30, 38),    # 17 x 15 x 19 = 4845 cells: the general path
    (8, 8, 128),     # thin
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("opts", [dict(), dict(n_cycles=2), dict(n_pre=1, n_post=3, n_coarse_sweeps=5, min_coarse_dim=3)],
                         ids=lambda o: "-".join(f"{k}={v}" for k, v in o.items()) or "default")
def test_small_levels_match_oracle(mg, shape, opts):
    print("small levels", shape, opts, flush=True)
    p = gen.random_small_problem(shape, 9, active_frac=0.8, blur=1.0)
    orc = O.Oracle(p.mask, p.h, min_coarse_dim=opts.get("min_coarse_dim", 4))
    oo = {"n_coarse" if k == "n_coarse_sweeps" else k: v for k, v in opts.items() if k != "min_coarse_dim"}
    act = p.mask == 1
    mask, rho, b = (torch.from_numpy(a).cuda() for a in (p.mask, p.rho, p.dirichlet))
    with mg.Hierarchy(mask, p.h, **opts) as H:
        assert H.nlevels() > 1
        for order in (1, 2):
            f = H.fold(rho, b)
            x, x_o = torch.zeros_like(f), np.zeros(shape)
            for _ in range(3):
                x = H.vcycle(x, f, order=order)
                x_o = orc.vcycle(x_o, p.rho, p.dirichlet, order=order, **oo)
                got = x.cpu().numpy()
                assert np.abs(got - x_o)[act].max() <= 1e-11 * np.abs(x_o[act]).max()
