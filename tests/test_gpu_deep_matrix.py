"""The deepest level of the one-workgroup call as a matrix product: values that
are not finite stay with the part of the domain that they belong to, as in the
relaxation the matrix stands for."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


# (shape, min_coarse_dim): the call holds 16^3, 8^3 and 4^3; 12^3 and 6^3; four
# levels down to 1 x 1 x 4 (the general path).  Two boxes, a quarter or more of
# the longest edge apart, so that no level couples them.
BOXES = [((64, 64, 64), 4), ((96, 96, 96), 4), ((64, 64, 256), 1)]


@pytest.mark.parametrize("shape,min_dim", BOXES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("order", [1, 2])
def test_nonfinite_values_stay_in_their_part(mg, shape, min_dim, value, order):
    print("parts", shape, min_dim, value, order, flush=True)
    nx = shape[2]
    lo = nx // 4 if nx == 256 or nx == 64 else nx // 3       # first part: [1, lo)
    hi = nx // 2 if nx == 256 else 3 * nx // 4 if nx == 64 else 2 * nx // 3
    mask = np.full(shape, -1, np.int8)
    mask[1:-1, 1:-1, 1:lo] = 1
    mask[1:-1, 1:-1, hi:nx - 1] = 1
    rng = np.random.default_rng(5)
    f = rng.standard_normal(shape) * (mask == 1)
    x = rng.standard_normal(shape) * (mask == 1)
    g = f.copy()
    g[shape[0] // 2, shape[1] // 2, lo // 2] = value
    t = lambda a: torch.from_numpy(a).cuda()
    with mg.Hierarchy(t(mask), 1.0 / nx, min_coarse_dim=min_dim) as H:
        assert H.nlevels(order) > 2
        clean, dirty = H.vcycle(t(x), t(f), order=order), H.vcycle(t(x), t(g), order=order)
    assert bool(torch.isfinite(clean).all())
    assert not bool(torch.isfinite(dirty[:, :, 1:lo]).all())
    assert torch.equal(dirty[:, :, hi:], clean[:, :, hi:])
