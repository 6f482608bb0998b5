"""Levels around the lines between cube passes and marches, which differ by pass,
level and precision: bit for bit the marches that the item-depth options select,
iterates and norms."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


MARCH = dict(item_depth_fine=16, item_depth_l1=4, item_depth_coarse=2)
# cubes of the finest level / of level 1: 2704, 3600, 4096, 4608 / 968 and 1152,
# 1512, 1728, 2128, 2704 (full boxes)
SHAPES = [(104, 104, 104), (120, 120, 120), (128, 128, 128), (128, 128, 144), (176, 176, 160), (128, 192, 192),
          (144, 224, 192), (192, 192, 192), (152, 224, 256), (208, 208, 208)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_lines_keep_the_iterates(mg, shape, precision):
    print("lines", shape, precision, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    mask = torch.full(shape, -1, dtype=torch.int8, device="cuda")
    mask[1:-1, 1:-1, 1:-1] = 1
    mask[40:47, 50:61, 30:44] = -1
    rho = torch.randn(shape, dtype=torch.float64, device="cuda", generator=g)
    o = dict(precision=precision, max_cycles=3, bc_order="second")
    with mg.Hierarchy(mask, 1.0 / shape[2], **o) as H, mg.Hierarchy(mask, 1.0 / shape[2], **o, **MARCH) as M:
        x, ix = H.solve(rho, tol=1e-12, check=False)
        y, iy = M.solve(rho, tol=1e-12, check=False)
        assert torch.equal(x, y)
        assert ix["history"] == iy["history"]
        assert H.residual_norm(rho, x) == M.residual_norm(rho, x)
