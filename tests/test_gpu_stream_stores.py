"""Finest passes on levels just below and just above the size from which they
store their result non-temporally (256 MiB touched by a pass): V-cycles against
the oracle in FP64, and the oracle's residual of the solution in mixed
precision."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.oracle import Oracle  # noqa: E402


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


def _problem(shape, seed):
    g = np.random.default_rng(seed)
    mask = np.full(shape, -1, np.int8)
    inner = (slice(1, -1),) * 3
    mask[inner] = np.where(g.random(tuple(s - 2 for s in shape)) < 1e-3, -1, 1)
    rho = np.where(mask == 1, g.standard_normal(shape), 0.0)
    return mask, rho, 1.0 / max(shape)


@pytest.mark.parametrize("shape", [(216, 224, 224), (232, 224, 216)], ids=["below", "above"])
def test_fp64_vcycles_match_oracle(mg, shape):
    mask, rho, h = _problem(shape, 11)
    bytes_ = int((mask == 1).sum()) * 25
    assert (bytes_ > 256 << 20) == (shape[0] == 232)
    print("stream stores", shape, bytes_, flush=True)
    orc = Oracle(mask, h)
    x_o = np.zeros(shape)
    with mg.Hierarchy(torch.from_numpy(mask).cuda(), h) as H:
        f = H.fold(torch.from_numpy(rho).cuda(), None)
        x_g = torch.zeros(shape, dtype=torch.float64, device="cuda")
        for _ in range(2):
            x_g = H.vcycle(x_g, f)
            x_o = orc.vcycle(x_o, rho, None)
        got = x_g.cpu().numpy()
    assert np.all(got[mask == -1] == 0)
    # two cycles of about 20 passes and transfers, each within a few units in
    # the last place of the largest value
    assert np.abs(got - x_o).max() <= 1e-12 * np.abs(x_o).max()


@pytest.mark.parametrize("shape", [(264, 272, 280), (288, 280, 272)], ids=["below", "above"])
def test_mixed_solution_has_the_residual_it_reports(mg, shape):
    mask, rho, h = _problem(shape, 12)
    bytes_ = int((mask == 1).sum()) * 13
    assert (bytes_ > 256 << 20) == (shape[0] == 288)
    print("stream stores mixed", shape, bytes_, flush=True)
    with mg.Hierarchy(torch.from_numpy(mask).cuda(), h, precision="mixed") as H:
        phi, info = H.solve(torch.from_numpy(rho).cuda(), tol=1e-9)
    assert info["r_final"] <= 1e-9 * info["r_ref"]
    r = Oracle(mask, h).residual_norm(rho, phi.cpu().numpy(), None)
    # sums of 2e7 squares in another order, and residuals 1e-9 of their terms'
    # scale over h^2: relative rounding of 1e-16 * 8e4 / 1e-9 of each
    assert abs(r - info["r_final"]) <= 1e-2 * info["r_final"]
