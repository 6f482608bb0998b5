"""Linear up-sampling of thin boxes, where a block takes several coarse planes:
planes of one cell, of a row, of just under, exactly and just over a block's
threads, numbers of planes that do not fill the last block, on the GPU against
the same sums in double precision on the host."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


def axis(a, ax):
    n = a.shape[ax]
    i = np.arange(2 * n)
    near, far = i // 2, np.clip(i // 2 + np.where(i % 2, 1, -1), 0, n - 1)
    return 0.75 * np.take(a, near, ax) + 0.25 * np.take(a, far, ax)


@pytest.mark.parametrize("shape", [(1, 1, 1), (5000, 1, 1), (257, 2, 3), (7, 1, 255), (7, 16, 16), (5, 1, 257),
                                   (70001, 1, 2), (3, 127, 2), (4, 43, 3), (33, 20, 18)],
                         ids=lambda s: "x".join(map(str, s)))
def test_thin_planes(mg, shape):
    print("up-sampling", shape, flush=True)
    rng = np.random.default_rng(3)
    c = rng.standard_normal(shape)
    m = np.where(rng.random([2 * s for s in shape]) < 0.6, 1, -1).astype(np.int8)
    got = mg.upsample_guess(torch.from_numpy(c).cuda(), torch.from_numpy(m).cuda()).cpu().numpy()
    want = np.where(m == 1, axis(axis(axis(c, 2), 1), 0), 0.0)
    # seven two-term sums of values of at most max |c|, each rounded at most twice
    assert np.abs(got - want).max() <= 14 * 2.0 ** -53 * np.abs(c).max()
