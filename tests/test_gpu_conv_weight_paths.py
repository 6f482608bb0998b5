"""Weight-gradient convolution on both of its kernels.  The kernel per tap (few
voxels, small or flat maps): every number of input-channel tiles, groups of 64
output channels that end inside, voxels that end inside a stage of 32, inputs
split inside an 8-channel piece.  The z march on maps large enough for it:
columns that leave the box, several z chunks, the same splits."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import test_gpu_conv_weight_grad as edges  # noqa: E402
from test_gpu_conv_weight_grad import mg  # noqa: E402,F401

# (n, d, h, w, ca, cb, cout, up)
PER_TAP = [
    (40, 2, 2, 2, 64, 0, 128, False),
    (5, 2, 3, 3, 8, 24, 16, False),
    (33, 1, 1, 1, 48, 0, 48, False),
    (2, 2, 4, 2, 8, 88, 80, True),
    (9, 1, 5, 7, 128, 0, 16, False),
    (3, 2, 2, 6, 128, 64, 144, True),
    (1, 1, 1, 77, 16, 0, 16, False),
]
MARCH = [
    (1, 6, 64, 66, 8, 40, 16, True),
    (2, 37, 65, 47, 16, 0, 32, False),
    (1, 40, 48, 81, 24, 8, 16, False),
    (1, 34, 48, 64, 16, 0, 16, False),
]


@pytest.mark.parametrize("case", PER_TAP + MARCH, ids=lambda c: "x".join(map(str, c[:4])) + f"-{c[4]}+{c[5]}-{c[6]}")
@pytest.mark.parametrize("inf", [False, True], ids=["finite", "inf"])
def test_weight_gradient(mg, case, inf):  # noqa: F811
    edges.test_weight_gradient_edges(mg, case, inf)
