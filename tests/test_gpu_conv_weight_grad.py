"""Weight-gradient convolution at the edges of its work split: columns of
16 x 16 voxels that end inside, at and past the box, chunks of z planes, a
single plane, input channels split between the two tensors inside a 16-channel
tile, and infinities at the faces of the box."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import unet_oracle as U  # noqa: E402


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


def bf16(a):
    t = torch.from_numpy(np.ascontiguousarray(a)).to(torch.bfloat16).cuda()
    return t, t.double().cpu().numpy()


# (n, d, h, w, ca, cb, cout, up)
CASES = [
    (1, 1, 1, 1, 16, 0, 16, False),
    (1, 2, 15, 17, 16, 0, 16, False),
    (1, 3, 16, 16, 8, 8, 16, False),
    (2, 37, 17, 16, 16, 0, 32, False),     # several z chunks, the last one shorter
    (1, 40, 16, 33, 8, 24, 16, False),
    (1, 6, 32, 18, 8, 40, 16, True),
    (3, 8, 16, 32, 128, 64, 16, True),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:4])) + f"-{c[4]}+{c[5]}-{c[6]}")
@pytest.mark.parametrize("inf", [False, True], ids=["finite", "inf"])
def test_weight_gradient_edges(mg, case, inf):
    n, d, h, w, ca, cb, cout, up = case
    print("weight gradient", case, inf, flush=True)
    rng = np.random.default_rng(7)
    a = rng.standard_normal((n, d // 2, h // 2, w // 2, ca) if up else (n, d, h, w, ca))
    if inf:  # first and last cell of the box: taps that reach past the face stay finite
        a[0, 0, 0, 0, 0] = np.inf
        a[-1, -1, -1, -1, -1] = np.inf
    a_t, a = bf16(a)
    b_t, b = bf16(rng.standard_normal((n, d, h, w, cb))) if cb else (None, None)
    g_t, g = bf16(rng.standard_normal((n, d, h, w, cout)))
    x = U.up2_nearest(a) if up else a
    if cb:
        x = np.concatenate([x, b], axis=-1)
    w0 = np.zeros((27, cout, ca + cb))
    fin = np.where(np.isfinite(x), x, 1.0)
    _, dw, db = U.conv3d_backward(fin, w0, g)
    _, dwa, dba = U.conv3d_backward(np.abs(fin), w0, np.abs(g))
    got_w, got_b = mg.nn.conv3d_bwd_weight(g_t, a_t, b=b_t, up_a=up)
    got_w, got_b = got_w.double().cpu().numpy(), got_b.double().cpu().numpy()
    # an infinity reaches the taps whose output voxel is in the box, no others
    hit = U.conv3d_backward(np.where(np.isfinite(x), 0.0, 1.0), w0, np.ones_like(g))[1] > 0
    assert np.array_equal(~np.isfinite(got_w), hit)
    # float32 sums of n d h w products of bfloat16 values (exact in float32)
    eps = n * d * h * w * 2.0 ** -24
    assert (np.abs(got_w - dw)[~hit] <= (eps * dwa)[~hit] + 1e-30).all()
    assert (np.abs(got_b - db) <= eps * dba + 1e-30).all()
