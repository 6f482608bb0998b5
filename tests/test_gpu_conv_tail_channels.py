"""Convolution with input channels that do not fill the last chunk of 32 (8, 24,
40, 56, 72): nothing of what follows the weights in memory reaches the output,
here NaNs behind the last weight, and the result is the oracle's."""
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


@pytest.mark.parametrize("ca,cb", [(8, 0), (24, 0), (16, 8), (40, 0), (8, 48), (72, 0)])
@pytest.mark.parametrize("cout,n", [(16, 1), (48, 1100), (64, 1100)], ids=["16", "48", "64"])
def test_channels_past_the_last(mg, ca, cb, cout, n):
    print("tail channels", ca, cb, cout, n, flush=True)
    rng = np.random.default_rng(3)
    d, h, w = (3, 5, 18) if n == 1 else (1, 2, 1)
    cin = ca + cb
    t = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()  # noqa: E731
    a, wt = t(rng.standard_normal((n, d, h, w, ca))), t(rng.standard_normal((27, cout, cin)) * 0.1)
    b = t(rng.standard_normal((n, d, h, w, cb))) if cb else None
    buf = torch.full((27 * cout * cin + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[:27 * cout * cin] = wt.flatten()
    got = mg.nn.conv3d(a, buf[:27 * cout * cin].view(27, cout, cin), None, b=b, relu=False).double().cpu().numpy()
    x = a.double().cpu().numpy()
    if cb:
        x = np.concatenate([x, b.double().cpu().numpy()], axis=-1)
    wd = wt.double().cpu().numpy()
    want = U.conv3d(x, wd, np.zeros(cout), relu=False)
    size = U.conv3d(np.abs(x), np.abs(wd), np.zeros(cout), relu=False)
    # sums of 27 cin exact products in float32, then one rounding to bfloat16
    assert np.all(np.abs(got - want) <= 27 * cin * 2.0 ** -24 * size + 2.0 ** -8 * np.abs(want) + 1e-30)
