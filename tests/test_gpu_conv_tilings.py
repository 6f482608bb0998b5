"""Convolution tilings of one to four channel groups a block: many small or flat
maps in one call take the wide tilings, a few of them at a time the narrow one,
with the same products in the same order, so the outputs agree bit for bit.
Whole chunks of 32 channels, trailing ones of 16, 16 channels in all,
up-sampled and concatenated inputs, maps of one voxel, row and plane."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


# channels (ca, cb, cout): 4, 4, 3, 3, 2 and 2 groups, then 16-channel inputs of 4 and 3
CHANNELS = [(32, 0, 64), (16, 32, 64), (32, 0, 96), (48, 0, 48), (96, 0, 32), (48, 0, 32), (16, 0, 64), (16, 0, 48)]
MAPS = [(1, 1, 1, False), (1, 1, 5, False), (1, 6, 3, False), (2, 2, 2, True), (5, 3, 17, False)]


@pytest.mark.parametrize("ca,cb,cout,d,h,w,up", [c + m for c in CHANNELS for m in MAPS if c[1] or not m[3]])
def test_wide_tilings_equal_narrow(mg, ca, cb, cout, d, h, w, up):
    n = 1030
    print("tilings", ca, cb, cout, d, h, w, up, flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16)  # noqa: E731
    a = rnd(n, d // 2, h // 2, w // 2, ca) if up else rnd(n, d, h, w, ca)
    b = rnd(n, d, h, w, cb) if cb else None
    wt, bias = rnd(27, cout, ca + cb) * 0.1, torch.randn(cout, device="cuda", generator=g)
    wide = mg.nn.conv3d(a, wt, bias, b=b, up_a=up, relu=False)
    assert bool(torch.isfinite(wide.float()).all())
    for k in (0, 500, 1020):
        s = slice(k, k + 10)
        part = mg.nn.conv3d(a[s].contiguous(), wt, bias, b=None if b is None else b[s].contiguous(), up_a=up,
                            relu=False)
        assert torch.equal(part, wide[s]), k
