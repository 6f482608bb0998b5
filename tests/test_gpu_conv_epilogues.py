"""The convolution's epilogues and the gated gradient kernels, bit for bit the
separate kernels: the gradient of an activation with the ReLU below it, the
split gradient of a concatenated input, the gated pooling gradient; output
tilings of 1 to 4 channel groups, partial voxel tiles, outputs that allow no
8-byte stores and channel counts that allow no 16-byte ones."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import unet_oracle as uo  # noqa: E402


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


@pytest.mark.parametrize("shape", [(2, 8, 24, 40), (1, 16, 8, 16), (3, 32, 40, 8)], ids=lambda s: "x".join(map(str, s)))
def test_backward_pass_equals_separate_kernels(mg, shape):
    print("epilogues", shape, flush=True)
    n, d, h, w = shape
    g = np.random.default_rng(7)
    rho, target = (torch.from_numpy(g.standard_normal(shape)).cuda() for _ in range(2))
    mask = torch.from_numpy(np.where(g.random(shape) < 0.6, 1, -1).astype(np.int8)).cuda()
    net = mg.UNet(seed=3)
    net.loss_grad(rho, mask, target)
    layers = uo.LAYERS
    idx = {L[0]: i for i, L in enumerate(layers)}
    shp = lambda c, lv: (n, d >> (lv - 1), h >> (lv - 1), w >> (lv - 1), c)  # noqa: E731
    A = {L[0]: net.tensor("act", i, shp(L[3], L[4])) for i, L in enumerate(layers)}
    G = {L[0]: net.tensor("act_grad", i, shp(L[3], L[4])) for i, L in enumerate(layers)}
    GP = [net.tensor("pool_grad", k, shp(16 << k, k + 2)) for k in range(3)]
    par = uo.unpack(net.params())

    def dgrad(l):
        wf = mg.nn.weight_flip(torch.from_numpy(par[l][0].copy()).cuda().bfloat16())
        return mg.nn.conv3d(G[l], wf, relu=False)

    for l, below in (("dec1b", "dec1a"), ("dec2b", "dec2a"), ("dec3b", "dec3a"), ("mid4b", "mid4a"),
                     ("enc3b", "enc3a"), ("enc2b", "enc2a"), ("enc1b", "enc1a")):
        assert torch.equal(mg.nn.relu_bwd(dgrad(l), A[below]), G[below]), below
    for l, below, skip, k in (("dec1a", "dec2b", "enc1b", 0), ("dec2a", "dec3b", "enc2b", 1),
                              ("dec3a", "mid4b", "enc3b", 2)):
        dup, dskip = mg.nn.split_grad(dgrad(l), layers[idx[l]][1])
        assert torch.equal(mg.nn.relu_bwd(dup, A[below]), G[below]), below
        assert torch.equal(mg.nn.relu_bwd(mg.nn.pool2_bwd(GP[k], dskip), A[skip]), G[skip]), skip
    for l, k in (("enc2a", 0), ("enc3a", 1), ("mid4a", 2)):
        assert torch.equal(dgrad(l), GP[k]), l
    net.close()


@pytest.mark.parametrize("cin,cout", [(16, 16), (8, 32), (16, 48), (16, 64), (32, 48), (48, 96), (64, 64)])
@pytest.mark.parametrize("size", [(1, 5, 6, 19), (4, 32, 32, 64)], ids=["small", "wide_tilings"])
def test_channel_tilings_and_unaligned_output(mg, cin, cout, size):
    print("tilings", cin, cout, size, flush=True)
    torch.manual_seed(cin * cout)
    x = torch.randn(*size, cin, device="cuda").bfloat16()
    w = (torch.randn(27, cout, cin, device="cuda") / (27 * cin) ** 0.5).bfloat16()
    bias = torch.randn(cout, device="cuda")
    got = mg.nn.conv3d(x, w, bias)
    # reference: the same convolution in 32 bits over the BF16 operands
    ref = torch.nn.functional.conv3d(x.float().permute(0, 4, 1, 2, 3).cpu(),
                                     w.float().view(3, 3, 3, cout, cin).permute(3, 4, 0, 1, 2).cpu(), bias.cpu(),
                                     padding=1).relu().permute(0, 2, 3, 4, 1)
    # sums of 27 cin products in 32 bits (1e-5 of the operands' scale) and one rounding to BF16
    assert bool(((got.cpu().float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all())
    # an output that starts on an odd 2-byte address: same values
    import ctypes as C
    buf = torch.zeros(got.numel() + 1, dtype=torch.bfloat16, device="cuda")
    st = mg.load_library().mg_nn_conv3d_fwd(x.data_ptr(), cin, 0, None, 0, w.data_ptr(), bias.data_ptr(),
                                            buf.data_ptr() + 2, cout, 1, *size,
                                            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    assert torch.equal(buf[1:].view_as(got), got)


@pytest.mark.parametrize("c", [3, 8, 12, 16])
def test_pool_gradient_channel_counts(mg, c):
    torch.manual_seed(c)
    g = torch.randn(2, 2, 4, 3, c, device="cuda").bfloat16()
    x = torch.randn(2, 4, 8, 6, c, device="cuda").bfloat16()
    got = mg.nn.pool2_bwd(g, x)
    up = g.float().repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)
    assert torch.equal(got, (x.float() + 0.125 * up).bfloat16())


@pytest.mark.parametrize("stride", [1, 2, 4, 8])
def test_guess_from_unaligned_fields(mg, stride):
    """Fields that start on no 16-byte (masks: 4-byte) address: same guess, bit for bit."""
    print("unaligned guess", stride, flush=True)
    g = np.random.default_rng(stride)
    shape = (16 * stride, 8 * stride, 24 * stride)
    n = int(np.prod(shape))
    rho, b = (torch.from_numpy(g.standard_normal(n + 1)).cuda() for _ in range(2))
    mask = torch.from_numpy(np.where(g.random(n + 1) < 0.5, 1, -1).astype(np.int8)).cuda()
    odd = [t[1:].view(shape) for t in (rho, mask, b)]
    net = mg.UNet(seed=5)
    out = torch.empty(n + 1, dtype=torch.float64, device="cuda")
    got = net.infer(odd[0], odd[1], odd[2], stride=stride, out=out[1:].view(shape))
    ref = net.infer(*(t.clone() for t in odd), stride=stride)
    assert bool((ref != 0).any()) and bool((ref[odd[1] != 1] == 0).all())
    # at stride 1 the input scale is summed by atomics: a last bit may differ
    assert torch.equal(got, ref) if stride > 1 else torch.allclose(got, ref, rtol=1e-2, atol=1e-3 * float(ref.abs().max()))
    net.close()


def test_upsample_of_more_planes_than_a_grid_dimension(mg):
    """A column of 65,540 coarse planes: more than one block row of the launch."""
    import ctypes as C
    nz = 65540
    c = torch.randn(nz, 1, 2, dtype=torch.float64, device="cuda")
    m = torch.ones(2 * nz, 2, 4, dtype=torch.int8, device="cuda")
    f = torch.full((2 * nz, 2, 4), float("nan"), dtype=torch.float64, device="cuda")
    st = mg.load_library().mg_upsample_guess(C.c_void_p(c.data_ptr()), 2, 1, nz, C.c_void_p(m.data_ptr()),
                                             C.c_void_p(f.data_ptr()),
                                             C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    # per axis 3/4 of the parent and 1/4 of the next cell on the child's side (edge cells repeated)
    ref = c
    for ax in range(3):
        n = ref.shape[ax]
        i = torch.arange(n, device="cuda")
        lo = ref.index_select(ax, (i - 1).clamp(min=0))
        hi = ref.index_select(ax, (i + 1).clamp(max=n - 1))
        ref = torch.stack([0.75 * ref + 0.25 * lo, 0.75 * ref + 0.25 * hi], dim=ax + 1).flatten(ax, ax + 1)
    assert float((f - ref).abs().max()) <= 1e-14 * float(ref.abs().max())
