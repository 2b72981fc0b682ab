"""Convolutions of a few images (conv_lat) against the tile kernels that run
the same layer at larger batches: same bits, row by row."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# dtype, C, H, W, K, k, stride, residual, images small / large, conv_lat form
CASES = [
    # whole 64-channel steps: one tap per step, several steps per tap
    ("f16", 64, 24, 24, 64, 3, 1, True, 2, 40, "<_Float16, false, true, 1>"),
    ("f16", 128, 29, 27, 72, 3, 2, False, 1, 33, "<_Float16, false, true, 1>"),
    # chunks of one step in different taps (72 and 8 channels), k tails,
    # 4 of 16 channels in the last tile, pixel tails
    ("f16", 72, 13, 11, 132, 3, 1, True, 3, 33, "<_Float16, false, false, 1>"),
    ("f16", 8, 17, 9, 260, 3, 2, False, 2, 64, "<_Float16, false, false, 1>"),
    # pointwise layers, conv_pw's among them
    ("f16", 960, 7, 7, 160, 1, 1, True, 1, 70, "<_Float16, false, true, 1>"),
    ("f16", 96, 14, 14, 512, 1, 1, False, 1, 8, "<_Float16, false, false, 1>"),
    ("f16", 40, 13, 11, 68, 1, 1, False, 3, 100, "<_Float16, false, false, 1>"),
    # whole-image layers: one to four planes, odd counts, stride 2
    ("f16", 64, 7, 7, 64, 3, 1, True, 3, 180, "<_Float16, true, true, 1>"),
    ("f16", 192, 7, 7, 128, 3, 1, False, 2, 90, "<_Float16, true, true, 1>"),
    ("f16", 256, 14, 14, 64, 3, 1, True, 1, 50, "<_Float16, true, true, 1>"),
    ("f16", 128, 14, 14, 64, 3, 2, False, 3, 190, "<_Float16, true, true, 1>"),
    # fp32
    ("f32", 128, 28, 28, 128, 3, 1, True, 1, 8, "<float, false, true, 1>"),
    ("f32", 20, 9, 37, 100, 3, 2, False, 2, 70, "<float, false, false, 1>"),
    # k ranges added in range order (with a workspace)
    ("f32", 512, 8, 8, 64, 3, 1, True, 3, 160, "<float, false, true, 4>"),
    ("f32", 516, 7, 7, 64, 3, 1, False, 2, 200, "<float, false, false, 4>"),
    ("f16", 512, 8, 8, 64, 3, 1, False, 2, 160, "<_Float16, false, true, 4>"),
]


@pytest.mark.parametrize("case", CASES)
def test_small_batches_give_the_bits_of_large_ones(case):
    import paper_2609_16742_amd as P
    ctc = P.ctc
    dtype, C, H, W, K, k, st, res, small, large, form = case
    print("small grid", case, flush=True)
    tdt = torch.float16 if dtype == "f16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(CASES.index(case))
    pad = k // 2
    p, q = ((d + 2 * pad - k) // st + 1 for d in (H, W))
    d = ctc.layer_desc(C, K, k, k, st, pad, 1, 1, ctc.CTC_ROLE_SUM)
    dt = ctc.DTYPES[dtype]

    def rnd(*shape):
        return torch.randn(shape, device="cuda", generator=g)

    x, w = rnd(large, H, W, C).to(tdt), (rnd(K, k, k, C) * 0.1).to(tdt)
    scale, shift = rnd(K), rnd(K)
    r = rnd(large, p, q, K).to(tdt) if res else None

    def run(n):
        nb = ctc.ctc_conv2d_workspace_bytes(d, dt, n, H, W)
        ws = torch.empty(max(nb, 1), dtype=torch.uint8, device="cuda")
        y = torch.full((n, p, q, K), float("nan"), dtype=tdt, device="cuda")
        ctc.ctc_conv2d_forward(d, dt, n, H, W, x[:n], w, scale, shift,
                               None if r is None else r[:n], 1, y,
                               workspace=ws if nb else None, ws_bytes=nb)
        return y, nb

    name = ctc.ctc_conv2d_kernel_name(d, dt, small, H, W)
    assert name == "conv_lat" + form.replace(" 4>", " 1>")
    assert not ctc.ctc_conv2d_kernel_name(d, dt, large, H,
                                          W).startswith("conv_lat")
    (ys, nb), (yl, _) = run(small), run(large)
    assert (nb > 0) == form.endswith("4>")
    torch.cuda.synchronize()
    bits = np.uint16 if dtype == "f16" else np.uint32
    a, b = (t.cpu().numpy().view(bits) for t in (ys, yl[:small]))
    assert np.array_equal(a, b)
    # and the values are the convolution's
    ref = torch.nn.functional.conv2d(
        x[:small].cpu().double().permute(0, 3, 1, 2),
        w.cpu().double().permute(0, 3, 1, 2), stride=st, padding=pad)
    ref = (ref * scale.cpu().double()[:, None, None]
           + shift.cpu().double()[:, None, None])
    if res:
        ref += r[:small].cpu().double().permute(0, 3, 1, 2)
    err = (ys.cpu().double().permute(0, 3, 1, 2) - ref.relu()).norm()
    # one rounding to 11 bits, or sums of K <= 4644 products in fp32
    assert err <= (2.0 ** -11 if dtype == "f16" else 1e-5) * ref.norm()


@pytest.mark.parametrize("dtype,protect,last", [("f32", "replace", 20), ("f16", "append", 4)])
def test_layers_split_over_k_leave_conv_lat_past_their_line(dtype, protect, last):
    """ResNet-18's 7x7 layers split k over four waves of conv_lat up to 2048
    tiles (fp32, whole steps of channels) or 512 (appended channels)."""
    import paper_2609_16742_amd as P
    from workloads import gen, nets
    net = nets.by_name("resnet18", dtype=dtype)
    print("split", dtype, protect, flush=True)
    cn = P.CtcNet(net.layers, net.in_shape, net.classes, dtype, gen.make_params(net),
                  protect=protect, max_batch=64)
    ops = [i for i, L in enumerate(net.layers)
           if L["op"] == "conv" and L["c_in"] == 512 and L["k"] == 3]
    for n in (1, last, last + 1, 64):
        names = {P.ctc.ctc_net_op_kernel(cn.h, i, n) for i in ops}
        assert len(names) == 1, names
        assert names.pop().startswith("conv_lat" if n <= last else "conv_dma"), n


# dtype, C, H, W, K, kernel, stride, residual, images, tile; ragged last pixel
# tiles, one or several channel tiles, 1 (fewer than the stages) to 36 steps
PP, PPR = "conv_pp<%d, %d, 0, false>", "conv_ppr<_Float16, %d, %d>"
TILES = [
    ("f16", 64, 25, 27, 128, 3, 1, True, 6, "conv_pp<128, 32, 0, false>"),
    ("f16", 64, 27, 25, 128, 1, 2, False, 40, "conv_pp<128, 32, 0, false>"),
    ("f16", 128, 27, 25, 256, 3, 2, True, 40, "conv_pp<128, 64, 0, false>"),
    ("f16", 256, 15, 17, 384, 1, 2, True, 90, "conv_pp<128, 64, 0, false>"),
    ("f16", 128, 29, 31, 128, 3, 1, True, 45, "conv_pp<128, 96, 0, false>"),
    ("f16", 192, 19, 21, 512, 3, 1, False, 33, "conv_pp<128, 128, 0, false>"),
    ("f16", 64, 39, 41, 128, 1, 2, True, 140, "conv_pp<128, 128, 0, false>"),
    ("f16", 64, 25, 27, 64, 3, 1, False, 13, "conv_pp<64, 32, 0, false>"),
    ("f16", 128, 25, 27, 192, 3, 1, True, 7, "conv_pp<64, 64, 0, false>"),
    ("f16", 64, 27, 25, 64, 5, 2, True, 250, "conv_pp<64, 96, 0, false>"),
    ("f16", 128, 41, 35, 256, 3, 2, True, 120, "conv_pp<256, 224, 0, false>"),
    ("f16", 256, 29, 27, 256, 3, 1, True, 57, "conv_pp<256, 224, 0, false>"),
    ("f16", 192, 13, 13, 384, 1, 1, True, 110, PP % (128, 128)),
    ("f16", 320, 13, 13, 384, 1, 1, False, 80, PP % (128, 96)),
    ("f16", 576, 13, 13, 128, 1, 1, True, 70, PP % (128, 64)),
    ("f16", 192, 13, 13, 256, 1, 1, False, 13, PP % (128, 32)),
    ("f16", 320, 13, 13, 192, 1, 1, True, 80, PP % (64, 96)),
    ("f16", 384, 13, 13, 64, 1, 1, False, 70, PP % (64, 64)),
    ("f16", 192, 13, 13, 64, 1, 1, True, 40, PP % (64, 32)),
    # channels that end within a step, channel tiles that end within a tile
    ("f16", 72, 25, 27, 136, 3, 1, True, 5, "conv_ppr<_Float16, 64, 32>"),
    ("f16", 104, 25, 27, 40, 3, 2, False, 60, "conv_ppr<_Float16, 64, 64>"),
    ("f16", 72, 31, 29, 40, 3, 1, True, 50, "conv_ppr<_Float16, 64, 96>"),
    ("f16", 72, 27, 25, 120, 3, 1, False, 5, "conv_ppr<_Float16, 128, 32>"),
    ("f16", 136, 27, 25, 232, 3, 1, True, 10, "conv_ppr<_Float16, 128, 64>"),
    ("f16", 72, 57, 53, 136, 3, 1, True, 9, "conv_ppr<_Float16, 128, 128>"),
    ("f16", 128, 27, 25, 192, 3, 1, False, 40, "conv_ppr<_Float16, 128, 128>"),
    ("f16", 64, 27, 25, 168, 5, 2, True, 18, "conv_ppr<_Float16, 64, 32>"),
    ("f16", 200, 13, 13, 232, 1, 1, True, 13, PPR % (128, 32)),
    ("f16", 264, 13, 13, 96, 1, 1, False, 70, PPR % (128, 64)),
    ("f16", 192, 13, 13, 232, 1, 1, True, 160, PPR % (128, 128)),
    # little more than one 128 x 128 tile per CU; an odd number of 64 channels
    ("f16", 136, 27, 25, 248, 3, 1, True, 25, PPR % (128, 128)),
    ("f16", 128, 27, 25, 256, 3, 1, False, 25, "conv_pp<128, 96, 0, false>"),
    ("f16", 72, 27, 25, 312, 3, 1, True, 23, PPR % (128, 128)),
    ("f16", 328, 13, 13, 136, 1, 1, True, 12, PPR % (64, 32)),
    ("f16", 576, 13, 13, 160, 1, 1, False, 25, PPR % (64, 64)),
    ("f16", 168, 13, 13, 160, 1, 1, True, 80, PPR % (64, 96)),
    ("f32", 36, 27, 25, 100, 3, 1, True, 9, "conv_ppr<float, 64, 32>"),
    ("f32", 44, 27, 25, 132, 3, 2, False, 60, "conv_ppr<float, 64, 32>"),
    ("f32", 36, 49, 51, 36, 3, 1, True, 40, "conv_ppr<float, 64, 64>"),
    ("f32", 96, 27, 25, 64, 3, 1, True, 13, "conv_pp32<64, 32>"),
    ("f32", 96, 27, 25, 128, 1, 2, False, 90, "conv_pp32<64, 32>"),
    ("f32", 128, 13, 15, 192, 3, 1, False, 20, "conv_pp32<64, 32>"),
    ("f32", 64, 49, 51, 64, 3, 1, True, 53, "conv_pp32<64, 64>"),
    ("f32", 32, 49, 51, 64, 1, 1, False, 54, "conv_pp32<64, 64>"),
]


@pytest.mark.parametrize("case", TILES)
def test_tiles_of_every_size_give_the_bits_of_one_image(case):
    import paper_2609_16742_amd as P
    ctc = P.ctc
    dtype, C, H, W, K, k, st, res, n, name = case
    print("tiles", case, flush=True)
    tdt = torch.float16 if dtype == "f16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(TILES.index(case))
    pad = k // 2
    p, q = ((d + 2 * pad - k) // st + 1 for d in (H, W))
    d = ctc.layer_desc(C, K, k, k, st, pad, 1, 1, ctc.CTC_ROLE_SUM)
    dt = ctc.DTYPES[dtype]

    def rnd(*shape):
        return torch.randn(shape, device="cuda", generator=g)

    x = rnd(n, H, W, C).to(tdt)
    w = (rnd(K, k, k, C) / (k * k * C) ** 0.5).to(tdt)
    scale, shift = rnd(K), rnd(K)
    r = rnd(n, p, q, K).to(tdt) if res else None
    y = torch.full((n, p, q, K), float("nan"), device="cuda").to(tdt)
    assert ctc.ctc_conv2d_kernel_name(d, dt, n, H, W) == name
    ctc.ctc_conv2d_forward(d, dt, n, H, W, x, w, scale, shift, r, 1, y)
    # the first, the last and a middle image alone
    for i in (0, n // 2, n - 1):
        one = torch.full((1, p, q, K), float("nan"), device="cuda").to(tdt)
        ctc.ctc_conv2d_forward(d, dt, 1, H, W, x[i:i + 1], w, scale, shift,
                               None if r is None else r[i:i + 1], 1, one)
        bits = torch.int16 if dtype == "f16" else torch.int32
        assert torch.equal(y[i:i + 1].view(bits), one.view(bits)), i
    ref = torch.nn.functional.conv2d(
        x.cpu().double().permute(0, 3, 1, 2), w.cpu().double().permute(0, 3, 1, 2),
        stride=st, padding=pad)
    ref = (ref * scale.cpu().double()[:, None, None]
           + shift.cpu().double()[:, None, None])
    if res:
        ref += r.cpu().double().permute(0, 3, 1, 2)
    ref = ref.relu()
    err = (y.cpu().double().permute(0, 3, 1, 2) - ref).flatten(1).norm(dim=1)
    # every image: one rounding to 11 bits, or sums of K <= 2304 in fp32
    assert bool((err <= (2.0 ** -11 if dtype == "f16" else 1e-5)
                 * ref.flatten(1).norm(dim=1)).all())


# maps taller or wider than the 16-bit coordinates of conv_pp's tiles, and the
# largest that fit (size + pad = 32768)
@pytest.mark.parametrize("dtype,H,W,K,pp", [
    ("f16", 33001, 2, 64, False), ("f16", 2, 33001, 256, False), ("f32", 2, 16500, 64, True),
    ("f32", 33001, 2, 64, False), ("f16", 2, 32767, 512, True), ("f16", 32767, 4, 512, True),
    ("f16", 4, 32768, 512, False), ("f32", 2, 32767, 64, True), ("f32", 2, 32768, 64, False)])
def test_long_maps_keep_their_kernel(dtype, H, W, K, pp):
    import paper_2609_16742_amd as P
    ctc = P.ctc
    print("long map", dtype, H, W, K, flush=True)
    d = ctc.layer_desc(64, K, 3, 3, 1, 1, 1, 1, ctc.CTC_ROLE_SUM)
    dt = ctc.DTYPES[dtype]
    assert ("conv_pp" in ctc.ctc_conv2d_kernel_name(d, dt, 1, H, W)) == pp
    tdt = torch.float16 if dtype == "f16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    x = torch.randn((1, H, W, 64), device="cuda", generator=g).to(tdt)
    w = (torch.randn((K, 3, 3, 64), device="cuda", generator=g) / 24).to(tdt)
    one, zero = torch.ones(K, device="cuda"), torch.zeros(K, device="cuda")
    y = torch.full((1, H, W, K), float("nan"), device="cuda").to(tdt)
    ctc.ctc_conv2d_forward(d, dt, 1, H, W, x, w, one, zero, None, 0, y)
    # the far end of the map
    hs, ws = slice(-20 if H > 20 else 0, None), slice(-20 if W > 20 else 0, None)
    ref = torch.nn.functional.conv2d(
        x[:, hs, ws].cpu().double().permute(0, 3, 1, 2),
        w.cpu().double().permute(0, 3, 1, 2), padding=1).permute(0, 2, 3, 1)
    ref, got = (ref[:, 1:], y[:, -19:]) if H > 20 else (ref[:, :, 1:], y[:, :, -19:])
    err = (got.cpu().double() - ref).norm()
    assert err <= (2.0 ** -11 if dtype == "f16" else 1e-5) * ref.norm()


# pooled layers of 256-channel tiles on maps up to and past conv_pp's coordinates
@pytest.mark.parametrize("H,W,pp", [(14, 16400, True), (14, 32767, True), (14, 32768, False),
                                    (33600, 8, False)])
def test_long_maps_keep_their_fused_pool(H, W, pp):
    import paper_2609_16742_amd as P
    ctc = P.ctc
    print("long map, pooled", H, W, flush=True)
    d = ctc.layer_desc(64, 256, 3, 3, 1, 1, 1, 1, ctc.CTC_ROLE_SUM)
    assert ("conv_pp" in ctc.ctc_conv2d_kernel_name(d, ctc.CTC_F16, 1, H, W, 2)) == pp
    g = torch.Generator(device="cuda")
    g.manual_seed(W)
    x = torch.randn((1, H, W, 64), device="cuda", generator=g).half()
    w = (torch.randn((256, 3, 3, 64), device="cuda", generator=g) / 24).half()
    scale, shift = (torch.rand(256, device="cuda", generator=g) for _ in range(2))
    y = torch.full((1, H, W, 256), float("nan"), device="cuda").half()
    yp = torch.full((1, H // 2, W // 2, 256), float("nan"), device="cuda").half()
    for pool, out in ((0, y), (2, yp)):
        ctc.ctc_conv2d_forward(d, ctc.CTC_F16, 1, H, W, x, w, scale, shift, None, 1, out,
                               pool=pool)
    win = y[:, :H // 2 * 2, :W // 2 * 2].unflatten(1, (-1, 2)).unflatten(3, (-1, 2))
    assert bool((win.amax(dim=(2, 4)) == yp).all())


# n, H, W, C, K: conv and 2x2 pool in one kernel; odd maps, strips of 16
# pixels that end in the map's middle, parts of strips per wave, even rows
# only, one and several 64-channel blocks
POOLED = [
    (9, 60, 60, 64, 64), (28, 47, 47, 64, 64), (5, 131, 45, 64, 64), (1, 182, 257, 64, 64),
    (9, 60, 60, 64, 40), (9, 60, 60, 64, 36), (9, 60, 60, 64, 24), (8, 64, 96, 128, 128), (30, 38, 47, 192, 128),
    (15, 39, 93, 96, 128), (30, 28, 56, 128, 256), (40, 42, 30, 128, 256),
    (4, 96, 112, 32, 64), (8, 64, 96, 72, 128),
]


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("case", POOLED)
def test_fused_pool_gives_the_bits_of_the_pooled_convolution(case, residual):
    import paper_2609_16742_amd as P
    ctc = P.ctc
    n, H, W, C, K = case
    print("pooled", case, "residual", residual, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(POOLED.index(case))
    d = ctc.layer_desc(C, K, 3, 3, 1, 1, 1, 1, ctc.CTC_ROLE_SUM)
    x = torch.randn((n, H, W, C), device="cuda", generator=g).half()
    w = (torch.randn((K, 3, 3, C), device="cuda", generator=g) / (9 * C) ** 0.5).half()
    scale = torch.rand(K, device="cuda", generator=g) + 0.5
    shift = torch.randn(K, device="cuda", generator=g)
    x[0, H // 2, W // 2, 3] = float("inf")
    r = torch.randn((n, H, W, K), device="cuda", generator=g).half() if residual else None
    for relu in (0, 1):
        y = torch.full((n, H, W, K), float("nan"), device="cuda").half()
        yp = torch.full((n, H // 2, W // 2, K), 7.0, device="cuda").half()
        ctc.ctc_conv2d_forward(d, ctc.CTC_F16, n, H, W, x, w, scale, shift, r, relu, y)
        ctc.ctc_conv2d_forward(d, ctc.CTC_F16, n, H, W, x, w, scale, shift, r, relu, yp,
                               pool=2)
        win = y[:, :H // 2 * 2, :W // 2 * 2].unflatten(1, (-1, 2)).unflatten(3, (-1, 2))
        ref = win.float().amax(dim=(2, 4)).half()      # amax keeps a NaN
        assert torch.equal(torch.isnan(ref), torch.isnan(yp))
        ok = ~torch.isnan(ref)
        assert torch.equal(ref[ok], yp[ok])


@pytest.mark.parametrize("C,H,W", [(64, 60, 60), (64, 45, 77), (128, 64, 96), (256, 56, 28)])
def test_residual_conv_with_a_fused_pool_in_a_network(C, H, W):
    """A residual block whose output only feeds a 2x2 pool: the pool runs in
    the kernel of the block's second conv, with the bits of the separate
    kernels."""
    import paper_2609_16742_amd as P
    import oracle
    from test_gpu_parity import _check_outputs, _net, _oracle_rows
    from workloads import gen
    from workloads.nets import Net, _B, _basic_block
    print("residual + pool", C, H, W, flush=True)
    b = _B()
    t = b.conv(0, 3, C, 3, 1, 1)
    t = _basic_block(b, t, C, C, 1)
    pool = b.maxpool(t, 2, 2, 0)
    b.fc(b.gap(pool), C, 10, final=True)
    n = 30 if C == 256 else 9
    net = Net("respool%d" % C, (3, H, W), b.layers, 10, "f16", n)
    params = gen.make_params(net, seed=C)
    cn = _net(P, net, params, max_batch=n)
    names = [P.ctc.ctc_net_op_kernel(cn.h, i, n) for i in (pool - 2, pool - 1)]
    assert names[0] == names[1], names              # the conv and its pool
    x = torch.from_numpy(gen.make_inputs(net, n, seed=C)).cuda()
    on = cn.forward(x).cpu().numpy()
    pooled = cn.tensor(pool, n).cpu().numpy().copy()
    cn.set_fusion(P.ctc.CTC_FUSE_BLOCK | P.ctc.CTC_FUSE_STEM)
    off = cn.forward(x).cpu().numpy()
    apart = cn.tensor(pool, n).cpu().numpy()
    same = bool((pooled.view(np.uint16) == apart.view(np.uint16)).all())
    assert same and np.array_equal(on.view(np.uint32), off.view(np.uint32))
    rows = [0, n - 1]
    _check_outputs(on[rows], _oracle_rows(net, oracle.protect_params(net, params),
                                          x.cpu().numpy(), rows), net.dtype)


# n, H, W, K, residual: layers of 64 input channels with filters in registers
ROWS = [
    (16, 60, 60, 64, True), (9, 60, 60, 128, False), (34, 33, 61, 64, False),
    (5, 150, 97, 64, True), (1, 181, 257, 128, True), (200, 18, 16, 64, True),
    (10, 57, 94, 192, False), (5, 57, 45, 256, True), (19, 57, 45, 40, True),
    (27, 57, 45, 12, True), (19, 45, 77, 32, False),
    (20, 60, 44, 96, False), (8, 60, 60, 100, True), (30, 33, 61, 68, True),
]


@pytest.mark.parametrize("case", ROWS)
def test_filters_in_registers_give_the_bits_of_one_image(case):
    import paper_2609_16742_amd as P
    ctc = P.ctc
    n, H, W, K, res = case
    print("rows", case, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(H)
    d = ctc.layer_desc(64, K, 3, 3, 1, 1, 1, 1, ctc.CTC_ROLE_SUM)
    assert ctc.ctc_conv2d_kernel_name(d, ctc.CTC_F16, n, H, W) == (
        "conv_rows<false, %s, false>" % ("false" if K % 8 else "true"))
    x = torch.randn((n, H, W, 64), device="cuda", generator=g).half()
    w = (torch.randn((K, 3, 3, 64), device="cuda", generator=g) / 24).half()
    scale = torch.rand(K, device="cuda", generator=g) + 0.5
    shift = torch.randn(K, device="cuda", generator=g)
    r = torch.randn((n, H, W, K), device="cuda", generator=g).half() if res else None
    y = torch.full((n, H, W, K), float("nan"), device="cuda").half()
    ctc.ctc_conv2d_forward(d, ctc.CTC_F16, n, H, W, x, w, scale, shift, r, 1, y)
    if n > 1:
        # single images and bands of rows run on kernels with smaller tiles
        for i in (0, n // 2, n - 1):
            one = torch.full((1, H, W, K), float("nan"), device="cuda").half()
            ctc.ctc_conv2d_forward(d, ctc.CTC_F16, 1, H, W, x[i:i + 1], w, scale, shift,
                                   None if r is None else r[i:i + 1], 1, one)
            assert torch.equal(y[i:i + 1].view(torch.int16), one.view(torch.int16)), i
    ref = torch.nn.functional.conv2d(x.cpu().float().permute(0, 3, 1, 2),
                                     w.cpu().float().permute(0, 3, 1, 2), padding=1)
    ref = (ref * scale.cpu()[:, None, None] + shift.cpu()[:, None, None]).permute(0, 2, 3, 1)
    if res:
        ref = ref + r.cpu().float()
    ref = ref.relu()
    err = (y.cpu().float() - ref).flatten(2).norm(dim=2)
    # every row of every image: one rounding to 11 bits
    assert bool((err <= 2.0 ** -11 * ref.flatten(2).norm(dim=2)).all())


@pytest.mark.parametrize("hw", [1, 3, 8, 9, 12])
def test_global_pool_over_part_and_whole_batches_of_pixels(hw):
    """Global average pools of maps that end within, at and past the sixteen
    pixels that a lane loads together."""
    import paper_2609_16742_amd as P
    import oracle
    from test_gpu_parity import _check_outputs, _net, _oracle_rows
    from workloads import gen
    from workloads.nets import Net, _B
    print("gap", hw, flush=True)
    b = _B()
    t = b.conv(0, 3, 32, 3, 2, 1)
    t = b.conv(t, 32, 584, 1, 1, 0)
    t = b.gap(t)
    b.fc(t, 584, 10, final=True)
    net = Net("gap%d" % hw, (3, 2 * hw, 2 * hw), b.layers, 10, "f16", 3)
    params = gen.make_params(net, seed=hw)
    cn = _net(P, net, params, max_batch=3)
    assert P.ctc.ctc_net_op_kernel(cn.h, 2, 3).startswith("gap_k")
    xh = gen.make_inputs(net, 3, seed=hw)
    y = cn.forward(torch.from_numpy(xh).cuda()).cpu().numpy()
    _check_outputs(y, _oracle_rows(net, oracle.protect_params(net, params), xh,
                                   [0, 1, 2]), net.dtype)
