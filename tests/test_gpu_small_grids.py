"""Convolutions of a few images (conv_lat) against the tile kernels that run
the same layer at larger batches: same bits, row by row."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# dtype, C, H, W, K, k, stride, residual, images small / large, conv_lat form
CASES = [
    # whole 64-channel steps: one tap per step, several steps per tap
    ("f16", 64, 56, 56, 64, 3, 1, True, 2, 8, "<_Float16, false, true, 1>"),
    ("f16", 128, 29, 27, 72, 3, 2, False, 1, 33, "<_Float16, false, true, 1>"),
    # chunks of one step in different taps (72 and 8 channels), k tails,
    # 4 of 16 channels in the last tile, pixel tails
    ("f16", 72, 13, 11, 132, 3, 1, True, 3, 33, "<_Float16, false, false, 1>"),
    ("f16", 8, 17, 9, 260, 3, 2, False, 2, 64, "<_Float16, false, false, 1>"),
    # pointwise layers, conv_pw's among them
    ("f16", 960, 7, 7, 160, 1, 1, True, 1, 70, "<_Float16, false, true, 1>"),
    ("f16", 96, 14, 14, 576, 1, 1, False, 1, 8, "<_Float16, false, false, 1>"),
    ("f16", 24, 13, 11, 36, 1, 1, False, 3, 100, "<_Float16, false, false, 1>"),
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


# C, H, W, K, stride, residual, images large (conv_pp) / small (conv_dma)
WIDE = [
    # one 128-channel tile, ragged last pixel tile; two tiles; 9, 18, 27 steps
    (64, 41, 35, 128, 2, True, 120, 90),
    (128, 27, 29, 128, 1, True, 55, 12),
    (192, 27, 29, 384, 1, False, 20, 8),
    (256, 29, 27, 256, 1, True, 56, 10),
]


@pytest.mark.parametrize("case", WIDE)
def test_wide_tiles_give_the_bits_of_small_ones(case):
    import paper_2609_16742_amd as P
    ctc = P.ctc
    C, H, W, K, st, res, large, small = case
    print("wide tiles", case, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(C + K)
    p, q = ((d - 1) // st + 1 for d in (H, W))
    d = ctc.layer_desc(C, K, 3, 3, st, 1, 1, 1, ctc.CTC_ROLE_SUM)

    def rnd(*shape):
        return torch.randn(shape, device="cuda", generator=g)

    x, w = rnd(large, H, W, C).half(), (rnd(K, 3, 3, C) * 0.05).half()
    scale, shift = rnd(K), rnd(K)
    r = rnd(large, p, q, K).half() if res else None
    x[1, H // 2, W // 2, 5] = float("inf")       # stays in its 3x3 windows

    def run(n):
        y = torch.full((n, p, q, K), float("nan"), device="cuda").half()
        ctc.ctc_conv2d_forward(d, ctc.CTC_F16, n, H, W, x[:n], w, scale, shift,
                               None if r is None else r[:n], 1, y)
        return y

    bn = 256 if K % 256 == 0 else 128
    names = [ctc.ctc_conv2d_kernel_name(d, ctc.CTC_F16, n, H, W)
             for n in (large, small)]
    assert names[0] == "conv_pp<%d, 224, 0, false>" % bn
    assert names[1].startswith("conv_dma<")
    yl, ys = run(large), run(small)
    torch.cuda.synchronize()
    a, b = (t.cpu().numpy().view(np.uint16) for t in (yl[:small], ys))
    nan = np.isnan(a.view(np.float16)) & np.isnan(b.view(np.float16))
    assert np.array_equal(a[~nan], b[~nan]) and nan.sum() < 9 * K + 1
    # every row past the small batch is written, and the inf stayed put
    assert bool(torch.isfinite(yl[small:]).all())
