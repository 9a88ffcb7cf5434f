"""GPU parity: convolution forward / data gradient / weight gradient against the oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
import synth
from gpu_util import TOL, assert_close, dev, host, inputs

pytestmark = pytest.mark.gpu
SEED = synth.DEFAULT_SEED


@pytest.fixture(scope="module")
def rn():
    import paper_1903_12650_amd as rn
    return rn


def check_sums(rn, y, handle, grad_of=None):
    """The batch-norm sums that a convolution leaves beside its output, against 64 bits of the stored values.  A channel's sums are
    float sums of at most 256 values per tile (at most 48 additions behind each other), added up in double: each within
    48 * 2^-24 < 1e-5 of the sum of its terms' sizes.  Forward: mean and variance (about a value of the channel itself, whose
    distance from the mean adds to the terms).  Gradients (grad_of: the BN layer's input, scale 1, shift 0, mean 0, 1/std 1):
    dbeta and dgamma under the layer's ReLU."""
    C = y.shape[-1]
    one, zero = torch.ones(C, device="cuda"), torch.zeros(C, device="cuda")
    y64 = y.double().reshape(-1, C)
    if grad_of is None:
        _, mean, rstd = rn.bn_relu_fwd_from_sums(y, handle, one, zero, None, 1e-5, 1)
        m64, var = y64.mean(0), y64.var(0, unbiased=False)
        spread = 2 * (var.sqrt() + (y64 - m64).abs().amax(0))
        assert bool(((mean.double() - m64).abs() <= 1e-5 * spread + 2.0 ** -23 * m64.abs()).all()), "mean"
        off = (rstd.double() ** -2 - 1e-5 - var).abs()
        assert bool((off <= 1e-5 * spread ** 2 + 2.0 ** -21 * (var + 1e-5)).all()), "variance"
        return
    x64 = grad_of.double().reshape(-1, C)
    _, _, dgamma, dbeta = rn.bn_relu_bwd_from_sums(y, grad_of, handle, one, zero, zero, one)
    g = torch.where(x64 > 0, y64, torch.zeros_like(y64))
    assert bool(((dbeta.double() - g.sum(0)).abs() <= 1e-5 * g.abs().sum(0) + 1e-30).all()), "dbeta"
    assert bool(((dgamma.double() - (g * x64).sum(0)).abs() <= 1e-5 * (g * x64).abs().sum(0) + 1e-30).all()), "dgamma"


def run_case(rn, mode_name, N, H, W, C, K, R, stride, pad, do_dgrad=True, tag=""):
    bf = mode_name == "bf16"
    tol = TOL[mode_name]
    x = synth.activation_nhwc(SEED, "x" + tag, N, C, H, W)
    w = synth.conv_weight_krsc(SEED, "w" + tag, K, C, R, R)
    x, w = inputs(mode_name, x, w)
    y_o = orc.conv_fwd(x, w, stride, pad)
    dy = synth.activation_nhwc(SEED, "dy" + tag, N, K, y_o.shape[1], y_o.shape[2])
    dy, = inputs(mode_name, dy)
    xd, wd, dyd = dev(x, bf), dev(w, bf), dev(dy, bf)
    errs = {}
    y = rn.conv_fwd(xd, wd, stride, pad)
    errs["y"] = assert_close(y, y_o, tol, f"y {tag}")
    dw = rn.conv_wgrad(xd, dyd, w.shape, stride, pad)
    assert dw.dtype == torch.float32
    errs["dw"] = assert_close(dw, orc.conv_wgrad(x, dy, w.shape, stride, pad), tol, f"dw {tag}")
    if do_dgrad:
        dx = rn.conv_dgrad(dyd, wd, x.shape, stride, pad)
        errs["dx"] = assert_close(dx, orc.conv_dgrad(dy, w, x.shape, stride, pad), tol, f"dx {tag}")
    return errs


SMALL = [  # N,H,W,C,K,R,stride,pad : ragged tiles, tails, every stride/pad/filter combination
    (2, 9, 7, 8, 8, 1, 1, 0),
    (1, 12, 12, 16, 24, 3, 1, 1),
    (3, 11, 13, 24, 40, 3, 2, 1),
    (2, 10, 10, 72, 136, 1, 2, 0),
    (1, 17, 15, 136, 72, 3, 1, 1),
    (2, 8, 8, 64, 64, 3, 2, 1),
    (1, 5, 5, 8, 200, 3, 1, 0),
    (5, 14, 14, 256, 64, 1, 1, 0),
    (2, 14, 14, 64, 256, 1, 1, 0),
    (1, 20, 20, 8, 8, 7, 2, 3),
    (2, 6, 6, 16, 16, 5, 1, 2),
    (1, 1, 1, 8, 8, 1, 1, 0),
    (2, 9, 7, 16, 16, 1, 2, 0),      # stride 2, odd sizes: the four pixel parity classes differ in size
    (1, 1, 5, 8, 8, 3, 2, 1),        # a single row: two parity classes are empty
    (2, 5, 4, 8, 16, 2, 2, 0),       # even filter, stride 2
    # 3x3 stride 1 pad 1 with whole 128-byte channel chunks, several tiles and images per case
    (3, 9, 9, 64, 64, 3, 1, 1),      # tiles that span two images, short last tile
    (2, 5, 12, 128, 72, 3, 1, 1),    # two channel chunks, ragged column tile
    (5, 7, 21, 192, 64, 3, 1, 1),    # three channel chunks (odd number of pipeline steps)
    (7, 4, 48, 64, 128, 3, 1, 1),    # wide, low images
    (2, 1, 56, 64, 64, 3, 1, 1),     # one-row images: every tap row but the middle one is padding
    (3, 8, 8, 128, 128, 3, 1, 1),    # one 64-pixel tile per image
    (1, 1, 1, 8, 8, 3, 1, 1),        # a single pixel: eight of the nine taps are padding
    (2, 2, 2, 16, 8, 3, 1, 1),       # 2x2 images: every pixel is a corner
    (1, 3, 100, 8, 8, 3, 1, 1),      # too wide for the one-run kernels (run of 2W + 2 rows): the general path
    (2, 3, 62, 8, 16, 3, 1, 1),      # wide, low images of few channels
]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("case", SMALL)
def test_small_shapes(rn, mode_name, case):
    N, H, W, C, K, R, stride, pad = case
    if mode_name == "f32":
        C = max(4, C // 2); K = max(4, K // 2)          # float needs only multiples of 4
    run_case(rn, mode_name, N, H, W, C, K, R, stride, pad, tag=str(case))


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,HW", [(2, 32), (1, 38), (3, 224)])
def test_stem(rn, mode_name, N, HW):
    """3-channel 7x7/2 pad-3 stem (appendix log: [3(4),224,224] -> (64,112,112))."""
    run_case(rn, mode_name, N, HW, HW, 3, 64, 7, 2, 3, do_dgrad=False, tag=f"stem{N}x{HW}")


# The 23 distinct convolution shapes of ResNet-50 v1.5: Cin, Cout, R, stride, Hin
RESNET_SHAPES = [
    (3, 64, 7, 2, 224), (64, 64, 1, 1, 56), (64, 64, 3, 1, 56), (64, 256, 1, 1, 56), (256, 64, 1, 1, 56),
    (256, 128, 1, 1, 56), (128, 128, 3, 2, 56), (128, 512, 1, 1, 28), (256, 512, 1, 2, 56), (512, 128, 1, 1, 28),
    (128, 128, 3, 1, 28), (512, 256, 1, 1, 28), (256, 256, 3, 2, 28), (256, 1024, 1, 1, 14), (512, 1024, 1, 2, 28),
    (1024, 256, 1, 1, 14), (256, 256, 3, 1, 14), (1024, 512, 1, 1, 14), (512, 512, 3, 2, 14), (512, 2048, 1, 1, 7),
    (1024, 2048, 1, 2, 14), (2048, 512, 1, 1, 7), (512, 512, 3, 1, 7),
]


@pytest.mark.parametrize("shape", RESNET_SHAPES)
def test_resnet50_shapes_batch40_bf16(rn, shape):
    """BASELINE config 3: every distinct conv shape at batch 40, bf16, fwd + dgrad + wgrad."""
    C, K, R, stride, H = shape
    errs = run_case(rn, "bf16", 40, H, H, C, K, R, stride, R // 2, do_dgrad=(C != 3), tag=str(shape))
    print(shape, {k: "%.2e" % v for k, v in errs.items()})


@pytest.mark.parametrize("shape", [(64, 64, 3, 1, 56), (256, 512, 1, 2, 56), (512, 512, 3, 2, 14), (3, 64, 7, 2, 224)])
def test_resnet50_shapes_f32(rn, shape):
    C, K, R, stride, H = shape
    run_case(rn, "f32", 4, H, H, C, K, R, stride, R // 2, do_dgrad=(C != 3), tag=str(shape))


def test_conv_reproducible_and_workspace_poison(rn):
    """Same inputs twice -> identical bits, with a NaN-poisoned workspace (nothing unwritten is read)."""
    x = dev(synth.activation_nhwc(SEED, "x", 8, 128, 28, 28), True)
    w = dev(synth.conv_weight_krsc(SEED, "w", 128, 128, 3, 3), True)
    dy = dev(synth.activation_nhwc(SEED, "dy", 8, 128, 14, 14), True)
    d = rn.ConvDesc(8, 28, 28, 128, 128, 3, 3, 2, 1, rn.BF16)
    outs = []
    for _ in range(2):
        ws = torch.full((max(rn.conv_wgrad_workspace_bytes(d), rn.conv_dgrad_workspace_bytes(d), 256) // 4,), float("nan"),
                        device="cuda").view(torch.uint8)
        outs.append((rn.conv_fwd(x, w, 2, 1), rn.conv_dgrad(dy, w, x.shape, 2, 1, workspace=ws.clone()),
                     rn.conv_wgrad(x, dy, w.shape, 2, 1, workspace=ws.clone())))
    for a, b in zip(*outs):
        assert torch.equal(a, b) and torch.isfinite(a.float()).all()


def test_conv_error_codes(rn):
    x = torch.zeros((1, 8, 8, 12), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((8, 3, 3, 12), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(rn.Rn50Error) as e:
        rn.conv_fwd(x, w, 1, 1)                              # Cin = 12 is not a multiple of 8
    assert e.value.code == -2
    x = torch.zeros((1, 8, 8, 16), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((8, 3, 3, 16), dtype=torch.bfloat16, device="cuda")
    dy = torch.zeros((1, 8, 8, 8), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(rn.Rn50Error) as e:
        rn.conv_dgrad(dy, w, x.shape, 1, 1, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    assert e.value.code == -3
    x3 = torch.zeros((1, 16, 16, 3), dtype=torch.bfloat16, device="cuda")
    w3 = torch.zeros((64, 7, 7, 3), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(rn.Rn50Error) as e:
        rn.conv_dgrad(torch.zeros((1, 8, 8, 64), dtype=torch.bfloat16, device="cuda"), w3, x3.shape, 2, 3)
    assert e.value.code == -2


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
def test_3x3_taps_never_reach_into_the_neighbouring_image(rn, mode_name):
    """The 3x3 / stride 1 kernels read one contiguous run of pixels per tile, which spans image borders: with one
    image of the batch all NaN (forward: of x; data gradient: of dy), the other images' outputs are bit for bit
    those of the batch where that image is zero."""
    bf = mode_name == "bf16"
    N, H, W, C, K = 3, 6, 10, (64 if bf else 32), (64 if bf else 32)
    x, w, dy = inputs(mode_name, synth.activation_nhwc(SEED, "x", N, C, H, W), synth.conv_weight_krsc(SEED, "w", K, C, 3, 3),
                      synth.activation_nhwc(SEED, "dy", N, K, H, W))
    wd = dev(w, bf)
    outs = []
    for poison in (0.0, float("nan")):
        xd, dyd = dev(x, bf).clone(), dev(dy, bf).clone()
        xd[1] = poison
        dyd[1] = poison
        outs.append((rn.conv_fwd(xd, wd, 1, 1), rn.conv_dgrad(dyd, wd, xd.shape, 1, 1)))
    for a, b in zip(*outs):
        assert torch.equal(a[0], b[0]) and torch.equal(a[2], b[2])
        assert torch.isnan(b[1]).any()


# The stem's own kernel: one and two output rows per tile, ragged pixel blocks, several tiles per workgroup, fewer than 64
# filters; shapes it leaves to the general kernel.
@pytest.mark.parametrize("N,H,W,K", [(1, 64, 64, 64), (40, 64, 64, 64), (2, 100, 100, 24), (1, 130, 130, 64), (2, 65, 140, 8),
                                     (1, 30, 300, 64), (1, 66, 66, 64), (1, 64, 64, 72), (1, 16, 700, 64)])
def test_stem_tiles(rn, N, H, W, K):
    x = synth.activation_nhwc(SEED, "x", N, 3, H, W)
    w = synth.conv_weight_krsc(SEED, "w", K, 3, 7, 7)
    x, w = inputs("bf16", x, w)
    y, handle = rn.conv_fwd_bn_sums(dev(x, True), dev(w, True), 2, 3)
    assert_close(y, orc.conv_fwd(x, w, 2, 3), TOL["bf16"], "y")
    assert torch.equal(y, rn.conv_fwd(dev(x, True), dev(w, True), 2, 3))
    g, b = torch.ones(K, device="cuda"), torch.zeros(K, device="cuda")
    _, mean, rstd = rn.bn_relu_fwd_from_sums(y, handle, g, b)
    _, mean2, rstd2 = rn.bn_relu_fwd(y, g, b)
    assert_close(mean, host(mean2), 1e-5, "mean")
    assert_close(rstd, host(rstd2), 1e-5, "rstd")


@pytest.mark.parametrize("N,HW,mean", [(4, 224, 5.0), (40, 224, 5.0), (256, 224, 0.0), (256, 224, 5.0)])
def test_stem_sums_against_64_bits(rn, N, HW, mean):
    """The stem's batch statistics over 1 to 28 tiles per workgroup, also where the images' mean is far from zero and the border
    pixels far from the others: within 2^-23 of the 64-bit values of the stored outputs (sums in double; one rounding of a
    workgroup's row, which averages out, and one of the result, 2^-24)."""
    gen = torch.Generator(device="cuda").manual_seed(SEED)
    x = (mean + torch.randn((N, HW, HW, 3), device="cuda", generator=gen)).bfloat16()
    w = dev(inputs("bf16", synth.conv_weight_krsc(SEED, "w", 64, 3, 7, 7))[0], True)
    y, handle = rn.conv_fwd_bn_sums(x, w, 2, 3)
    _, m, r = rn.bn_relu_fwd_from_sums(y, handle, torch.ones(64, device="cuda"), torch.zeros(64, device="cuda"))
    y64 = y.view(-1, 64).double()
    mean_o = y64.mean(0)
    var_o = (y64 - mean_o).square().mean(0)
    rstd_o = (var_o + 1e-5).rsqrt()
    assert float((m.double() - mean_o).abs().div(mean_o.abs() + var_o.sqrt()).max()) <= 2.0 ** -23
    assert float((r.double() / rstd_o - 1).abs().max()) <= 2.0 ** -23


# Where the waves of a workgroup split the reduction (few output tiles, at least four 128-byte chunks): chunk counts that
# are and are not multiples of four, ragged channels, the tile counts at which the tile changes, stride-2 pixel classes,
# the channel count beyond which the linear forward kernel keeps the shared ring.
K_SPLIT = [  # N,H,W,C,K,R,stride,pad (channels in 128-byte chunks of the bf16 type)
    (1, 7, 7, 256, 64, 1, 1, 0),       # four chunks, one ragged row tile
    (1, 5, 5, 320, 72, 1, 1, 0),       # five chunks, ragged columns
    (2, 6, 7, 424, 136, 1, 1, 0),      # seven chunks, the last one ragged
    (1, 32, 32, 256, 512, 1, 1, 0),    # 128 tiles of 64x64
    (1, 32, 33, 256, 512, 1, 1, 0),    # 136
    (2, 32, 32, 256, 512, 1, 1, 0),    # 256
    (2, 32, 33, 256, 512, 1, 1, 0),    # 264: the shared ring
    (1, 9, 8, 8, 16, 3, 1, 1),         # nine chunks of one ragged tap each
    (2, 9, 7, 136, 72, 3, 1, 1),       # taps of three chunks, wave ranges that begin inside a tap
    (3, 9, 11, 72, 40, 3, 2, 1),       # stride 2: classes of one, two and four taps
    (2, 7, 6, 264, 520, 1, 2, 0),      # stride 2 without taps in three of the classes
    (1, 4, 4, 2048, 64, 1, 1, 0),      # the most channels of a linear forward layer
    (1, 4, 4, 2056, 64, 1, 1, 0),      # one vector more
]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("case", K_SPLIT)
def test_k_split_edges(rn, mode_name, case):
    N, H, W, C, K, R, stride, pad = case
    if mode_name == "f32":
        C = C if C > 2000 else max(4, C // 2)          # the same number of 128-byte chunks
    run_case(rn, mode_name, N, H, W, C, K, R, stride, pad, tag="ks" + str(case))


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K", [(1, 1, 1, 8, 8), (1, 2, 1, 8, 8), (1, 1, 2, 8, 8), (2, 16, 16, 64, 64), (3, 17, 9, 136, 72),
                                       (2, 7, 6, 264, 520), (5, 31, 30, 256, 512), (9, 56, 56, 256, 128)])
def test_strided_1x1_data_gradient_stores_every_pixel(rn, mode_name, N, H, W, C, K):
    """Tiles hold the pixels with the tap and store the zeros beside them: rows, columns and tiles at the edges, into a buffer
    of NaNs."""
    dt = torch.bfloat16 if mode_name == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(H * W + C)
    dy = torch.randn(N, (H - 1) // 2 + 1, (W - 1) // 2 + 1, K, device="cuda", generator=gen).to(dt)
    w = (torch.randn(K, 1, 1, C, device="cuda", generator=gen) * 0.1).to(dt)
    dx = torch.full((N, H, W, C), float("nan"), device="cuda", dtype=dt)
    rn.conv_dgrad(dy, w, dx.shape, 2, 0, dx=dx)
    want = torch.zeros(N, H, W, C, device="cuda", dtype=torch.float64)
    want[:, ::2, ::2] = (dy.double().reshape(-1, K) @ w.double().reshape(K, C)).reshape(dy.shape[:3] + (C,))
    assert_close(dx, host(want), TOL[mode_name], "dx")
    assert torch.equal(dx == 0, want == 0)


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K,R,pad", [(1, 1, 1, 8, 8, 3, 1), (2, 5, 4, 24, 40, 3, 1), (3, 57, 55, 72, 64, 3, 1), (2, 96, 97, 264, 64, 3, 1),
                                             (5, 33, 35, 136, 128, 2, 0), (2, 61, 62, 520, 32, 5, 2)])
def test_strided_data_gradient_takes_every_class_of_every_range_once(rn, mode_name, N, H, W, C, K, R, pad):
    """The order of the four parity classes changes along the grid: images of one tile per class to many turns, one to nine column
    tiles; into a buffer of NaNs."""
    dt = torch.bfloat16 if mode_name == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(H * W + C)
    w = (torch.randn(K, R, R, C, generator=gen) / (R * R * K) ** 0.5).to(dt)
    dy = torch.randn(N, (H + 2 * pad - R) // 2 + 1, (W + 2 * pad - R) // 2 + 1, K, generator=gen).to(dt)
    x = torch.zeros(N, C, H, W, dtype=torch.float64, requires_grad=True)
    torch.nn.functional.conv2d(x, w.permute(0, 3, 1, 2).double(), stride=2, padding=pad).backward(dy.permute(0, 3, 1, 2).double())
    dx = torch.full((N, H, W, C), float("nan"), device="cuda", dtype=dt)
    rn.conv_dgrad(dy.cuda(), w.cuda(), dx.shape, 2, pad, dx=dx)
    assert_close(dx, x.grad.permute(0, 2, 3, 1).contiguous().numpy(), TOL[mode_name], "dx")


@pytest.mark.parametrize("N,H,W,C,K,R,stride", [(3, 120, 123, 64, 136, 1, 1), (3, 120, 123, 72, 136, 3, 1), (3, 241, 239, 16, 136, 3, 2),
                                                (1, 200, 210, 8, 264, 1, 1), (2, 56, 57, 256, 840, 1, 1), (7, 224, 220, 3, 64, 7, 2)])
def test_outputs_written_through(rn, N, H, W, C, K, R, stride):
    """bf16 outputs of 10.1 to 22 MB: ragged rows and columns of every store path (plain, halo, strided, the stem), forward with
    and without sums, the data gradient with the same sizes in the other direction; into buffers of NaNs."""
    gen = torch.Generator().manual_seed(H + K)
    pad = R // 2
    x = torch.randn(N, H, W, C, generator=gen).bfloat16()
    w = (torch.randn(K, R, R, C, generator=gen) / (R * R * C) ** 0.5).bfloat16()
    want = torch.nn.functional.conv2d(x.permute(0, 3, 1, 2).double(), w.permute(0, 3, 1, 2).double(), stride=stride, padding=pad)
    want = want.permute(0, 2, 3, 1).contiguous().numpy()
    assert 2 * want.size >= 10 << 20
    y = torch.full(want.shape, float("nan"), device="cuda", dtype=torch.bfloat16)
    rn.conv_fwd(x.cuda(), w.cuda(), stride, pad, y=y)
    assert_close(y, want, TOL["bf16"], "y")
    y2, _ = rn.conv_fwd_bn_sums(x.cuda(), w.cuda(), stride, pad)
    assert torch.equal(y, y2)
    if stride == 1:
        wt = w.flip(1, 2).permute(3, 1, 2, 0).contiguous()  # the same convolution as a data gradient
        dx = torch.full(want.shape, float("nan"), device="cuda", dtype=torch.bfloat16)
        rn.conv_dgrad(x.cuda(), wt.cuda(), want.shape, 1, pad, dx=dx)
        assert_close(dx, want, TOL["bf16"], "dx")


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K", [(3, 128, 130, 16, 72), (2, 191, 129, 40, 136)])
def test_images_too_wide_for_the_halo_loop(rn, mode_name, N, H, W, C, K):
    """3x3 / stride 1 on the eight-wave tile (from 192 of them on) where its run of pixels has no room: the gathering loop, forward with
    and without sums, data gradient with and without."""
    dt = torch.bfloat16 if mode_name == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(W + K)
    rand = lambda *shape, scale=1.0: (torch.randn(*shape, generator=gen) * scale).to(dt)
    nchw = lambda t: t.double().permute(0, 3, 1, 2)
    x, w, dy, wt = rand(N, H, W, C), rand(K, 3, 3, C, scale=(9 * C) ** -0.5), rand(N, H, W, C), rand(C, 3, 3, K, scale=(9 * C) ** -0.5)
    want = torch.nn.functional.conv2d(nchw(x), nchw(w), padding=1).permute(0, 2, 3, 1).contiguous()
    y = rn.conv_fwd(x.cuda(), w.cuda(), 1, 1)
    assert_close(y, want.numpy(), TOL[mode_name], "y")
    y2, sums = rn.conv_fwd_bn_sums(x.cuda(), w.cuda(), 1, 1)
    assert torch.equal(y, y2)
    check_sums(rn, y, sums)
    want = torch.nn.grad.conv2d_input((N, K, H, W), nchw(wt), nchw(dy), padding=1).permute(0, 2, 3, 1).contiguous()
    dx = rn.conv_dgrad(dy.cuda(), wt.cuda(), y.shape, 1, 1)
    assert_close(dx, want.numpy(), TOL[mode_name], "dx")
    one, zero = torch.ones(K, device="cuda"), torch.zeros(K, device="cuda")
    dx2, sums = rn.conv_dgrad_bn_sums(dy.cuda(), wt.cuda(), y.shape, 1, 1, y, one, zero, zero, one)
    assert torch.equal(dx, dx2)
    check_sums(rn, dx, sums, grad_of=y)


# 3x3 / stride 1 layers by the filter row: tiles of 32 rows (at most 128 tiles of 64x64), of 64 rows with the reduction split over the
# waves (to 256) and 2x2 waves (to 512, 513 the tap by tap loop), one to four chunks of channels (ragged ones too), image widths on
# either side of those whose runs of pixels still fit, images narrower than the filter.
HALO_ROWS = [(1, 1, 1, 8, 8), (1, 2, 1, 64, 64), (2, 5, 3, 72, 40), (1, 3, 111, 64, 64), (1, 3, 112, 64, 64), (1, 30, 95, 136, 24), (1, 30, 96, 136, 24),
             (1, 90, 95, 64, 64), (1, 90, 96, 64, 64), (1, 120, 79, 72, 64), (1, 120, 80, 72, 64), (40, 14, 14, 200, 128), (60, 13, 15, 200, 128),
             (60, 13, 16, 136, 128), (6, 57, 56, 64, 64), (3, 83, 79, 64, 64), (3, 83, 80, 64, 64), (81, 14, 14, 72, 128), (84, 14, 14, 72, 128)]
# ... and the tap by tap loop of the tallest tile (256x64, from 384 of them on): whole and ragged, the widest image it takes and one column
# more, images of one column, more channels than a chunk (bf16: 64).
HALO_TALL = [(32, 56, 56, 64, 64), (25, 63, 63, 40, 24), (25, 62, 64, 40, 24), (33, 3000, 1, 16, 64), (1, 1, 98400, 8, 8), (33, 56, 54, 72, 64)]

# ... and of 128x128 tiles, two workgroups per compute unit: the widest image they take and one column more, one chunk, images of one column,
# whole images and tiles, the longest rest that still counts as half a round (768 tiles) and one row of tiles more.
HALO_PAIRS = [(1, 265, 31, 72, 1000), (1, 257, 32, 72, 1000), (1, 265, 31, 8, 1000), (1, 8200, 1, 64, 1016), (42, 14, 14, 136, 1024),
              (48, 16, 16, 64, 1024), (1, 12300, 1, 8, 1024)]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K", HALO_ROWS + HALO_TALL + HALO_PAIRS)
def test_3x3_by_filter_rows(rn, mode_name, N, H, W, C, K):
    """Forward with and without sums, data gradient with and without, into buffers of NaNs, against 64 bits."""
    dt = torch.bfloat16 if mode_name == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(N + W + C)
    rand = lambda *shape, scale=1.0: (torch.randn(*shape, generator=gen) * scale).to(dt)
    nchw = lambda t: t.double().permute(0, 3, 1, 2)
    x, w, dy, wt = rand(N, H, W, C), rand(K, 3, 3, C, scale=(9 * C) ** -0.5), rand(N, H, W, C), rand(C, 3, 3, K, scale=(9 * C) ** -0.5)
    want = torch.nn.functional.conv2d(nchw(x), nchw(w), padding=1).permute(0, 2, 3, 1).contiguous()
    y = torch.full(want.shape, float("nan"), device="cuda", dtype=dt)
    rn.conv_fwd(x.cuda(), w.cuda(), 1, 1, y=y)
    assert_close(y, want.numpy(), TOL[mode_name], "y")
    y2, sums = rn.conv_fwd_bn_sums(x.cuda(), w.cuda(), 1, 1)
    assert torch.equal(y, y2)
    check_sums(rn, y, sums)
    want = torch.nn.grad.conv2d_input((N, K, H, W), nchw(wt), nchw(dy), padding=1).permute(0, 2, 3, 1).contiguous()
    dx = torch.full(want.shape, float("nan"), device="cuda", dtype=dt)
    rn.conv_dgrad(dy.cuda(), wt.cuda(), y.shape, 1, 1, dx=dx)
    assert_close(dx, want.numpy(), TOL[mode_name], "dx")
    one, zero = torch.ones(K, device="cuda"), torch.zeros(K, device="cuda")
    dx2, sums = rn.conv_dgrad_bn_sums(dy.cuda(), wt.cuda(), y.shape, 1, 1, y, one, zero, zero, one)
    assert torch.equal(dx, dx2)
    check_sums(rn, dx, sums, grad_of=y)


# Output pixel grids whose tensor is one column below, exactly and one column above the 1 MB from which convolutions write their
# outputs through: columns, filter, stride, channels on the other side (64x64 tiles; the two K splits; the halo loop; the
# strided gather and data gradient; 1x1 / stride 2 with its zeros; the stem).
WRITE_LINE = [(64, 1, 1, 64), (64, 1, 1, 264), (64, 3, 1, 64), (8, 3, 1, 16), (72, 3, 2, 24), (64, 1, 2, 128), (64, 7, 2, 3)]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("K,R,stride,C", WRITE_LINE)
@pytest.mark.parametrize("beside", [-1, 0, 1])
def test_outputs_on_either_side_of_the_write_through_line(rn, mode_name, K, R, stride, C, beside):
    dt = torch.bfloat16 if mode_name == "bf16" else torch.float32
    es, pad = 2 if mode_name == "bf16" else 4, R // 2
    P = (1 << 20) // (es * K * 32)  # (narrow: the halo loop's run fits)
    Q = -(-(1 << 20) // (es * K * P)) + beside
    size = es * K * P * Q
    assert (size < 1 << 20) == (beside < 0) and (beside or K == 72 or size == 1 << 20)
    gen = torch.Generator().manual_seed(K + R + C)
    rand = lambda *shape, scale=1.0: (torch.randn(*shape, generator=gen) * scale).to(dt)
    nchw = lambda t: t.double().permute(0, 3, 1, 2)
    nan = lambda shape: torch.full(shape, float("nan"), device="cuda", dtype=dt)
    # forward: the output has the grid
    x, w = rand(1, stride * P, stride * Q, C), rand(K, R, R, C, scale=(R * R * C) ** -0.5)
    want = torch.nn.functional.conv2d(nchw(x), nchw(w), stride=stride, padding=pad).permute(0, 2, 3, 1).contiguous()
    y = nan((1, P, Q, K))
    assert want.shape == y.shape
    rn.conv_fwd(x.cuda(), w.cuda(), stride, pad, y=y)
    assert_close(y, want.numpy(), TOL[mode_name], "y")
    y2 = nan(y.shape)
    rn.conv_fwd_bn_sums(x.cuda(), w.cuda(), stride, pad, y=y2)
    assert torch.equal(y, y2)
    if C == 3:
        return
    # data gradient: the input has the grid
    w, po, qo = rand(C, R, R, K, scale=(R * R * C) ** -0.5), (P + 2 * pad - R) // stride + 1, (Q + 2 * pad - R) // stride + 1
    dy = rand(1, po, qo, C)
    want = torch.nn.grad.conv2d_input((1, K, P, Q), nchw(w), nchw(dy), stride=stride, padding=pad).permute(0, 2, 3, 1).contiguous()
    dx = nan((1, P, Q, K))
    rn.conv_dgrad(dy.cuda(), w.cuda(), dx.shape, stride, pad, dx=dx)
    assert_close(dx, want.numpy(), TOL[mode_name], "dx")
    one, zero = torch.ones(K, device="cuda"), torch.zeros(K, device="cuda")
    dx2 = nan(dx.shape)
    rn.conv_dgrad_bn_sums(dy.cuda(), w.cuda(), dx.shape, stride, pad, torch.ones_like(dx), one, zero, zero, one, dx=dx2)
    assert torch.equal(dx, dx2)


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("C,K,R", [(64, 64, 1), (72, 72, 1), (128, 136, 1), (136, 128, 1), (200, 264, 1), (64, 72, 3), (64, 64, 3), (56, 64, 3), (64, 56, 3)])
@pytest.mark.parametrize("N,hw", [(1, 7), (6, 28)])
def test_weight_gradient_whole_and_ragged_tiles(rn, mode_name, C, K, R, N, hw):
    """Whole tiles are stored row by row from a scalar offset, ragged ones element by element, side by side in one result:
    channel counts with either and both, one split (the result itself) and many (partial sums), into NaNs; twice the same bits."""
    dt = torch.bfloat16 if mode_name == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(C + K)
    x, dy = torch.randn(N, hw, hw, C, generator=gen).to(dt), torch.randn(N, hw, hw, K, generator=gen).to(dt)
    nchw = lambda t: t.double().permute(0, 3, 1, 2)
    want = torch.nn.grad.conv2d_weight(nchw(x), (K, C, R, R), nchw(dy), padding=R // 2).permute(0, 2, 3, 1).contiguous()
    d = rn.ConvDesc(N, hw, hw, C, K, R, R, 1, R // 2, rn.BF16 if mode_name == "bf16" else rn.F32)
    got = []
    for _ in range(2):
        dw = torch.full((K, R, R, C), float("nan"), device="cuda")
        ws = torch.full((max(rn.conv_wgrad_workspace_bytes(d), 256),), 0xFF, dtype=torch.uint8, device="cuda")
        got.append(rn.conv_wgrad(x.cuda(), dy.cuda(), dw.shape, 1, R // 2, dw=dw, workspace=ws))
    assert_close(got[0], want.numpy(), TOL[mode_name], "dw")
    assert torch.equal(got[0], got[1])


# Weight gradient: tiles that span filter taps, channel counts at the edges of the tile widths, pixel ranges of less than one
# chunk, one chunk more than a whole number of splits, and the most splits.
WGRAD_EDGES = [(1, 3, 3, 40, 64, 3, 1, 1), (2, 8, 8, 64, 72, 1, 1, 0), (2, 8, 8, 72, 64, 1, 1, 0), (1, 1, 1, 128, 128, 3, 1, 1),
               (5, 23, 29, 64, 64, 1, 1, 0), (3, 40, 41, 8, 8, 3, 2, 1), (1, 9, 9, 56, 136, 5, 1, 2), (2, 14, 14, 512, 1024, 1, 2, 0)]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("case", WGRAD_EDGES)
def test_wgrad_plan_edges(rn, mode_name, case):
    run_case(rn, mode_name, *case, tag="wg" + str(case))


# Output grids along which the gathering weight gradient steps by a chunk (64 pixels, 32 in float): one pixel an image, one column,
# one row, rows on either side of a chunk, an image exactly one, several images in one, with strides and filters of either parity.
WGRAD_STEPS = [(70, 1, 1, 16, 24, 3, 1, 1), (70, 2, 2, 16, 24, 3, 2, 1), (3, 70, 1, 16, 24, 3, 1, 1), (3, 1, 70, 16, 24, 3, 1, 1), (2, 5, 31, 40, 72, 3, 1, 1),
               (2, 5, 32, 40, 72, 3, 1, 1), (2, 5, 33, 40, 72, 3, 1, 1), (2, 3, 63, 72, 8, 3, 1, 1), (2, 3, 64, 72, 8, 3, 1, 1), (2, 3, 65, 72, 8, 3, 1, 1),
               (2, 3, 130, 72, 8, 3, 1, 1), (5, 8, 8, 136, 72, 3, 1, 1), (5, 4, 8, 136, 72, 3, 1, 1), (11, 7, 7, 136, 72, 3, 1, 1), (9, 13, 15, 72, 136, 3, 2, 1),
               (3, 29, 27, 64, 64, 1, 2, 0), (3, 17, 21, 24, 40, 2, 1, 1), (2, 33, 18, 24, 40, 5, 3, 2), (2, 9, 11, 16, 16, 1, 1, 0),
               # (64 channels and fewer: images of less than a chunk and more, widths from one column to one more than a chunk)
               (11, 7, 7, 64, 64, 3, 1, 1), (9, 6, 6, 16, 24, 3, 1, 1), (5, 8, 7, 64, 64, 3, 1, 1), (40, 2, 1, 64, 48, 3, 1, 1), (3, 9, 14, 64, 64, 3, 1, 1),
               (3, 9, 15, 64, 64, 3, 1, 1), (3, 9, 30, 64, 64, 3, 1, 1), (3, 9, 31, 64, 64, 3, 1, 1), (3, 5, 62, 64, 64, 3, 1, 1), (3, 5, 63, 64, 64, 3, 1, 1),
               (2, 3, 64, 64, 64, 3, 1, 1)]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K,R,stride,pad", WGRAD_STEPS)
def test_weight_gradient_steps_over_rows_and_images(rn, mode_name, N, H, W, C, K, R, stride, pad):
    dt = torch.bfloat16 if mode_name == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(N + H + W + C)
    x = torch.randn(N, H, W, C, generator=gen).to(dt)
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    dy = torch.randn(N, P, Q, K, generator=gen).to(dt)
    nchw = lambda t: t.double().permute(0, 3, 1, 2)
    want = torch.nn.grad.conv2d_weight(nchw(x), (K, C, R, R), nchw(dy), stride=stride, padding=pad).permute(0, 2, 3, 1).contiguous()
    dw = torch.full((K, R, R, C), float("nan"), device="cuda")
    rn.conv_wgrad(x.cuda(), dy.cuda(), (K, R, R, C), stride, pad, dw=dw)
    assert_close(dw, want.numpy(), 1e-5, "dw", elementwise=None)  # (products of the inputs as they are, float sums of at most 3,000)


# All nine taps in one workgroup (bf16, at most 64 channels each way, from 65,536 positions of the images padded by a row and a column on; the
# third case has fewer: one tile per tap, in short splits): an image of exactly a chunk of 64 padded positions, of fewer, of one more row, of a
# column; widths on both sides of every count of passes over the run of x (14, 30, 62), and the first that no run holds; grids of at most one
# workgroup per compute unit (131,072 positions) and of more.
NINE_TAPS = [(1024, 7, 7, 64, 64), (1338, 6, 6, 48, 24), (1023, 7, 7, 64, 64), (911, 8, 7, 64, 64), (10923, 2, 1, 64, 48), (437, 9, 14, 64, 64), (410, 9, 15, 40, 8),
             (212, 9, 30, 64, 64), (205, 9, 31, 64, 64), (40, 56, 56, 64, 56), (174, 5, 62, 64, 64), (171, 5, 63, 64, 64), (347, 5, 62, 64, 64), (128, 56, 56, 16, 64)]


@pytest.mark.parametrize("N,H,W,C,K", NINE_TAPS)
def test_weight_gradient_of_nine_taps_at_once(rn, N, H, W, C, K):
    gen = torch.Generator(device="cuda").manual_seed(N + W)
    x = torch.randn(N, H, W, C, device="cuda", generator=gen).bfloat16()
    dy = torch.randn(N, H, W, K, device="cuda", generator=gen).bfloat16()
    dw = [torch.full((K, 3, 3, C), float("nan"), device="cuda") for _ in range(2)]
    for d in dw:
        rn.conv_wgrad(x, dy, d.shape, 1, 1, dw=d)
    assert torch.equal(dw[0], dw[1])
    xp = torch.nn.functional.pad(x.float(), (0, 0, 1, 1, 1, 1))
    rows = dy.double().reshape(-1, K)
    for r in range(3):
        for s in range(3):
            want = rows.t().contiguous() @ xp[:, r:r + H, s:s + W].reshape(-1, C).double()
            # (float sums of products that are exact in float: at most 1,100 per workgroup, 384 workgroups)
            assert_close(dw[0][:, r, s], want.cpu().numpy(), 1e-5, f"dw tap {r},{s}", elementwise=None)


# Forward on the 128x128 tile (from 384 of them on), whose two rings are of different depth (float: three buffers of A, two of B; bf16: two and
# one): reductions of two chunks (no third buffer of A), three, four and more, ragged channels on both sides, a strided gather with one chunk and with several per tap, a last row tile of one row.
DEEP_RING = [(8, 56, 56, 128, 256, 1, 1), (8, 56, 56, 136, 200, 1, 1), (8, 56, 56, 200, 256, 1, 1), (1, 157, 157, 328, 136, 1, 1), (8, 112, 112, 40, 200, 3, 2),
             (8, 111, 112, 72, 136, 3, 2), (2, 159, 157, 64, 128, 2, 1)]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K,R,stride", DEEP_RING)
def test_forward_with_rings_of_different_depth(rn, mode_name, N, H, W, C, K, R, stride):
    dt, pad = torch.bfloat16 if mode_name == "bf16" else torch.float32, R // 2
    gen = torch.Generator().manual_seed(C + K)
    x, w = torch.randn(N, H, W, C, generator=gen).to(dt), (torch.randn(K, R, R, C, generator=gen) / (R * R * C) ** 0.5).to(dt)
    want = torch.nn.functional.conv2d(x.float().permute(0, 3, 1, 2), w.float().permute(0, 3, 1, 2), stride=stride, padding=pad).permute(0, 2, 3, 1).contiguous()
    y = torch.full(want.shape, float("nan"), device="cuda", dtype=dt)
    rn.conv_fwd(x.cuda(), w.cuda(), stride, pad, y=y)
    assert_close(y, want.numpy(), TOL[mode_name], "y")
    y2, sums = rn.conv_fwd_bn_sums(x.cuda(), w.cuda(), stride, pad)
    assert torch.equal(y, y2)
    check_sums(rn, y, sums)


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K", [(21, 56, 56, 64, 200), (1, 257, 255, 24, 136), (16, 64, 64, 32, 264), (6, 64, 64, 16, 256), (1, 505, 504, 64, 264)])
def test_one_chunk_on_large_tiles(rn, mode_name, N, H, W, C, K):
    """1x1 layers whose reduction is one chunk and whose grid has at least 384 tiles of 128x128 (the second: 512 rows of tiles, the last of 127 rows):
    forward with and without sums, the data gradient likewise, with a second branch and at stride 2, into buffers of NaNs.  In bf16 a data
    gradient's sums come from 64x64 tiles, and from 128 MB of output on (the last one, just above; at stride 2 both of 264 columns)
    from 128x128, with a second branch from 128x64: the same rows of sums."""
    dt = torch.bfloat16 if mode_name == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(C + K)
    rand = lambda *shape, scale=1.0: (torch.randn(*shape, generator=gen) * scale).to(dt)
    nan = lambda *shape: torch.full(shape, float("nan"), device="cuda", dtype=dt)
    x, w, wt, add = rand(N, H, W, C), rand(K, 1, 1, C, scale=C ** -0.5), rand(C, 1, 1, K, scale=C ** -0.5), rand(N, H, W, K)
    y = rn.conv_fwd(x.cuda(), w.cuda(), 1, 0, y=nan(N, H, W, K))
    want = x.float().reshape(-1, C) @ w.float().reshape(K, C).t()
    assert_close(y.view(-1, K), want.numpy(), TOL[mode_name], "y")
    y2, sums = rn.conv_fwd_bn_sums(x.cuda(), w.cuda(), 1, 0)
    assert torch.equal(y, y2)
    check_sums(rn, y, sums)
    dx = rn.conv_dgrad(x.cuda(), wt.cuda(), (N, H, W, K), 1, 0, dx=nan(N, H, W, K))
    want = x.float().reshape(-1, C) @ wt.float().reshape(C, K)
    assert_close(dx.view(-1, K), want.numpy(), TOL[mode_name], "dx")
    one, zero = torch.ones(K, device="cuda"), torch.zeros(K, device="cuda")
    dx2, sums = rn.conv_dgrad_bn_sums(x.cuda(), wt.cuda(), (N, H, W, K), 1, 0, y, one, zero, zero, one, dx=nan(N, H, W, K))
    assert torch.equal(dx, dx2)
    check_sums(rn, dx, sums, grad_of=y)
    both, sums = rn.conv_dgrad_bn_sums(x.cuda(), wt.cuda(), (N, H, W, K), 1, 0, y, one, zero, zero, one, addend=add.cuda(), dx=nan(N, H, W, K))
    assert_close(both.view(-1, K), (want + add.float().reshape(-1, K)).numpy(), TOL[mode_name], "dx + addend")
    check_sums(rn, both, sums, grad_of=y)
    dx2 = rn.conv_dgrad(x.cuda(), wt.cuda(), (N, 2 * H, 2 * W, K), 2, 0, dx=nan(N, 2 * H, 2 * W, K))
    assert torch.equal(dx2[:, ::2, ::2], dx) and not dx2[:, 1::2].any() and not dx2[:, :, 1::2].any()
    below = torch.randn(dx2.shape, device="cuda").to(dt)
    dx3, sums = rn.conv_dgrad_bn_sums(x.cuda(), wt.cuda(), dx2.shape, 2, 0, below, one, zero, zero, one, dx=nan(*dx2.shape))
    assert torch.equal(dx2, dx3)
    check_sums(rn, dx3, sums, grad_of=below)
