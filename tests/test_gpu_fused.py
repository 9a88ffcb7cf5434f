"""GPU parity of the convolution + batch-norm pairs whose per-channel sums are taken in the
convolution's output stage (conv_fwd_bn_sums -> bn_relu_fwd_from_sums, conv_dgrad_bn_sums ->
bn_relu_bwd_from_sums), against the oracle's separate operations, through the C ABI."""
import numpy as np
import pytest
import torch

import oracle as orc
import synth
from gpu_util import impose_relu_decisions, TOL, assert_close, dev, host, inputs

pytestmark = pytest.mark.gpu
SEED = synth.DEFAULT_SEED


@pytest.fixture(scope="module")
def rn():
    import paper_1903_12650_amd as rn
    return rn


# (N, H, W, Cin, Cout, R, stride, pad): several row tiles with a ragged last one, ragged channel tiles,
# both strides, the stem, and a single-tile case
FUSED_SHAPES = [(2, 14, 14, 64, 64, 1, 1, 0), (3, 13, 9, 24, 40, 3, 1, 1), (2, 28, 28, 32, 136, 3, 2, 1),
                (5, 28, 28, 128, 128, 1, 1, 0), (2, 30, 30, 64, 256, 1, 2, 0), (1, 5, 5, 8, 8, 3, 1, 1),
                (2, 64, 64, 3, 64, 7, 2, 3), (40, 7, 7, 256, 64, 1, 1, 0), (3, 11, 13, 24, 40, 3, 2, 1),
                (2, 9, 7, 16, 16, 1, 2, 0),
                # 3x3 stride 1 pad 1, whole channel chunks, tiles spanning images
                (3, 9, 9, 64, 64, 3, 1, 1), (2, 5, 12, 128, 72, 3, 1, 1), (5, 7, 21, 192, 64, 3, 1, 1),
                (7, 4, 48, 64, 128, 3, 1, 1), (40, 14, 14, 64, 64, 3, 1, 1),
                # ... large enough for the eight-wave 256x128 tile (forward / data gradient): the sums' row count follows
                (16, 28, 28, 64, 512, 3, 1, 1), (16, 28, 28, 512, 64, 3, 1, 1)]


def _vec(tag, C, scale, shift):
    return (shift + scale * synth.normal(SEED, tag, (C,))).astype(np.float32)


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("shape", FUSED_SHAPES)
def test_conv_fwd_bn_sums(rn, mode_name, shape):
    bf = mode_name == "bf16"
    tol = TOL[mode_name]
    N, H, W, C, K, R, stride, pad = shape
    x = synth.activation_nhwc(SEED, "x", N, C, H, W)
    w = synth.conv_weight_krsc(SEED, "w", K, C, R, R)
    x, w = inputs(mode_name, x, w)
    gamma, beta = _vec("g", K, 0.3, 1.0), _vec("b", K, 0.2, 0.0)
    xd, wd = dev(x, bf), dev(w, bf)
    y, sums = rn.conv_fwd_bn_sums(xd, wd, stride, pad)
    assert torch.equal(y, rn.conv_fwd(xd, wd, stride, pad)), "the sums must not change the convolution"
    assert_close(y, orc.conv_fwd(x, w, stride, pad), tol, "y")
    yh = host(y)
    res = inputs(mode_name, synth.normal(SEED, "r", yh.shape))[0]
    for mode in (0, 1, 2):
        r = res if mode == 2 else None
        z, mean, rstd = rn.bn_relu_fwd_from_sums(y, sums, dev(gamma), dev(beta), dev(r, bf) if r is not None else None,
                                                 1e-5, mode)
        z_o, mean_o, rstd_o = orc.bn_relu_fwd(yh, gamma, beta, r, 1e-5, mode)   # on the GPU path's own y
        if yh.size // K > 1:
            assert_close(z, z_o, tol, f"z mode {mode}")
            assert_close(mean, mean_o, 1e-5, "mean")
            assert_close(rstd, rstd_o, 1e-4, "rstd")
        # and the separate-pass kernels agree to rounding of the float sums
        z_u, mean_u, rstd_u = rn.bn_relu_fwd(y, dev(gamma), dev(beta), dev(r, bf) if r is not None else None, 1e-5, mode)
        assert_close(mean, host(mean_u), 1e-5, "mean vs separate pass")
        assert_close(rstd, host(rstd_u), 1e-5, "rstd vs separate pass")


def test_conv_fwd_bn_sums_large_mean_and_running_stats(rn):
    # all-positive operands: every output channel's mean is many standard deviations from zero and the
    # tiles' shifts differ, so the change of shift in the final sum is exercised
    N, H, W, C, K = 4, 20, 20, 64, 72
    x = np.abs(synth.activation_nhwc(SEED, "x", N, C, H, W)) + 3.0
    w = np.abs(synth.conv_weight_krsc(SEED, "w", K, C, 3, 3)) + 0.05
    g, b = np.ones(K, np.float32), np.zeros(K, np.float32)
    y, sums = rn.conv_fwd_bn_sums(dev(x), dev(w), 1, 1)
    yh = host(y)
    rm0 = synth.normal(SEED, "rm", (K,)); rv0 = np.abs(synth.normal(SEED, "rv", (K,))) + 1
    rm, rv = dev(rm0), dev(rv0)
    z, mean, rstd = rn.bn_relu_fwd_from_sums(y, sums, dev(g), dev(b), None, 1e-5, 0, running_mean=rm, running_var=rv,
                                             momentum=0.9)
    z_o, mean_o, rstd_o = orc.bn_relu_fwd(yh, g, b, None, 1e-5, 0)
    rm_o, rv_o = orc.bn_running_update(yh, rm0, rv0, 0.9)
    assert float(np.min(np.abs(mean_o) * rstd_o)) > 3.0, "the case must have |mean| >> std"
    assert_close(mean, mean_o, 1e-6, "mean")
    assert_close(rstd, rstd_o, 1e-4, "rstd")
    assert_close(z, z_o, 1e-3, "z")
    assert_close(rm, rm_o, 1e-6, "running_mean")
    assert_close(rv, rv_o, 1e-4, "running_var")


@pytest.mark.parametrize("N,H,C,K", [(40, 28, 64, 72), (8, 28, 64, 72)])
def test_conv_fwd_bn_sums_mean_far_from_zero(rn, N, H, C, K):
    """Outputs 4000 +- 0.5 in float: the statistics stay within 2^-22 of their 64-bit values, summed by the finalize launch (490
    tile rows) and by the apply pass (98)."""
    x = synth.activation_nhwc(SEED, "x", N, C, H, H) * 4.0 + 4000.0
    w = np.full((K, 1, 1, C), 1.0 / C, np.float32)
    y, sums = rn.conv_fwd_bn_sums(dev(x), dev(w), 1, 0)
    _, mean, rstd = rn.bn_relu_fwd_from_sums(y, sums, dev(np.ones(K, np.float32)), dev(np.zeros(K, np.float32)), None, 1e-5, 0)
    y64 = host(y).reshape(-1, K).astype(np.float64)
    mean_o, rstd_o = y64.mean(0), 1.0 / np.sqrt(y64.var(0) + 1e-5)
    assert (mean_o * rstd_o).min() > 4000
    assert np.all(np.abs(host(mean) - mean_o) <= 2.0 ** -24 * mean_o + 2.0 ** -22 / rstd_o)
    assert np.abs(host(rstd) / rstd_o - 1).max() <= 2.0 ** -22, np.abs(host(rstd) / rstd_o - 1).max() * 2 ** 24


@pytest.mark.parametrize("mode_name,C", [("bf16", 8), ("bf16", 24), ("f32", 12)])
@pytest.mark.parametrize("H,W", [(512, 512), (512, 513), (577, 611)])
def test_many_tile_rows_are_reduced_by_their_producer(rn, mode_name, C, H, W):
    """Above 4096 tile rows (of 64 pixels here; 4096, 4104 and 5509 of them) the convolutions leave rows of doubles.  Statistics
    and backward sums against 64 bits: per-tile sums in float over 64 values, everything behind them in double."""
    bf = mode_name == "bf16"
    dt = torch.bfloat16 if bf else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(H + C)
    x = (torch.randn(1, H, W, 8, device="cuda", generator=gen) + 3.0).to(dt)
    w = (torch.randn(C, 1, 1, 8, device="cuda", generator=gen) * 0.3 + 0.5).to(dt)
    y, sums = rn.conv_fwd_bn_sums(x, w, 1, 0)
    gamma, beta = torch.ones(C, device="cuda"), torch.zeros(C, device="cuda")
    _, mean, rstd = rn.bn_relu_fwd_from_sums(y, sums, gamma, beta, None, 1e-5, 1)
    y64 = y.double().reshape(-1, C)
    mean_o = y64.mean(0)
    rstd_o = 1.0 / torch.sqrt(y64.var(0, unbiased=False) + 1e-5)
    assert ((mean - mean_o).abs() <= 2.0 ** -23 * mean_o.abs() + 2.0 ** -22 / rstd_o).all()
    assert ((rstd / rstd_o - 1).abs() <= 2.0 ** -22).all()
    # backward: dy [1][H][W][8] of a 1x1 layer with C input channels, whose input is that BN's output
    dy = torch.randn(1, H, W, 8, device="cuda", generator=gen).to(dt)
    wb = (torch.randn(8, 1, 1, C, device="cuda", generator=gen) * 0.3).to(dt)
    dx, bsums = rn.conv_dgrad_bn_sums(dy, wb, (1, H, W, C), 1, 0, y, gamma, beta, mean, rstd)
    _, _, dgamma, dbeta = rn.bn_relu_bwd_from_sums(dx, y, bsums, gamma, beta, mean, rstd, mode=1)
    xhat = (y64 - mean.double()) * rstd.double()
    # (the decision as the kernel takes it, in float: y * rstd - mean * rstd > 0)
    on = torch.addcmul(-(mean * rstd).double(), y64, rstd.double()).float() > 0
    g64 = dx.double().reshape(-1, C) * on
    # a tile's float sum of 64 terms is off by at most 64 * 2^-24 of the sum of their magnitudes
    for got, terms in ((dbeta, g64), (dgamma, g64 * xhat)):
        assert ((got.double() - terms.sum(0)).abs() <= 64 * 2.0 ** -24 * terms.abs().sum(0)).all()


DGRAD_SHAPES = [s for s in FUSED_SHAPES if s[3] != 3]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("shape", DGRAD_SHAPES)
def test_conv_dgrad_bn_sums(rn, mode_name, shape):
    bf = mode_name == "bf16"
    tol = TOL[mode_name]
    N, H, W, C, K, R, stride, pad = shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    # the BN layer below the convolution: input bx [N,H,W,C], output z feeds the convolution
    bx = synth.activation_nhwc(SEED, "bx", N, C, H, W) * 1.3 + 0.2
    dy = synth.activation_nhwc(SEED, "dy", N, K, P, Q)
    w = synth.conv_weight_krsc(SEED, "w", K, C, R, R)
    bx, dy, w = inputs(mode_name, bx, dy, w)
    gamma, beta = _vec("g", C, 0.3, 1.0), _vec("b", C, 0.2, 0.0)
    z_o, mean_o, rstd_o = orc.bn_relu_fwd(bx, gamma, beta, None, 1e-5, 1)
    z_o = inputs(mode_name, z_o)[0]
    dyd, wd, bxd = dev(dy, bf), dev(w, bf), dev(bx, bf)
    gd, bd = dev(gamma), dev(beta)
    # The backward kernels recompute the ReLU decision from bx: with the GPU forward pass's statistics that is
    # that pass's decision bit for bit, which is recorded here and imposed on the oracle's backward pass wherever a
    # pre-activation within rounding of zero landed on the other side.
    bits = rn.relu_mask_like(bxd)
    _, md, rd = rn.bn_relu_fwd(bxd, gd, bd, None, 1e-5, 1, relu_mask=bits)
    assert_close(md, mean_o, 1e-5, "mean")
    assert_close(rd, rstd_o, 1e-4, "rstd")
    z_o, _ = impose_relu_decisions(z_o, bits)
    dz, sums = rn.conv_dgrad_bn_sums(dyd, wd, (N, H, W, C), stride, pad, bxd, gd, bd, md, rd)
    assert torch.equal(dz, rn.conv_dgrad(dyd, wd, (N, H, W, C), stride, pad)), "the sums must not change the gradient"
    assert_close(dz, orc.conv_dgrad(dy, w, (N, H, W, C), stride, pad), tol, "dz")
    dx, _, dg, db = rn.bn_relu_bwd_from_sums(dz, bxd, sums, gd, bd, md, rd)
    dx_o, _, dg_o, db_o = orc.bn_relu_bwd(host(dz).astype(np.float32), bx, z_o, gamma, mean_o, rstd_o, 1)
    if N * H * W > 1:
        assert_close(dx, dx_o, tol, "dx")
        assert_close(dg, dg_o, tol, "dgamma")
        assert_close(db, db_o, tol, "dbeta")
    # the separate-pass kernels (same mask rule) agree to rounding of the float sums
    dx_u, _, dg_u, db_u = rn.bn_relu_bwd(dz, bxd, None, gd, md, rd, 1, beta=bd)
    assert_close(dg, host(dg_u), 1e-5, "dgamma vs separate pass")
    assert_close(db, host(db_u), 1e-5, "dbeta vs separate pass")
    assert_close(dx, host(dx_u), max(1e-5, tol / 4), "dx vs separate pass")


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("shape", DGRAD_SHAPES)
def test_conv_dgrad_bn_sums_residual_layer_with_addend(rn, mode_name, shape):
    """The BN layer below is a residual-add layer (mode 2) whose output has a second consumer: the data
    gradient adds that consumer's gradient (one rounding of the sum), takes the mask from the recorded bits."""
    bf = mode_name == "bf16"
    tol = TOL[mode_name]
    N, H, W, C, K, R, stride, pad = shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    bx = synth.activation_nhwc(SEED, "bx", N, C, H, W) * 1.3 + 0.2
    res = synth.activation_nhwc(SEED, "res", N, C, H, W)
    dy = synth.activation_nhwc(SEED, "dy", N, K, P, Q)
    add = synth.activation_nhwc(SEED, "add", N, C, H, W) * 0.7
    w = synth.conv_weight_krsc(SEED, "w", K, C, R, R)
    bx, res, dy, add, w = inputs(mode_name, bx, res, dy, add, w)
    gamma, beta = _vec("g", C, 0.3, 1.0), _vec("b", C, 0.2, 0.0)
    bxd, resd = dev(bx, bf), dev(res, bf)
    gd, bd = dev(gamma), dev(beta)
    bits = rn.relu_mask_like(bxd)
    z, md, rd = rn.bn_relu_fwd(bxd, gd, bd, resd, 1e-5, 2, relu_mask=bits)      # the layer's own forward pass
    dz, sums = rn.conv_dgrad_bn_sums(dev(dy, bf), dev(w, bf), (N, H, W, C), stride, pad, bxd, gd, bd, md, rd,
                                     addend=dev(add, bf), relu_mask=bits)
    want = orc.conv_dgrad(dy, w, (N, H, W, C), stride, pad) + add
    assert_close(dz, want, tol, "dz = data gradient + addend")
    if bf:   # one rounding of the float sum: never further from it than rounding the exact sum twice would be
        plain = host(rn.conv_dgrad(dev(dy, bf), dev(w, bf), (N, H, W, C), stride, pad))
        assert orc.rel_l2(host(dz), want) <= orc.rel_l2(synth.round_bf16(plain + add), want) * 1.05 + 1e-7
    dx, dres, dg, db = rn.bn_relu_bwd_from_sums(dz, bxd, sums, gd, bd, md, rd, mode=2, relu_mask=bits)
    dx_o, dres_o, dg_o, db_o = orc.bn_relu_bwd(host(dz).astype(np.float32), bx, host(z), gamma, host(md), host(rd), 2)
    if N * H * W > 1:
        assert_close(dx, dx_o, tol, "dx")
        assert_close(dres, dres_o, tol, "dresidual")
        assert_close(dg, dg_o, max(tol, 1e-3), "dgamma")
        assert_close(db, db_o, max(tol, 1e-3), "dbeta")
    # an addend that counts only under recorded ReLU bits (the identity shortcut's gradient, taken without
    # a masked copy) gives the bits of the call with the masked tensor
    V = 8 if bf else 4
    rng = np.random.default_rng(11)
    abits = rng.integers(0, 1 << V, size=add.size // V).astype(np.uint8)
    keep = ((abits[:, None] >> np.arange(V)[None, :]) & 1).astype(add.dtype).reshape(add.shape)
    nbytes = rn.conv_bn_sums_bytes(rn.ConvDesc(N, H, W, C, K, R, R, stride, pad, rn.BF16 if bf else rn.F32))
    zeros = lambda: torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    dz_m, sums_m = rn.conv_dgrad_bn_sums(dev(dy, bf), dev(w, bf), (N, H, W, C), stride, pad, bxd, gd, bd, md, rd,
                                         addend=dev(add, bf), relu_mask=bits, addend_mask=dev(abits), sums=zeros())
    dz_p, sums_p = rn.conv_dgrad_bn_sums(dev(dy, bf), dev(w, bf), (N, H, W, C), stride, pad, bxd, gd, bd, md, rd,
                                         addend=dev(add * keep, bf), relu_mask=bits, sums=zeros())
    assert torch.equal(dz_m, dz_p) and torch.equal(sums_m[1], sums_p[1])
    # the separate-pass kernels agree to rounding of the float sums
    dx_u, dres_u, dg_u, db_u = rn.bn_relu_bwd(dz, bxd, z, gd, md, rd, 2, beta=bd)
    assert torch.equal(dres, dres_u)
    assert_close(dg, host(dg_u), 1e-5, "dgamma vs separate pass")
    assert_close(db, host(db_u), 1e-5, "dbeta vs separate pass")
    assert_close(dx, host(dx_u), max(1e-5, tol / 4), "dx vs separate pass")


# Whole tiles only, a last tile of one row, of all rows but one, and columns that end inside a tile; 1x1 and 3x3 (one run and classes); the large tiles of
# the 3x3 / stride 1 layers, whole and with ragged rows and columns: pairs of 128x128, 256x128, 256x64.
@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K,R,stride", [(50, 32, 32, 128, 128, 1, 1), (1, 1, 49153, 128, 64, 1, 1), (1, 1, 25727, 136, 200, 1, 1),
                                                (16, 31, 31, 128, 64, 3, 1), (13, 32, 32, 256, 64, 3, 2), (1, 1, 65, 40, 24, 1, 1),
                                                (48, 16, 16, 1024, 64, 3, 1), (1, 265, 31, 1000, 72, 3, 1), (8, 32, 32, 1024, 64, 3, 1),
                                                (1, 257, 32, 1000, 72, 3, 1), (32, 56, 56, 64, 32, 3, 1), (25, 63, 63, 40, 24, 3, 1)])
@pytest.mark.parametrize("recorded,second", [(True, True), (True, False), (False, True)])
def test_conv_dgrad_bn_sums_of_whole_and_ragged_tiles(rn, mode_name, N, H, W, C, K, R, stride, recorded, second):
    """Random ReLU decisions of both layers, every bit position of a vector among them; sums against 64 bits."""
    bf = mode_name == "bf16"
    dt, V = (torch.bfloat16, 8) if bf else (torch.float32, 4)
    gen = torch.Generator().manual_seed(5)
    rand = lambda *s: torch.randn(*s, generator=gen).to(dt).cuda()
    P, Q = (H - 1) // stride + 1, (W - 1) // stride + 1
    dy, w, x, add = rand(N, P, Q, K), (torch.randn(K, R, R, C, generator=gen) / (K * R * R) ** 0.5).to(dt).cuda(), rand(N, H, W, C), rand(N, H, W, C)
    gamma, beta = (torch.randn(C, generator=gen).cuda() for _ in range(2))
    mean, rstd = 0.2 * torch.randn(C, generator=gen).cuda(), 0.5 + torch.rand(C, generator=gen).cuda()
    bits, abits = (torch.randint(0, 1 << V, (N * H * W * C // V,), generator=gen, dtype=torch.uint8).cuda() for _ in range(2))
    decisions = lambda b: ((b[:, None] >> torch.arange(V, device="cuda", dtype=torch.uint8)) & 1).view(N * H * W, C).bool()
    extra = dict(relu_mask=bits) if recorded else {}
    if second:
        extra.update(addend=add, addend_mask=abits)
    dz, sums = rn.conv_dgrad_bn_sums(dy, w, (N, H, W, C), stride, R // 2, x, gamma, beta, mean, rstd, dx=torch.full_like(x, float("nan")), **extra)
    want = rn.conv_dgrad(dy, w, (N, H, W, C), stride, R // 2).double().view(-1, C)
    if second:
        want = want + torch.where(decisions(abits), add.view(-1, C), torch.zeros_like(add.view(-1, C))).double()
        assert_close(dz.view(-1, C), want.cpu().numpy(), TOL[mode_name], "dx + second branch")
    else:
        assert torch.equal(dz.double().view(-1, C), want)
    scale = gamma * rstd   # the kernels' decision: fma(x, scale, fma(-mean, scale, beta)) > 0
    pre = x.double().view(-1, C) * scale.double() + (beta.double() - mean.double() * scale.double()).float().double()
    on = decisions(bits) if recorded else pre > 0
    g = torch.where(on, dz.double().view(-1, C), 0.0)
    xhat = (x.double().view(-1, C) - mean.double()) * rstd.double()
    _, _, dgamma, dbeta = rn.bn_relu_bwd_from_sums(dz, x, sums, gamma, beta, mean, rstd, mode=2 if recorded else 1, **(dict(relu_mask=bits) if recorded else {}))
    # A tile's float sum adds at most 40 terms one behind another: the rows of a thread (tile rows / row groups), then the row groups of a column (8 + 32 at
    # bf16 tiles of 256 rows, 2 + 32 at 64x64, 16 + 16 in float).  Beside them the normalised value's two roundings, of at most 1 + |mean * rstd| / |xhat|
    # units each: 64 in all.  Without recorded bits a decision within a rounding of zero may fall either way.
    near = torch.where(pre.abs() <= 2.0 ** -22 * (1 + pre.abs()), dz.double().view(-1, C).abs(), 0.0) if not recorded else torch.zeros_like(g)
    for got, terms, slack in ((dbeta, g, near), (dgamma, g * xhat, near * xhat.abs())):
        assert ((got.double() - terms.sum(0)).abs() <= 64 * 2.0 ** -24 * terms.abs().sum(0) + slack.sum(0)).all()


# A last tile with rows past the last, in one run of pixels (64x64, K split over the waves, 128x128 tiles), in classes and in 3x3 / stride 1 layers.
@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K,R,stride", [(1, 1, 65, 40, 24, 1, 1), (1, 5, 13, 64, 512, 1, 1), (1, 1, 24577, 136, 128, 1, 1), (3, 15, 15, 40, 24, 3, 2),
                                                (3, 13, 13, 40, 24, 3, 1)])
@pytest.mark.parametrize("recorded,second", [(True, True), (True, False), (False, True), (False, False)])
def test_an_infinity_in_a_ragged_tile_counts_once(rn, mode_name, N, H, W, C, K, R, stride, recorded, second):
    """An infinite input of the BN layer under an open ReLU makes its channel's dgamma infinite, with the sign of its gradient, as in a whole tile;
    rows past the last, which read a pixel of the image, do not add zero times it (not a number)."""
    bf = mode_name == "bf16"
    dt, V = (torch.bfloat16, 8) if bf else (torch.float32, 4)
    gen = torch.Generator().manual_seed(9)
    rand = lambda *s: torch.randn(*s, generator=gen).to(dt).cuda()
    P, Q = (H - 1) // stride + 1, (W - 1) // stride + 1
    dy, w, x = rand(N, P, Q, K), (torch.randn(K, R, R, C, generator=gen) / (K * R * R) ** 0.5).to(dt).cuda(), rand(N, H, W, C)
    hit = [(0, 0), (N * H * W - 1, C - 1), (N * H * W - 1, 3)]     # (pixel, channel): the pixels that rows past the last read
    for p, c in hit:
        x.view(-1, C)[p, c] = float("inf")
    gamma, beta, mean, rstd = torch.ones(C).cuda(), torch.zeros(C).cuda(), torch.zeros(C).cuda(), torch.ones(C).cuda()
    extra = dict(relu_mask=torch.full((N * H * W * C // V,), (1 << V) - 1, dtype=torch.uint8, device="cuda")) if recorded else {}
    if second:
        extra["addend"] = rand(N, H, W, C)
    dz, sums = rn.conv_dgrad_bn_sums(dy, w, (N, H, W, C), stride, R // 2, x, gamma, beta, mean, rstd, **extra)
    _, _, dgamma, dbeta = rn.bn_relu_bwd_from_sums(dz, x, sums, gamma, beta, mean, rstd, mode=2 if recorded else 1,
                                                   **(dict(relu_mask=extra["relu_mask"]) if recorded else {}))
    g = dz.double().view(-1, C)
    for p, c in hit:
        assert float(g[p, c]) != 0.0 and float(dgamma[c]) == float("inf") * (1 if float(g[p, c]) > 0 else -1), (p, c, float(dgamma[c]))
    others = torch.ones(C, dtype=torch.bool, device="cuda")
    others[[c for _, c in hit]] = False
    assert torch.isfinite(dgamma[others]).all() and torch.isfinite(dbeta).all()


def test_fused_sums_reproducible_and_independent_of_buffer_contents(rn):
    N, H, W, C, K = 6, 28, 28, 64, 128
    x = dev(synth.activation_nhwc(SEED, "x", N, C, H, W), True)
    w = dev(synth.conv_weight_krsc(SEED, "w", K, C, 3, 3), True)
    g, b = dev(_vec("g", K, 0.3, 1.0)), dev(_vec("b", K, 0.2, 0.0))
    d = rn.ConvDesc(N, H, W, C, K, 3, 3, 1, 1, rn.BF16)
    outs = []
    for fill in (0, 0xFF):
        sums = torch.full((rn.conv_bn_sums_bytes(d),), fill, dtype=torch.uint8, device="cuda")
        y, h = rn.conv_fwd_bn_sums(x, w, 1, 1, sums=sums)
        outs.append(rn.bn_relu_fwd_from_sums(y, h, g, b, None, 1e-5, 1))
    for a, c in zip(*outs):
        assert torch.equal(a, c)


def test_fused_abi_errors(rn):
    N, H, W, C, K = 2, 8, 8, 16, 16
    x = dev(synth.activation_nhwc(SEED, "x", N, C, H, W), True)
    w = dev(synth.conv_weight_krsc(SEED, "w", K, C, 1, 1), True)
    g, b = dev(np.ones(K, np.float32)), dev(np.zeros(K, np.float32))
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    with pytest.raises(rn.Rn50Error) as e:
        rn.conv_fwd_bn_sums(x, w, 1, 0, sums=small)
    assert e.value.code == -3                                   # RN50_ERR_WORKSPACE
    y, h = rn.conv_fwd_bn_sums(x, w, 1, 0)
    other = (rn.ConvDesc(N, H, W, C, 2 * K, 1, 1, 1, 0, rn.BF16), h[1])
    with pytest.raises(rn.Rn50Error) as e:
        rn.bn_relu_fwd_from_sums(y, other, g, b)
    assert e.value.code == -1                                   # RN50_ERR_INVALID: not this layer's producer
    with pytest.raises(rn.Rn50Error) as e:
        rn.bn_relu_fwd_from_sums(y, h, g, b, None, 1e-5, 2)     # mode 2 without residual
    assert e.value.code == -1
    # addend_mask without addend: rejected before the first launch, so workspace, dx and sums stay as they were
    dy = dev(synth.activation_nhwc(SEED, "dy", N, K, H, W), True)
    mask = torch.full((N * H * W * C // 8,), 0xff, dtype=torch.uint8, device="cuda")
    d = rn.ConvDesc(N, H, W, C, K, 1, 1, 1, 0, rn.BF16)
    wsb = torch.full((rn.conv_dgrad_workspace_bytes(d),), 0x5a, dtype=torch.uint8, device="cuda")
    sums = torch.full((rn.conv_bn_sums_bytes(d),), 0x5a, dtype=torch.uint8, device="cuda")
    dx = torch.full((N, H, W, C), 3.0, dtype=torch.bfloat16, device="cuda")
    gc, bc = dev(np.ones(C, np.float32)), dev(np.zeros(C, np.float32))
    with pytest.raises(rn.Rn50Error) as e:
        rn.conv_dgrad_bn_sums(dy, w, (N, H, W, C), 1, 0, x, gc, bc, bc, gc, dx=dx, workspace=wsb, sums=sums,
                              addend=None, addend_mask=mask)
    assert e.value.code == -1
    torch.cuda.synchronize()
    assert bool((wsb == 0x5a).all()) and bool((sums == 0x5a).all()) and bool((dx == 3.0).all())


# ------------------------------------------------- BN+ReLU applied in the consumer convolution's operand load
BN_IN_SHAPES = [(2, 9, 7, 24, 40), (3, 14, 14, 64, 256), (40, 14, 14, 256, 1024), (2, 8, 8, 72, 136), (40, 7, 7, 512, 2048),
                (1, 5, 5, 8, 8)]


@pytest.mark.parametrize("mode_name", ["f32", "bf16"])
@pytest.mark.parametrize("shape", BN_IN_SHAPES)
def test_conv_bn_in_equals_the_unfused_pair_and_the_oracle(rn, mode_name, shape):
    """conv_fwd_bn_in / conv_wgrad_bn_in read the BN layer's INPUT and apply BN+ReLU on the fly: bit for bit the
    convolution of the tensor bn_relu_fwd stores, and that tensor's convolution by the oracle at the mode's bar."""
    N, H, W, C, K = shape
    bf = mode_name == "bf16"
    if not bf and (C % 4 or K % 4):
        pytest.skip("channel counts must be multiples of the 16-byte vector")
    if bf and (C % 8 or K % 8):
        pytest.skip("channel counts must be multiples of the 16-byte vector")
    x, w, dy = inputs(mode_name, synth.activation_nhwc(SEED, "x", N, C, H, W) * 1.5 + 0.3,
                      synth.conv_weight_krsc(SEED, "w", K, C, 1, 1), synth.activation_nhwc(SEED, "dy", N, K, H, W))
    gamma = (1.0 + 0.2 * synth.normal(SEED, "g", (C,))).astype(np.float32)
    beta = (0.1 * synth.normal(SEED, "b", (C,))).astype(np.float32)
    xd, wd, dyd, gd, bd = dev(x, bf), dev(w, bf), dev(dy, bf), dev(gamma), dev(beta)
    z, mean, rstd = rn.bn_relu_fwd(xd, gd, bd, None, 1e-5, 1)
    y_ref = rn.conv_fwd(z, wd, 1, 0)
    dw_ref = rn.conv_wgrad(z, dyd, wd.shape, 1, 0)
    y, handle = rn.conv_fwd_bn_in(xd, gd, bd, mean, rstd, wd, with_sums=True)
    dw = rn.conv_wgrad_bn_in(xd, gd, bd, mean, rstd, dyd, wd.shape)
    torch.cuda.synchronize()
    assert torch.equal(y, y_ref), "forward differs from the convolution of the stored BN output"
    assert torch.equal(dw, dw_ref), "weight gradient differs from that of the stored BN output"
    assert_close(y, orc.conv_fwd(host(z), host(wd), 1, 0), TOL[mode_name], "y")
    assert_close(dw, orc.conv_wgrad(host(z), host(dyd), tuple(wd.shape), 1, 0), TOL[mode_name], "dw")
    # the sums it leaves for the BN layer behind it are those of conv_fwd_bn_sums on the stored tensor
    g2, b2 = dev(np.ones(K, np.float32)), dev(np.zeros(K, np.float32))
    z2, m2, r2 = rn.bn_relu_fwd_from_sums(y, handle, g2, b2)
    y3, h3 = rn.conv_fwd_bn_sums(z, wd, 1, 0)
    z3, m3, r3 = rn.bn_relu_fwd_from_sums(y3, h3, g2, b2)
    assert torch.equal(z2, z3) and torch.equal(m2, m3) and torch.equal(r2, r3)


def test_conv_bn_in_rejects_other_filters(rn):
    x = torch.zeros((1, 8, 8, 16), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((16, 3, 3, 16), dtype=torch.bfloat16, device="cuda")
    v = torch.ones(16, device="cuda")
    d = rn.ConvDesc(1, 8, 8, 16, 16, 3, 3, 1, 1, rn.BF16)
    import ctypes
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = rn.raw.conv_fwd_bn_in(ctypes.byref(d), p(x), p(v), p(v), p(v), p(v), p(w), p(x), None, ctypes.c_size_t(0), None)
    assert rc == -2 and b"1x1" in rn.raw.rn50_last_error()
