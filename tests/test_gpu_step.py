"""GPU parity of the composed paths: one bottleneck block through the operation-level ABI
(BASELINE config 1) and resnet_step against the oracle's training step."""
import numpy as np
import pytest
import torch

import oracle as orc
import synth
from oracle import net
from gpu_util import TOL, assert_close, dev, host, inputs

pytestmark = pytest.mark.gpu
SEED = synth.DEFAULT_SEED


@pytest.fixture(scope="module")
def rn():
    import paper_1903_12650_amd as rn
    return rn


def test_config1_bottleneck_block_f32(rn):
    """One bottleneck block with projection shortcut, fp32, batch 2, input 2x64x56x56, loss = sum(out*T),
    then one LARS step (eta 0.001, momentum 0.9, wd 5e-5 on conv weights, lr 1.0)."""
    N, H, C, Wd = 2, 56, 64, 64
    x = synth.activation_nhwc(SEED, "x", N, C, H, H)
    shapes = [(Wd, 1, 1, C), (Wd, 3, 3, Wd), (4 * Wd, 1, 1, Wd), (4 * Wd, 1, 1, C)]
    table, params = [], []
    for i, s in enumerate(shapes):
        table += [(f"c{i}.w", s, "conv"), (f"c{i}.gamma", (s[0],), "gamma"), (f"c{i}.beta", (s[0],), "beta")]
        params += [synth.conv_weight_krsc(SEED, f"c{i}", s[0], s[3], s[1], s[2]), np.ones(s[0], np.float32),
                   np.zeros(s[0], np.float32)]
    T = synth.activation_nhwc(SEED, "T", N, 4 * Wd, H, H)
    out_o, tape = net.bottleneck_fwd(x, params, 1, True)

    P = [dev(p) for p in params]
    xd, Td = dev(x), dev(T)

    def cbn(inp, i, stride, pad, mode, res=None):
        y = rn.conv_fwd(inp, P[3 * i], stride, pad)
        z, mean, rstd = rn.bn_relu_fwd(y, P[3 * i + 1], P[3 * i + 2], res, 1e-5, mode)
        return dict(x=inp, y=y, z=z, mean=mean, rstd=rstd, i=i, stride=stride, pad=pad, mode=mode)

    def cbn_bwd(dz, t, dz2=None):
        i = t["i"]
        dy, dres, dg, db = rn.bn_relu_bwd(dz, t["y"], t["z"], P[3 * i + 1], t["mean"], t["rstd"], t["mode"],
                                          beta=P[3 * i + 2], dz2=dz2)
        dw = rn.conv_wgrad(t["x"], dy, P[3 * i].shape, t["stride"], t["pad"])
        dx = rn.conv_dgrad(dy, P[3 * i], t["x"].shape, t["stride"], t["pad"])
        return dx, dres, [dw, dg, db]

    t1 = cbn(xd, 0, 1, 0, 1); t2 = cbn(t1["z"], 1, 1, 1, 1); tp = cbn(xd, 3, 1, 0, 0)
    t3 = cbn(t2["z"], 2, 1, 0, 2, res=tp["z"])
    assert_close(t3["z"], out_o, TOL["f32"], "block output")
    # A pre-activation within float rounding of zero may land on either side of the ReLU (a handful of the
    # block's 1.2 million do, depending on the summation order of the convolution in front), and one differing
    # decision moves the gradients by more than the float bar.  Both outcomes are valid: the decisions are
    # checked to differ only where the value is within rounding of zero, then the oracle's backward pass runs
    # with the decisions of the forward pass under test.
    for t_g, t_o in ((t1, tape[0]), (t2, tape[1]), (t3, tape[2])):
        zg, zo = host(t_g["z"]), t_o["z"]
        differ = (zg > 0) != (zo > 0)
        assert differ.sum() <= 8 and (not differ.any() or
                                      max(np.abs(zg[differ]).max(), np.abs(zo[differ]).max()) <= 1e-5 * np.sqrt(np.mean(zo * zo)))
        t_o["z"] = np.where(zg > 0, np.maximum(zo, np.float32(1e-30)), np.float32(0)).astype(zo.dtype)
    dx_o, grads_o = net.bottleneck_bwd(T, tape)
    wds = net.lars_hyper(table, 5e-5)
    vel = [np.zeros_like(p) for p in params]
    w_o, v_o, _ = orc.lars_update(params, grads_o, vel, 0.001, 0.9, 1.0, wds)
    d2, dsc, g3 = cbn_bwd(Td, t3)
    d1, _, g2 = cbn_bwd(d2, t2)
    dxa, _, g1 = cbn_bwd(d1, t1)
    dxb, _, gp = cbn_bwd(dsc, tp)
    assert_close(dxa + dxb, dx_o, TOL["f32"], "dx")
    grads = g1 + g2 + g3 + gp
    for (name, _, _), g, go in zip(table, grads, grads_o):
        assert_close(g, go, TOL["f32"], name)
    V = [torch.zeros_like(p) for p in P]
    Wn = [p.clone() for p in P]
    rn.lars_update(rn.LarsTable(Wn, grads, V, wds), 0.001, 0.9, 1.0)
    for (name, _, _), w, v, wo, vo in zip(table, Wn, V, w_o, v_o):
        assert_close(w, wo, TOL["lars"], name + " w_new")
        assert_close(v, vo, TOL["f32"], name + " v_new (inherits the gradient's tolerance)")
    # the update itself at the fp32 LARS tolerance, from identical gradients
    V = [torch.zeros_like(p) for p in P]
    Wn = [p.clone() for p in P]
    rn.lars_update(rn.LarsTable(Wn, [dev(g) for g in grads_o], V, wds), 0.001, 0.9, 1.0)
    for (name, _, _), w, v, wo, vo in zip(table, Wn, V, w_o, v_o):
        assert_close(w, wo, TOL["lars"], name + " w_new")
        assert_close(v, vo, TOL["lars"], name + " v_new")


@pytest.mark.parametrize("N,H", [(2, 56), (4, 41), (8, 56)])
def test_bottleneck_block_f32_against_the_double_oracle(rn, N, H):
    """The float block at sizes whose 3x3 layer splits its reduction over the waves (98 and 106 tiles of 64x64) and at one
    whose does not (392).  Another summation order puts a pre-activation within rounding of zero on the other side of the
    ReLU, and one such decision moves a gradient by up to 2e-3; that is all that may differ.  So the decisions are counted
    against the oracle in double, and with the same decisions every value is held to float rounding: a sum of n terms carries
    about sqrt(n) roundings of 2^-24, and the longest sequential sums here (pixels of a split, tile rows) stay below 4096
    terms, 4e-6.  (Seen: at most two decisions, |z| <= 8e-7; outputs 4e-7, gradients 1.4e-6.)"""
    bar = 2.0 ** -24 * 4096 ** 0.5
    C, Wd = 64, 64
    x, T = synth.activation_nhwc(SEED, "x", N, C, H, H), synth.activation_nhwc(SEED, "T", N, 4 * Wd, H, H)
    shapes = [(Wd, 1, 1, C), (Wd, 3, 3, Wd), (4 * Wd, 1, 1, Wd), (4 * Wd, 1, 1, C)]
    params = []
    for i, s in enumerate(shapes):
        params += [synth.conv_weight_krsc(SEED, f"c{i}", s[0], s[3], s[1], s[2]), np.ones(s[0], np.float32),
                   (0.1 * synth.normal(SEED, f"b{i}", (s[0],))).astype(np.float32)]
    _, tape = net.bottleneck_fwd(x.astype(np.float64), [p.astype(np.float64) for p in params], 1, True)
    P, xd = [dev(p) for p in params], dev(x)

    def fwd(inp, i, pad, mode, res=None):
        y = rn.conv_fwd(inp, P[3 * i], 1, pad)
        z, mean, rstd = rn.bn_relu_fwd(y, P[3 * i + 1], P[3 * i + 2], res, 1e-5, mode)
        return dict(x=inp, y=y, z=z, mean=mean, rstd=rstd, i=i, pad=pad, mode=mode)

    def bwd(dz, t):
        i = t["i"]
        dy, dres, dg, db = rn.bn_relu_bwd(dz, t["y"], t["z"], P[3 * i + 1], t["mean"], t["rstd"], t["mode"], beta=P[3 * i + 2])
        return (rn.conv_dgrad(dy, P[3 * i], t["x"].shape, 1, t["pad"]), dres,
                [rn.conv_wgrad(t["x"], dy, P[3 * i].shape, 1, t["pad"]), dg, db])

    t1 = fwd(xd, 0, 0, 1); t2 = fwd(t1["z"], 1, 1, 1); tp = fwd(xd, 3, 0, 0); t3 = fwd(t2["z"], 2, 0, 2, tp["z"])
    differing = 0
    for t_g, t_o in ((t1, tape[0]), (t2, tape[1]), (t3, tape[2])):
        zg, zo = host(t_g["z"]).astype(np.float64), t_o["z"]
        assert_close(zg, zo, bar, "z", elementwise=False)
        differ = (zg > 0) != (zo > 0)
        rms = np.sqrt(np.mean(zo * zo))
        assert not differ.any() or np.maximum(zg, zo)[differ].max() <= bar * rms
        differing += int(differ.sum())
        t_o["z"] = np.where(zg > 0, np.maximum(zo, 1e-300), 0.0)
    # a value of size rms lies within bar * rms of zero with a density of 0.4 per rms: a handful of the block's values
    assert differing <= max(8, int(2 * 0.4 * bar * N * H * H * (2 * Wd + 4 * Wd))), differing
    dx_o, grads_o = net.bottleneck_bwd(T.astype(np.float64), tape)
    d2, dsc, g3 = bwd(dev(T), t3)
    d1, _, g2 = bwd(d2, t2)
    dxa, _, g1 = bwd(d1, t1)
    dxb, _, gp = bwd(dsc, tp)
    assert_close(dxa + dxb, dx_o, bar, "dx")
    for k, (g, go) in enumerate(zip(g1 + g2 + g3 + gp, grads_o)):
        assert_close(g, go, bar, f"gradient {k}")


def setup_step(rn, mode_name, N, hw, widths, blocks, stem, classes, expansion=4, ls=0.0):
    bf = mode_name == "bf16"
    plan = rn.ResnetPlan(N, rn.BF16 if bf else rn.F32, hw, classes, widths, blocks, stem, expansion,
                         label_smoothing=ls)
    table = net.param_table(widths, blocks, stem, classes, 3, expansion)
    assert plan.num_tensors == len(table)
    for (name, shape, _), pshape in zip(table, plan.shapes):
        assert tuple(shape) == tuple(pshape), name
    master = synth.params_from_table(SEED, table)
    images = synth.activation_nhwc(SEED, "img", N, 3, hw, hw)
    labels = synth.labels(SEED, "lab", N, classes)
    if bf:
        images = synth.round_bf16(images)
    model = [synth.round_bf16(p) for p in master] if bf else master

    def arena(arrs, dtype=torch.float32):
        a = torch.zeros(plan.arena_elems, dtype=torch.float32)
        for off, p in zip(plan.offsets, arrs):
            a[off:off + p.size] = torch.from_numpy(p.ravel())
        return a.cuda().to(dtype)

    M = arena(master); V = torch.zeros_like(M); G = torch.zeros(plan.arena_elems, device="cuda")
    Mod = arena(model, torch.bfloat16) if bf else M
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
    ws.view(torch.float32)[:] = float("nan")          # nothing unwritten may be read
    return dict(plan=plan, table=table, master=master, model=model, images=images, labels=labels, M=M, V=V, G=G,
                Mod=Mod, ws=ws, bf=bf, N=N, classes=classes, widths=widths, blocks=blocks, ls=ls)


def run_step_vs_oracle(rn, mode_name, *cfg, ls=0.0, tol=None, grad_tol=None, flip_bound=False):
    """End to end against the oracle's training step.

    The forward results (loss, logits) are held to the mode's bar.  Gradients are held to it only
    where no ReLU decision can differ: a pre-activation that is off by delta flips a fraction
    ~delta of the masks z > 0, and every flipped element is wrong by its full value, so the
    rel-L2 error of a gradient is ~sqrt(delta * density) whatever the implementation (measured
    between the oracle's own float and double builds at full depth: 4e-3 from delta = 1.7e-5).
    `grad_tol` states the bound used when that applies; the per-operation bar is enforced with
    identical masks in run_step_vs_chain.

    flip_bound: derive each gradient's bound from measurements instead.  The oracle's float and double builds differ
    in their pre-activations by delta_fd (seen at the logits) and, through the flipped masks alone, in gradient i by
    e_fd[i].  The GPU's pre-activations differ from the float oracle's by delta_gpu (float accumulation over up to
    4,608 terms against one rounding of a double sum), so a fraction delta_gpu/delta_fd times larger flips and the
    gradient noise, which goes with the square root of that fraction, is sqrt(delta_gpu/delta_fd) * e_fd[i];
    the bound is three times that plus the float bar."""
    S = setup_step(rn, mode_name, *cfg, ls=ls)
    tol = TOL[mode_name] if tol is None else tol
    grad_tol = tol if grad_tol is None else grad_tol
    plan, table, master = S["plan"], S["table"], S["master"]
    vel = [np.zeros_like(p) for p in master]
    o = net.train_step(S["images"], S["labels"], master, S["model"], vel, table, widths=S["widths"],
                       blocks=S["blocks"], label_smoothing=ls)
    logits = torch.empty((S["N"], S["classes"]), device="cuda")
    loss = rn.resnet_step(plan, dev(S["images"], S["bf"]), dev(S["labels"]), S["M"], S["V"], S["G"], S["Mod"], 1.0,
                          S["ws"], update=True, logits_out=logits)
    torch.cuda.synchronize()
    assert abs(float(loss.item()) - o["loss"]) <= tol * abs(o["loss"]), (float(loss.item()), o["loss"])
    assert_close(logits, o["logits"], tol, "logits", elementwise=False)   # (end to end: many roundings deep)
    bounds = None
    if flip_bound:
        o64 = net.forward_backward(S["images"].astype(np.float64), S["labels"], [p.astype(np.float64) for p in S["model"]],
                                   S["widths"], S["blocks"], label_smoothing=ls)
        delta_fd = orc.rel_l2(o["logits"], o64["logits"])
        delta_gpu = orc.rel_l2(host(logits), o64["logits"])
        e_fd = [orc.rel_l2(a, b) for a, b in zip(o["grads"], o64["grads"])]
        scale = float(np.sqrt(max(delta_gpu / max(delta_fd, 1e-12), 1.0)))
        bounds = [3.0 * scale * e + tol for e in e_fd]
        print(f"flip bound: delta_fd {delta_fd:.2e}, delta_gpu {delta_gpu:.2e} (x{scale ** 2:.0f}), float-vs-double "
              f"gradient noise {min(e_fd):.1e} .. {max(e_fd):.1e}, bounds {min(bounds):.1e} .. {max(bounds):.1e}")
    worst = {}
    for i, (name, shape, kind) in enumerate(table):
        e = orc.rel_l2(host(plan.view(S["G"], i)), o["grads"][i])
        worst[name] = e
        if bounds is not None:
            grad_tol = bounds[i]
        assert e <= grad_tol, f"grad {name}: rel-L2 {e:.3e} > {grad_tol:.1e}"
        # w_new = w - v: an error of `tol` in the gradient moves w_new by at most tol*|v|/|w_new| (+ LARS rounding)
        dn = np.linalg.norm((o["w_new"][i].astype(np.float64) - master[i]).ravel())
        wn = np.linalg.norm(o["w_new"][i].astype(np.float64).ravel())
        assert_close(plan.view(S["M"], i), o["w_new"][i], 2 * grad_tol * dn / wn + TOL["lars"], name + " w_new")
    top = sorted(worst.items(), key=lambda kv: -kv[1])[:4]
    print(f"{mode_name} {cfg}: loss {float(loss.item()):.6f} vs {o['loss']:.6f}; worst grads:",
          ", ".join(f"{k} {v:.2e}" for k, v in top))


def run_step_vs_chain(rn, mode_name, *cfg, ls=0.0, loss_band=0.05):
    """resnet_step must be bitwise equal to the operation-by-operation chain, whose every operation
    is checked against the oracle on the same inputs, at the mode's bar (see step_chain.py)."""
    from step_chain import run_chain
    S = setup_step(rn, mode_name, *cfg, ls=ls)
    plan, table = S["plan"], S["table"]
    bf = S["bf"]
    img, lab = dev(S["images"], bf), dev(S["labels"])
    M0 = S["M"].clone()
    logits = torch.empty((S["N"], S["classes"]), device="cuda")
    loss = rn.resnet_step(plan, img, lab, S["M"], S["V"], S["G"], S["Mod"], 1.0, S["ws"], update=True,
                          logits_out=logits)
    model = [dev(p, bf) for p in S["model"]]
    vecs = [dev(p) for p in S["master"]]
    c_loss, c_logits, c_grads, ch = run_chain(rn, img, lab, model, vecs, S["blocks"], ls, TOL[mode_name])
    assert torch.equal(loss, c_loss) and torch.equal(logits, c_logits)
    for i, (name, _, _) in enumerate(table):
        assert torch.equal(plan.view(S["G"], i), c_grads[i]), f"grad {name} differs from the op-by-op chain"
    # LARS from the same gradients through the table form of the ABI: bitwise equal too, and at the
    # float LARS bar against the oracle given these gradients
    Wn = [plan.view(M0, i).clone() for i in range(len(table))]
    Vn = [torch.zeros_like(w) for w in Wn]
    wds = net.lars_hyper(table, 5e-5)
    rn.lars_update(rn.LarsTable(Wn, c_grads, Vn, wds), 0.001, 0.9, 1.0)
    w_o, v_o, _ = orc.lars_update(S["master"], [host(g) for g in c_grads], [np.zeros_like(p) for p in S["master"]],
                                  0.001, 0.9, 1.0, wds)
    for i, (name, _, _) in enumerate(table):
        assert torch.equal(plan.view(S["M"], i), Wn[i]) and torch.equal(plan.view(S["V"], i), Vn[i]), name
        assert_close(Wn[i], w_o[i], TOL["lars"], name + " w_new"); assert_close(Vn[i], v_o[i], TOL["lars"], name + " v_new")
        if bf:
            assert np.array_equal(host(plan.view(S["Mod"], i)), synth.round_bf16(host(Wn[i]))), name
    # end to end the oracle's loss is reproduced within a loose band only (chaotic amplification of bf16 rounding)
    vel = [np.zeros_like(p) for p in S["master"]]
    o = net.forward_backward(S["images"], S["labels"], S["model"], S["widths"], S["blocks"], label_smoothing=ls)
    le = abs(float(loss.item()) - o["loss"]) / abs(o["loss"])
    top = sorted(ch.worst.items(), key=lambda kv: -kv[1])[:5]
    print(f"{mode_name} {cfg}: loss {float(loss.item()):.5f} vs oracle {o['loss']:.5f} (rel {le:.2e}); end-to-end logits rel-L2 "
          f"{orc.rel_l2(host(logits), o['logits']):.2e}; {len(ch.worst)} per-op checks, worst:",
          ", ".join(f"{k} {v:.2e}" for k, v in top))
    assert le <= loss_band


def test_step_small_net_f32(rn):
    run_step_vs_oracle(rn, "f32", 4, 64, (8, 12, 16, 24), (2, 1, 2, 1), 8, 10)


def test_step_resnet50_f32_batch4_end_to_end(rn):
    """Full-depth ResNet-50 at 224x224 in float mode, end to end against the oracle: forward at the
    float bar, every gradient within the ReLU-flip bound computed from the measured pre-activation differences
    (see run_step_vs_oracle)."""
    run_step_vs_oracle(rn, "f32", 4, 224, (64, 128, 256, 512), (3, 4, 6, 3), 64, 1000, flip_bound=True)


def test_step_resnet50_f32_batch4_per_op(rn):
    run_step_vs_chain(rn, "f32", 4, 224, (64, 128, 256, 512), (3, 4, 6, 3), 64, 1000, loss_band=1e-4)


def test_step_shallow_net_bf16_end_to_end(rn):
    """A shallow net (one block per stage, 128x128 input): the forward pass stays within the bf16 bar
    end to end.  Gradients are not compared end to end in bf16: with pre-activations off by ~2e-3 the
    ReLU-flip bound is ~5% per layer and compounds (36% at the stem here); they are compared per
    operation, with identical masks, in the *_per_op / batch40 tests."""
    run_step_vs_oracle(rn, "bf16", 8, 128, (8, 16, 24, 32), (1, 1, 1, 1), 8, 16, ls=0.1, grad_tol=np.inf)


def test_step_small_net_bf16(rn):
    run_step_vs_chain(rn, "bf16", 4, 64, (8, 16, 24, 32), (2, 1, 2, 1), 8, 16, ls=0.1, loss_band=0.2)


@pytest.mark.parametrize("mode_name,loss_band", [("f32", 1e-4), ("bf16", 0.3)])
@pytest.mark.parametrize("hw", [33, 35, 38, 64])
def test_step_small_net_odd_images(rn, mode_name, loss_band, hw):
    """The stem's BN + ReLU + max-pool in one pass (two pooled rows per thread) at odd and even numbers of rows and columns before
    and after the pool, 17 / 18 / 19 / 32 -> 9 / 9 / 10 / 16: bitwise the separate operations, values and winners."""
    run_step_vs_chain(rn, mode_name, 3, hw, (8, 16, 24, 32), (1, 1, 1, 1), 8, 16, loss_band=loss_band)


def test_step_resnet50_batch40_bf16(rn):
    """BASELINE config 4: the full ResNet-50 v1.5 step at batch 40, mixed precision."""
    run_step_vs_chain(rn, "bf16", 40, 224, (64, 128, 256, 512), (3, 4, 6, 3), 64, 1000)


def test_step_resnet50_batch40_bf16_forward_end_to_end_against_bf16_storage_oracle(rn):
    """BASELINE config 4, end to end: the logits and the loss of resnet_step at batch 40 in bf16 mode against the
    oracle's operations composed with the activations rounded to bf16 at the points where the step stores them
    (tests/bf16_storage.py; every convolution output, every BN output, the pooled features).  Both sides make the
    same roundings; what is left is float-vs-double accumulation, which a network that re-rounds at every layer
    amplifies too (a value that rounds the other way is off by a whole bf16 step).  That floor is measured here, by
    jittering every stored tensor of the reference in the last bit of a float before its rounding, and the GPU path
    must be within 1.5 times it -- and clearly nearer to the bf16-storage reference than to the unrounded oracle,
    from which bf16 storage alone moves the logits by about 10 % (tests/test_oracle_bf16_storage.py)."""
    import bf16_storage
    S = setup_step(rn, "bf16", 40, 224, (64, 128, 256, 512), (3, 4, 6, 3), 64, 1000)
    plan = S["plan"]
    logits = torch.empty((S["N"], S["classes"]), device="cuda")
    loss = rn.resnet_step(plan, dev(S["images"], True), dev(S["labels"]), S["M"], S["V"], S["G"], S["Mod"], 1.0, S["ws"],
                          update=False, logits_out=logits)
    torch.cuda.synchronize()
    want = bf16_storage.forward(S["images"], S["model"], S["master"], S["blocks"], rounded=True)
    floor = orc.rel_l2(bf16_storage.forward(S["images"], S["model"], S["master"], S["blocks"], rounded=True, jitter=1e-7), want)
    exact = bf16_storage.forward(S["images"], S["model"], S["master"], S["blocks"], rounded=False)
    err, err_exact = orc.rel_l2(host(logits), want), orc.rel_l2(host(logits), exact)
    print("batch-40 bf16 logits: rel-L2 %.3e against the bf16-storage reference (floor from a 1e-7 jitter: %.3e), %.3e "
          "against the unrounded oracle (the reference itself is %.3e away from it)"
          % (err, floor, err_exact, orc.rel_l2(want, exact)))
    assert err <= 1.5 * floor + TOL["bf16"], (err, floor)
    assert err <= 0.75 * err_exact, (err, err_exact)
    lo = bf16_storage.loss_of(want, S["labels"])
    assert abs(float(loss.item()) - lo) <= 5e-3 * abs(lo), (float(loss.item()), lo)


def test_step_gradients_only_and_reproducible(rn):
    plan = rn.ResnetPlan(4, rn.BF16, 64, 16, (8, 16, 24, 32), (1, 1, 1, 1), 8, 4)
    table = net.param_table((8, 16, 24, 32), (1, 1, 1, 1), 8, 16, 3, 4)
    master = synth.params_from_table(SEED, table)
    M = torch.zeros(plan.arena_elems)
    for off, p in zip(plan.offsets, master):
        M[off:off + p.size] = torch.from_numpy(p.ravel())
    M = M.cuda(); Mod = M.to(torch.bfloat16); V = torch.zeros_like(M)
    img = dev(synth.activation_nhwc(SEED, "img", 4, 3, 64, 64), True)
    lab = dev(synth.labels(SEED, "lab", 4, 16))
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
    outs = []
    for _ in range(2):
        G = torch.zeros(plan.arena_elems, device="cuda")
        M0 = M.clone()
        loss = rn.resnet_step(plan, img, lab, M0, V, G, Mod, 1.0, ws, update=False)
        assert torch.equal(M0, M)                        # update=0: weights untouched
        outs.append((loss.clone(), G))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


def test_profile_hooks_and_plan_lifecycle(rn):
    """The launch-timing aid counts exactly the tagged launches of the steps it is enabled for (pause
    skips a step), and plans with their private streams can be created, used and destroyed in turn."""
    import gc
    for rep in range(2):
        N, hw, widths, blocks, stem, classes = 2, 32, (8, 8, 8, 8), (1, 2, 1, 1), 8, 10
        plan = rn.ResnetPlan(N, rn.BF16, hw, classes, widths, blocks, stem, 4)
        M = torch.randn(plan.arena_elems, device="cuda") * 0.1
        V = torch.zeros_like(M); G = torch.zeros_like(M); Mod = M.to(torch.bfloat16)
        ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
        img = torch.randn(N, hw, hw, 3, device="cuda").to(torch.bfloat16)
        lab = torch.zeros(N, dtype=torch.int32, device="cuda")
        step = lambda: rn.resnet_step(plan, img, lab, M, V, G, Mod, 0.1, ws)
        step()
        torch.cuda.synchronize()
        n_units = 1 + sum(blocks) * 3 + 4                       # stem, three per block, one projection per stage
        rn.profile_begin("conv_wgrad", 1000)
        step()
        rn.profile_pause(True)
        step()
        rn.profile_pause(False)
        step()
        torch.cuda.synchronize()
        ms = rn.profile_end()
        assert len(ms) == 2 * n_units                           # two timed steps, one weight gradient per unit
        assert all(0.0 < t < 50.0 for t in ms), ms
        # the timeline form: when every launch of one step began, after the first one, and how long it ran
        rn.profile_begin("", 4000)
        step()
        torch.cuda.synchronize()
        tl = rn.profile_end_timeline()
        tags = rn.profile_tags()
        assert len(tl) == len(tags) > 5 * n_units and tl[0][0] == 0.0
        assert all(at >= 0.0 and 0.0 < dur < 50.0 for at, dur in tl)
        assert {"conv_fwd", "conv_dgrad", "conv_wgrad", "bn_apply", "bn_bwd_apply", "lars_apply"} <= set(tags)
        assert max(at for at, _ in tl) > max(dur for _, dur in tl)      # the launches are spread over the step
        loss = step()
        torch.cuda.synchronize()
        assert np.isfinite(float(loss.item()))
        del plan
        gc.collect()


def test_step_on_a_caller_stream_matches_the_default_stream(rn):
    """resnet_step forks its private streams from whatever stream the caller passes and joins them back:
    the same step on a non-default stream, followed only by that stream's synchronization, gives the same bits."""
    N, hw, widths, blocks, stem, classes = 4, 64, (8, 16, 16, 24), (2, 1, 1, 1), 8, 10
    plan = rn.ResnetPlan(N, rn.BF16, hw, classes, widths, blocks, stem, 4)
    M0 = torch.randn(plan.arena_elems, device="cuda") * 0.1
    img = torch.randn(N, hw, hw, 3, device="cuda").to(torch.bfloat16)
    lab = torch.arange(N, dtype=torch.int32, device="cuda") % classes
    outs = []
    for use_stream in (False, True):
        M = M0.clone(); V = torch.zeros_like(M); G = torch.zeros_like(M); Mod = M.to(torch.bfloat16)
        ws = torch.full((plan.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
        loss = torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        if use_stream:
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                for _ in range(2):
                    rn.resnet_step(plan, img, lab, M, V, G, Mod, 0.1, ws, loss_out=loss)
            st.synchronize()
        else:
            for _ in range(2):
                rn.resnet_step(plan, img, lab, M, V, G, Mod, 0.1, ws, loss_out=loss)
            torch.cuda.current_stream().synchronize()
        outs.append((M.clone(), V.clone(), G.clone(), Mod.clone(), loss.clone()))
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    assert torch.isfinite(outs[0][2][: plan.sizes[0]]).all()


@pytest.mark.parametrize("mode", ["bf16", "f32"])
def test_step_with_conv3_input_fusion_gives_the_same_bits(rn, mode):
    """With conv3 applying conv2's BN+ReLU in its operand load (forward and weight gradient) the step's
    weights, momenta, gradients, loss and logits are bit for bit those of the step that stores conv2's
    normalised output: two blocks per stage, ragged widths, two steps in a row."""
    bf = mode == "bf16"
    N, hw, widths, blocks, stem, classes = 4, 64, (8, 16, 24, 40), (2, 1, 2, 1), 8, 10
    outs = []
    for fused in (False, True):
        plan = rn.ResnetPlan(N, rn.BF16 if bf else rn.F32, hw, classes, widths, blocks, stem, 4)
        plan.fuse_conv3_input(fused)
        table = net.param_table(widths, blocks, stem, classes, 3, 4)
        M = torch.zeros(plan.arena_elems)
        for off, p in zip(plan.offsets, synth.params_from_table(SEED, table)):
            M[off:off + p.size] = torch.from_numpy(p.ravel())
        M = M.cuda(); V = torch.zeros_like(M); G = torch.zeros_like(M); Mod = M.to(torch.bfloat16) if bf else M
        img = dev(synth.activation_nhwc(SEED, "img", N, 3, hw, hw), bf)
        lab = dev(synth.labels(SEED, "lab", N, classes))
        ws = torch.full((plan.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
        loss = torch.zeros(1, device="cuda"); logits = torch.zeros(N, classes, device="cuda")
        for _ in range(2):
            rn.resnet_step(plan, img, lab, M, V, G, Mod, 0.5, ws, loss_out=loss, logits_out=logits)
        torch.cuda.synchronize()
        outs.append((M.clone(), V.clone(), G.clone(), Mod.clone(), loss.clone(), logits.clone()))
    for name, a, b in zip(("master", "velocity", "grads", "model", "loss", "logits"), *outs):
        assert torch.equal(a, b), name
    assert torch.isfinite(outs[0][2]).all()


@pytest.mark.parametrize("mode,N", [("bf16", 6), ("f32", 4), ("bf16", 90)])
def test_step_computes_the_same_statistics_whoever_computes_them(rn, mode, N):
    """Apply passes whose launch also finalizes (the 56x56 layers here): a workgroup that never asks for another one's results
    computes them itself, to the same bits; weights, statistics and loss of two training steps.  At batch 90 the apply passes have up to
    16,384 workgroups, of which 1024 run at a time, and the 56x56 layer on 64x64 tiles has 4410 rows of sums, which its producer adds up to 64 rows of
    doubles first (more than 4096)."""
    bf = mode == "bf16"
    out = []
    for polls in (2000, 0):
        plan = rn.ResnetPlan(N, rn.BF16 if bf else rn.F32)
        assert rn.raw.rn50_internal_wait_polls(plan.handle, polls) == 0
        M = torch.empty(plan.arena_elems, device="cuda"); V = torch.empty_like(M); G = torch.zeros_like(M)
        rn.resnet_init_params(plan, SEED, M, V)
        Mod = M.to(torch.bfloat16) if bf else M
        gen = torch.Generator(device="cuda").manual_seed(1)
        img = torch.randn(N, 224, 224, 3, device="cuda", generator=gen).to(Mod.dtype)
        lab = torch.randint(0, 1000, (N,), device="cuda", generator=gen, dtype=torch.int32)
        ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
        state = rn.TrainState(plan)
        for _ in range(2):
            loss = rn.resnet_train_step(plan, rn.LrSchedule(base_lr=0.1), state, img, lab, M, V, G, Mod, ws)
        out.append([loss.clone(), M, V, G] + [t.clone() for t in state.running_mean + state.running_var])
    for a, b in zip(*out):
        assert torch.equal(a, b)


def test_step_resnet50_batch256_bf16_equals_the_chain(rn):
    """The large-batch configuration (batch 256, 6.4 times the measured one: tensors of up to 411 MB, tens
    of thousands of output tiles): resnet_step is bit for bit the operation-by-operation chain, whose
    operations are held to the oracle at batch 40 and below and, here, at batch 256 for a third of the network; the loss of the untrained network is near
    ln(1000) and every gradient is finite and non-zero."""
    from step_chain import run_chain
    cfg = (256, 224, (64, 128, 256, 512), (3, 4, 6, 3), 64, 1000)
    S = setup_step(rn, "bf16", *cfg)
    plan, table = S["plan"], S["table"]
    img, lab = dev(S["images"], True), dev(S["labels"])
    logits = torch.empty((S["N"], S["classes"]), device="cuda")
    loss = rn.resnet_step(plan, img, lab, S["M"], S["V"], S["G"], S["Mod"], 1.0, S["ws"], update=False, logits_out=logits)
    torch.cuda.synchronize()
    assert abs(float(loss.item()) - np.log(1000.0)) < 1.0, float(loss.item())
    model = [dev(p, True) for p in S["model"]]
    vecs = [dev(p) for p in S["master"]]
    # ... and at this size the operations of the stem, of the first block of every stage, of the last block and of
    # the head are compared with the oracle on the chain's own inputs (rel-L2 and every element), as at batch 40
    checked = ("stem", "s0b0", "s1b0", "s2b0", "s3b0", "s3b2", "head")
    c_loss, c_logits, c_grads, ch = run_chain(rn, img, lab, model, vecs, S["blocks"], 0.0, TOL["bf16"], check=checked)
    assert len(ch.worst) >= 100, len(ch.worst)
    top = sorted(ch.worst.items(), key=lambda kv: -kv[1])[:4]
    print("batch 256: %d per-op checks against the oracle, worst rel-L2: %s; worst element excess %.2f"
          % (len(ch.worst), ", ".join(f"{k} {v:.2e}" for k, v in top), max(ch.worst_elem.values())))
    assert torch.equal(loss, c_loss) and torch.equal(logits, c_logits)
    for i, (name, _, _) in enumerate(table):
        g = plan.view(S["G"], i)
        assert torch.equal(g, c_grads[i]), f"grad {name} differs from the op-by-op chain"
        assert torch.isfinite(g).all() and float(g.abs().max()) > 0, name
