"""GPU parity: the HIP library (through its C ABI) against the CPU fp64 oracle, element by element, on the
same seeded inputs.

Tolerances (stated by the benchmark spec): activations and loss within 1e-4, gradients and weights after 10 steps
within 1e-3, as max|gpu - ref| / max|ref| per tensor; the loss as a relative difference.

Sub-gradient choices.  ReLU and max-pool are kinks: an element whose pre-activation is closer to zero than
fp32 can resolve (a few 1e-6 after a K=500..4600 accumulation) may fall on either side, and with only
512..32768 elements per channel one such element moves that channel's gradient by 1/sqrt(count), far more
than 1e-3.  Both outcomes are correct gradients of the same continuous loss.  So the forward quantities are
compared directly, and for the backward pass the oracle is told which side the GPU took for every element
(rebuilt here bit for bit from the z, scale and shift tensors the library exposes: the kernels decide on
b = fmaf(z, scale, shift)); the oracle verifies that every choice differing from its own lies within 1e-4
of max|b| -- the activation tolerance -- and refuses anything else, then differentiates with those choices.
The tests bound what that lets through far below that margin: at most max(4, 4e-6 of all decisions) may differ
(none at all on the small blocks), and the farthest differing element must lie within 1e-5 of max|b| of the
kink, so a kernel whose b were off systematically would fail here long before the oracle's own margin.
Where 4e-6 comes from: an fp32 accumulation over K terms leaves z with a relative error of about sqrt(K) * 2^-24
(1.4e-6 for the 512-channel pointwise layers, K = 512 + 9), and over ten steps the two sides' weights drift apart
by a few 1e-6 relative, which moves b by as much; b is close to standard normal, so it lies within +-e of zero
with probability 0.8 e: up to about 0.8 * (1.4e-6 + 3e-6) = 3.5e-6 of the decisions.  Measured: at most 2.0e-6
(the 2x2x512 block of the five-block schedule after ten steps; 7e-8 on the 16x16 block), farthest 2.7e-6 of max|b|.
"""
from dataclasses import replace

import numpy as np
import pytest

from oracle import block as ob
from paper_2012_03096_amd import workloads as wl

pytestmark = pytest.mark.gpu

ACT_TOL = 1e-4
GRAD_TOL = 1e-3


def relerr(got, ref):
    ref = np.asarray(ref, dtype=np.float64)
    got = np.asarray(got, dtype=np.float64)
    assert got.shape == ref.shape, (got.shape, ref.shape)
    if not np.all(np.isfinite(got)):
        return float("inf")
    d = np.abs(got - ref).max() if ref.size else 0.0
    return float(d / max(np.abs(ref).max(), 1e-30)) if ref.size else 0.0


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2012_03096_amd import binding
    binding.lib()
    return torch, binding


def _ref_block(w, tp, sp, **kw):
    return ob.RefBlock(w.teacher, tp, w.student, sp, momentum=w.momentum, **kw)


def _layer_act_shapes(arch):
    res = []
    for (ci, hi, wi, co, ho, wo), L in zip(wl.layer_shapes(arch), arch.layers):
        res.append(((arch.n, ci, ho, wo), (arch.n, co, ho, wo), L.kind))
    return res


def gpu_decisions(pb, blk, arch, x=None):
    """ReLU masks per layer and pool argmax as the GPU took them in its last student forward.
    x: the block input (fp32), needed when the block has an identity skip."""
    relu = []
    nl = len(arch.layers)
    b = None
    for l, (ushape, zshape, kind) in enumerate(_layer_act_shapes(arch)):
        c = zshape[1]

        def bn(layer):
            z = blk.get_tensor(pb.STUDENT_ACT, layer, 1, zshape).astype(np.float64)
            sc = blk.get_tensor(pb.STUDENT_ACT, layer, 4, (c,)).astype(np.float64)[None, :, None, None]
            sh = blk.get_tensor(pb.STUDENT_ACT, layer, 5, (c,)).astype(np.float64)[None, :, None, None]
            return (z * sc + sh).astype(np.float32)      # product exact in fp64: the sign is fmaf's sign

        b = bn(l)
        if l == nl - 1 and arch.shortcut == 1:
            b = b + bn(nl)                                # fp32 add, as in the kernel
        elif l == nl - 1 and arch.shortcut == 2:
            b = b + x.astype(np.float32)                  # identity skip: fmaf(x, 1, 0) = x, then the fp32 add
        relu.append(b > 0)
    pool_arg = None
    if arch.pool == 2:
        y = np.maximum(b, np.float32(0))
        N, C, H, W = y.shape
        Hp, Wp = H // 2, W // 2
        win = y[:, :, :2 * Hp, :2 * Wp].reshape(N, C, Hp, 2, Wp, 2).transpose(0, 1, 2, 4, 3, 5).reshape(N, C, Hp, Wp, 4)
        pool_arg = np.argmax(win, axis=-1)                # first maximum, like the kernel's strict '>'
    return {"relu": relu, "pool_arg": pool_arg}


DECISION_LOG = []
BN_DECAY = float(np.float32(0.9))
DIFFERING_FRACTION = 4e-6      # of all ReLU / pool decisions of a run may be taken differently from the oracle's own
DIFFERING_FLOOR = 4
DIFFERING_WORST_REL = 1e-5     # and each of those lies this close to the kink, as a fraction of max|b|


class DecisionTally:
    """Sums, over the steps of one run, what the oracle reports about the decisions it was handed."""

    def __init__(self):
        self.total = self.differing = 0
        self.worst_rel = 0.0

    def add(self, cache):
        self.total += cache["decisions_total"]
        self.differing += cache["decisions_differing"]
        self.worst_rel = max(self.worst_rel, cache["decisions_worst_rel"])

    def failures(self, none_allowed=False):
        out = {}
        allowed = 0 if none_allowed else max(DIFFERING_FLOOR, int(DIFFERING_FRACTION * self.total))
        if self.differing > allowed:
            out["decisions.differing"] = (self.differing, self.total, allowed)
        if self.worst_rel > DIFFERING_WORST_REL:
            out["decisions.worst_rel"] = self.worst_rel
        return out


def run_parity(gpu, w, steps, random_affine=True, loss_reduction=0, check_intermediates=True, x_override=None,
               no_differing_decisions=False):
    """Runs teacher forward + `steps` student steps on both sides and returns a dict of failures."""
    torch, pb = gpu
    x, tp, sp = w.tensors(random_affine=random_affine)
    if x_override is not None:
        x = x_override
    # a short memory for the running statistics, so that ten steps outweigh their starting values
    ref = _ref_block(w, tp, sp, loss_reduction=loss_reduction, bn_decay=BN_DECAY)
    blk = pb.Block(w.teacher, tp, w.student, sp, momentum=w.momentum, loss_reduction=loss_reduction, bn_decay=BN_DECAY)
    fails = {}

    def check(name, got, want, tol):
        e = relerr(got, want)
        if not e <= tol:
            fails[name] = e

    xd = torch.from_numpy(x).cuda()
    td = torch.empty(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda")
    t_ref, tcache = ob.block_forward(w.teacher, ref.tp, x, keep=True)
    blk.teacher_forward(xd, td)
    torch.cuda.synchronize()
    if check_intermediates:
        for l, (ushape, zshape, kind) in enumerate(_layer_act_shapes(w.teacher)):
            rec = tcache["layers"][l]
            check(f"teacher.z{l}", blk.get_tensor(pb.TEACHER_ACT, l, 1, zshape), rec["z"], ACT_TOL)
            check(f"teacher.mean{l}", blk.get_tensor(pb.TEACHER_ACT, l, 2, (zshape[1],)), rec["mean"], ACT_TOL)
            check(f"teacher.rstd{l}", blk.get_tensor(pb.TEACHER_ACT, l, 3, (zshape[1],)), rec["rstd"], ACT_TOL)
        if w.teacher.shortcut == 1:
            nl = len(w.teacher.layers)
            zs = tcache["layers"][-1]["zs"]
            check("teacher.zs", blk.get_tensor(pb.TEACHER_ACT, nl, 1, zs.shape), zs, ACT_TOL)
    check("teacher.target", td.cpu().numpy(), t_ref, ACT_TOL)

    # the student trains against the oracle's target rounded to fp32 on both sides, so that a teacher
    # discrepancy does not leak into the student comparison
    t32 = t_ref.astype(np.float32)
    td.copy_(torch.from_numpy(t32))
    out = torch.empty_like(td)
    blk.student_forward(xd, out)
    torch.cuda.synchronize()
    check("student.forward_out", out.cpu().numpy(), ref.student_forward(x), ACT_TOL)

    tally = DecisionTally()
    for step in range(steps):
        l_gpu = blk.student_step(xd, td, w.lr)
        l_ref = ref.student_step(x, t32, w.lr, decisions=gpu_decisions(pb, blk, w.student, x))
        tally.add(ref.cache)
        e = abs(l_gpu - l_ref) / max(abs(l_ref), 1e-30)
        if not e <= ACT_TOL:
            fails[f"loss[{step}]"] = (e, l_gpu, l_ref)
        if step == 0:
            assert abs(blk.last_loss() - l_gpu) == 0.0
            if check_intermediates:
                for l, (ushape, zshape, kind) in enumerate(_layer_act_shapes(w.student)):
                    rec = ref.cache["layers"][l]
                    if kind == wl.DWSEP3X3:
                        check(f"student.u{l}", blk.get_tensor(pb.STUDENT_ACT, l, 0, ushape), rec["u"], ACT_TOL)
                    check(f"student.z{l}", blk.get_tensor(pb.STUDENT_ACT, l, 1, zshape), rec["z"], ACT_TOL)
                    check(f"student.mean{l}", blk.get_tensor(pb.STUDENT_ACT, l, 2, (zshape[1],)), rec["mean"], ACT_TOL)
                    check(f"student.rstd{l}", blk.get_tensor(pb.STUDENT_ACT, l, 3, (zshape[1],)), rec["rstd"], ACT_TOL)
            grads = blk.student_grads()
            for l, L in enumerate(w.student.layers):
                if not L.trainable:
                    continue
                for k, (g_gpu, g_ref) in enumerate(zip(grads[l], ref.grads[l])):
                    check(f"grad[{l}][{k}]", g_gpu, g_ref, GRAD_TOL)
    params = blk.student_params()
    for l, (lp, lr_) in enumerate(zip(params, ref.sp)):
        for k, (a, b) in enumerate(zip(lp, lr_)):
            check(f"weights_after_{steps}[{l}][{k}]", a, b, GRAD_TOL)
    # running statistics: moved once per student step (not by the plain forward passes above), the teacher's never
    for l, (rm, rv) in enumerate(ref.s_running):
        c = rm.shape
        check(f"running_mean_after_{steps}[{l}]", blk.get_tensor(pb.STUDENT_BN_RUNNING, l, 0, c), rm, ACT_TOL)
        check(f"running_var_after_{steps}[{l}]", blk.get_tensor(pb.STUDENT_BN_RUNNING, l, 1, c), rv, ACT_TOL)
    for l, (rm, rv) in enumerate(ref.t_running):
        if not (np.all(blk.get_tensor(pb.TEACHER_BN_RUNNING, l, 0, rm.shape) == 0) and
                np.all(blk.get_tensor(pb.TEACHER_BN_RUNNING, l, 1, rm.shape) == 1)):
            fails[f"teacher_running[{l}]"] = "moved"
    blk.close()
    fails.update(tally.failures(none_allowed=no_differing_decisions))
    DECISION_LOG.append((w.name, steps, tally.differing, tally.total, tally.worst_rel))
    print(f"[parity] {w.name}: {steps} steps, {tally.differing} of {tally.total} decisions taken differently, "
          f"farthest from the kink {tally.worst_rel:.2e} of max|b|", flush=True)
    return fails


def test_cfg1_tiny_block_ten_steps(gpu):
    fails = run_parity(gpu, wl.cfg1_tiny(), steps=10, random_affine=False, no_differing_decisions=True)
    assert not fails, fails


@pytest.mark.parametrize("name", [w.name for w in wl.small_variants()])
def test_small_ragged_variants_ten_steps(gpu, name):
    w = {v.name: v for v in wl.small_variants()}[name]
    fails = run_parity(gpu, w, steps=10, no_differing_decisions=True)
    assert not fails, fails


@pytest.mark.parametrize("name", [w.name for w in wl.degenerate_variants()])
def test_degenerate_shapes_three_steps(gpu, name):
    """1x1 maps, single rows and columns, two channels, one image, pools and strides that end in one pixel."""
    w = {v.name: v for v in wl.degenerate_variants()}[name]
    fails = run_parity(gpu, w, steps=3, no_differing_decisions=True)
    assert not fails, fails


@pytest.mark.parametrize("fused", [1, 0])
@pytest.mark.parametrize("name", [w.name for w in wl.fused_forward_variants()])
def test_fused_depthwise_pointwise_forward(gpu, monkeypatch, name, fused):
    """The one-kernel depthwise + pointwise forward (PBKD_DWPW=1 takes it wherever the shape allows, 0 never) on small
    blocks ragged in batch and channels; depthwise outputs, pre-BatchNorm outputs, statistics, loss, gradients, weights."""
    monkeypatch.setenv("PBKD_DWPW", str(fused))
    w = {v.name: v for v in wl.fused_forward_variants()}[name]
    fails = run_parity(gpu, w, steps=5, no_differing_decisions=True)
    assert not fails, fails


def test_eq3_loss_reduction(gpu):
    w = wl.small_variants()[0]
    fails = run_parity(gpu, w, steps=3, loss_reduction=1)
    assert not fails, fails


def test_cfg2_vgg_block2_full_size(gpu):
    fails = run_parity(gpu, wl.cfg2_vgg_block2(), steps=10, random_affine=False)
    assert not fails, fails


def test_cfg3_resnet_down_full_size(gpu):
    fails = run_parity(gpu, wl.cfg3_resnet_down(), steps=10, random_affine=False)
    assert not fails, fails


def test_cfg4_imagenet_block_batch4_ten_steps(gpu):
    fails = run_parity(gpu, wl.cfg4_imagenet_vgg_block1(n=4), steps=10, random_affine=False)
    assert not fails, fails


def test_cfg4_imagenet_block_full_size_one_step(gpu):
    fails = run_parity(gpu, wl.cfg4_imagenet_vgg_block1(), steps=1, random_affine=False)
    assert not fails, fails


@pytest.mark.parametrize("k", range(13))
def test_paper_granularity_tasks(gpu, k):
    """Each of the thirteen per-convolution VGG16 tasks (one conv teacher, two DS layers student; section 4.4), batch 16."""
    tasks = wl.paper_granularity_vgg16_tasks(n=16)
    assert len(tasks) == 13
    fails = run_parity(gpu, tasks[k], steps=3)
    assert not fails, (tasks[k].name, fails)


def test_cfg4_shape_with_four_row_depthwise_strips_three_steps(gpu):
    """The ImageNet-shaped block at batch 11: the smallest batch at which the depthwise kernels take four rows per
    thread (N * H/4 * W/4 >= 32768 strips per channel), over several steps."""
    w = wl.cfg4_imagenet_vgg_block1(n=11)
    assert w.teacher.n * (w.teacher.h // 4) * (w.teacher.w // 4) >= 32768
    fails = run_parity(gpu, w, steps=3, random_affine=True)
    assert not fails, fails


@pytest.mark.parametrize("name", ["cfg2_batch16", "ragged_pool", "ragged_residual_s2", "fullconv_first"])
def test_large_mean_channels(gpu, name):
    """Block input 30 + N(0,1) instead of a post-ReLU map: every pre-BatchNorm channel of the first layers then has
    |mean| of the order of 30 standard deviations, where a one-pass variance E[z^2] - mean^2 loses (mean/sigma)^2 ~ 1e3
    times the rounding error of its sums.  The statistics, activations, loss and gradients must still meet the bounds."""
    w = wl.cfg2_vgg_block2(n=16) if name == "cfg2_batch16" else {v.name: v for v in wl.small_variants()}[name]
    rng = np.random.default_rng(30)
    x = (30.0 + rng.standard_normal((w.teacher.n, w.teacher.c, w.teacher.h, w.teacher.w))).astype(np.float32)
    fails = run_parity(gpu, w, steps=3, x_override=x)
    assert not fails, fails


@pytest.mark.parametrize("n,h,w_,value", [(16, 14, 14, 3.5), (32, 7, 7, 3.75), (10, 14, 21, 3.5), (4, 49, 8, 3.25)])
def test_statistics_are_sums_divided_by_the_count(gpu, n, h, w_, value):
    """A channel's mean is the rounded quotient of its sum and its count, not a product with the count's rounded reciprocal.  Half of
    the images are zero, half `value`, and one pixel of the first puts the mean halfway between two fp32 numbers: every sum is exact,
    so the quotient is, and goes to the even number; for half of the channels the product falls below it (counts 49 * 2^k and 2940)."""
    torch, pb = gpu
    c, count = 64, n * h * w_
    t, s = wl.Arch(n, c, h, w_, wl._convs([c, c])), wl.Arch(n, c, h, w_, wl._dws([c, c]))
    x, tp, sp = wl.Workload("means", t, s, seed=3).tensors(random_affine=True)
    sp = [[a.copy() for a in lp] for lp in sp]
    sp[0][0].reshape(c, 9)[:] = np.eye(9)[4]                # z = x
    sp[0][1].reshape(c, c)[:] = np.eye(c)
    odd = 2.0 * np.arange(c) + 1
    x = np.zeros_like(x)
    x[n // 2:] = value
    x[0, :, h // 2, w_ // 2] = count * odd * 2.0 ** -24
    blk = pb.Block(t, tp, s, sp)
    blk.student_forward(torch.from_numpy(x).cuda(), torch.empty((n, c, h, w_), device="cuda"))
    got = blk.get_tensor(pb.STUDENT_ACT, 0, 2, (c,))
    blk.close()
    want = value / 2 + odd * 2.0 ** -24
    assert (want.astype(np.float32) != ((count * want) * (1.0 / count)).astype(np.float32)).sum() == c // 2
    np.testing.assert_array_equal(got, want.astype(np.float32))


def test_sums_over_a_wave_have_one_order(gpu):
    """The fp64 sum over a wave adds lanes 32, 16, 8, 4, 2 and 1 apart, in that order: the feature error of 65536 numbers (256
    workgroups of 256 threads, one number a thread, then one workgroup over their sums) to the last bit."""
    torch, pb = gpu

    def group(v):                                           # [..., 256] -> [...]
        v = v.reshape(*v.shape[:-1], 4, 64)
        while v.shape[-1] > 1:
            v = v[..., :v.shape[-1] // 2] + v[..., v.shape[-1] // 2:]
        v = v[..., 0]
        return (v[..., 0] + v[..., 1]) + (v[..., 2] + v[..., 3])

    rng = np.random.default_rng(8)
    for _ in range(8):
        a, b = rng.standard_normal((2, 65536)).astype(np.float32)
        d = a.astype(np.float64) - b.astype(np.float64)
        want = group(group((d * d).reshape(256, 256))) * (1.0 / 65536)
        assert pb.feature_mse_noalloc(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()) == want


FORCED = ([("PBKD_PW_VARIANT", v) for v in range(10)] + [("PBKD_CONV_TILE", v) for v in range(4)] +
          [("PBKD_WGRAD_VARIANT", v) for v in range(4)] + [("PBKD_CONV_KSPLIT", v) for v in (2, 3)])


@pytest.mark.parametrize("var,value", FORCED, ids=[f"{k[5:].lower()}{v}" for k, v in FORCED])
def test_every_tile_variant_on_ragged_blocks(gpu, monkeypatch, var, value):
    """The library picks tile shapes and kernel variants from the layer's shape; the benchmark shapes reach only some of
    them.  Its tuning overrides (read when a block is created) force each one in turn onto small blocks whose sizes are
    multiples of no tile: odd channel counts, 2x2 to 12x12 maps, pixel counts that leave ragged tails."""
    monkeypatch.setenv(var, str(value))
    by_name = {v.name: v for v in wl.small_variants()}
    for name in ("ragged_pool", "three_layers_oddc", "paper_task_2x2", "fullconv_first", "ragged_residual_s2"):
        fails = run_parity(gpu, by_name[name], steps=2, check_intermediates=(name == "three_layers_oddc"))
        assert not fails, (var, value, name, fails)


def pointwise_split_blocks():
    """Blocks for the 1x1 kernels that form fp32 products from bf16 pieces (at least 16 input channels): chunks of 16
    channels that end ragged (17, 20, 33 channels) or whole (16, 64), channel tiles of one and several blocks of 32 with
    ragged last ones, pixel counts that leave tails for one, two and four pixels a lane, a strided shortcut, more than one
    stage of 128 input channels."""
    by_name = {v.name: v for v in wl.small_variants()}
    t = wl.Arch(3, 19, 9, 11, wl._convs([19, 37, 37], stride0=2), shortcut=1, shortcut_stride=2)
    s = wl.Arch(3, 19, 9, 11, wl._dws([19, 37, 37], stride0=2), shortcut=1, shortcut_stride=2)
    res = wl.Workload("residual_19ch", t, s, seed=51, copy_shortcut=True)
    t = wl.Arch(3, 64, 8, 12, wl._convs([64, 145]))
    s = wl.Arch(3, 64, 8, 12, wl._dws([64, 270, 145]))
    return [by_name["three_layers_oddc"], by_name["paper_task_2x2"], wl.cfg1_tiny(), res, wl.Workload("wide_270ch", t, s, seed=52)]


@pytest.mark.parametrize("variant", range(10, 16))
def test_pointwise_split_variants_on_ragged_blocks(gpu, monkeypatch, variant):
    """Every tile of the split 1x1 kernels, forced onto ragged blocks: forward, data gradient and the weights that the
    update kernel re-packs for them, against the oracle."""
    monkeypatch.setenv("PBKD_PW_VARIANT", str(variant))
    for w in pointwise_split_blocks():
        fails = run_parity(gpu, w, steps=3)
        assert not fails, (variant, w.name, fails)


def test_pointwise_split_is_as_accurate_as_fp32(gpu, monkeypatch):
    """The six bf16 products of three-way split operands leave out at most 2^-24 of each product, so against the fp64 oracle
    the split 1x1 kernels must not be worse than the fp32 MFMA one by more than rounding noise: z of two layers (K = 512
    and 260, many-pixel and K-over-waves tiles)."""
    t = wl.Arch(6, 512, 8, 8, wl._convs([512, 96]))
    s = wl.Arch(6, 512, 8, 8, wl._dws([512, 260, 96]))
    w = wl.Workload("pointwise_accuracy", t, s, seed=53)
    torch, pb = gpu
    x, tp, sp = w.tensors(random_affine=True)
    ref = _ref_block(w, tp, sp)
    t_ref = ref.teacher_forward(x)
    ref.student_step(x, t_ref, w.lr)
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(t_ref.astype(np.float32)).cuda()
    errs = {}
    for variant in (3, 10, 14):
        monkeypatch.setenv("PBKD_PW_VARIANT", str(variant))
        blk = pb.Block(w.teacher, tp, w.student, sp)
        blk.student_step(xd, td, w.lr)
        zs = [blk.get_tensor(pb.STUDENT_ACT, l, 1, shp) for l, (_, shp, _) in enumerate(_layer_act_shapes(w.student))]
        errs[variant] = [relerr(z, r["z"]) for z, r in zip(zs, ref.cache["layers"])]
        blk.close()
    print("[pointwise accuracy] max|err|/max|ref| of z0, z1:", errs)
    for variant in (10, 14):
        for a, b in zip(errs[3], errs[variant]):
            assert b <= 2.0 * a + 2e-7, errs


def fp32_matrix_product(P, u, parts):
    """P @ u as the fp32 matrix instructions sum it, a fused multiply-add per product (the kernels that used them measured
    1.97e-7 and 2.0e-7 against fp64 at K = 433 and 512 in four parts, which this gives); K in `parts` contiguous parts,
    added in order."""
    k = P.shape[1]
    step = -(-k // parts)
    total = None
    for k0 in range(0, k, step):
        acc = np.zeros((P.shape[0], u.shape[1]), dtype=np.float32)
        for i in range(k0, min(k, k0 + step)):
            acc = (acc + np.multiply.outer(P[:, i].astype(np.float64), u[i].astype(np.float64))).astype(np.float32)
        total = acc if total is None else total + acc
    return total


@pytest.mark.parametrize("n,h,w_,ci,co,parts", [(7, 41, 48, 433, 169, 4), (21, 14, 14, 512, 512, 4), (16, 4, 4, 512, 512, 4), (33, 16, 16, 128, 130, 1),
                                                (8, 27, 23, 67, 100, 1), (4, 13, 11, 16, 24, 1), (20, 41, 48, 64, 33, 1), (130, 32, 32, 160, 64, 1),
                                                (32, 32, 34, 128, 24, 4), (8, 17, 40, 128, 328, 4), (33, 32, 34, 180, 32, 4)])
def test_pointwise_split_leaves_no_larger_error_than_fp32_products(gpu, n, h, w_, ci, co, parts):
    """rms error of the 1x1 kernel the library chooses, against fp64 on its own input, for 400 of its
    pixels: not larger than that of fp32 multiply-adds summed in `parts` parts (4: as the fp32 kernels did with long sums
    over few pixels)."""
    torch, pb = gpu
    t, s = wl.Arch(n, ci, h, w_, wl._convs([ci, co])), wl.Arch(n, ci, h, w_, wl._dws([ci, co]))
    x, tp, sp = wl.Workload("pointwise_error", t, s, seed=31).tensors(random_affine=True)
    blk = pb.Block(t, tp, s, sp)
    td = torch.zeros(wl.output_shape(t), dtype=torch.float32, device="cuda")
    blk.student_step(torch.from_numpy(x).cuda(), td, 0.0, want_loss=False)
    u = blk.get_tensor(pb.STUDENT_ACT, 0, 0, (n, ci, h, w_)).transpose(1, 0, 2, 3).reshape(ci, -1)
    z = blk.get_tensor(pb.STUDENT_ACT, 0, 1, (n, co, h, w_)).transpose(1, 0, 2, 3).reshape(co, -1)
    blk.close()
    some = np.unique(np.linspace(0, u.shape[1] - 1, 400).astype(int))
    P, u, z = sp[0][1].reshape(co, ci), u[:, some], z[:, some]
    ref = P.astype(np.float64) @ u.astype(np.float64)
    got, fp32 = rms_error(z, ref), rms_error(fp32_matrix_product(P, u, parts), ref)
    print(f"[pointwise error] {ci}->{co} {h}x{w_}x{n}: rms {got:.3e}, fp32 products {fp32:.3e}")
    assert got <= 1.02 * fp32


def value_classes(a):
    """0 for numbers, 1 and -1 for infinities, 2 for NaN."""
    return np.where(np.isnan(a), 2, np.where(np.isinf(a), np.sign(a), 0)).astype(int)


def same_nonfinite(got, want, what):
    """The same elements are infinite or NaN, and the others agree (each to the scale of its channel: some are past 1e36)."""
    g, w = value_classes(got), value_classes(want)
    assert (g == w).all(), (what, int((g != w).sum()), "differ, first", got[g != w][0], want[g != w][0])
    with np.errstate(all="ignore"):
        ok = np.isfinite(want)
        scale = np.max(np.where(ok, np.abs(want.astype(np.float64)), 0), axis=(0, 2, 3), keepdims=True)
        err = np.where(ok, np.abs(got.astype(np.float64) - want), 0) / np.maximum(scale, 1e-30)
    assert err.max() <= ACT_TOL, (what, err.max())


@pytest.mark.parametrize("variant", [-1] + list(range(10, 16)))
@pytest.mark.parametrize("n,h,w_,chans,stride", [(2, 6, 8, (20, 33, 40), 1), (40, 32, 32, (24, 70, 17), 1), (3, 9, 7, (130, 65, 30), 2)])
def test_pointwise_split_infinities(gpu, monkeypatch, n, h, w_, chans, stride, variant):
    """Infinities, NaNs and numbers past bfloat16's largest in the activations and the weights of 1x1 convolutions (pointwise and
    strided shortcut): every output is the number, infinity or NaN that plain products of the kernel's own input make,
    with the batch's and with running statistics."""
    torch, pb = gpu
    rng = np.random.default_rng(7)
    t = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans), stride0=stride), shortcut=1, shortcut_stride=stride)
    s = wl.Arch(n, chans[0], h, w_, wl._dws(list(chans), stride0=stride), shortcut=1, shortcut_stride=stride)
    x, tp, sp = wl.Workload("infinities", t, s, seed=41, copy_shortcut=True).tensors(random_affine=True)
    x = x.copy()
    for v in (np.inf, -np.inf, np.nan, 3.4e38):
        x[rng.integers(n), rng.integers(chans[0]), rng.integers(h), rng.integers(w_)] = v
    x[-1, -1, -1, -1] = np.inf
    for l in range(2):                     # (depthwise outputs of a few hundredths: 3.4e38 times them stays a number)
        sp[l][0] = sp[l][0] * np.float32(1e-2)
        sp[l][1] = sp[l][1].copy()
        sp[l][1][3, 1], sp[l][1][5, 2] = np.inf, -3.4e38
    if variant >= 0:
        monkeypatch.setenv("PBKD_PW_VARIANT", str(variant))
    blk = pb.Block(t, tp, s, sp)
    xd = torch.from_numpy(x).cuda()
    out = torch.empty(wl.output_shape(s), dtype=torch.float32, device="cuda")
    shapes = _layer_act_shapes(s)
    for mode in (0, 1):
        pb.network_forward([blk], [1], xd, [out], bn_mode=mode)
        torch.cuda.synchronize()
        for l in range(2 if stride == 2 and variant in (12, 13) else 3):     # (those tiles take no strided shortcut)
            if l < 2:
                u, P = blk.get_tensor(pb.STUDENT_ACT, l, 0, shapes[l][0]), sp[l][1]
            else:
                u, P = x[:, :, ::stride, ::stride], sp[2][0]
            co, ci = P.shape[:2]
            with np.errstate(all="ignore"):
                want = P.reshape(co, ci).astype(np.float64) @ u.astype(np.float64).transpose(1, 0, 2, 3).reshape(ci, -1)
                want = want.astype(np.float32).reshape(co, n, *u.shape[2:]).transpose(1, 0, 2, 3)
            got = blk.get_tensor(pb.STUDENT_ACT, l, 1, want.shape)
            same_nonfinite(got, want, (mode, l))
    blk.close()


FIRST_LAYER_SWITCHES = [("PBKD_CF_TH", 4), ("PBKD_CF_TH", 8), ("PBKD_CF_OCC", 1), ("PBKD_CF_OCC", 6), ("PBKD_DW_EDGE", 0),
                        ("PBKD_DW_EDGE", 2), ("PBKD_WGRAD_BN_FUSED", 0), ("PBKD_FIRST_BWD", 0)]


@pytest.mark.parametrize("var,value", FIRST_LAYER_SWITCHES, ids=[f"{k[5:].lower()}{v}" for k, v in FIRST_LAYER_SWITCHES])
def test_first_layer_and_depthwise_switches(gpu, monkeypatch, var, value):
    """Both tile heights and several grid sizes of the first-layer convolution, both ways the depthwise kernels get
    their edge columns on widths that do not fill 16-lane rows (12, 20, 36), and the first layer's weight gradient
    with and without its BatchNorm backward folded in (the default folds): each against the oracle on the blocks with a
    full first convolution (one, two and three input channels, a ragged second channel block, widths 12 to 36) and on
    two depthwise-only blocks."""
    monkeypatch.setenv(var, str(value))
    by_name = {v.name: v for v in wl.small_variants()}
    for name in ("fullconv_first", "fullconv_first_2ch", "fullconv_first_w36_70ch", "fullconv_first_w11", "ragged_pool", "wide_rows"):
        fails = run_parity(gpu, by_name[name], steps=3)
        assert not fails, (var, value, name, fails)


@pytest.mark.parametrize("split", [0, 1], ids=["fp32_mfma", "bf16_split"])
def test_teacher_convolution_both_arithmetics(gpu, monkeypatch, split):
    """The teacher's 3x3 convolutions through the fp32 MFMA kernel (PBKD_CONV_SPLIT=0) and through the bf16 MFMA
    kernel that splits every fp32 operand three ways (the default), each against the oracle at the activation
    tolerance: ragged channel counts (5, 7, 33, 40, 70: chunks of 8 with a zero-weight tail), stride 2, several images
    per pixel tile (2x2, 6x6, 8x8 maps), a K split (2x2 maps), tiles that end inside the image (9x11, 12x12), a
    projection shortcut beside it; stride 2 and rows of two tiles on widths the split kernel takes (12, 16, 40)."""
    monkeypatch.setenv("PBKD_CONV_SPLIT", str(split))
    by_name = {v.name: v for v in wl.small_variants()}
    for name in ("ragged_pool", "ragged_residual_s2", "three_layers_oddc", "paper_task_2x2", "two_layers_skip",
                 "second_layer_s2_w16", "fullconv_first_w36_70ch", "fullconv_first_7ch", "split_s2_first_w12",
                 "split_s2_second_w16", "split_two_tiles_w40"):
        fails = run_parity(gpu, by_name[name], steps=1)
        assert not fails, (split, name, fails)
    fails = run_parity(gpu, wl.cfg1_tiny(), steps=1)
    assert not fails, (split, fails)


def test_split_convolution_on_drawn_shapes(gpu):
    """Teacher forward of two-layer 3x3 blocks whose shapes are drawn (fixed seed) from what the bf16-split kernel takes:
    widths that are multiples of 4 up to 72 (rows of one to three tiles), heights 2 to 20, whole-image maps whose H*W is a
    multiple of 4 while the width is not (6x6, 2x14, 10x10), batches that leave the last pixel tile partly empty, 9 to 70
    input channels (ragged last chunk), stride 2 in either layer, with and without a projection shortcut."""
    torch, pb = gpu
    rng = np.random.default_rng(2024)
    shapes = [(6, 6), (2, 14), (10, 10)]
    while len(shapes) < 14:
        shapes.append((int(rng.integers(2, 21)), 4 * int(rng.integers(1, 19))))
    for k, (h, w_) in enumerate(shapes):
        n = int(rng.integers(1, 8))
        c0, c1, c2 = (int(rng.integers(9, 71)) for _ in range(3))
        s0 = 2 if (k % 4 == 1 and h >= 4 and w_ >= 8 and w_ % 8 == 0) else 1
        s1 = 2 if (k % 4 == 3 and h >= 4 and w_ >= 8 and w_ % 8 == 0) else 1
        sc = 1 if (k % 3 == 0) else 0
        layers = [wl.Layer(wl.CONV3X3, c0, c1, s0, 0), wl.Layer(wl.CONV3X3, c1, c2, s1, 0)]
        slayers = [wl.Layer(wl.DWSEP3X3, c0, c1, s0, 1), wl.Layer(wl.DWSEP3X3, c1, c2, s1, 1)]
        t = wl.Arch(n, c0, h, w_, layers, shortcut=sc, shortcut_stride=s0 * s1)
        s = wl.Arch(n, c0, h, w_, slayers, shortcut=sc, shortcut_stride=s0 * s1)
        wk = wl.Workload(f"drawn_{k}", t, s, seed=100 + k, copy_shortcut=bool(sc))
        x, tp, sp = wk.tensors(random_affine=True)
        t_ref, tcache = ob.block_forward(t, tp, x, keep=True)
        blk = pb.Block(t, tp, s, sp)
        xd = torch.from_numpy(x).cuda()
        td = torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda")
        blk.teacher_forward(xd, td)
        torch.cuda.synchronize()
        what = (k, n, c0, c1, c2, h, w_, s0, s1, sc)
        for l in range(2):
            rec = tcache["layers"][l]
            z = blk.get_tensor(pb.TEACHER_ACT, l, 1, rec["z"].shape)
            assert relerr(z, rec["z"]) <= ACT_TOL, (what, l, relerr(z, rec["z"]))
            assert relerr(blk.get_tensor(pb.TEACHER_ACT, l, 2, rec["mean"].shape), rec["mean"]) <= ACT_TOL, (what, l, "mean")
            assert relerr(blk.get_tensor(pb.TEACHER_ACT, l, 3, rec["rstd"].shape), rec["rstd"]) <= ACT_TOL, (what, l, "rstd")
        assert relerr(td.cpu().numpy(), t_ref) <= ACT_TOL, (what, "target")
        blk.close()


# (n, channels, h, w, strides): tiles of stacked rows that run over several images and end with the batch (14x14, 27x23,
# 7x7), K split over workgroups (7x7 with 300 channels), several column tiles with a ragged last one (5x131, 9x70 at 64
# channels), a width and height of one, stride 2 on odd and even sizes, one output row per image
STACKED_ROWS = [(3, (40, 72, 33), 14, 14, (1, 1)), (4, (67, 100, 67), 27, 23, (1, 1)), (5, (300, 130, 20), 7, 7, (1, 1)),
                (2, (17, 9, 70), 5, 131, (1, 1)), (1, (64, 64, 64), 9, 70, (1, 1)), (6, (12, 20, 9), 13, 1, (1, 1)),
                (9, (10, 33, 16), 1, 11, (1, 1)), (3, (24, 40, 31), 15, 17, (2, 1)), (2, (9, 65, 48), 18, 30, (1, 2)),
                (7, (16, 16, 16), 2, 3, (2, 1)), (1, (129, 9, 10), 3, 3, (1, 1)), (9, (17, 24, 40), 20, 24, (1, 1)),
                (30, (16, 30, 200), 5, 5, (1, 1))]


@pytest.mark.parametrize("wgs", [0, 1, 3])
@pytest.mark.parametrize("n,chans,h,w_,strides", STACKED_ROWS)
def test_split_convolution_on_any_map(gpu, monkeypatch, n, chans, h, w_, strides, wgs):
    """Teacher forward on maps whose rows are not whole 16-byte groups, where the bf16-split kernel takes tiles out of the
    stacked rows of all images: every layer's pre-activation and statistics against the fp64 oracle at ACT_TOL.  With a
    workgroup per tile, and with one and three workgroups that walk all of them: tiles of two, three and more chunks behind one
    another, odd and even numbers of chunks in all, scalar and 16-byte stores, K split and not."""
    torch, pb = gpu
    monkeypatch.setenv("PBKD_CONV_ROWS", "1")
    if wgs:
        monkeypatch.setenv("PBKD_SPLIT_WGS", str(wgs))
    layers = [wl.Layer(wl.CONV3X3, a, b, st, 0) for a, b, st in zip(chans[:-1], chans[1:], strides)]
    slayers = [wl.Layer(wl.DWSEP3X3, a, b, st, 1) for a, b, st in zip(chans[:-1], chans[1:], strides)]
    t, s = wl.Arch(n, chans[0], h, w_, layers), wl.Arch(n, chans[0], h, w_, slayers)
    x, tp, sp = wl.Workload("any_map", t, s, seed=7).tensors(random_affine=True)
    t_ref, tcache = ob.block_forward(t, tp, x, keep=True)
    blk = pb.Block(t, tp, s, sp)
    xd = torch.from_numpy(x).cuda()
    td = torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda")
    blk.teacher_forward(xd, td)
    torch.cuda.synchronize()
    for l, rec in enumerate(tcache["layers"]):
        for k, key in ((1, "z"), (2, "mean"), (3, "rstd")):
            got = blk.get_tensor(pb.TEACHER_ACT, l, k, rec[key].shape)
            assert relerr(got, rec[key]) <= ACT_TOL, (l, key, relerr(got, rec[key]))
    assert relerr(td.cpu().numpy(), t_ref) <= ACT_TOL
    blk.close()


@pytest.mark.parametrize("n,c,h,w_", [(5, 9, 6, 5), (3, 7, 5, 6), (4, 6, 3, 7), (2, 5, 14, 14), (7, 4, 27, 23), (1, 3, 1, 9), (3, 4, 9, 67),
                                      (130, 2, 128, 33)])
def test_depthwise_on_widths_that_are_no_multiple_of_four(gpu, n, c, h, w_):
    """Forward and backward of two depthwise-separable layers where the last four-column strip of a row overlaps the one
    before it by one, two or three columns (and on 33x128 maps with four-row strips): gradients must count those once."""
    t = wl.Arch(n, c, h, w_, wl._convs([c, c + 1, c]))
    s = wl.Arch(n, c, h, w_, wl._dws([c, c + 1, c]))
    fails = run_parity(gpu, wl.Workload("dw_any_width", t, s, seed=13), steps=2)
    assert not fails, fails


@pytest.mark.parametrize("n,h,w_,chans", [(3, 2, 2, (5, 70, 6)), (7, 1, 5, (9, 8, 66)), (2, 14, 14, (40, 33, 64)), (5, 3, 3, (20, 129, 5)),
                                          (4, 23, 27, (7, 66, 9)), (2, 3, 1, (6, 5, 4)), (1, 1, 4, (3, 5, 7)), (300, 2, 3, (8, 9, 10))])
def test_pointwise_weight_gradient_on_any_map(gpu, n, h, w_, chans):
    """Pointwise weight gradients where an image is no whole number of 32-pixel chunks: its last group of four pixels
    overlaps the one before it by zero to three, a chunk spans several images (4, 5, 6 and 9 pixels), and maps of three
    pixels keep the kernel that loads single values."""
    t, s = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans))), wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)))
    fails = run_parity(gpu, wl.Workload("wgrad_any_map", t, s, seed=17), steps=2)
    assert not fails, fails


@pytest.mark.parametrize("huge", [False, True])
@pytest.mark.parametrize("n,h,w_,ci,co", [(32, 14, 14, 96, 130), (40, 8, 8, 64, 33), (6, 27, 23, 67, 100), (3, 5, 3, 5, 70), (96, 2, 2, 130, 64),
                                          (1, 1, 4, 3, 5), (17, 16, 32, 20, 24)])
def test_pointwise_weight_gradient_leaves_no_larger_error_than_fp32_products(gpu, monkeypatch, n, h, w_, ci, co, huge):
    """rms error of dP against fp64 (dz formed in fp64 from the kernel's own z, u its own): from split operands not above what the
    fp32 matrix cores leave.  Both sum the same products in the same parts, but a sum is rounded 6 times per 16 pixels for 8, and
    both take over the roundings of dz and u; 5 % for the drawing of them, and 3e-8 of rms where a sum is a few pixels and nearly
    exact either way.  A number past bfloat16's largest (u = 3.4e38, weights of its channel small enough for z to be ordinary)
    leaves a number, not a NaN.  No output reaches ReLU's corner: beta = 5, gamma = 0.1."""
    torch, pb = gpu
    t, s = wl.Arch(n, ci, h, w_, wl._convs([ci, co])), wl.Arch(n, ci, h, w_, wl._dws([ci, co]))
    x, tp, sp = wl.Workload("wgrad_error", t, s, seed=37).tensors(random_affine=True)
    x, sp = x.copy(), [[a.copy() for a in lp] for lp in sp]
    sp[0][2][:], sp[0][3][:] = 0.1, 5.0
    if huge:
        sp[0][0].reshape(ci, 9)[1] = np.eye(9)[4]
        sp[0][1].reshape(co, ci)[:, 1] *= np.float32(1e-38)
        x[:, 1, -1, -1] = 3.4e38
    td = torch.from_numpy((5 + np.random.default_rng(3).standard_normal((n, co, h, w_))).astype(np.float32)).cuda()
    errs = {}
    for split in (0, 1):
        monkeypatch.setenv("PBKD_WGRAD_SPLIT", str(split))
        blk = pb.Block(t, tp, s, sp)
        blk.student_step(torch.from_numpy(x).cuda(), td, 0.0, want_loss=False)
        u = blk.get_tensor(pb.STUDENT_ACT, 0, 0, (n, ci, h, w_)).astype(np.float64).transpose(1, 0, 2, 3).reshape(ci, -1)
        z = blk.get_tensor(pb.STUDENT_ACT, 0, 1, (n, co, h, w_)).astype(np.float64).transpose(1, 0, 2, 3).reshape(co, -1)
        dP = blk.get_tensor(pb.STUDENT_GRAD, 0, 1, (co, ci)).astype(np.float64)
        blk.close()
        rstd = 1 / np.sqrt(z.var(1, keepdims=True) + s.bn_eps)
        xhat = (z - z.mean(1, keepdims=True)) * rstd
        g = 2 * (0.1 * xhat + 5 - td.cpu().numpy().astype(np.float64).transpose(1, 0, 2, 3).reshape(co, -1)) / z.size
        dz = 0.1 * rstd * (g - g.mean(1, keepdims=True) - xhat * (g * xhat).mean(1, keepdims=True))
        ref = dz @ u.T
        scale = np.abs(dz) @ np.abs(u.T) if n * h * w_ < 64 else np.sqrt((dz ** 2) @ (u ** 2).T)      # (of a sum: few pixels may cancel)
        assert np.isfinite(dP).all()
        errs[split] = float(np.sqrt(np.mean(((dP - ref) / scale) ** 2)))
    print(f"[pointwise weight gradient error] {ci}->{co} {h}x{w_}x{n} huge={huge}: fp32 products {errs[0]:.3e}, split {errs[1]:.3e}")
    assert errs[1] <= 1.05 * errs[0] + 3e-8, errs


@pytest.mark.parametrize("n,h,w_,ci,co,split", [(4, 16, 16, 16, 16, 0), (128, 16, 16, 16, 16, 0), (160, 16, 16, 16, 16, 1), (32, 4, 4, 512, 512, 0),
                                                (33, 4, 4, 512, 512, 1), (5, 7, 7, 67, 100, 0), (170, 7, 7, 67, 100, 1)])
def test_pointwise_weight_gradient_of_few_chunks_keeps_fp32_products(gpu, monkeypatch, n, h, w_, ci, co, split):
    """Weight gradients whose workgroups sum at most four chunks of 32 pixels are those of the fp32 products, bit for bit, longer
    ones those of the split products: on both kinds of map, one chunk, the last size below the line and the first above it."""
    torch, pb = gpu
    t, s = wl.Arch(n, ci, h, w_, wl._convs([ci, co])), wl.Arch(n, ci, h, w_, wl._dws([ci, co]))
    x, tp, sp = wl.Workload("wgrad_route", t, s, seed=5).tensors(random_affine=True)
    xd = torch.from_numpy(x).cuda()
    td = torch.zeros(wl.output_shape(t), dtype=torch.float32, device="cuda")
    got = {}
    for asked in ("", "0", "1"):
        if asked:
            monkeypatch.setenv("PBKD_WGRAD_SPLIT", asked)
        blk = pb.Block(t, tp, s, sp)
        blk.student_step(xd, td, 0.0, want_loss=False)
        got[asked] = blk.get_tensor(pb.STUDENT_GRAD, 0, 1, (co, ci))
        blk.close()
    assert (got["0"] != got["1"]).any()
    np.testing.assert_array_equal(got[""], got[str(split)])


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("variant", range(4))
def test_every_weight_gradient_tile_with_both_products(gpu, monkeypatch, variant, split):
    """Each tile of the pointwise weight gradient with fp32 and with split products, forced: tiles and channels that end ragged,
    whole chunks per image and groups of four pixels that overlap, and one to ten chunks a workgroup (the loaders take them one
    by one, in twos or in fours, with every remainder)."""
    monkeypatch.setenv("PBKD_WGRAD_VARIANT", str(variant))
    monkeypatch.setenv("PBKD_WGRAD_SPLIT", str(split))
    for n, h, w_, chans in ((3, 8, 8, (20, 70, 33)), (40, 8, 12, (20, 300, 130)), (30, 5, 6, (260, 390, 140)), (6, 8, 8, (520, 515)),
                            (10, 8, 8, (520, 515)), (17, 7, 7, (515, 520))):
        t, s = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans))), wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)))
        fails = run_parity(gpu, wl.Workload("wgrad_tiles", t, s, seed=29), steps=2)
        assert not fails, (n, h, w_, chans, fails)


@pytest.mark.parametrize("variant", range(4))
@pytest.mark.parametrize("n,h,w_,ci,co", [(32, 14, 14, 96, 130), (40, 8, 8, 64, 33), (6, 27, 23, 67, 100), (3, 5, 3, 5, 70)])
def test_pointwise_weight_gradient_infinities(gpu, monkeypatch, n, h, w_, ci, co, variant):
    """A NaN or an infinity in the target's last channel (a row that tiles past the last channel repeat), in an image's last pixel
    (which the last group of four shares with the one before it), makes that row of dP NaN and leaves the others bit for bit;
    a sum past fp32's largest (u = 3.4e38) is the infinity that fp32 products make of it; an infinite input makes all NaN."""
    torch, pb = gpu
    t, s = wl.Arch(n, ci, h, w_, wl._convs([ci, co])), wl.Arch(n, ci, h, w_, wl._dws([ci, co]))
    x, tp, sp = wl.Workload("wgrad_infinities", t, s, seed=61).tensors(random_affine=True)
    x, sp = np.maximum(x, 0), [[a.copy() for a in lp] for lp in sp]
    sp[0][2][:], sp[0][3][:] = 0.1, 5.0                                     # (no output reaches ReLU's corner)
    sp[0][0].reshape(ci, 9)[1] = np.eye(9)[4]
    sp[0][1].reshape(co, ci)[:, 1] *= np.float32(1e-38)
    td = (5 + np.random.default_rng(4).standard_normal((n, co, h, w_))).astype(np.float32)
    monkeypatch.setenv("PBKD_WGRAD_VARIANT", str(variant))

    def gradient(split, xv, tv):
        monkeypatch.setenv("PBKD_WGRAD_SPLIT", str(split))
        blk, xd, tgt = pb.Block(t, tp, s, sp), torch.from_numpy(xv).cuda(), torch.from_numpy(tv).cuda()
        blk.student_step(xd, tgt, 0.0, want_loss=False)
        dP = blk.get_tensor(pb.STUDENT_GRAD, 0, 1, (co, ci))
        blk.close()
        return dP

    past, infinite = x.copy(), x.copy()
    past[0, 1, -1, -1] = 3.4e38
    infinite[n // 2, ci - 1, 0, 0] = np.inf
    for split in (0, 1):
        base = gradient(split, x, td)
        assert np.isfinite(base).all()
        for v in (np.nan, np.inf, -np.inf):
            bad = td.copy()
            bad[n // 2, co - 1, -1, -1] = v
            got = gradient(split, x, bad)
            assert np.isnan(got[co - 1]).all(), (split, v)
            np.testing.assert_array_equal(got[:co - 1], base[:co - 1])
        assert np.isnan(gradient(split, infinite, td)).all(), split
    # dz of the order of 1e12 / rstd: products with 3.4e38 overflow, the other channels' stay numbers
    far = (td * np.float32(1e12)).astype(np.float32)
    fp32, split = gradient(0, past, far), gradient(1, past, far)
    assert np.isinf(fp32[:, 1]).any() and np.isfinite(np.delete(fp32, 1, 1)).all()
    np.testing.assert_array_equal(value_classes(split), value_classes(fp32))


def launched_kinds(gpu, w):
    """{kernel kind: launches} of one student step of a new block."""
    torch, pb = gpu
    x, tp, sp = w.tensors()
    blk = pb.Block(w.teacher, tp, w.student, sp)
    blk.profile_enable(None, 200)
    blk.student_step(torch.from_numpy(x).cuda(), torch.zeros(wl.output_shape(w.teacher), device="cuda"), 0.0, want_loss=False)
    got = {k: n for k, (_, n) in blk.profile_read().items()}
    blk.close()
    return got


@pytest.mark.parametrize("n,h,w_,chans,pool,shortcut", [
    (1, 1, 4, (3, 16), 0, 0), (3, 2, 2, (5, 70, 16), 0, 0), (2, 4, 4, (64, 64), 2, 0), (3, 6, 8, (16, 65, 128), 2, 0), (2, 5, 7, (40, 17, 33), 2, 0),
    (9, 27, 23, (67, 100, 67), 0, 2), (5, 8, 12, (20, 128, 64), 2, 1), (7, 9, 5, (130, 127, 63), 0, 1), (40, 16, 16, (64, 128, 128), 2, 0),
    (33, 12, 20, (70, 64, 64), 2, 2), (150, 7, 7, (64, 100), 0, 0), (20, 30, 28, (200, 48, 64), 2, 0)])
def test_pointwise_gradients_in_one_kernel(gpu, monkeypatch, n, h, w_, chans, pool, shortcut):
    """Pointwise weight and data gradient from one kernel that forms dz from g and z, from the head's inputs with and without a
    pool and a second input, or reads it (a pool without aligned windows): 64 and 128 rows of weights, ragged channels, one to six
    column tiles, images that end in overlapping groups of four pixels, units that wrap, one to five chunks a workgroup (see the next
    test for more)."""
    monkeypatch.setenv("PBKD_PW_BWD", "1")
    chans = tuple(chans) if shortcut != 2 else (chans[0], *chans[1:-1], chans[0])
    t = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans)), shortcut=1 if shortcut == 1 else 0, shortcut_stride=1, pool=pool)
    s = wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)), shortcut=shortcut, shortcut_stride=1, pool=pool)
    w = wl.Workload("pw_bwd", t, s, seed=41)
    assert launched_kinds(gpu, w)["pw_bwd"] == sum(co >= 16 for co in chans[1:])
    fails = run_parity(gpu, w, steps=2)
    assert not fails, fails


@pytest.mark.parametrize("co", [64, 40, 128, 100])
@pytest.mark.parametrize("source,n,h,w_,pool,shortcut,chunks", [
    ("given", 8, 30, 30, 2, 0, 8), ("inside", 9, 32, 32, 0, 0, 9), ("head", 7, 32, 32, 0, 0, 7), ("head_skip", 5, 32, 32, 0, 1, 5),
    ("pooled_head", 8, 32, 32, 2, 0, 8), ("pooled_head_skip", 6, 32, 32, 2, 1, 6)])
def test_pointwise_gradients_in_one_kernel_of_many_chunks(gpu, source, n, h, w_, pool, shortcut, chunks, co):
    """Every source of dz, with 64 and 128 rows of weights, whole and ragged, where the loaders take their register sets (three, two
    with a second head input) a second time round and more, and with every remainder: 1024 input channels leave 16 workgroups to the
    pixels, each with `chunks` chunks of 64 pixels (maps half as high and chunks of 32 with more than 64 output channels)."""
    px = 64 if co <= 64 else 32
    h = h if co <= 64 or source == "given" else h // 2
    n = n if co <= 64 or source != "given" else n // 2
    unit = 8 if pool and source != "given" else 4
    nchunks = -(-n * -(-h * w_ // unit) // (px // unit))
    assert -(-nchunks // (256 // (1024 // 64))) == chunks
    chans = (1024, co, 16) if source == "inside" else (1024, co)
    t = wl.Arch(n, 1024, h, w_, wl._convs(list(chans)), shortcut=shortcut, shortcut_stride=1, pool=pool)
    s = wl.Arch(n, 1024, h, w_, wl._dws(list(chans)), shortcut=shortcut, shortcut_stride=1, pool=pool)
    w = wl.Workload("pw_bwd_chunks", t, s, seed=43)
    assert launched_kinds(gpu, w).get("pw_bwd", 0) >= 1
    fails = run_parity(gpu, w, steps=2)
    assert not fails, fails


@pytest.mark.parametrize("n,h,w_,ci,co,pool", [(8, 16, 16, 512, 16, 0), (8, 16, 16, 300, 33, 0), (3, 9, 7, 300, 64, 0), (8, 16, 16, 300, 64, 2),
                                               (3, 9, 7, 512, 100, 0), (8, 16, 16, 512, 128, 0), (8, 16, 16, 512, 128, 2), (64, 16, 16, 300, 64, 0)])
def test_pointwise_data_gradient_leaves_no_larger_error_than_the_kernel_apart(gpu, monkeypatch, n, h, w_, ci, co, pool):
    """rms error of du against fp64 (dz formed in fp64 from the kernel's own z) with the gradients in one kernel, not above what the
    pointwise kernel leaves.  A block's input that is one at a single pixel of each channel makes the depthwise weight gradient's
    nine sums single values of du.  Where both sum in the same order they are equal, else 1 % for the drawing of the 10 to 18
    thousand values.  No output reaches ReLU's corner: beta = 5, and gamma = 0.03 (xhat is at most the root of the 16384 pixels)."""
    torch, pb = gpu
    gamma = float(np.float32(0.03))
    t, s = wl.Arch(n, ci, h, w_, wl._convs([ci, co]), pool=pool), wl.Arch(n, ci, h, w_, wl._dws([ci, co]), pool=pool)
    err = {"0": [], "1": []}
    for seed in range(4):
        x, tp, sp = wl.Workload("du_error", t, s, seed=37 + seed).tensors(random_affine=True)
        sp = [[a.copy() for a in lp] for lp in sp]
        sp[0][2][:], sp[0][3][:] = gamma, 5.0
        rng, ch = np.random.default_rng(seed), np.arange(ci)
        py, px = rng.integers(1, h - 1, ci), rng.integers(1, w_ - 1, ci)
        x = np.zeros_like(x)
        x[n // 2, ch, py, px] = 1.0
        td = (5 + rng.standard_normal(wl.output_shape(t))).astype(np.float32)
        t64, P = td.astype(np.float64).transpose(1, 0, 2, 3), sp[0][1].reshape(co, ci).astype(np.float64)
        for mode in err:
            monkeypatch.setenv("PBKD_PW_BWD", mode)
            blk = pb.Block(t, tp, s, sp)
            blk.profile_enable(["pw_bwd"], 4)
            blk.student_step(torch.from_numpy(x).cuda(), torch.from_numpy(td).cuda(), 0.0, want_loss=False)
            assert ("pw_bwd" in blk.profile_read()) == (mode == "1")
            z = blk.get_tensor(pb.STUDENT_ACT, 0, 1, (n, co, h, w_)).astype(np.float64).transpose(1, 0, 2, 3)
            mean, rstd = (blk.get_tensor(pb.STUDENT_ACT, 0, k, (co, 1)).astype(np.float64) for k in (2, 3))
            dec = gpu_decisions(pb, blk, s)
            dD = blk.get_tensor(pb.STUDENT_GRAD, 0, 0, (ci, 9)).astype(np.float64)
            blk.close()
            assert dec["relu"][0].all()
            xhat = (z.reshape(co, -1) - mean) * rstd
            b = (gamma * xhat + 5).reshape(co, n, h, w_)
            if pool:
                win = lambda v: v.reshape(co, n, h // 2, 2, w_ // 2, 2).transpose(0, 1, 2, 4, 3, 5).reshape(co, n, h // 2, w_ // 2, 4)
                arg = dec["pool_arg"].transpose(1, 0, 2, 3)[..., None]
                g = np.zeros((co, n, h // 2, w_ // 2, 4))
                np.put_along_axis(g, arg, 2 * (np.take_along_axis(win(b), arg, -1) - t64[..., None]) / td.size, -1)
                g = g.reshape(co, n, h // 2, w_ // 2, 2, 2).transpose(0, 1, 2, 4, 3, 5)
            else:
                g = 2 * (b - t64) / td.size
            g = g.reshape(co, -1)
            dz = gamma * rstd * (g - g.mean(1, keepdims=True) - xhat * (g * xhat).mean(1, keepdims=True))
            at = np.stack([(n // 2 * h + py - (k // 3 - 1)) * w_ + px - (k % 3 - 1) for k in range(9)], 1)       # [ci, 9]
            dzs = dz[:, at]                                                                                # [co, ci, 9]
            ref = np.einsum("oc,ock->ck", P, dzs)
            err[mode].append((dD - ref) / np.sqrt(np.einsum("oc,ock->ck", P ** 2, dzs ** 2)))
    rms = {k: float(np.sqrt(np.mean(np.square(v)))) for k, v in err.items()}
    print(f"[pointwise data gradient error] {ci}->{co} {h}x{w_}x{n} pool={pool}: apart {rms['0']:.3e}, in one {rms['1']:.3e}")
    assert rms["1"] <= 1.01 * rms["0"], rms


@pytest.mark.parametrize("n,h,w_,chans,pool", [(6, 27, 23, (40, 100, 67), 0), (40, 8, 8, (20, 33, 64), 2), (3, 5, 3, (17, 70, 70), 0)])
def test_pointwise_gradients_in_one_kernel_infinities(gpu, monkeypatch, n, h, w_, chans, pool):
    """A target that holds a NaN or an infinity in its last channel's last pixel, an infinite input, and a depthwise output past
    bfloat16's largest: every gradient of the block has its infinities and NaNs where the kernels apart have them."""
    torch, pb = gpu
    t = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans)), pool=pool)
    s = wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)), pool=pool)
    x, tp, sp = wl.Workload("pw_bwd_infinities", t, s, seed=61).tensors(random_affine=True)
    x, sp = np.maximum(x, 0), [[a.copy() for a in lp] for lp in sp]
    sp[-1][2][:], sp[-1][3][:] = 0.1, 5.0                                   # (no output reaches ReLU's corner)
    sp[0][0].reshape(chans[0], 9)[1] = np.eye(9)[4]
    sp[0][1].reshape(chans[1], chans[0])[:, 1] *= np.float32(1e-38)
    td = (5 + np.random.default_rng(4).standard_normal(wl.output_shape(t))).astype(np.float32)

    def gradients(mode, xv, tv):
        monkeypatch.setenv("PBKD_PW_BWD", mode)
        blk, xd, tgt = pb.Block(t, tp, s, sp), torch.from_numpy(xv).cuda(), torch.from_numpy(tv).cuda()
        blk.student_step(xd, tgt, 0.0, want_loss=False)
        got = [blk.get_tensor(pb.STUDENT_GRAD, l, k, shape) for l, shapes in enumerate(wl.param_shapes(s)) for k, shape in enumerate(shapes)]
        blk.close()
        return got

    past, infinite = x.copy(), x.copy()
    past[0, 1, -1, -1] = 3.4e38
    infinite[n // 2, chans[0] - 1, 0, 0] = np.inf
    cases = [(past, td), (infinite, td), (past, (td * np.float32(1e12)).astype(np.float32))]
    for v in (np.nan, np.inf, -np.inf):
        bad = td.copy()
        bad[n // 2, -1, -1, -1] = v
        cases.append((x, bad))
    for i, (xv, tv) in enumerate(cases):
        for a, b in zip(gradients("1", xv, tv), gradients("0", xv, tv)):
            np.testing.assert_array_equal(value_classes(a), value_classes(b), err_msg=str(i))


@pytest.mark.parametrize("n,h,w_,chans,pool", [
    (1, 1, 4, (3, 5, 16), 0), (2, 3, 4, (1, 33, 20), 0), (3, 2, 8, (2, 16, 16, 16), 2), (5, 7, 12, (3, 31, 17), 0), (1, 4, 32, (3, 32, 32), 2),
    (7, 6, 36, (1, 65, 16), 2), (9, 13, 20, (3, 100, 24), 0), (4, 33, 64, (3, 64, 64), 0), (37, 10, 28, (2, 40, 16), 2),
    (6, 30, 44, (3, 520, 20), 0), (40, 10, 28, (2, 1000, 16), 2)])
def test_first_layers_gradients_in_one_kernel(gpu, n, h, w_, chans, pool):
    """A full first layer and the depthwise convolution behind it: one to 32 groups of channels, ragged ones; one, two and three input
    channels; rows past the map in the last patch; patches that wrap from row to row and from image to image within a tile of eight; one
    tile of which most is past the end, and (520 and 1000 channels) two and four tiles a workgroup."""
    t = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans)), pool=pool)
    s = wl.Arch(n, chans[0], h, w_, [wl.Layer(wl.CONV3X3, chans[0], chans[1], 1, 1)] + wl._dws(list(chans[1:])), pool=pool)
    w = wl.Workload("first_bwd", t, s, seed=43)
    assert launched_kinds(gpu, w).get("first_bwd") == 1
    fails = run_parity(gpu, w, steps=2)
    assert not fails, fails


def shifted(torch, v, dy, dx):
    """v at (y + dy, x + dx), zero outside the map."""
    H, W = v.shape[-2:]
    out = torch.zeros_like(v)
    out[..., max(0, -dy):H - max(0, dy), max(0, -dx):W - max(0, dx)] = v[..., max(0, dy):H - max(0, -dy), max(0, dx):W - max(0, -dx)]
    return out


@pytest.mark.parametrize("n,h,w_,ci,c,off,seeds", [(1, 16, 16, 3, 64, 1, 8), (2, 32, 32, 3, 32, 1, 8), (16, 32, 32, 3, 64, 0, 4), (5, 27, 36, 2, 40, 2, 4),
                                                   (8, 32, 32, 3, 1024, 0, 1), (8, 112, 112, 1, 1024, 0, 1), (8, 112, 112, 1, 1024, 30, 1)])
def test_first_layers_gradients_leave_no_larger_error_than_the_kernels_apart(gpu, monkeypatch, n, h, w_, ci, c, off, seeds):
    """rms errors of the first layer's weight, gamma and beta gradients and of the depthwise weight gradient behind it against fp64, from
    the kernels' own z and statistics, each relative to the root of its terms' squares: with all from one kernel not above what the
    kernels apart leave, at one, two and 25 tiles a workgroup, with inputs around 0, 1, 2 and 30.  5 % for the drawing of the values (32
    to 64 of gamma and beta a seed: their ratio has a standard error of 1 to 2 % over 8 seeds)."""
    torch, pb = gpu
    d, co = torch.float64, 16
    t = wl.Arch(n, ci, h, w_, wl._convs([ci, c, co]))
    s = wl.Arch(n, ci, h, w_, [wl.Layer(wl.CONV3X3, ci, c, 1, 1)] + wl._dws([c, co]))
    err = {"0": [], "1": []}
    for seed in range(seeds):
        x, tp, sp = wl.Workload("first_error", t, s, seed=seed).tensors(random_affine=True)
        xd = torch.from_numpy((x + np.float32(off)).astype(np.float32)).cuda()
        td = torch.from_numpy(np.random.default_rng(1).standard_normal((n, co, h, w_)).astype(np.float32)).cuda()
        P, D = (torch.from_numpy(sp[1][k].reshape(shape)).cuda().to(d) for k, shape in ((1, (co, c)), (0, (c, 9))))
        for mode in err:
            monkeypatch.setenv("PBKD_FIRST_BWD", mode)
            blk = pb.Block(t, tp, s, sp)
            blk.profile_enable(["first_bwd"], 4)
            blk.student_step(xd, td, 0.0, want_loss=False)
            assert ("first_bwd" in blk.profile_read()) == (mode == "1")
            get = lambda which, l, k, shape: torch.from_numpy(blk.get_tensor(which, l, k, shape)).cuda().to(d)
            z, zn = get(pb.STUDENT_ACT, 0, 1, (n, c, h, w_)), get(pb.STUDENT_ACT, 1, 1, (n, co, h, w_))
            (mean, rstd, sc, sh), (mn, rn, scn, shn) = ([get(pb.STUDENT_ACT, l, k, (1, k_, 1, 1)) for k in (2, 3, 4, 5)] for l, k_ in ((0, c), (1, co)))
            got = [get(pb.STUDENT_GRAD, 0, 0, (c, 9 * ci)), get(pb.STUDENT_GRAD, 0, 1, (c, 1)), get(pb.STUDENT_GRAD, 0, 2, (c, 1)), get(pb.STUDENT_GRAD, 1, 0, (c, 9))]
            blk.close()
            over = (0, 2, 3)
            bn = zn * scn + shn
            gn = (bn.float() > 0) * 2 * (bn - td.to(d)) / td.numel()
            xn = (zn - mn) * rn
            dzn = scn * (gn - gn.mean(over, keepdim=True) - xn * (gn * xn).mean(over, keepdim=True))
            du = (P.t() @ dzn.transpose(0, 1).reshape(co, -1)).reshape(c, n, h, w_).transpose(0, 1)
            b = z * sc + sh
            on = b.float() > 0
            taps = [(k // 3 - 1, k % 3 - 1) for k in range(9)]
            g, terms = torch.zeros_like(z), [[], [], [], []]                # of dW, dgamma, dbeta, dD: (sum, root of the squares' sum)
            both = lambda v: (v.sum(over), (v * v).sum(over).sqrt())
            for k, (dy, dx) in enumerate(taps):
                v = shifted(torch, du, -dy, -dx)
                g += D[:, k].reshape(1, c, 1, 1) * v
                terms[3].append(both(b * on * v))
            g *= on
            xhat = (z - mean) * rstd
            terms[1].append(both(g * xhat))
            terms[2].append(both(g))
            dz = sc * (g - g.mean(over, keepdim=True) - xhat * (g * xhat).mean(over, keepdim=True))
            for i in range(ci):
                for dy, dx in taps:
                    terms[0].append(both(dz * shifted(torch, xd[:, i:i + 1].to(d), dy, dx)))
            err[mode].append([float((((a - torch.stack([q[0] for q in v], 1)) / torch.stack([q[1] for q in v], 1)) ** 2).mean()) for a, v in zip(got, terms)])
    rms = {k: np.sqrt(np.mean(v, 0)) for k, v in err.items()}
    print(f"[first layers' gradient errors] {ci}->{c} {h}x{w_}x{n} off={off}: apart {rms['0']}, in one {rms['1']}")
    assert (rms["1"] <= 1.05 * rms["0"]).all(), rms


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_first_layers_gradients_not_numbers(gpu, monkeypatch, bad):
    """An input or a target that holds a NaN or an infinity: numbers where the kernels apart have numbers, in every gradient of the
    block.  (Not so for a number near the largest: whether fp32 sums that hold it pass the largest on the way depends on their
    order, and here the parts are put together in 64 bits.)"""
    torch, pb = gpu
    chans, n, h, w_ = (3, 40, 33), 3, 9, 12
    t = wl.Arch(n, 3, h, w_, wl._convs(list(chans)))
    s = wl.Arch(n, 3, h, w_, [wl.Layer(wl.CONV3X3, 3, 40, 1, 1)] + wl._dws(list(chans[1:])))
    x, tp, sp = wl.Workload("first_bwd_not_numbers", t, s, seed=47).tensors(random_affine=True)
    td = np.random.default_rng(5).standard_normal(wl.output_shape(t)).astype(np.float32)

    def gradients(mode, xv, tv):
        monkeypatch.setenv("PBKD_FIRST_BWD", mode)
        blk, xd, tgt = pb.Block(t, tp, s, sp), torch.from_numpy(xv).cuda(), torch.from_numpy(tv).cuda()
        blk.student_step(xd, tgt, 0.0, want_loss=False)
        got = [blk.get_tensor(pb.STUDENT_GRAD, l, k, shape) for l, shapes in enumerate(wl.param_shapes(s)) for k, shape in enumerate(shapes)]
        blk.close()
        return got

    xb, tb = x.copy(), td.copy()
    xb[1, 2, 4, 11] = bad
    tb[2, 32, -1, -1] = bad
    for xv, tv in ((xb, td), (x, tb)):
        for a, b in zip(gradients("1", xv, tv), gradients("0", xv, tv)):
            np.testing.assert_array_equal(np.isfinite(a), np.isfinite(b))


def test_teacher_weights_replaced_after_creation(gpu):
    """pbkd_block_set_tensor on a teacher's convolution weights re-packs them for whichever kernel the layer runs (the
    bf16-split kernel keeps three bf16 images of them): the forward pass then follows the new weights."""
    torch, pb = gpu
    w = wl.cfg1_tiny()
    x, tp, sp = w.tensors(random_affine=True)
    _, tp2, _ = replace(w, seed=w.seed + 7).tensors(random_affine=True)
    blk = pb.Block(w.teacher, tp, w.student, sp)
    for l in range(len(tp2)):
        blk.set_tensor(pb.TEACHER_PARAM, l, 0, tp2[l][0])           # the convolution weights only
    mixed = [[tp2[l][0]] + [a for a in tp[l][1:]] for l in range(len(tp))]
    t_ref = ob.block_forward(w.teacher, mixed, x)
    xd = torch.from_numpy(x).cuda()
    td = torch.empty(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda")
    blk.teacher_forward(xd, td)
    torch.cuda.synchronize()
    assert relerr(td.cpu().numpy(), t_ref) <= ACT_TOL
    blk.close()


@pytest.mark.parametrize("env", [{"PBKD_CONV_WINO": "1"}, {"PBKD_CONV_WINO": "0"}, {"PBKD_CONV_ROWS": "1"}])
@pytest.mark.parametrize("n,h,w_,chans", [(3, 12, 16, (40, 72, 33)), (5, 8, 8, (64, 130, 17)), (2, 14, 14, (300, 16, 65))])
def test_teacher_weights_replaced_reach_every_split_kernel(gpu, monkeypatch, n, h, w_, chans, env):
    """pbkd_block_set_tensor on the weights of layers on transformed tiles, aligned maps and stacked rows: a block with its weights
    replaced gives bit for bit what a block created with them gives, and what the fp64 oracle gives at ACT_TOL."""
    torch, pb = gpu
    for name, value in env.items():
        monkeypatch.setenv(name, value)
    t, s = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans))), wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)))
    w = wl.Workload("replaced", t, s, seed=67)
    x, tp, sp = w.tensors(random_affine=True)
    _, tp2, _ = replace(w, seed=68).tensors(random_affine=True)
    xd, got = torch.from_numpy(x).cuda(), []
    for first in (tp, tp2):
        blk = pb.Block(t, first, s, sp)
        td = torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda")
        blk.teacher_forward(xd, td)
        for l, lp in enumerate(tp2):
            for k, a in enumerate(lp):
                blk.set_tensor(pb.TEACHER_PARAM, l, k, a)
        blk.teacher_forward(xd, td)
        torch.cuda.synchronize()
        got.append([blk.get_tensor(pb.TEACHER_ACT, l, 1, shp) for l, (_, shp, _) in enumerate(_layer_act_shapes(t))] + [td.cpu().numpy()])
        blk.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    t_ref, cache = ob.block_forward(t, [[a.astype(np.float64) for a in lp] for lp in tp2], x.astype(np.float64), keep=True)
    for z, ref in zip(got[0], [rec["z"] for rec in cache["layers"]] + [t_ref]):
        assert relerr(z, ref) <= ACT_TOL


def test_split_convolution_is_as_accurate_as_fp32(gpu, monkeypatch):
    """Six bf16 products of three-way split operands leave out terms of at most 2^-24 of each product, so against the fp64
    oracle the split kernel must not be worse than the fp32 MFMA kernel by more than rounding noise.  Two layers with
    long dot products (K = 9*128 and 9*256), BatchNorm between them, several workgroup tiles in a persistent grid."""
    torch, pb = gpu
    t = wl.Arch(24, 128, 16, 16, wl._convs([128, 256, 96]))
    s = wl.Arch(24, 128, 16, 16, wl._dws([128, 256, 96]))
    w = wl.Workload("accuracy_probe", t, s, seed=11)
    x, tp, sp = w.tensors(random_affine=True)
    t_ref, tcache = ob.block_forward(w.teacher, [[a.astype(np.float64) for a in lp] for lp in tp], x.astype(np.float64), keep=True)
    xd = torch.from_numpy(x).cuda()
    errs = {}
    for split in (0, 1):
        monkeypatch.setenv("PBKD_CONV_SPLIT", str(split))
        blk = pb.Block(w.teacher, tp, w.student, sp)
        td = torch.empty(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda")
        blk.teacher_forward(xd, td)
        torch.cuda.synchronize()
        e = []
        for l in range(2):
            z = blk.get_tensor(pb.TEACHER_ACT, l, 1, tcache["layers"][l]["z"].shape)
            e.append(relerr(z, tcache["layers"][l]["z"]))
        e.append(relerr(td.cpu().numpy(), t_ref))
        errs[split] = e
        blk.close()
    print(f"[split accuracy] max|err|/max|ref| of z0, z1, target: fp32 MFMA {errs[0]}, bf16 split {errs[1]}")
    for a, b in zip(errs[0], errs[1]):
        assert a <= ACT_TOL and b <= ACT_TOL, errs
        assert b <= 2.0 * a + 2e-7, errs


def rms_error(got, ref):
    got, ref = np.asarray(got, dtype=np.float64), np.asarray(ref, dtype=np.float64)
    return float(np.sqrt(np.mean((got - ref) ** 2) / np.mean(ref ** 2)))


def teacher_layer_errors(gpu, w, tp, x):
    """rms error against fp64 of each pre-activation of a two-layer teacher, the second layer's against what fp64 makes of the
    first layer's own output (so that it holds that layer's error alone)."""
    torch, pb = gpu
    t = w.teacher
    blk = pb.Block(t, tp, w.student, w.tensors(random_affine=True)[2])
    td = torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda")
    blk.teacher_forward(torch.from_numpy(x).cuda(), td)
    torch.cuda.synchronize()
    shapes = [shp for _, shp, _ in _layer_act_shapes(t)]
    z = [blk.get_tensor(pb.TEACHER_ACT, l, 1, shp) for l, shp in enumerate(shapes)]
    blk.close()
    p64 = [[a.astype(np.float64) for a in lp] for lp in tp]
    z0 = z[0].astype(np.float64)
    mean = z0.mean((0, 2, 3), keepdims=True)
    var = ((z0 - mean) ** 2).mean((0, 2, 3), keepdims=True)
    act = np.maximum((z0 - mean) / np.sqrt(var + t.bn_eps) * p64[0][1][None, :, None, None] + p64[0][2][None, :, None, None], 0)
    errs = []
    for l, inp in enumerate((x.astype(np.float64), act)):
        one = wl.Arch(t.n, t.layers[l].cin, t.h, t.w, [replace(t.layers[l])])
        ref = ob.block_forward(one, [p64[l]], inp, keep=True)[1]["layers"][0]["z"]
        errs.append(rms_error(z[l], ref))
    return errs


@pytest.mark.parametrize("kind", ["plain", "small_variance", "large_channel_off"])
@pytest.mark.parametrize("n,h,w_,chans", [(24, 16, 16, (128, 256, 96)), (6, 13, 11, (16, 9, 40)), (9, 7, 7, (64, 500, 512)),
                                          (6, 27, 23, (67, 100, 67))])
def test_convolution_behind_a_batchnorm_keeps_fp32_accuracy(gpu, monkeypatch, n, h, w_, chans, kind):
    """Whatever the scale of a BatchNorm's output and of the weights behind it, the split products' error against fp64 stays
    that of fp32 products: relative to each product, never to a channel's bound or to its row's largest weight.  Beside
    ordinary values: a producer whose variance is far below eps (outputs of a hundredth of gamma), and one input channel
    whose weights are 1e6 times the others' and whose activations are all zero.  At most twice the fp32 MFMA kernel's rms
    error: the split leaves out 2^-27 (rms) of a product, and with one running sum it rounds 27 times per eight channels at that
    sum's size, the fp32 kernel 72 times, half of them adding exact zeros (post-ReLU operands) and over shorter sums where
    it splits K: alike to within 1.4.  Pieces held relative to a bound stand at 2.4 to 38 times."""
    t, s = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans))), wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)))
    w = wl.Workload("behind_batchnorm", t, s, seed=21)
    x, tp, _ = w.tensors(random_affine=True)
    x = np.maximum(x, 0)
    if kind == "small_variance":
        tp[0][0] = tp[0][0] * np.float32(1e-5)
        tp[0][2] = np.zeros_like(tp[0][2])
    if kind == "large_channel_off":
        tp[1][0] = tp[1][0].copy()
        tp[1][0][:, 0] *= np.float32(1e6)
        tp[0][2] = tp[0][2].copy()
        tp[0][2][0] = -1e3
    errs = {}
    for split in (0, 1):
        monkeypatch.setenv("PBKD_CONV_SPLIT", str(split))
        errs[split] = teacher_layer_errors(gpu, w, tp, x)[1]
    print(f"[behind a BatchNorm] {kind} {chans} {h}x{w_}: rms error of z1, fp32 MFMA {errs[0]:.3e}, split {errs[1]:.3e}")
    assert errs[1] <= 2.0 * errs[0], errs


@pytest.mark.parametrize("n,h,w_,chans", [(6, 13, 11, (16, 9, 40)), (9, 7, 7, (64, 500, 512)), (6, 27, 23, (67, 100, 67)), (4, 14, 14, (512, 128, 130)),
                                          (2, 55, 57, (33, 64, 48)), (40, 5, 5, (256, 260, 20)), (64, 2, 1, (48, 64, 64))])
def test_stacked_rows_are_no_less_accurate_than_fp32(gpu, monkeypatch, n, h, w_, chans):
    """On maps whose rows are not whole 16-byte groups the split kernel stands in for the fp32 MFMA kernel, so its rms error
    against fp64 must not be the larger one, in a layer on the block input and one behind a BatchNorm.  It sums a chunk's 27
    MFMAs from zero and adds that to the running sum: n chunks leave about 27/2 + n/2 squared roundings at the size of the
    result where the fp32 kernel's leave 36 n/2 (72 products a chunk, half of them zeros) over its K split of up to eight, four
    chunks a split at least.  (2 %: what
    the rms of a thousand elements of either kernel is uncertain by.)"""
    t, s = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans))), wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)))
    w = wl.Workload("stacked_rows_accuracy", t, s, seed=23)
    x, tp, _ = w.tensors(random_affine=True)
    x = np.maximum(x, 0)
    errs = {}
    for split in (0, 1):
        monkeypatch.setenv("PBKD_CONV_SPLIT", str(split))
        monkeypatch.setenv("PBKD_CONV_ROWS", str(split))
        errs[split] = teacher_layer_errors(gpu, w, tp, x)
    print(f"[stacked rows accuracy] {chans} {h}x{w_}: rms error of z0, z1: fp32 MFMA {errs[0]}, split {errs[1]}")
    for a, b in zip(errs[0], errs[1]):
        assert b <= 1.02 * a, errs


@pytest.mark.parametrize("tile", [-1, 0, 1, 2, 3])
@pytest.mark.parametrize("n,h,w_,chans,strides", [(3, 13, 15, (40, 72, 33), (1, 1)), (5, 7, 7, (300, 130, 20), (1, 1)), (3, 17, 13, (24, 40, 31), (2, 1)),
                                                  (2, 5, 131, (17, 9, 70), (1, 1)), (6, 13, 1, (12, 20, 9), (1, 1))])
def test_stacked_rows_infinities(gpu, monkeypatch, n, h, w_, chans, strides, tile):
    """Infinities and numbers past bfloat16's largest in the block's input, in a layer's output (running statistics) and in the
    weights: every pre-activation is the number, infinity or NaN that plain products make of them, K split or not."""
    torch, pb = gpu
    layers = [wl.Layer(wl.CONV3X3, a, b, st, 0) for a, b, st in zip(chans[:-1], chans[1:], strides)]
    slayers = [wl.Layer(wl.DWSEP3X3, a, b, st, 1) for a, b, st in zip(chans[:-1], chans[1:], strides)]
    t, s = wl.Arch(n, chans[0], h, w_, layers), wl.Arch(n, chans[0], h, w_, slayers)
    x, tp, sp = wl.Workload("infinities", t, s, seed=43).tensors(random_affine=True)
    rng = np.random.default_rng(9)
    x = np.maximum(x, 0)
    for v in (np.inf, 3.4e38, -np.inf):
        x[rng.integers(n), rng.integers(chans[0]), rng.integers(h), rng.integers(w_)] = v
    x[-1, -1, -1, -1] = np.inf
    tp[0][0] = tp[0][0].copy()
    tp[0][0][3] *= np.float32(1e-3)
    tp[0][0][3, 1, 1, 1], tp[0][0][5, 2, 0, 0] = np.inf, np.float32(3.4e38)
    x[:, 2] = np.minimum(x[:, 2], np.float32(0.5))          # (times 3.4e38: a number)
    monkeypatch.setenv("PBKD_CONV_ROWS", "1")
    if tile >= 0:
        monkeypatch.setenv("PBKD_CONV_TILE", str(tile))
    blk = pb.Block(t, tp, s, sp)
    xd = torch.from_numpy(x).cuda()
    out = torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda")
    for mode in (0, 1):
        pb.network_forward([blk], [0], xd, [out], bn_mode=mode)
        torch.cuda.synchronize()
        a = x
        for l, (_, shp, _) in enumerate(_layer_act_shapes(t)):
            got = blk.get_tensor(pb.TEACHER_ACT, l, 1, shp)
            st, (ho, wo) = strides[l], shp[2:]
            xp = np.pad(a.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
            want = np.zeros((chans[l + 1], n * ho * wo))
            with np.errstate(all="ignore"):
                for tap in range(9):
                    i, j = tap // 3, tap % 3
                    part = xp[:, :, i:i + st * (ho - 1) + 1:st, j:j + st * (wo - 1) + 1:st].transpose(1, 0, 2, 3).reshape(chans[l], -1)
                    want += tp[l][0][:, :, i, j].astype(np.float64) @ part
                want = want.astype(np.float32).reshape(chans[l + 1], n, ho, wo).transpose(1, 0, 2, 3)
                same_nonfinite(got, want, (mode, l))
                sc, sh = (blk.get_tensor(pb.TEACHER_ACT, l, k, (chans[l + 1],))[None, :, None, None].astype(np.float64) for k in (4, 5))
                a = np.fmax((got * sc + sh).astype(np.float32), 0)          # fmaxf: a NaN becomes 0
    blk.close()


@pytest.mark.parametrize("env,n,h,w_,chans", [({"PBKD_CONV_WINO": "1"}, 4, 8, 12, (48, 32)), ({"PBKD_CONV_WINO": "1"}, 6, 13, 11, (18, 70)),
                                              ({"PBKD_CONV_WINO": "1"}, 40, 2, 2, (300, 64)), ({"PBKD_CONV_WINO": "0"}, 4, 8, 12, (48, 32)),
                                              ({"PBKD_CONV_WINO": "0"}, 3, 13, 15, (40, 72)), ({"PBKD_CONV_ROWS": "1"}, 5, 7, 7, (300, 130))])
def test_a_nan_in_the_input_of_a_convolution_stays_one(gpu, monkeypatch, env, n, h, w_, chans):
    """NaNs in a block's input, beside an infinity: every output of the first layer that they reach is a NaN, the others are what
    plain products make of them, on transformed tiles, aligned maps and stacked rows."""
    torch, pb = gpu
    t, s = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans))), wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)))
    x, tp, sp = wl.Workload("nan_input", t, s, seed=47).tensors(random_affine=True)
    rng = np.random.default_rng(11)
    for v in (np.nan, np.nan) + ((np.inf,) if env != {"PBKD_CONV_WINO": "0"} or w_ % 4 else ()):
        x[rng.integers(n), rng.integers(chans[0]), rng.integers(h), rng.integers(w_)] = v
    x[0, -1, 0, 0] = x[-1, 0, -1, -1] = np.nan
    for name, value in env.items():
        monkeypatch.setenv(name, value)
    blk = pb.Block(t, tp, s, sp)
    xd, out = torch.from_numpy(x).cuda(), torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda")
    blk.teacher_forward(xd, out)
    got = blk.get_tensor(pb.TEACHER_ACT, 0, 1, (n, chans[1], h, w_))
    blk.close()
    xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
    want = np.zeros((chans[1], n * h * w_))
    with np.errstate(all="ignore"):
        for tap in range(9):
            i, j = tap // 3, tap % 3
            want += tp[0][0][:, :, i, j].astype(np.float64) @ xp[:, :, i:i + h, j:j + w_].transpose(1, 0, 2, 3).reshape(chans[0], -1)
    same_nonfinite(got, want.astype(np.float32).reshape(chans[1], n, h, w_).transpose(1, 0, 2, 3), env)


# whole-image, several and ragged workgroup tiles (a tile has 64 2x2 output tiles), odd heights and widths (half-empty 2x2 tiles;
# 16-, 8- and 4-byte stores), images that end inside a workgroup tile, a last chunk of 16 channels that reaches back, K split
# (7x7, 4x4), maps of one row, one column and more than 128 rows
TRANSFORMED = [(3, (40, 72, 33), 14, 14), (4, (67, 100, 67), 27, 23), (5, (300, 130, 20), 7, 7), (2, (17, 16, 70), 5, 131), (6, (18, 20, 16), 13, 1),
               (9, (16, 33, 16), 1, 11), (20, (64, 48, 32), 4, 4), (2, (48, 64, 65), 16, 32), (1, (16, 31, 16), 150, 3), (3, (32, 16, 16), 40, 36),
               (33, (16, 64, 16), 2, 2), (1, (16, 128, 128), 12, 16)]


@pytest.mark.parametrize("n,chans,h,w_", TRANSFORMED + [(6, (16, 19, 40), 13, 11), (9, (64, 200, 96), 7, 7), (4, (48, 32, 130), 8, 12), (40, (48, 64, 64), 2, 2)])
def test_forced_transformed_tiles_run(gpu, monkeypatch, n, chans, h, w_):
    """The shapes of the tests below do run on transformed tiles when these are forced, and their pre-activations differ from the
    other kernels' in rounding."""
    torch, pb = gpu
    t, s = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans))), wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)))
    x, tp, sp = wl.Workload("forced", t, s, seed=7).tensors(random_affine=True)
    monkeypatch.setenv("PBKD_CONV_ROWS", "1")
    xd, td, z = torch.from_numpy(x).cuda(), torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda"), []
    for wino in ("0", "1"):
        monkeypatch.setenv("PBKD_CONV_WINO", wino)
        assert all((pb.arch_conv_kernel(t, l)[0] == "transformed") == (wino == "1") for l in range(2))
        blk = pb.Block(t, tp, s, sp)
        blk.teacher_forward(xd, td)
        z.append([blk.get_tensor(pb.TEACHER_ACT, l, 1, shp) for l, (_, shp, _) in enumerate(_layer_act_shapes(t))])
        blk.close()
    assert all((a != b).any() for a, b in zip(*z))


@pytest.mark.parametrize("wgs", [0, 1, 3])
@pytest.mark.parametrize("n,chans,h,w_", TRANSFORMED)
def test_transformed_tiles_on_any_map(gpu, monkeypatch, n, chans, h, w_, wgs):
    """Teacher forward on transformed 2x2 tiles, forced: every layer's pre-activation and statistics against the fp64 oracle at
    ACT_TOL, with a workgroup per tile and with one and three workgroups that walk all of them."""
    monkeypatch.setenv("PBKD_CONV_WINO", "1")
    test_split_convolution_on_any_map(gpu, monkeypatch, n, chans, h, w_, (1, 1), wgs)


@pytest.mark.parametrize("n,h,w_,chans", [(6, 13, 11, (16, 19, 40)), (9, 7, 7, (64, 200, 96)), (4, 8, 12, (48, 32, 130)), (40, 2, 2, (48, 64, 64))])
def test_transformed_tiles_infinities(gpu, monkeypatch, n, h, w_, chans):
    """Infinities and numbers past bfloat16's largest through the transformed tiles: what plain products make of them, also in the
    outputs that share a window with one without depending on it."""
    monkeypatch.setenv("PBKD_CONV_WINO", "1")
    test_stacked_rows_infinities(gpu, monkeypatch, n, h, w_, chans, (1, 1), -1)


@pytest.mark.parametrize("kind", ["plain", "small_variance", "large_channel_off", "large_mean"])
@pytest.mark.parametrize("n,h,w_,chans", [(24, 16, 16, (128, 256, 96)), (2, 56, 56, (64, 64, 64)), (64, 4, 4, (512, 512, 256)), (3, 36, 40, (118, 48, 32)),
                                          (8, 12, 20, (16, 32, 24))])
def test_transformed_tiles_are_no_less_accurate_than_the_direct_kernel(gpu, monkeypatch, n, h, w_, chans, kind):
    """On the maps where the transformed tiles stand in for the aligned direct kernel their rms error against fp64 must not be
    the larger one.  A sum's roundings at its own size: 6 per 16 channels for 54, and 1.75 times a sum's error passes through the
    output transform: 1.75 sqrt(6 / 54) = 0.58 of the direct kernel's, plus what does not grow with the channels (the two
    roundings of B^T d B and of the transform back, 0.9e-7 in all: as much as 16 channels leave the direct kernel, whose sums
    are then exact in part: 5 % for that)."""
    t, s = wl.Arch(n, chans[0], h, w_, wl._convs(list(chans))), wl.Arch(n, chans[0], h, w_, wl._dws(list(chans)))
    w = wl.Workload("transformed_accuracy", t, s, seed=27)
    x, tp, _ = w.tensors(random_affine=True)
    x = np.maximum(x, 0) + np.float32(30 if kind == "large_mean" else 0)
    if kind == "small_variance":
        tp[0][0] = tp[0][0] * np.float32(1e-5)
        tp[0][2] = np.zeros_like(tp[0][2])
    if kind == "large_channel_off":
        tp[1][0] = tp[1][0].copy()
        tp[1][0][:, 0] *= np.float32(1e6)
        tp[0][2] = tp[0][2].copy()
        tp[0][2][0] = -1e3
    errs = {}
    for wino in (0, 1):
        monkeypatch.setenv("PBKD_CONV_WINO", str(wino))
        errs[wino] = teacher_layer_errors(gpu, w, tp, x)
    print(f"[transformed tiles accuracy] {kind} {chans} {h}x{w_}: rms error of z0, z1: direct {errs[0]}, transformed {errs[1]}")
    for a, b in zip(errs[0], errs[1]):
        assert b <= 1.05 * a, errs


def conv3x3_fp64(x, w):
    n, c, h, wd = x.shape
    xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
    z = np.zeros((w.shape[0], n * h * wd))
    for tap in range(9):
        i, j = tap // 3, tap % 3
        z += w[:, :, i, j].astype(np.float64) @ xp[:, :, i:i + h, j:j + wd].transpose(1, 0, 2, 3).reshape(c, -1)
    return z.reshape(w.shape[0], n, h, wd).transpose(1, 0, 2, 3)


@pytest.mark.parametrize("n,h,w_,ci,co", [(2, 12, 16, 64, 48), (3, 13, 11, 40, 72), (20, 4, 4, 300, 33)])
def test_transformed_tiles_error_is_relative_to_window_and_filter(gpu, monkeypatch, n, h, w_, ci, co):
    """Pixels 1e5 times the others, taps that are zero or a thousandth of the others: an error of the transformed tiles is at most
    2^-24 of 64 (11 + 6 channels / 16) times the window's largest pixel x the filter's largest tap, summed over the channels
    (conv_wino_kernel.h derives it), and so much larger than the direct kernel's where only such taps meet such pixels: that
    kernel's is at most 2^-24 of (27 channels / 8 + 5) times the sum of its own products' sizes (27 roundings per eight channels;
    products left out, K split)."""
    torch, pb = gpu
    t, s = wl.Arch(n, ci, h, w_, wl._convs([ci, co])), wl.Arch(n, ci, h, w_, wl._dws([ci, co]))
    x, tp, sp = wl.Workload("uneven", t, s, seed=73).tensors(random_affine=True)
    rng = np.random.default_rng(13)
    x = np.maximum(x, 0) * np.where(rng.random(x.shape) < 0.002, np.float32(1e5), np.float32(1))
    r = rng.random(tp[0][0].shape)
    tp[0][0] = tp[0][0] * np.where(r < 0.2, 0, np.where(r < 0.4, 1e-3, 1)).astype(np.float32)
    w = tp[0][0]
    ref, products = conv3x3_fp64(x, w), conv3x3_fp64(np.abs(x), np.abs(w))
    # the window of a 2x2 tile: four rows and columns around it
    xp = np.pad(np.abs(x), ((0, 0), (0, 0), (1, 2 + h % 2), (1, 2 + w_ % 2)))
    largest = np.max([xp[:, :, i:i + h + h % 2:2, j:j + w_ + w_ % 2:2] for i in range(4) for j in range(4)], axis=0)
    tiles = np.einsum("oc,nchw->nohw", np.abs(w).max((2, 3)).astype(np.float64), largest.astype(np.float64))
    tiles = np.repeat(np.repeat(tiles, 2, 2), 2, 3)[:, :, :h, :w_]
    xd, td, worst = torch.from_numpy(x).cuda(), torch.empty(wl.output_shape(t), device="cuda"), {}
    for wino, bound in ((1, 64 * (11 + 6 * ci / 16) * tiles), (0, (27 * ci / 8 + 5) * products)):
        monkeypatch.setenv("PBKD_CONV_WINO", str(wino))
        blk = pb.Block(t, tp, s, sp)
        blk.teacher_forward(xd, td)
        err = np.abs(blk.get_tensor(pb.TEACHER_ACT, 0, 1, ref.shape) - ref)
        blk.close()
        if wino or (h * w_) % 4 == 0:
            worst[wino] = float(np.max(err / (bound * 2.0 ** -24)))
            assert worst[wino] <= 1, worst
    print(f"[uneven taps and pixels] {ci}->{co} {h}x{w_}: worst share of its bound {worst}")


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("n,c,h,w_", [(30, 80, 52, 52), (64, 272, 8, 8)])
def test_weights_that_are_mostly_zero_keep_the_direct_kernel(gpu, monkeypatch, n, c, h, w_, graph):
    """A layer whose shape asks for transformed tiles runs them with weights of which half are not zero, and the direct kernel bit
    for bit where fewer are, single taps or whole filters: at creation and after pbkd_block_set_tensor, in captured steps too,
    those of a schedule that another block owns among them."""
    torch, pb = gpu
    t, s = wl.Arch(n, c, h, w_, wl._convs([c, c])), wl.Arch(n, c, h, w_, wl._dws([c, c]))
    assert pb.arch_conv_kernel(t, 0)[0] == "transformed"
    x, tp, sp = wl.Workload("pruned", t, s, seed=79).tensors(random_affine=True)
    x = np.maximum(x, 0)
    rng = np.random.default_rng(17)
    full = tp[0][0]
    keep = np.argsort(rng.random((c, c, 9)), axis=2).reshape(full.shape)
    weights = {"all": full, "five": full * (keep < 5), "four": full * (keep < 4), "tenth": full * (rng.random(full.shape) < 0.1),
               "filters": full * (rng.random((c, c, 1, 1)) < 0.1)}
    tiles = {"all": True, "five": True, "four": False, "tenth": False, "filters": False}
    xd, td = torch.from_numpy(x).cuda(), torch.zeros(wl.output_shape(t), device="cuda")
    other = torch.zeros(wl.output_shape(t), device="cuda")
    st = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()

    def labels(w, wino):
        if wino is None:
            monkeypatch.delenv("PBKD_CONV_WINO", raising=False)
        else:
            monkeypatch.setenv("PBKD_CONV_WINO", wino)
        blk = pb.Block(t, [[w] + tp[0][1:]], s, sp)
        blk.teacher_forward(xd, td)
        torch.cuda.synchronize()
        blk.close()
        return td.cpu().numpy()

    want = {name: labels(w, "1" if tiles[name] else "0") for name, w in weights.items()}
    for name, w in weights.items():
        assert (labels(w, "0" if tiles[name] else "1") != want[name]).any(), name
        np.testing.assert_array_equal(labels(w, None), want[name], err_msg=name)
    monkeypatch.delenv("PBKD_CONV_WINO", raising=False)
    blk, first = (pb.Block(t, tp, s, sp) for _ in range(2))
    for b in (blk, first):
        b.set_graph_mode(graph)
    for name in ("all", "tenth", "filters", "four", "five", "all"):
        blk.set_tensor(pb.TEACHER_PARAM, 0, 0, weights[name])
        for call in range(2):
            for all_at_once in (False, True):
                td.zero_()
                torch.cuda.synchronize()
                if all_at_once:
                    pb.distill_step_all([first, blk], [xd, xd], [other, td], 0.0, st, [0, 1], [0, 0], False, None)
                else:
                    blk.teacher_forward(xd, td, stream=st[0])
                torch.cuda.synchronize()
                np.testing.assert_array_equal(td.cpu().numpy(), want[name], err_msg=f"{name} {call} {all_at_once}")
    blk.close()
    first.close()


def test_batchnorm_parameters_replaced_rescale_the_layer_behind(gpu):
    """pbkd_block_set_tensor on a teacher's gamma and beta, by seven orders of magnitude: the convolution behind follows."""
    torch, pb = gpu
    t, s = wl.Arch(3, 12, 10, 10, wl._convs([12, 20, 17])), wl.Arch(3, 12, 10, 10, wl._dws([12, 20, 17]))
    x, tp, sp = wl.Workload("rescale", t, s, seed=3).tensors(random_affine=True)
    blk = pb.Block(t, tp, s, sp)
    tp[0][1] = tp[0][1] * np.float32(3e7)
    tp[0][2] = tp[0][2] * np.float32(1e-3)
    for slot in (1, 2):
        blk.set_tensor(pb.TEACHER_PARAM, 0, slot, tp[0][slot])
    t_ref = ob.block_forward(t, tp, x)
    xd = torch.from_numpy(x).cuda()
    td = torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda")
    blk.teacher_forward(xd, td)
    torch.cuda.synchronize()
    assert relerr(td.cpu().numpy(), t_ref) <= ACT_TOL
    blk.close()


def test_zero_loss_when_student_is_the_factored_teacher(gpu):
    torch, pb = gpu
    chans = [6, 8, 5]
    t_arch = wl.Arch(3, 6, 8, 8, [wl.Layer(wl.CONV3X3, ci, co, 2 if i == 0 else 1, 0) for i, (ci, co) in enumerate(zip(chans[:-1], chans[1:]))],
                     shortcut=1, shortcut_stride=2, pool=2)
    s_arch = wl.Arch(3, 6, 8, 8, [wl.Layer(wl.DWSEP3X3, ci, co, 2 if i == 0 else 1, 1) for i, (ci, co) in enumerate(zip(chans[:-1], chans[1:]))],
                     shortcut=1, shortcut_stride=2, pool=2)
    sp = wl.make_params(s_arch, 1, True)
    tp = []
    for l in range(2):
        D, P, g, b = sp[l]
        tp.append([(P[:, :, None, None] * D[None, :, 0]).astype(np.float32), g.copy(), b.copy()])
    tp.append([q.copy() for q in sp[2]])
    x = wl.make_input(t_arch, 5)
    blk = pb.Block(t_arch, tp, s_arch, sp)
    xd = torch.from_numpy(x).cuda()
    td = torch.empty(wl.output_shape(t_arch), dtype=torch.float32, device="cuda")
    blk.teacher_forward(xd, td)
    loss = blk.student_step(xd, td, 0.1)
    # fp32 rounding of P*D and of two differently ordered sums: activations are O(1), so the mean squared
    # difference sits at the fp32 epsilon squared times a modest factor
    assert 0.0 <= loss < 1e-10, loss
    after = blk.student_params()
    for lp, lq in zip(after, sp):
        for a, b in zip(lp, lq):
            assert np.abs(a - b).max() < 1e-5
    blk.close()


def test_checkpoint_resume_is_bit_exact(gpu):
    torch, pb = gpu
    w = wl.small_variants()[1]
    x, tp, sp = w.tensors(random_affine=True)
    xd = torch.from_numpy(x).cuda()
    td = torch.empty(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda")
    a = pb.Block(w.teacher, tp, w.student, sp, momentum=0.9)
    a.teacher_forward(xd, td)
    for _ in range(10):
        a.student_step(xd, td, 0.02)
    ten = a.student_params()
    b = pb.Block(w.teacher, tp, w.student, sp, momentum=0.9)
    for _ in range(5):
        b.student_step(xd, td, 0.02)
    shapes = wl.param_shapes(w.student)
    saved_p = b.student_params()
    saved_v = [[b.get_tensor(pb.STUDENT_MOMENTUM, l, k, shp) for k, shp in enumerate(lp)] for l, lp in enumerate(shapes)]
    c = pb.Block(w.teacher, tp, w.student, sp, momentum=0.9)
    for l, lp in enumerate(shapes):
        for k, _ in enumerate(lp):
            c.set_tensor(pb.STUDENT_PARAM, l, k, saved_p[l][k])
            c.set_tensor(pb.STUDENT_MOMENTUM, l, k, saved_v[l][k])
    for _ in range(5):
        c.student_step(xd, td, 0.02)
    for lp, lq in zip(c.student_params(), ten):
        for p, q in zip(lp, lq):
            np.testing.assert_array_equal(p, q)
    for blk in (a, b, c):
        blk.close()


def test_create_errors(gpu):
    torch, pb = gpu
    import ctypes
    w = wl.cfg1_tiny()
    x, tp, sp = w.tensors()
    ta, sa = pb.make_arch(w.teacher), pb.make_arch(w.student)
    need = pb.workspace_bytes(w.teacher, w.student)
    ws = torch.empty(need + 512, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) & ~255
    tpa, k1 = pb._params_array(tp)
    spa, k2 = pb._params_array(sp)
    train = pb.TrainDesc(0.9, 0)
    h = ctypes.c_void_p()
    L = pb.lib()
    st = L.pbkd_block_create(ctypes.byref(ta), tpa, ctypes.byref(sa), spa, ctypes.byref(train), ctypes.c_void_p(base), need - 256,
                             None, ctypes.byref(h))
    assert st == pb.ENOMEM and "smaller" in pb.last_error()
    st = L.pbkd_block_create(ctypes.byref(ta), tpa, ctypes.byref(sa), spa, ctypes.byref(train), ctypes.c_void_p(base + 4), need,
                             None, ctypes.byref(h))
    assert st == pb.ENOMEM
    bad_train = pb.TrainDesc(1.5, 0)
    st = L.pbkd_block_create(ctypes.byref(ta), tpa, ctypes.byref(sa), spa, ctypes.byref(bad_train), ctypes.c_void_p(base), need,
                             None, ctypes.byref(h))
    assert st == pb.EINVAL
    st = L.pbkd_block_create(ctypes.byref(ta), tpa, ctypes.byref(sa), spa, ctypes.byref(train), ctypes.c_void_p(base), need,
                             None, ctypes.byref(h))
    assert st == pb.OK
    loss = ctypes.c_float()
    assert L.pbkd_block_last_loss(h, ctypes.byref(loss)) == pb.ESTATE
    assert L.pbkd_teacher_forward(h, None, None, None) == pb.EINVAL
    buf = np.empty(3, np.float32)
    assert L.pbkd_block_get_tensor(h, pb.STUDENT_PARAM, 0, 0, buf.ctypes.data_as(ctypes.POINTER(ctypes.c_float)), 3) == pb.ESHAPE
    assert L.pbkd_block_get_tensor(h, pb.STUDENT_PARAM, 9, 0, buf.ctypes.data_as(ctypes.POINTER(ctypes.c_float)), 3) == pb.EINVAL
    # running statistics have two slots; activations and gradients cannot be set
    c = np.empty(16, np.float32)
    cp = c.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
    assert L.pbkd_block_get_tensor(h, pb.STUDENT_BN_RUNNING, 0, 1, cp, 16) == pb.OK and np.all(c == 1)
    assert L.pbkd_block_get_tensor(h, pb.TEACHER_BN_RUNNING, 0, 2, cp, 16) == pb.EINVAL
    assert L.pbkd_block_set_tensor(h, pb.STUDENT_ACT, 0, 2, cp, 16) == pb.EINVAL
    assert L.pbkd_block_set_tensor(h, pb.STUDENT_GRAD, 0, 2, cp, 16) == pb.EINVAL
    # device tensors must be 16-byte aligned: refused before anything is launched
    xd = torch.zeros(4 * 16 * 16 * 16 + 4, dtype=torch.float32, device="cuda")
    td = torch.zeros(4 * 16 * 16 * 16 + 4, dtype=torch.float32, device="cuda")
    xp, tpd = ctypes.c_void_p(xd.data_ptr()), ctypes.c_void_p(td.data_ptr())
    xo, to = ctypes.c_void_p(xd.data_ptr() + 4), ctypes.c_void_p(td.data_ptr() + 4)
    assert L.pbkd_teacher_forward(h, xo, tpd, None) == pb.EINVAL and "aligned" in pb.last_error()
    assert L.pbkd_student_step(h, xp, to, ctypes.c_float(0.1), None, None) == pb.EINVAL
    assert L.pbkd_distill_step(h, xo, tpd, ctypes.c_float(0.1), None, None, None) == pb.EINVAL
    assert L.pbkd_block_last_loss(h, ctypes.byref(loss)) == pb.ESTATE      # none of the refused calls ran a step
    assert L.pbkd_teacher_forward(h, xp, tpd, None) == pb.OK
    torch.cuda.synchronize()
    L.pbkd_block_destroy(h)
    bad_decay = pb.TrainDesc(0.9, 0, 1.0)
    st = L.pbkd_block_create(ctypes.byref(ta), tpa, ctypes.byref(sa), spa, ctypes.byref(bad_decay), ctypes.c_void_p(base), need,
                             None, ctypes.byref(h))
    assert st == pb.EINVAL and "bn_decay" in pb.last_error()


def _all_blocks_setup(gpu, ws, tensors, n_streams, policy):
    torch, pb = gpu
    blocks = [pb.Block(w.teacher, tp, w.student, sp, momentum=w.momentum) for w, (x, tp, sp) in zip(ws, tensors)]
    x0 = torch.from_numpy(tensors[0][0]).cuda()
    ts = [torch.empty(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda") for w in ws]
    xs = [x0] + ts[:-1]
    streams = [torch.cuda.Stream() for _ in range(n_streams)]
    tstream = torch.cuda.Stream()
    sob, order, load = pb.schedule_blocks(None, n_streams, policy, blocks=blocks)
    torch.cuda.synchronize()
    return blocks, xs, ts, streams, tstream, sob, order


def test_all_vgg16_blocks_concurrently(gpu):
    """The whole CIFAR-shaped VGG16 at batch 128: the teacher chain feeds every block, the five student
    blocks train independently on three streams assigned by worst-fit-decreasing; ten steps against the
    oracle, and the result must not depend on the number of streams or the policy (blocks share nothing)."""
    torch, pb = gpu
    from oracle import schedule as osched
    ws = wl.cfg5_vgg16_blocks()
    tensors = [w.tensors() for w in ws]
    steps, lr = 10, 0.01
    tallies = [DecisionTally() for _ in ws]
    blocks, xs, ts, streams, tstream, sob, order = _all_blocks_setup(gpu, ws, tensors, 3, 0)
    weights = [osched.block_weight(w.teacher, w.student) for w in ws]
    assert sob == osched.wfd(weights, 3)[0]
    # oracle chain: block k's input is the fp32-rounded oracle output of block k-1
    refs, x_ref, t_ref = [], [], []
    x = tensors[0][0]
    for w, (_, tp, sp) in zip(ws, tensors):
        ref = ob.RefBlock(w.teacher, tp, w.student, sp, momentum=w.momentum)
        t = ref.teacher_forward(x)
        refs.append(ref); x_ref.append(x); t_ref.append(t)
        x = t.astype(np.float32)
    fails = {}
    losses = []
    for s in range(steps):
        pb.distill_step_all(blocks, xs, ts, lr, streams, sob, order, True, tstream)
        torch.cuda.synchronize()
        losses.append([b.last_loss() for b in blocks])
        for b, (w, ref) in enumerate(zip(ws, refs)):
            if s == 0:
                e = relerr(ts[b].cpu().numpy(), t_ref[b])
                if not e <= ACT_TOL:
                    fails[f"block{b}.target"] = e
            l_ref = ref.student_step(x_ref[b], t_ref[b].astype(np.float32), lr, decisions=gpu_decisions(pb, blocks[b], w.student))
            tallies[b].add(ref.cache)
            e = abs(losses[s][b] - l_ref) / abs(l_ref)
            if not e <= ACT_TOL:
                fails[f"block{b}.loss[{s}]"] = (e, losses[s][b], l_ref)
    params = [b.student_params() for b in blocks]
    for b, ref in enumerate(refs):
        for l, (lp, lr_) in enumerate(zip(params[b], ref.sp)):
            for k, (a, r) in enumerate(zip(lp, lr_)):
                e = relerr(a, r)
                if not e <= GRAD_TOL:
                    fails[f"block{b}.weights[{l}][{k}]"] = e
    for b in blocks:
        b.close()
    for b, tally in enumerate(tallies):
        print(f"[parity] cfg5 block {b}: {steps} steps, {tally.differing} of {tally.total} decisions taken differently, "
              f"farthest from the kink {tally.worst_rel:.2e} of max|b|", flush=True)
        for k, v in tally.failures().items():
            fails[f"block{b}.{k}"] = v
    assert not fails, fails
    # same work on one stream, round robin: bit-identical (deterministic reductions, no shared state)
    blocks1, xs1, ts1, streams1, tstream1, sob1, order1 = _all_blocks_setup(gpu, ws, tensors, 1, 1)
    losses1 = []
    for s in range(steps):
        pb.distill_step_all(blocks1, xs1, ts1, lr, streams1, sob1, order1, True, tstream1)
        losses1.append([b.last_loss() for b in blocks1])
    assert losses1 == losses
    for pa, blk1 in zip(params, blocks1):
        for lp, lq in zip(pa, blk1.student_params()):
            for a, c in zip(lp, lq):
                np.testing.assert_array_equal(a, c)
    for b in blocks1:
        b.close()
    # two sets of target buffers taken in turn and no host synchronisation between the steps: the next step's teacher
    # chain then runs ahead of this step's students (a teacher launch waits only for the steps that read the buffer it
    # overwrites); same bits again
    blocks2, xs2, ts2, streams2, tstream2, sob2, order2 = _all_blocks_setup(gpu, ws, tensors, 3, 0)
    ts2b = [torch.empty_like(t) for t in ts2]
    sets = [(xs2, ts2), ([xs2[0]] + ts2b[:-1], ts2b)]
    for s in range(steps):
        xs_, ts_ = sets[s % 2]
        pb.distill_step_all(blocks2, xs_, ts_, lr, streams2, sob2, order2, True, tstream2)
    torch.cuda.synchronize()
    assert [b.last_loss() for b in blocks2] == losses[-1]
    for pa, blk2 in zip(params, blocks2):
        for lp, lq in zip(pa, blk2.student_params()):
            for a, c in zip(lp, lq):
                np.testing.assert_array_equal(a, c)
    for b in blocks2:
        b.close()


def test_distill_step_on_two_streams_is_bit_identical(gpu, monkeypatch):
    """pbkd_distill_step overlaps teacher and student on two streams; its results must be those of
    pbkd_teacher_forward + pbkd_student_step on one stream, bit for bit, over several consecutive steps
    (the teacher of step i+1 runs while the student of step i is still in its backward pass), also with the teacher
    held back until the student step before the previous one has ended (PBKD_TEACHER_LAG=1)."""
    torch, pb = gpu
    w = wl.cfg2_vgg_block2()
    x, tp, sp = w.tensors()
    xd = torch.from_numpy(x).cuda()
    results = []
    for mode in ("one_stream", "two_streams", "two_streams_teacher_lag"):
        if mode == "two_streams_teacher_lag":
            monkeypatch.setenv("PBKD_TEACHER_LAG", "1")
        else:
            monkeypatch.delenv("PBKD_TEACHER_LAG", raising=False)
        blk = pb.Block(w.teacher, tp, w.student, sp, momentum=w.momentum)
        td = torch.zeros(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda")
        s1, s2, s3 = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
        if mode == "two_streams":
            blk.set_aux_stream(s3)      # weight gradients on a third stream
        torch.cuda.synchronize()
        losses = []
        for step in range(6):
            if mode != "one_stream":
                blk.distill_step(xd, td, w.lr, want_loss=False, student_stream=s1, teacher_stream=s2)
            else:
                blk.teacher_forward(xd, td, stream=s1)
                blk.student_step(xd, td, w.lr, want_loss=False, stream=s1)
            if step in (2, 5):
                losses.append(blk.last_loss())
        torch.cuda.synchronize()
        results.append((losses, [np.concatenate([a.ravel() for a in lp]) for lp in blk.student_params()], td.cpu().numpy()))
        blk.close()
    monkeypatch.delenv("PBKD_TEACHER_LAG", raising=False)
    l0, p0, t0 = results[0]
    for l1, p1, t1 in results[1:]:
        assert l0 == l1
        assert np.array_equal(t0, t1)
        for a, b in zip(p0, p1):
            assert np.array_equal(a, b)


AUX_BLOCKS = {  # channels, first layer a full convolution, variables, launches a step of weight gradients of their own and with another one
    "one_kernel": ((64, 128, 128), False, {}, {"pw_bwd": 2}),
    "first_in_one_kernel": ((3, 32, 64), True, {}, {"pw_bwd": 1, "first_bwd": 1}),
    "apart": ((64, 160, 192, 144), False, {}, {"pw_wgrad_mfma": 3}),
    "made_apart": ((3, 64, 128, 64), True, {"PBKD_PW_BWD": "0", "PBKD_FIRST_BWD": "0"}, {"pw_wgrad_mfma": 2, "conv3x3_wgrad": 1}),
    "mixed": ((64, 128, 160, 128), False, {}, {"pw_bwd": 2, "pw_wgrad_mfma": 1}),
    "mixed_first": ((3, 32, 160, 64), True, {}, {"pw_bwd": 1, "pw_wgrad_mfma": 1, "first_bwd": 1})}


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("name", AUX_BLOCKS)
def test_auxiliary_stream_is_bit_identical(gpu, monkeypatch, name, graph):
    """Six steps with an auxiliary stream, alone and beside the teacher, eager and captured: bit for bit those on one stream, where both
    gradients of every layer come from one kernel, from two, and in turn.  The stream gets work exactly where there is a weight
    gradient of its own: while the step's stream is kept busy it is idle otherwise (a captured step puts none on it)."""
    torch, pb = gpu
    chans, full, env, launches = AUX_BLOCKS[name]
    used = any(k.endswith(("wgrad", "wgrad_mfma")) for k in launches)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    layers = wl._dws(list(chans))
    if full:
        layers[0] = wl.Layer(wl.CONV3X3, chans[0], chans[1], 1, 1)
    t, s = wl.Arch(160, chans[0], 16, 16, wl._convs(list(chans))), wl.Arch(160, chans[0], 16, 16, layers)
    w = wl.Workload("aux", t, s, seed=19)
    x, tp, sp = w.tensors()
    xd = torch.from_numpy(x).cuda()
    results = []
    for mode in ("plain", "aux", "aux_two_streams"):
        s1, s2, s3 = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
        td = torch.zeros(wl.output_shape(t), device="cuda")
        blk = pb.Block(t, tp, s, sp, momentum=w.momentum)
        blk.set_graph_mode(graph)
        if mode != "plain":
            blk.set_aux_stream(s3)
        torch.cuda.synchronize()
        for step in range(6):
            blk.distill_step(xd, td, w.lr, want_loss=False, student_stream=s1, teacher_stream=s2 if mode == "aux_two_streams" else s1)
        torch.cuda.synchronize()
        results.append([blk.last_loss()] + [a for lp in blk.student_params() for a in lp])
        if mode == "aux" and not graph:
            with torch.cuda.stream(s1):
                torch.cuda._sleep(100_000_000)
            blk.student_step(xd, td, w.lr, want_loss=False, stream=s1)
            assert not s1.query() and s3.query() == (not used)
            torch.cuda.synchronize()
            blk.profile_enable(["pw_bwd", "first_bwd", "pw_wgrad_mfma", "conv3x3_wgrad"], 8)
            blk.student_step(xd, td, w.lr, want_loss=False, stream=s1)
            assert {k: n for k, (_, n) in blk.profile_read().items()} == launches
        blk.close()
    for got in results[1:]:
        for a, b in zip(got, results[0]):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("n,c,h,w_", [(96, 144, 20, 24), (84, 48, 40, 40), (64, 272, 8, 8)])
def test_transformed_tiles_beside_other_streams_are_bit_identical(gpu, n, c, h, w_, graph):
    """Beside other streams' kernels the transformed tiles run on fewer workgroups (more tiles than these here, with and without
    K split): labels and trained students of two blocks are bit for bit those of calls on one stream, from pbkd_distill_step on
    two streams, from all blocks at once, chained and not, and from whole tasks, eager and captured."""
    torch, pb = gpu
    t, s = wl.Arch(n, c, h, w_, wl._convs([c, c])), wl.Arch(n, c, h, w_, wl._dws([c, c]))
    assert pb.arch_conv_kernel(t, 0)[0] == "transformed"
    ws = [wl.Workload("beside", t, s, seed=71 + k) for k in range(2)]
    params = [w.tensors(random_affine=True) for w in ws]
    xd = torch.from_numpy(np.maximum(params[0][0], 0)).cuda()
    st = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    got = {}
    for mode in ("one", "two", "chain", "all", "tasks"):
        blocks = [pb.Block(t, tp, s, sp) for _, tp, sp in params]
        td = [torch.zeros(wl.output_shape(t), device="cuda") for _ in range(2)]
        xs = [xd, td[0] if mode == "chain" else xd]
        torch.cuda.synchronize()
        for b in blocks:
            b.set_graph_mode(graph)
        for _ in range(3):
            if mode in ("one", "two"):
                for b, o in zip(blocks, td):
                    b.distill_step(xd, o, 0.01, want_loss=False, student_stream=st[0], teacher_stream=st[0 if mode == "one" else 1])
            elif mode == "tasks":
                pb.run_tasks_work_stealing(blocks, xs, td, 0.01, [1, 1], st[:2], [0, 1])
            else:
                pb.distill_step_all(blocks, xs, td, 0.01, st[:2], [0, 1], [0, 0], mode == "chain", st[2] if mode == "chain" else None)
            torch.cuda.synchronize()
        got[mode] = [o.cpu().numpy() for o in td] + [a.copy() for b in blocks for lp in b.student_params() for a in lp]
        if mode == "chain":                      # (the second block's input is the first one's labels there)
            blocks[1].teacher_forward(td[0], td[1])
            torch.cuda.synchronize()
            np.testing.assert_array_equal(got[mode][1], td[1].cpu().numpy())
        for b in blocks:
            b.close()
    first = 1 + 1 + len([a for lp in params[0][2] for a in lp])
    for mode in ("two", "chain", "all", "tasks"):
        for k, (a, b) in enumerate(zip(got[mode], got["one"])):
            if mode != "chain" or k == 0 or 2 <= k < first:
                np.testing.assert_array_equal(a, b, err_msg=f"{mode} {k}")


@pytest.mark.parametrize("name", ["cfg1", "ragged_residual_s2", "three_layers_skip_pool", "cfg2"])
def test_graph_mode_replays_are_bit_identical_to_eager_steps(gpu, name):
    """pbkd_block_set_graph_mode: the captured step is replayed several times, with the program's own eager work and
    synchronisations between the replays, and every replay must leave exactly what the eager step leaves: losses, the
    teacher's target, and all weights.  One-stream steps (pbkd_teacher_forward + pbkd_student_step), the two-stream
    pbkd_distill_step, and a change of learning rate (a second capture) are all covered."""
    torch, pb = gpu
    w = {"cfg1": wl.cfg1_tiny(), "cfg2": wl.cfg2_vgg_block2(n=32)}.get(name) or {v.name: v for v in wl.small_variants()}[name]
    x, tp, sp = w.tensors(random_affine=True)
    xd = torch.from_numpy(x).cuda()
    lrs = [0.01, 0.01, 0.01, 0.02, 0.02, 0.01, 0.01]
    results = []
    for mode in ("eager", "graph_one_stream", "graph_two_streams"):
        blk = pb.Block(w.teacher, tp, w.student, sp, momentum=w.momentum)
        td = torch.zeros(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda")
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        blk.set_graph_mode(mode != "eager")
        torch.cuda.synchronize()
        losses, targets = [], []
        for step, lr in enumerate(lrs):
            if mode == "graph_two_streams":
                blk.distill_step(xd, td, lr, want_loss=False, student_stream=s1, teacher_stream=s2)
            else:
                blk.teacher_forward(xd, td, stream=s1)
                blk.student_step(xd, td, lr, want_loss=False, stream=s1)
            # eager work and a synchronisation between the replays
            losses.append(blk.last_loss())
            with torch.cuda.stream(s1):
                targets.append(float(td.double().sum().item()))
        torch.cuda.synchronize()
        results.append((losses, targets, [np.concatenate([a.ravel() for a in lp]) for lp in blk.student_params()],
                        [blk.get_tensor(pb.STUDENT_BN_RUNNING, 0, k, (w.student.layers[0].cout,)) for k in (0, 1)]))
        blk.close()
    ref = results[0]
    assert ref[0][0] != ref[0][-1]                      # the steps did train
    for got in results[1:]:
        assert got[0] == ref[0]
        assert got[1] == ref[1]
        for a, b in zip(got[2], ref[2]):
            assert np.array_equal(a, b)
        for a, b in zip(got[3], ref[3]):
            assert np.array_equal(a, b)


def test_graph_mode_all_block_step_is_bit_identical(gpu):
    """pbkd_distill_step_all with every block in graph mode: the whole teacher chain + five student steps as one
    graph, replayed with eager work between the replays, against the same steps issued eagerly (batch 16)."""
    torch, pb = gpu
    ws = wl.cfg5_vgg16_blocks(n=16)
    tensors = [w.tensors() for w in ws]
    out = []
    for graph in (False, True):
        blocks, xs, ts, streams, tstream, sob, order = _all_blocks_setup(gpu, ws, tensors, 3, 0)
        for b in blocks:
            b.set_graph_mode(graph)
        losses = []
        for s in range(5):
            pb.distill_step_all(blocks, xs, ts, 0.01, streams, sob, order, True, tstream)
            losses.append([b.last_loss() for b in blocks])
            with torch.cuda.stream(tstream):
                losses.append(float(ts[-1].double().sum().item()))
        torch.cuda.synchronize()
        out.append((losses, [[np.concatenate([a.ravel() for a in lp]) for lp in b.student_params()] for b in blocks]))
        # without a chain (every block its own stream, round robin), graph against eager as well
        xs2 = [x.clone() for x in xs]
        sob2, order2, _ = pb.schedule_blocks(None, 3, 1, blocks=blocks)
        for s in range(3):
            pb.distill_step_all(blocks, xs2, ts, 0.01, streams, sob2, order2, False, None)
        torch.cuda.synchronize()
        out[-1] = out[-1] + ([b.last_loss() for b in blocks],)
        for b in blocks:
            b.close()
    (l0, p0, n0), (l1, p1, n1) = out
    assert l0 == l1 and n0 == n1
    for pa, pb_ in zip(p0, p1):
        for a, b in zip(pa, pb_):
            assert np.array_equal(a, b)


def test_work_stealing_runs_every_task_once_with_identical_results(gpu):
    """pbkd_run_tasks_work_stealing (section 3.3): all tasks start in worker 0's queue, so the other workers
    must steal; whoever runs a task, its block ends with exactly the weights of the same steps run statically."""
    torch, pb = gpu
    ws = wl.small_variants()
    steps = [(3, 1, 4, 2, 5, 2, 1, 3)[i % 8] for i in range(len(ws))]

    def make():
        blocks, xs, ts = [], [], []
        for w in ws:
            x, tp, sp = w.tensors()
            blocks.append(pb.Block(w.teacher, tp, w.student, sp, momentum=w.momentum))
            xs.append(torch.from_numpy(x).cuda())
            ts.append(torch.empty(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda"))
        return blocks, xs, ts

    # static reference: every task on one stream, in order
    blocks, xs, ts = make()
    s0 = torch.cuda.Stream()
    for b, x, t, k, w in zip(blocks, xs, ts, steps, ws):
        for _ in range(k):
            b.teacher_forward(x, t, stream=s0)
            b.student_step(x, t, w.lr, want_loss=False, stream=s0)
    torch.cuda.synchronize()
    ref = [[np.concatenate([a.ravel() for a in lp]) for lp in b.student_params()] for b in blocks]
    ref_loss = [b.last_loss() for b in blocks]
    for b in blocks:
        b.close()

    blocks, xs, ts = make()
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    ran_on, n_steals = pb.run_tasks_work_stealing(blocks, xs, ts, ws[0].lr, steps, streams, [0] * len(ws))
    assert all(0 <= r < 3 for r in ran_on)
    assert n_steals >= 1 and len(set(ran_on)) >= 2
    for b, r, rl in zip(blocks, ref, ref_loss):
        got = [np.concatenate([a.ravel() for a in lp]) for lp in b.student_params()]
        for a, c in zip(got, r):
            assert np.array_equal(a, c)
        assert b.last_loss() == rl
        b.close()


def test_reassembled_network_forward_and_feature_error(gpu):
    """pbkd_network_forward / pbkd_feature_mse (Algorithm 1's reassembly and its evaluation, label free): the five
    VGG16 blocks at batch 16 with their seeded weights on both sides; the network with no, some and all blocks
    replaced -- every block output and the feature error against the oracle."""
    torch, pb = gpu
    ws = wl.cfg5_vgg16_blocks(n=16)
    blocks, refs, ts = [], [], []
    x0 = None
    for i, w in enumerate(ws):
        x, tp, sp = w.tensors(random_affine=True)
        blocks.append(pb.Block(w.teacher, tp, w.student, sp, momentum=w.momentum))
        refs.append(_ref_block(w, tp, sp))
        if i == 0:
            x0 = x
        ts.append(torch.empty(wl.output_shape(w.teacher), dtype=torch.float32, device="cuda"))
    xd = torch.from_numpy(x0).cuda()
    s = torch.cuda.Stream()
    t_ref = ob.network_forward(refs, [0] * 5, x0)
    outs = [torch.empty_like(t) for t in ts]
    pb.network_forward(blocks, [0] * 5, xd, ts, stream=s)
    for mask in ([0, 0, 0, 0, 0], [1, 0, 1, 0, 1], [0, 1, 0, 0, 0], [1, 1, 1, 1, 1]):
        pb.network_forward(blocks, mask, xd, outs, stream=s)
        torch.cuda.synchronize()
        want = ob.network_forward(refs, mask, x0)
        for k, (o, r) in enumerate(zip(outs, want)):
            e = relerr(o.cpu().numpy(), r)
            assert e <= ACT_TOL, (mask, k, e)
        got = pb.feature_mse(blocks[0], outs[-1], ts[-1], stream=s)
        ref = ob.feature_mse(want[-1], t_ref[-1])
        if ref == 0.0:
            assert got == 0.0, mask
        else:
            assert abs(got - ref) <= 1e-3 * ref, (mask, got, ref)
    # shapes that do not chain are refused
    with pytest.raises(Exception):
        pb.network_forward([blocks[0], blocks[2]], [0, 0], xd, [ts[0], ts[2]], stream=s)
    # inference mode: seeded running statistics on both sides (the teacher's come with its weights; the students'
    # stand for what training would have left), every mask again
    rng = np.random.default_rng(2012)
    for blk, ref in zip(blocks, refs):
        for kind, pairs in ((pb.TEACHER_BN_RUNNING, ref.t_running), (pb.STUDENT_BN_RUNNING, ref.s_running)):
            for l, pair in enumerate(pairs):
                pair[0] = (rng.normal(size=pair[0].shape) * 0.3).astype(np.float32).astype(np.float64)
                pair[1] = rng.uniform(0.5, 2.0, pair[1].shape).astype(np.float32).astype(np.float64)
                blk.set_tensor(kind, l, 0, pair[0])
                blk.set_tensor(kind, l, 1, pair[1])
    for mask in ([0, 0, 0, 0, 0], [1, 0, 1, 0, 1], [1, 1, 1, 1, 1]):
        pb.network_forward(blocks, mask, xd, outs, stream=s, bn_mode=1)
        torch.cuda.synchronize()
        want = ob.network_forward(refs, mask, x0, bn_mode=1)
        for k, (o, r) in enumerate(zip(outs, want)):
            e = relerr(o.cpu().numpy(), r)
            assert e <= ACT_TOL, ("inference", mask, k, e)
    # the batch-statistics forward still gives what it gave before, and the running pairs were only read
    pb.network_forward(blocks, [1, 0, 1, 0, 1], xd, outs, stream=s)
    torch.cuda.synchronize()
    want = ob.network_forward(refs, [1, 0, 1, 0, 1], x0)
    assert relerr(outs[-1].cpu().numpy(), want[-1]) <= ACT_TOL
    for blk, ref in zip(blocks, refs):
        for l, pair in enumerate(ref.s_running):
            assert np.array_equal(blk.get_tensor(pb.STUDENT_BN_RUNNING, l, 0, pair[0].shape), pair[0].astype(np.float32))
            assert np.array_equal(blk.get_tensor(pb.STUDENT_BN_RUNNING, l, 1, pair[1].shape), pair[1].astype(np.float32))
    with pytest.raises(Exception):
        pb.network_forward(blocks, [0] * 5, xd, outs, stream=s, bn_mode=2)
    # Algorithm 1's selection in both modes: per-block errors, the choice at a threshold inside the widest gap between
    # consecutive sorted errors (far from both of its ends), and the error of the network reassembled from the chosen blocks
    for mode in (0, 1):
        _, errs_ref, _ = ob.select_blocks(refs, x0, threshold=0.0, bn_mode=mode)
        srt = sorted(errs_ref)
        i = max(range(4), key=lambda j: srt[j + 1] / srt[j])
        assert srt[i + 1] > 1.1 * srt[i] > 0, srt
        thr = float(np.sqrt(srt[i] * srt[i + 1]))
        use_ref, _, final_ref = ob.select_blocks(refs, x0, threshold=thr, bn_mode=mode)
        use, errs, final = pb.select_blocks(blocks, xd, ts, outs, thr, stream=s, bn_mode=mode)
        assert use == use_ref and sum(use) == i + 1, (mode, use, use_ref)
        for k in range(5):
            assert abs(errs[k] - errs_ref[k]) <= 1e-3 * errs_ref[k], (mode, k, errs[k], errs_ref[k])
        assert abs(final - final_ref) <= 1e-3 * final_ref, (mode, final, final_ref)
    for b in blocks:
        b.close()


@pytest.mark.parametrize("n,h,w_,chans", [(1, 14, 14, ((40, 64, 40), (40, 72, 40))), (5, 27, 23, ((67, 100, 67), (67, 33, 20))), (2, 7, 5, ((16, 9, 16),) * 17)])
def test_inference_on_any_map(gpu, n, h, w_, chans):
    """Forward with running statistics on maps whose rows are not whole 16-byte groups, teacher's, student's and mixed blocks,
    and through more layers (34) than one launch turns running pairs into scales for: every block's output."""
    torch, pb = gpu
    blocks, refs, outs = [], [], []
    rng = np.random.default_rng(5)
    for i, ch in enumerate(chans):
        t, s = wl.Arch(n, ch[0], h, w_, wl._convs(list(ch))), wl.Arch(n, ch[0], h, w_, wl._dws(list(ch)))
        w = wl.Workload(f"inference_{i}", t, s, seed=60 + i)
        x, tp, sp = w.tensors(random_affine=True)
        if i == 0:
            x0 = x
        blocks.append(pb.Block(t, tp, s, sp))
        refs.append(_ref_block(w, tp, sp))
        outs.append(torch.empty(wl.output_shape(t), dtype=torch.float32, device="cuda"))
        for kind, pairs in ((pb.TEACHER_BN_RUNNING, refs[-1].t_running), (pb.STUDENT_BN_RUNNING, refs[-1].s_running)):
            for l, pair in enumerate(pairs):
                pair[0] = (rng.normal(size=pair[0].shape) * 0.3).astype(np.float32).astype(np.float64)
                pair[1] = rng.uniform(0.5, 2.0, pair[1].shape).astype(np.float32).astype(np.float64)
                blocks[-1].set_tensor(kind, l, 0, pair[0])
                blocks[-1].set_tensor(kind, l, 1, pair[1])
    xd = torch.from_numpy(x0).cuda()
    k = len(chans)
    for mask in ([0] * k, [1] * k, [i % 2 for i in range(k)]):
        pb.network_forward(blocks, mask, xd, outs, bn_mode=1)
        torch.cuda.synchronize()
        for i, (o, r) in enumerate(zip(outs, ob.network_forward(refs, mask, x0, bn_mode=1))):
            assert relerr(o.cpu().numpy(), r) <= ACT_TOL, (mask, i, relerr(o.cpu().numpy(), r))
    for b in blocks:
        b.close()


def test_offsets_past_two_gib(gpu):
    """Tensors of 3.9 GB (300 images of 64 channels, 225x225, no aligned rows): teacher's 3x3 and student's depthwise and 1x1
    kernels address them with 32-bit byte offsets.  Running statistics keep images apart, so the first, one across the
    2 GiB line and the last are compared with the same images alone; and the weight gradients of 160 images (2.07 GB,
    the largest the grouped kernel takes) that repeat two must be those of the two."""
    torch, pb = gpu
    c, h = 64, 225

    def block(n, seed):
        t, s = wl.Arch(n, c, h, h, wl._convs([c, c])), wl.Arch(n, c, h, h, wl._dws([c, c]))
        w = wl.Workload("offsets", wl.Arch(1, c, 8, 8, t.layers), wl.Arch(1, c, 8, 8, s.layers), seed=seed)
        _, tp, sp = w.tensors(random_affine=True)
        return pb.Block(t, tp, s, sp)

    def forward(x):
        blk = block(x.shape[0], 71)
        outs = []
        for use in (0, 1):
            out = torch.empty_like(x)
            pb.network_forward([blk], [use], x, [out], bn_mode=1)
            torch.cuda.synchronize()
            outs.append(out)
        blk.close()
        return outs

    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((300, c, h, h), generator=gen, device="cuda")
    some = [0, 165, 166, 299]                      # (image 165 holds byte 2^31)
    assert 165 * c * h * h * 4 < 2 ** 31 <= 166 * c * h * h * 4
    large, small = forward(x), forward(x[some].contiguous())
    for l, s in zip(large, small):
        assert relerr(l[some].cpu().numpy(), s.cpu().numpy()) <= 1e-6
    del large, small
    grads = []
    for n in (2, 160):
        blk = block(n, 72)
        xn = x[:2].repeat(n // 2, 1, 1, 1)
        target = torch.linspace(0, 1, h, device="cuda").expand(n, c, h, h).contiguous()
        blk.student_step(xn, target, 0.0)
        grads.append([g for layer in blk.student_grads() for g in layer])
        blk.close()
        del xn, target
    for a, b in zip(*grads):
        assert relerr(b, a) <= GRAD_TOL
    torch.cuda.empty_cache()


def test_fused_gradients_of_two_gib(gpu):
    """The largest tensors the kernels of fused gradients take, 2 GiB to the byte (128 images of 64 channels, 256x256): offsets reach
    the one from which on theirs are past every buffer.  128 images that repeat two have the gradients of the two."""
    torch, pb = gpu
    c, h = 64, 256
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((2, 3, h, h), generator=gen, device="cuda")
    target = torch.randn((2, c, h, h), generator=gen, device="cuda")
    t = wl.Arch(1, 3, 8, 8, wl._convs([3, c, c]))
    s = wl.Arch(1, 3, 8, 8, [wl.Layer(wl.CONV3X3, 3, c, 1, 1)] + wl._dws([c, c]))
    _, tp, sp = wl.Workload("two_gib", t, s, seed=73).tensors(random_affine=True)
    grads = []
    for n in (2, 128):
        assert n < 128 or n * c * h * h * 4 == 2 ** 31
        t, s = replace(t, n=n, h=h, w=h), replace(s, n=n, h=h, w=h)
        blk = pb.Block(t, tp, s, sp)
        blk.profile_enable(["pw_bwd", "first_bwd"], 4)
        blk.student_step(x.repeat(n // 2, 1, 1, 1), target.repeat(n // 2, 1, 1, 1), 0.0)
        assert {k: m for k, (_, m) in blk.profile_read().items()} == {"pw_bwd": 1, "first_bwd": 1}
        grads.append([g for layer in blk.student_grads() for g in layer])
        blk.close()
    for a, b in zip(*grads):
        assert relerr(b, a) <= GRAD_TOL
    torch.cuda.empty_cache()
