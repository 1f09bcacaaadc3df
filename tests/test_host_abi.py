"""CPU-only checks of the C ABI: the library loads, exports every declared symbol, and its host-side
logic (descriptor validation, workspace sizing, FLOP counts, the block scheduler) agrees with the
oracle.  No kernel is launched here."""
import os
import re

import numpy as np
import pytest

from oracle import schedule as osched
from paper_2012_03096_amd import binding as pb
from paper_2012_03096_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "pbkd.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(pbkd_[a-z_]+)\s*\(", header))
    assert declared == set(pb.EXPORTS), declared ^ set(pb.EXPORTS)
    L = pb.lib()
    for name in declared:
        assert getattr(L, name) is not None


def _all_workloads():
    return [wl.cfg1_tiny(), wl.cfg2_vgg_block2(), wl.cfg3_resnet_down(), wl.cfg4_imagenet_vgg_block1()] + \
        wl.cfg5_vgg16_blocks() + wl.small_variants() + wl.paper_granularity_vgg16_tasks()


def test_validate_accepts_all_workloads_and_sizes_workspace():
    for w in _all_workloads():
        assert pb.arch_validate(w.teacher, w.student) == pb.OK, (w.name, pb.last_error())
        nbytes = pb.workspace_bytes(w.teacher, w.student)
        assert nbytes > 0 and nbytes % 256 == 0
    # the ImageNet-shaped block: seven 411 MB activation-sized tensors (teacher z1 z2; student z1 u2 z2; gradient ping-pong gz du)
    big = pb.workspace_bytes(*(lambda w: (w.teacher, w.student))(wl.cfg4_imagenet_vgg_block1()))
    assert 2.5e9 < big < 4e9


def test_flops_match_oracle_definition():
    for w in _all_workloads():
        assert pb.arch_flops(w.teacher, False) == osched.arch_flops(w.teacher, False), w.name
        assert pb.arch_flops(w.student, False) == osched.arch_flops(w.student, False), w.name
        assert pb.arch_flops(w.student, True) == osched.arch_flops(w.student, True), w.name


def test_validation_errors():
    w = wl.cfg1_tiny()
    bad = wl.Arch(4, 16, 16, 16, [wl.Layer(wl.DWSEP3X3, 16, 16, 1, 1), wl.Layer(wl.DWSEP3X3, 8, 16, 1, 1)])
    assert pb.arch_validate(w.teacher, bad) == pb.ESHAPE and "cin" in pb.last_error()
    bad = wl.Arch(4, 16, 16, 16, [wl.Layer(wl.DWSEP3X3, 16, 16, 1, 1), wl.Layer(wl.DWSEP3X3, 16, 8, 1, 1)])
    assert pb.arch_validate(w.teacher, bad) == pb.ESHAPE
    bad = wl.Arch(4, 16, 16, 16, [wl.Layer(wl.DWSEP3X3, 16, 16, 3, 1), wl.Layer(wl.DWSEP3X3, 16, 16, 1, 1)])
    assert pb.arch_validate(w.teacher, bad) == pb.EINVAL
    bad = wl.Arch(4, 16, 16, 16, [wl.Layer(wl.DWSEP3X3, 16, 16, 1, 1), wl.Layer(wl.CONV3X3, 16, 16, 1, 1)])
    assert pb.arch_validate(w.teacher, bad) == pb.EUNSUPPORTED
    bad = wl.Arch(4, 16, 16, 16, [wl.Layer(wl.DWSEP3X3, 16, 16, 1, 1), wl.Layer(wl.DWSEP3X3, 16, 16, 1, 0)])
    assert pb.arch_validate(w.teacher, bad) == pb.EUNSUPPORTED
    bad = wl.Arch(4, 16, 16, 16, [])
    assert pb.arch_validate(w.teacher, bad) == pb.EINVAL
    bad = wl.Arch(4, 16, 16, 16, w.student.layers, pool=3)
    assert pb.arch_validate(w.teacher, bad) == pb.EINVAL
    bad = wl.Arch(2, 16, 16, 16, w.student.layers)
    assert pb.arch_validate(w.teacher, bad) == pb.ESHAPE
    bad = wl.Arch(4, 16, 16, 16, w.student.layers, shortcut=1, shortcut_stride=2)
    assert pb.arch_validate(w.teacher, bad) == pb.ESHAPE
    assert pb.workspace_bytes(w.teacher, bad) == 0
    bad = wl.Arch(4, 16, 1, 1, w.student.layers, pool=2)
    assert pb.arch_validate(bad, bad) in (pb.ESHAPE, pb.EUNSUPPORTED)


@pytest.mark.parametrize("seed", range(10))
@pytest.mark.parametrize("policy", [0, 1])
def test_scheduler_matches_oracle(seed, policy):
    rng = np.random.default_rng(seed)
    n = int(rng.integers(0, 14))
    m = int(rng.integers(1, 6))
    weights = [int(v) for v in rng.integers(1, 50, n)]       # small range: many ties
    got = pb.schedule_blocks(weights, m, policy)
    ref = (osched.wfd if policy == 0 else osched.round_robin)(weights, m)
    assert got[0] == ref[0] and got[1] == ref[1] and got[2] == ref[2]


def test_scheduler_on_vgg16_blocks_and_errors():
    blocks = wl.cfg5_vgg16_blocks()
    weights = [pb.arch_flops(b.teacher, False) + pb.arch_flops(b.student, True) for b in blocks]
    for m in (1, 2, 3, 4, 5, 7):
        got = pb.schedule_blocks(weights, m, 0)
        ref = osched.wfd(weights, m)
        assert got[0] == ref[0] and got[2] == ref[2]
    with pytest.raises(pb.PbkdError) as e:
        pb.schedule_blocks(weights, 0, 0)
    assert e.value.status == pb.EINVAL
    with pytest.raises(pb.PbkdError):
        pb.schedule_blocks(weights, 2, 5)


@pytest.mark.parametrize("pixels", [32768, 100352, 262144, 401408, 1605632])
def test_pointwise_tiles_of_few_channels_are_not_half_empty(pixels):
    """Up to 32 output channels of a 1x1 convolution take a tile of 32 channels, not the 64-channel one that more take."""
    import ctypes
    choice = pb.lib()._ZN4pbkd15pw_split_choiceExiii            # (pixels, output channels, pixels per image, stride)
    choice.restype, choice.argtypes = ctypes.c_int, [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    for cout in (1, 16, 24, 32):
        assert choice(pixels, cout, 1024, 1) != choice(pixels, 64, 1024, 1), cout


@pytest.mark.parametrize("n,h,w,c,fp32", [(512, 1, 1, 96, True), (512, 2, 1, 64, True), (128, 1, 3, 256, True), (8, 7, 7, 128, True), (64, 2, 3, 192, True), (512, 1, 1, 384, True),
                                          (64, 5, 5, 128, False), (128, 7, 7, 64, False), (8, 7, 7, 512, False), (32, 15, 13, 64, False)])
def test_few_pixels_of_tiny_maps_keep_the_fp32_convolution(monkeypatch, n, h, w, c, fp32):
    """The split kernels keep another weight image than the fp32 one, so the workspace tells which a teacher layer runs."""
    t, s = wl.Arch(n, c, h, w, wl._convs([c, c])), wl.Arch(n, c, h, w, wl._dws([c, c]))
    chosen = pb.workspace_bytes(t, s)
    monkeypatch.setenv("PBKD_CONV_SPLIT", "0")
    assert (chosen == pb.workspace_bytes(t, s)) == fp32


def conv_kernel(n, cin, cout, h, w, stride=1):
    return pb.arch_conv_kernel(wl.Arch(n, cin, h, w, [wl.Layer(wl.CONV3X3, cin, cout, stride, 0)]), 0)


@pytest.mark.parametrize("n,cin,cout,h,w,stride,name", [
    (8, 3, 64, 32, 32, 1, "first"), (8, 8, 64, 13, 13, 1, "fp32"), (4, 64, 64, 1, 1, 1, "fp32"), (32, 64, 128, 15, 13, 1, "rows"), (16, 128, 128, 16, 16, 2, "aligned"),
    (75, 512, 512, 16, 16, 1, "transformed"), (31, 112, 112, 112, 112, 1, "transformed"), (122, 64, 64, 36, 36, 1, "transformed"),
    (42, 32, 32, 64, 68, 1, "aligned"), (69, 32, 32, 36, 36, 1, "transformed"), (128, 512, 512, 4, 4, 1, "aligned"), (64, 272, 272, 8, 8, 1, "transformed"),
    (5, 160, 160, 16, 16, 1, "aligned"), (20, 48, 48, 180, 156, 1, "aligned"), (1, 64, 64, 32, 32, 1, "aligned")])
def test_each_convolution_runs_the_kernel_its_shape_asks_for(n, cin, cout, h, w, stride, name):
    """Without tuning overrides: the direct kernels where a map is not aligned, strided, tiny or has few channels, transformed tiles
    only where they are priced well below the aligned kernel."""
    assert conv_kernel(n, cin, cout, h, w, stride)[0] == name


def test_transformed_tiles_where_asked_for_and_where_they_cannot_run(monkeypatch):
    shapes = [(1, 16, 16, 1, 1), (3, 40, 33, 14, 14), (2, 17, 70, 5, 131), (1, 31, 16, 150, 3), (33, 16, 64, 2, 2), (4, 300, 130, 12, 16)]
    monkeypatch.setenv("PBKD_CONV_WINO", "0")
    assert all(conv_kernel(*s)[0] != "transformed" for s in shapes + [(75, 512, 512, 16, 16)])
    monkeypatch.setenv("PBKD_CONV_WINO", "1")
    assert all(conv_kernel(*s)[0] == "transformed" for s in shapes)
    assert conv_kernel(4, 512, 64, 4, 4)[1] == 8                              # (K split over up to eight workgroups)
    # at most 15 input channels, a stride, outputs of 4 GiB, weight images of 4 GiB
    for s in ((8, 15, 64, 16, 16), (8, 32, 64, 16, 16, 2), (64, 16, 128, 400, 400), (1, 6912, 6912, 8, 8)):
        assert conv_kernel(*s)[0] not in ("transformed", ""), s
    assert conv_kernel(64, 16, 127, 362, 364)[0] == "transformed"             # 4.28 GB, 0.01 below 4 GiB
    for name in ("PBKD_CONV_TILE", "PBKD_CONV_KSPLIT", "PBKD_CONV_ROWS"):     # another forced geometry leaves them out by default
        monkeypatch.delenv("PBKD_CONV_WINO", raising=False)
        monkeypatch.setenv(name, "1")
        assert conv_kernel(75, 512, 512, 16, 16)[0] != "transformed"
        monkeypatch.delenv(name)
    monkeypatch.setenv("PBKD_CONV_SPLIT", "0")
    assert conv_kernel(75, 512, 512, 16, 16)[0] == "fp32"
    # no 3x3 convolution, no layer, no descriptor
    t = wl.Arch(2, 16, 8, 8, [wl.Layer(wl.DWSEP3X3, 16, 16, 1, 0)])
    assert pb.arch_conv_kernel(t, 0) == ("", 0) and pb.arch_conv_kernel(t, 1) == ("", 0) and pb.arch_conv_kernel(t, -1) == ("", 0)
    assert pb.lib().pbkd_arch_conv_kernel(None, 0, None) == b""


def test_split_weights_that_do_not_fit_their_index_keep_the_fp32_kernels(monkeypatch):
    """Split copies take 6 bytes a weight and are addressed in 32 bits (a 3x3 image, a 1x1 image) or, all of a student's
    together, in 31 bits of 2-byte units.  Sizes past that are still accepted, with the fp32 copies."""
    # a teacher's 3x3 layer of 9600 x 9600 channels: 5.5 GB split, 3.3 GB in fp32 (the workspace tells which is kept)
    small = wl.Arch(1, 9600, 5, 5, [wl.Layer(wl.DWSEP3X3, 9600, 9600, 1, 1)])
    t = wl.Arch(1, 9600, 5, 5, [wl.Layer(wl.CONV3X3, 9600, 9600, 1, 0)])
    chosen = pb.workspace_bytes(t, small)
    monkeypatch.setenv("PBKD_CONV_SPLIT", "0")
    assert chosen == pb.workspace_bytes(t, small) > 0
    monkeypatch.delenv("PBKD_CONV_SPLIT")

    # 1x1 weights: the workspace grows with them while the kind of copy stays the same, by less where it changes.  A teacher
    # keeps one image a layer (4 GiB split at 26752 x 26752), a student two copies in one arena (2^30 floats at 18944 x 18944).
    def workspace(tc, sc):
        return pb.workspace_bytes(wl.Arch(1, tc, 1, 1, [wl.Layer(wl.DWSEP3X3, tc, tc, 1, 0)]), wl.Arch(1, sc, 1, 1, [wl.Layer(wl.DWSEP3X3, sc, sc, 1, 1)]))

    def per_weight(c):
        return workspace(c, c) / c ** 2

    split, past_arena = per_weight(16384), per_weight(20480)
    assert 3.5 < split - past_arena < 4.5                # two student copies of 4 bytes a weight instead of 6
    assert 1.5 < past_arena - per_weight(28672) < 2.5    # and the teacher's


def test_bench_reads_the_tuning_variables_as_the_library_does(monkeypatch):
    """The peaks that the benchmark reports rates against are those of the products in use: one chunk of pixels a workgroup (fp32
    products), eight and more (split ones), and variables that are no numbers, which the library takes for 0."""
    import bench
    for name in ("PBKD_WGRAD_SPLIT", "PBKD_CONV_SPLIT"):
        monkeypatch.delenv(name, raising=False)
    tiny, large = wl.cfg1_tiny(), [wl.cfg2_vgg_block2(), wl.cfg3_resnet_down(), wl.cfg4_imagenet_vgg_block1()]
    assert not bench.weight_gradient_split_in_use(tiny) and all(bench.weight_gradient_split_in_use(w) for w in large)
    assert bench.conv_split_in_use()
    for value, wgrad in (("0", [False] * 4), ("", [False] * 4), ("off", [False] * 4), ("1", [True] * 4), ("2", [False] + [True] * 3)):
        monkeypatch.setenv("PBKD_WGRAD_SPLIT", value)
        monkeypatch.setenv("PBKD_CONV_SPLIT", value)
        assert [bench.weight_gradient_split_in_use(w) for w in [tiny] + large] == wgrad, value
        t = wl.Arch(32, 64, 224, 224, [wl.Layer(wl.CONV3X3, 64, 64, 1, 0)])
        assert bench.conv_split_in_use() == (pb.arch_conv_kernel(t, 0)[0] != "fp32"), value
