"""GPU parity, layer by layer and block by block, at full size: every tensor the device keeps for
back-propagation, for every block and micro-batch of the benchmark configurations, against the plain CPU oracle
(float64, nothing rounded) fed the device's own layer inputs / block inputs (tests/teacher.py).  Element-wise,
2e-2 (bf16 operands) / 1e-4 (fp32 check mode), in the launch configuration bench.py times (all micro-batches of
the batch in one group call per direction)."""
import time

import numpy as np
import pytest

from paper_1911_05146_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: these tests need a real MI355X")
    from paper_1911_05146_amd import hpf
    return hpf


def layerwise(oracle, spec, mode, grouped=True, fusion=2, randomize_affine=True, blockwise=True):
    from parity import run_gpu_step
    from teacher import blockwise_check, layerwise_check
    print(f"\n[case] layer-wise {spec.name} b={spec.microbatch} m={spec.num_microbatches} mode={mode} grouped={grouped} "
          f"fusion={fusion} seed={spec.seed}", flush=True)
    inp = W.make_inputs(spec, randomize_affine=randomize_affine)
    t0 = time.time()
    seen, res = run_gpu_step(spec, inp, mode, grouped=grouped, fusion=fusion, keep=True)
    part = res.pop("part")
    try:
        rep = layerwise_check(oracle, part, spec, seen, res, mode)
        print(f"[layer-wise] {spec.name} {mode}: {rep.summary()} ({time.time() - t0:.0f} s)", flush=True)
        if blockwise:
            t0 = time.time()
            rb = blockwise_check(oracle, part, spec, seen, res, mode)
            print(f"[block-wise] {spec.name} {mode}: {rb.summary()}; {rb.extra} ({time.time() - t0:.0f} s)", flush=True)
    finally:
        part.close()
    return rep


@pytest.mark.parametrize("mode", ["bf16", "f32"])
def test_single_blocks_layerwise(gpu, oracle, mode):
    """Every block kind at its full micro-batch, first seed, no retries."""
    cases = {
        "bottleneck-identity-r1001-stage2": (W.Block(W.BOTTLENECK, 128, 32, 128, 1), 16, 32),
        "bottleneck-entry-stride2-proj": (W.Block(W.BOTTLENECK, 64, 32, 128, 2), 16, 8),
        "bottleneck-widen-proj-stride1": (W.Block(W.BOTTLENECK, 16, 16, 64, 1), 32, 8),
        "bottleneck-wide-identity": (W.Block(W.BOTTLENECK, 128, 64, 128, 1), 16, 8),
        "basic-identity": (W.Block(W.BASIC, 32, 32, 32, 1), 16, 16),
        "basic-identity-64": (W.Block(W.BASIC, 64, 64, 64, 1), 8, 16),
        "basic-entry-stride2-proj": (W.Block(W.BASIC, 32, 64, 64, 2), 16, 16),
        "bottleneck-r152-stage3": (W.Block(W.BOTTLENECK, 1024, 256, 1024, 1), 14, 4),
        "bottleneck-r152-entry": (W.Block(W.BOTTLENECK, 512, 256, 1024, 2), 28, 2),
    }
    for name, (blk, hw, b) in cases.items():
        spec = W.PartitionSpec(name=name, in_h=hw, in_w=hw, in_c=blk.c_in, blocks=(blk,), microbatch=b,
                               num_microbatches=2, seed=21)
        layerwise(oracle, spec, mode)


@pytest.mark.parametrize("images,grouped", [(1, True), (4, False), (5, True)])
@pytest.mark.parametrize("fusion", [0, 1])
@pytest.mark.parametrize("blk,hw", [(W.Block(W.BOTTLENECK, 64, 32, 128, 2), 32),   # 64 channels x 64 / 80 rows of records: either side of the limit
                                    (W.Block(W.BASIC, 48, 80, 80, 2), 16),         # channel counts that divide no work-group, a second slab of 16
                                    (W.Block(W.POSTACT, 16, 48, 48, 2), 8)])       # fewer rows than row groups
def test_statistics_from_records_layerwise(gpu, oracle, blk, hw, fusion, images, grouped):
    """BatchNorm statistics and backward sums that the consuming kernel adds up from the producer's records, or a launch in between."""
    spec = W.PartitionSpec(name=f"records-{blk.kind}-{blk.c_in}-{blk.c_out}", in_h=hw, in_w=hw, in_c=blk.c_in, blocks=(blk,),
                           microbatch=images, num_microbatches=2, seed=23)
    layerwise(oracle, spec, "bf16", grouped=grouped, fusion=fusion, blockwise=False)


@pytest.mark.parametrize("fusion", [0, 1])
@pytest.mark.parametrize("blk,hw", [(W.Block(W.BOTTLENECK, 160, 128, 64, 1), 10),    # five and four steps of 32 behind a BatchNorm, with and without statistics behind
                                    (W.Block(W.BOTTLENECK, 96, 48, 192, 2), 14),     # three, two; a projection of three
                                    (W.Block(W.BOTTLENECK, 192, 160, 192, 1), 6),    # six (steps of 64) and five, identity shortcut
                                    (W.Block(W.BASIC, 16, 16, 16, 1), 12)])          # 3x3 in five
def test_short_reductions_layerwise(gpu, oracle, blk, hw, fusion):
    """Reductions that are in flight as a whole, with the BatchNorm in front, the statistics, the sums of a backward pass and the residual."""
    spec = W.PartitionSpec(name=f"short-{blk.c_in}-{blk.c_mid}-{blk.c_out}", in_h=hw, in_w=hw, in_c=blk.c_in, blocks=(blk,),
                           microbatch=3, num_microbatches=2, seed=37)
    layerwise(oracle, spec, "bf16", grouped=True, fusion=fusion, blockwise=False)


@pytest.mark.parametrize("images,micro", [(1, 1), (3, 3), (1, 8), (4, 7)])
def test_weight_gradients_of_several_classes_in_one_launch_layerwise(gpu, oracle, images, micro):
    """Five tile classes and the whole-image one, few items each: one launch whose micro-batches go to work-groups in even and odd shares."""
    blocks = (W.Block(W.BASIC, 16, 16, 16, 1), W.Block(W.BASIC, 16, 32, 32, 2), W.Block(W.BOTTLENECK, 32, 64, 128, 2),
              W.Block(W.BOTTLENECK, 128, 16, 64, 1))
    spec = W.PartitionSpec(name="classes", in_h=32, in_w=32, in_c=16, blocks=blocks, microbatch=images, num_microbatches=micro, seed=29)
    layerwise(oracle, spec, "bf16", grouped=True, fusion=1, blockwise=False)


def test_row_band_runs_layerwise(gpu, oracle):
    """Runs of 64-16-16-64 bottlenecks at 32x32 (the first stage of ResNet-1001): each image is cut into four bands of
    eight rows, one work-group each, and the rows next to a band travel with the BatchNorm records.  Three blocks, so
    that every exchange of the loop runs; an odd number of images; one and several micro-batches per launch."""
    blocks = tuple(W.Block(W.BOTTLENECK, 64, 16, 64, 1) for _ in range(3))
    for b, m, grouped in ((8, 2, True), (3, 2, True), (5, 3, False)):
        spec = W.PartitionSpec(name=f"bands-3x(64-16-64)@32x32-b{b}", in_h=32, in_w=32, in_c=64, blocks=blocks, microbatch=b,
                               num_microbatches=m, seed=23)
        layerwise(oracle, spec, "bf16", grouped=grouped)
    spec = W.PartitionSpec(name="bands-3x(64-16-64)@32x32-level1", in_h=32, in_w=32, in_c=64, blocks=blocks, microbatch=4,
                           num_microbatches=2, seed=23)
    layerwise(oracle, spec, "bf16", fusion=1)


def test_runs_with_weights_through_lds_layerwise(gpu, oracle):
    """Register-resident runs, whose weight matrices the work-group stages through LDS: 128-64 and 128-32 bottlenecks at
    16x16 (conv2's matrix in one piece or in three, conv1's and conv3's in turn in one area), basic and post-activation blocks of
    32 channels at 16x16 and of 16 channels at 32x32 (one matrix at a time).
    Three blocks, so that the staging of the first block, of a following block and of the last one all run; an odd
    number of images; one call per micro-batch and one for all."""
    runs = {
        "wide-3x(128-64-128)@16x16": (tuple(W.Block(W.BOTTLENECK, 128, 64, 128, 1) for _ in range(3)), 16, 128, True),
        "3x(128-32-128)@16x16": (tuple(W.Block(W.BOTTLENECK, 128, 32, 128, 1) for _ in range(3)), 16, 128, True),
        "3x basic32@16x16": (tuple(W.Block(W.BASIC, 32, 32, 32, 1) for _ in range(3)), 16, 32, True),
        "3x basic16@32x32": (tuple(W.Block(W.BASIC, 16, 16, 16, 1) for _ in range(3)), 32, 16, True),
        "3x postact32@16x16": (tuple(W.Block(W.POSTACT, 32, 32, 32, 1) for _ in range(3)), 16, 32, False),
        "3x postact16@32x32": (tuple(W.Block(W.POSTACT, 16, 16, 16, 1) for _ in range(3)), 32, 16, False),
    }
    # 40 images per micro-batch: two chunks of polled members in the forward, three in the exchanges of a 128-64 block's backward; the
    # largest size of the 128-32 runs
    spec = W.PartitionSpec(name="wide-3x(128-64-128)@16x16-b40", in_h=16, in_w=16, in_c=128, blocks=runs["wide-3x(128-64-128)@16x16"][0],
                           microbatch=40, num_microbatches=2, seed=37)
    layerwise(oracle, spec, "bf16", blockwise=False)
    spec = W.PartitionSpec(name="3x(128-32-128)@16x16-b40", in_h=16, in_w=16, in_c=128, blocks=runs["3x(128-32-128)@16x16"][0],
                           microbatch=40, num_microbatches=2, seed=37)
    layerwise(oracle, spec, "bf16", blockwise=False)
    # 100 images per micro-batch: four chunks of polled members
    for name, blocks, hw, c in (("3x basic32@16x16-b100", runs["3x basic32@16x16"][0], 16, 32),
                                ("3x basic64@8x8-b100", tuple(W.Block(W.BASIC, 64, 64, 64, 1) for _ in range(3)), 8, 64),
                                ("3x postact32@16x16-b100", runs["3x postact32@16x16"][0], 16, 32)):
        spec = W.PartitionSpec(name=name, in_h=hw, in_w=hw, in_c=c, blocks=blocks, microbatch=100, num_microbatches=2, seed=37)
        layerwise(oracle, spec, "bf16", blockwise=False)
    for name, (blocks, hw, c, blockwise) in runs.items():
        for b, m, grouped in ((3, 2, True), (4, 3, False)):
            spec = W.PartitionSpec(name=f"{name}-b{b}", in_h=hw, in_w=hw, in_c=c, blocks=blocks, microbatch=b,
                                   num_microbatches=m, seed=37)
            layerwise(oracle, spec, "bf16", grouped=grouped, blockwise=blockwise)


@pytest.mark.parametrize("kind,c,mid,h,w,images",
                         # records in an idle tile | in an area of their own, in front of the staged matrix
                         [(k, 32, 32, 8, 16, b) for k in (W.BASIC, W.POSTACT) for b in (3, 44)] +
                         # as above | weights fetched where they are used in the forward | in both directions
                         [(k, 64, 64, 8, 16, b) for k in (W.BASIC, W.POSTACT) for b in (3, 40, 60, 90)] +
                         [(W.BOTTLENECK, 128, 32, 8, 16, b) for b in (3, 24)] + [(W.BOTTLENECK, 128, 64, 8, 8, b) for b in (3, 20)] +
                         # staged weights | fetched where they are used, records in an idle tile / an area of their own
                         [(W.BOTTLENECK, 256, 64, 4, 16, 3), (W.BOTTLENECK, 256, 64, 8, 16, 3), (W.BOTTLENECK, 256, 64, 4, 16, 12)] +
                         # staged weights behind an area of records | in the forward only
                         [(W.BOTTLENECK, 256, 64, 4, 8, b) for b in (6, 18)])
def test_lds_tile_resident_runs_layerwise(gpu, oracle, kind, c, mid, h, w, images):
    """Image-resident runs of the shapes that the register kernels do not take, whose images and gathered BatchNorm records lie in LDS
    tiles: every kernel and every place of the records and of the weights, which depend on the number of images.  Three blocks: the
    first, a following one and the last."""
    spec = W.PartitionSpec(name=f"tile-{kind}-{c}-{mid}@{h}x{w}-b{images}", in_h=h, in_w=w, in_c=c, blocks=(W.Block(kind, c, mid, c, 1),) * 3,
                           microbatch=images, num_microbatches=2 if images < 40 else 1, seed=59)
    layerwise(oracle, spec, "bf16", blockwise=False)


@pytest.mark.parametrize("kind,c,hw,images,micro", [(W.CONV_RELU, 256, 7, 4, 2), (W.CONV_RELU, 64, 10, 2, 1), (W.CONV_RELU, 16, 32, 2, 1),   # a class in its own kernel
                                                    (W.CONV_RELU, 128, 7, 4, 7), (W.CONV_RELU, 64, 10, 2, 7), (W.DENSE, 512, 1, 5, 8),   # in two, four shares
                                                    (W.CONV_RELU, 16, 24, 16, 3)])   # many items that add to one tile
def test_weight_gradients_of_one_class_layerwise(gpu, oracle, kind, c, hw, images, micro):
    """One tile class with few items: in the kernel of the class, or its micro-batches dealt to work-groups in shares that do not divide them."""
    spec = W.PartitionSpec(name=f"class-{kind}-{c}", in_h=hw, in_w=hw, in_c=c, blocks=(W.Block(kind, c, c if kind != W.DENSE else 1, c, 1),),
                           microbatch=images, num_microbatches=micro, seed=31)
    layerwise(oracle, spec, "bf16", grouped=True, fusion=1, blockwise=False)


@pytest.mark.parametrize("kind,c,mid,h,w,images",
                         [(W.BASIC, 64, 64, 12, 8, 5), (W.POSTACT, 64, 64, 8, 8, 6),             # two and four images at a time, the last batch not full
                          (W.BASIC, 32, 32, 4, 16, 9), (W.BOTTLENECK, 128, 32, 4, 16, 3),        # fewer images than fit a batch
                          (W.BOTTLENECK, 256, 64, 4, 8, 15), (W.BOTTLENECK, 128, 64, 8, 32, 3)])  # as many as fit the LDS; rows of 32 pixels
def test_weight_gradients_of_small_images_layerwise(gpu, oracle, kind, c, mid, h, w, images):
    """Weight gradients of resident runs that stage several images of a micro-batch at a time, in shares that cross micro-batches."""
    spec = W.PartitionSpec(name=f"batches-{kind}-{c}-{mid}@{h}x{w}-b{images}", in_h=h, in_w=w, in_c=c, blocks=(W.Block(kind, c, mid, c, 1),) * 2,
                           microbatch=images, num_microbatches=3, seed=67)
    layerwise(oracle, spec, "bf16", blockwise=False)


@pytest.mark.parametrize("images", [1, 8, 9, 16, 17, 31, 33])
@pytest.mark.parametrize("kind,c,mid,hw", [(W.BASIC, 16, 16, 32), (W.BASIC, 32, 32, 16), (W.BASIC, 64, 64, 8),
                                           (W.POSTACT, 16, 16, 32), (W.POSTACT, 32, 32, 16), (W.POSTACT, 64, 64, 8),
                                           (W.BOTTLENECK, 128, 32, 16), (W.BOTTLENECK, 128, 64, 16)])
def test_register_resident_runs_around_the_polled_chunk_layerwise(gpu, oracle, kind, c, mid, hw, images):
    """Image-resident runs with the residual stream in registers collect the BatchNorm words of 32 images at a time, basic blocks those of 16 where there
    are no more, bottlenecks of eight: one image (no partner), full chunks, chunks that are not full, one word beyond a chunk,
    either side of each change of kernel.  Two blocks: the first and the last."""
    spec = W.PartitionSpec(name=f"reg-{kind}-{c}@{hw}x{hw}-b{images}", in_h=hw, in_w=hw, in_c=c,
                           blocks=(W.Block(kind, c, mid, c, 1),) * 2, microbatch=images, num_microbatches=1, seed=43)
    layerwise(oracle, spec, "bf16", blockwise=False)


@pytest.mark.parametrize("images,micro,grouped", [(1, 1, True), (3, 2, True), (8, 3, True), (9, 2, False), (12, 2, True), (16, 1, True), (17, 1, True), (33, 2, True)])
def test_register_resident_runs_of_8x8_bottlenecks_layerwise(gpu, oracle, images, micro, grouped):
    """256-64 bottlenecks on 8x8: words of 8, 16 or 32 images at a time, full chunks and one image beyond.  Three blocks: the first, a following
    one and the last."""
    spec = W.PartitionSpec(name=f"reg8-256-64@8x8-b{images}", in_h=8, in_w=8, in_c=256, blocks=(W.Block(W.BOTTLENECK, 256, 64, 256, 1),) * 3,
                           microbatch=images, num_microbatches=micro, seed=73)
    layerwise(oracle, spec, "bf16", grouped=grouped, blockwise=False)


@pytest.mark.parametrize("images,blocks", [(1, 1), (1, 3), (4, 2), (5, 2), (8, 2), (9, 2), (16, 2)])
def test_row_bands_around_the_polled_chunk_layerwise(gpu, oracle, images, blocks):
    """64-16 bottlenecks at 32x32 collect the words of 32 bands at a time, of 16 where there are no more: the four bands of one image alone, one block
    alone, the last image of the one kernel and the first of the other, more than one chunk (36 bands) and whole chunks (32, 64)."""
    spec = W.PartitionSpec(name=f"bands-{blocks}-b{images}", in_h=32, in_w=32, in_c=64, blocks=(W.Block(W.BOTTLENECK, 64, 16, 64, 1),) * blocks,
                           microbatch=images, num_microbatches=1, seed=79)
    layerwise(oracle, spec, "bf16", blockwise=False)


@pytest.mark.parametrize("before,behind,images,micro", [(0, 1, 5, 2), (1, 0, 1, 1), (1, 2, 33, 1), (0, 3, 4, 3), (1, 1, 16, 1), (0, 1, 17, 1)])
@pytest.mark.parametrize("kind,c,mid,hw", [(W.BASIC, 16, 32, 32), (W.BASIC, 32, 64, 16), (W.POSTACT, 16, 32, 32), (W.POSTACT, 32, 64, 16),
                                           (W.BOTTLENECK, 64, 32, 32), (W.BOTTLENECK, 64, 64, 32)])
def test_runs_led_in_by_a_block_that_halves_the_image_layerwise(gpu, oracle, kind, c, mid, hw, before, behind, images, micro):
    """A strided block with a projection runs in the launch of the identity blocks behind it, or in one of its own at the end of a
    partition: between the caller's tensors, behind another run, one image and one word beyond a polled chunk."""
    first = W.Block(kind, c, 16 if kind == W.BOTTLENECK else c, c, 1)
    blocks = (first,) * before + (W.Block(kind, c, mid, 2 * c, 2),) + (W.Block(kind, 2 * c, mid, 2 * c, 1),) * behind
    spec = W.PartitionSpec(name=f"lead-{kind}-{c}-{mid}@{hw}-{before}+{behind}-b{images}", in_h=hw, in_w=hw, in_c=c, blocks=blocks,
                           microbatch=images, num_microbatches=micro, seed=71)
    layerwise(oracle, spec, "bf16", grouped=micro != 3, blockwise=False)


@pytest.mark.parametrize("kind,c,mid,hw", [(W.BASIC, 16, 16, 32), (W.BASIC, 32, 32, 16), (W.BASIC, 64, 64, 8),
                                           (W.BOTTLENECK, 128, 32, 16), (W.BOTTLENECK, 128, 64, 16), (W.BOTTLENECK, 256, 64, 8), (W.BOTTLENECK, 64, 16, 32)])
def test_statistics_of_channels_whose_mean_jumps_between_blocks(gpu, oracle, kind, c, mid, hw):
    """The first block of a run moves every fourth channel of the residual stream by 40 standard deviations.  The next block's
    statistics must not feel it: squares summed about any value d standard deviations from the mean lose a factor d^2 = 1600
    of the variance's digits (measured then: 1.1e-4 ... 1.6e-4).  Bound for invstd: about 20 roundings of 2^-24 in a sum of squares about one of its own
    pixels (amplified by 1 + 4^2 at most), half of that in the root: 1e-5."""
    from parity import run_gpu_step
    from teacher import layerwise_check
    spec = W.PartitionSpec(name=f"jump-{kind}-{c}-{mid}@{hw}x{hw}", in_h=hw, in_w=hw, in_c=c, blocks=(W.Block(kind, c, mid, c, 1),) * 2,
                           microbatch=5, num_microbatches=1, seed=47)
    print(f"\n[case] {spec.name}", flush=True)
    inp = W.make_inputs(spec, randomize_affine=True)
    lay = {e.name: e for e in W.param_layout(spec)}
    P = lambda n: inp.params[lay[n].offset:lay[n].offset + lay[n].size].reshape(lay[n].shape)
    last = 2 if kind == W.BASIC else 3
    P(f"block0.bn{last}.gamma")[:] = 0.02      # the last convolution's operand is 4 +- 0.02 everywhere
    P(f"block0.bn{last}.beta")[:] = 4.0
    w = P(f"block0.W{last}")
    w[..., ::4] = 0.0
    w[w.shape[0] // 2, w.shape[1] // 2, :, ::4] = 10.0 / w.shape[2]   # the centre tap alone, or the border would differ
    seen, res = run_gpu_step(spec, inp, "bf16", grouped=True, keep=True)
    part = res.pop("part")
    try:
        rep = layerwise_check(oracle, part, spec, seen, res, "bf16")
    finally:
        part.close()
    assert rep.worst["bn.invstd"][0] <= 1e-5, rep.worst["bn.invstd"]


@pytest.mark.parametrize("kind,c,mid,hw", [(W.BASIC, 16, 16, 32), (W.BASIC, 32, 32, 16), (W.BASIC, 64, 64, 8),
                                           (W.BOTTLENECK, 128, 32, 16), (W.BOTTLENECK, 128, 64, 16), (W.BOTTLENECK, 256, 64, 8), (W.BOTTLENECK, 64, 16, 32)])
def test_a_channel_whose_variance_overflows_is_switched_off(gpu, kind, c, mid, hw):
    """Values of +-3e18 have a sum of squares beyond float32: the variance is infinite, 1 / sqrt of it is 0 (not NaN), the channel's
    BatchNorm gives beta and every other channel is as without it."""
    import torch
    spec = W.PartitionSpec(name=f"overflow-{kind}-{c}-{mid}@{hw}x{hw}", in_h=hw, in_w=hw, in_c=c, blocks=(W.Block(kind, c, mid, c, 1),),
                           microbatch=5, num_microbatches=1, seed=53)
    print(f"\n[case] {spec.name}", flush=True)
    inp = W.make_inputs(spec, randomize_affine=True)
    x = inp.act_in[0].copy().reshape(5, hw * hw, c)
    x[..., 0] = np.where(np.arange(hw * hw) % 2, 3e18, -3e18)
    part = gpu.Partition(spec, inp.params)
    try:
        y = part.forward_microbatch(0, torch.from_numpy(x.reshape(inp.act_in[0].shape)).to("cuda:0", torch.bfloat16))
        torch.cuda.synchronize()
        st = part.stash_read(0, 0, gpu.HPF_T_STATS0)
        v = torch.from_numpy(x).to(torch.bfloat16).double().numpy().reshape(-1, c)[:, 1:]
        assert st[c] == 0.0
        assert np.allclose(st[c + 1:], 1.0 / np.sqrt(v.var(axis=0) + spec.bn_eps), rtol=1e-5)
        assert bool(torch.isfinite(y).all())
    finally:
        part.close()


def test_convolutions_with_split_reductions_layerwise(gpu, oracle):
    """Plain 3x3 convolution units with long reductions into few output tiles (VGG-16's last two groups: 512 channels on
    4x4 and 2x2 pixels) run with every reduction split over two to four work-groups whose fp32 partial sums a second
    launch adds up, in both directions.  Group sizes 1 and several (the split count depends on it), a ragged last
    tile (48 pixel rows), 9 x 256 and 9 x 512 reduction elements (36 and 72 steps: splits of unequal length)."""
    cases = (("512@4x4", 512, 512, 4, 16, 2, True), ("512@4x4-single-calls", 512, 512, 4, 16, 2, False),
             ("512@2x2-ragged", 512, 512, 2, 12, 3, True), ("256-512@4x4", 256, 512, 4, 8, 2, True))
    for name, cin, cout, hw, b, m, grouped in cases:
        blocks = (W.Block(W.CONV_RELU, cin, cout, cout, 1), W.Block(W.CONV_RELU, cout, cout, cout, 1))
        spec = W.PartitionSpec(name=f"splitk-{name}-b{b}", in_h=hw, in_w=hw, in_c=cin, blocks=blocks, microbatch=b,
                               num_microbatches=m, seed=41)
        layerwise(oracle, spec, "bf16", grouped=grouped, blockwise=False)
    layerwise(oracle, spec, "bf16", fusion=0, blockwise=False)   # every step a kernel of its own: the same convolution launches


def test_whole_image_weight_gradient_of_16_channel_convolutions_layerwise(gpu, oracle):
    """3x3 convolutions between 16 and 16 channels on 1024-pixel images take the weight-gradient kernel that forms all
    nine taps from one staging of an image.  Square images (32 pixels per row: one image row per MFMA step) and the
    two other row lengths it accepts (16 and 8 pixels: two and four image rows per step, other border lanes); image
    counts that do not divide into equal work items; one image; pre- and post-activation operands (with and without
    the BatchNorm recomputed while staging); one call per micro-batch and one for all."""
    basic = tuple(W.Block(W.BASIC, 16, 16, 16, 1) for _ in range(2))
    for (h, w), b, m, grouped in (((32, 32), 5, 3, True), ((32, 32), 1, 2, False), ((64, 16), 3, 2, True), ((128, 8), 2, 2, True)):
        spec = W.PartitionSpec(name=f"t9-basic16@{h}x{w}-b{b}", in_h=h, in_w=w, in_c=16, blocks=basic, microbatch=b,
                               num_microbatches=m, seed=29)
        layerwise(oracle, spec, "bf16", grouped=grouped)
    # many convolutions of the class in one partition: the work items then take several images each (here 3, 3, ..., 2)
    many = tuple(W.Block(W.BASIC, 16, 16, 16, 1) for _ in range(40))
    spec = W.PartitionSpec(name="t9-40xbasic16@32x32-b32", in_h=32, in_w=32, in_c=16, blocks=many, microbatch=32,
                           num_microbatches=2, seed=29)
    layerwise(oracle, spec, "bf16", blockwise=False)
    post = tuple(W.Block(W.POSTACT, 16, 16, 16, 1) for _ in range(2))
    for fusion in (2, 1, 0):
        spec = W.PartitionSpec(name=f"t9-postact16@32x32-level{fusion}", in_h=32, in_w=32, in_c=16, blocks=post, microbatch=6,
                               num_microbatches=2, seed=31)
        layerwise(oracle, spec, "bf16", fusion=fusion, blockwise=False)   # the block-wise harness covers pre-activation blocks


def test_config1_resnet20_layerwise(gpu, oracle):
    for mode in ("bf16", "f32"):
        layerwise(oracle, W.config(1), mode, grouped=False)
        layerwise(oracle, W.config(1), mode, grouped=True)


def test_config2_resnet110_partition_full_size_layerwise(gpu, oracle):
    """Full size in the launch configuration bench.py times; the other fusion level and the fp32 mode on two of the eight
    micro-batches (same micro-batch size, same kernels)."""
    layerwise(oracle, W.config(2), "bf16")
    small = W.with_microbatching(W.config(2), 16, 2, loss_divisor=128)
    layerwise(oracle, small, "bf16", fusion=1)
    layerwise(oracle, small, "f32")


def test_config3_resnet1001_partition_full_size_layerwise(gpu, oracle):
    """The benchmark configuration: 21 blocks x 8 micro-batches x 32 images through the image-resident kernels."""
    layerwise(oracle, W.config(3), "bf16")


def test_config3_other_schedules_layerwise(gpu, oracle):
    spec = W.with_microbatching(W.config(3), 32, 2, loss_divisor=256)
    layerwise(oracle, spec, "bf16", fusion=1, blockwise=False)
    layerwise(oracle, spec, "bf16", fusion=0, blockwise=False)
    layerwise(oracle, spec, "bf16", grouped=False)
    layerwise(oracle, W.with_microbatching(W.config(3), 8, 2, loss_divisor=256), "f32")


def test_config6_wide_resnet1001_partition_full_size_layerwise(gpu, oracle):
    """Layer by layer at full size; block by block on two of the eight micro-batches."""
    layerwise(oracle, W.config(6), "bf16", blockwise=False)
    layerwise(oracle, W.with_microbatching(W.config(6), 32, 2, loss_divisor=256), "bf16")


def test_config4_resnet1001_whole_full_size_layerwise(gpu, oracle):
    """333 blocks + stem + head, 8 micro-batches of 8 images."""
    layerwise(oracle, W.config(4), "bf16", blockwise=False)


def test_config5_resnet152_stage3_full_size_layerwise(gpu, oracle):
    """36 blocks at 14x14x1024, 4 micro-batches of 16 images (3 TFLOP per oracle pass)."""
    layerwise(oracle, W.config(5), "bf16", blockwise=False)
