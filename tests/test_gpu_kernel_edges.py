"""Small problems at the edges of the kernels' tiles and of the rules that choose between them, against the oracle.

Tolerances: the ones of tests/parity.py (tiny = toy networks, where fp32 rounding is all there is)."""
import numpy as np
import pytest
import torch

from dds_inputs import make_params, workload
from dds_inputs.configs import Workload, ring_mixing, tiny_resnet
from parity import bf16_round, check_parity, flat_init, run_hip, run_oracle
from test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,B", [(1, 63), (2, 32), (3, 85), (2, 128)])
def test_update_ranges_by_split_count(W, B):
    # 16-channel layers at 16 x 16 pixels have one split per image: 63 and 64 of them are summed by tiles of 256 weights; of 255 and 256
    # images one per two, summed by tiles of 64 (the lines themselves: test_update_tiles_by_split_count)
    _compare(tiny_resnet(K=1, W=W, B=B, hw=16, c=16, precision="bf16"), seed=20, T=2)


@pytest.mark.parametrize("c,hw,B", [(4, 2, 3), (20, 6, 2), (1028, 2, 2)])
def test_global_average_pool_chunk_and_pixel_remainders(c, hw, B):
    # channel chunks that do not divide the workgroup, fewer pixels than pixel lanes, more than 256 chunks
    ops = [{"op": "conv", "cin": 3, "cout": c, "k": 1, "stride": 1, "pad": 0}, {"op": "relu"}, {"op": "gap"},
           {"op": "linear", "cin": c, "cout": 10}, {"op": "softmax_ce"}]
    _compare(Workload(name=f"gap_{c}", ops=ops, bounds=[0, len(ops)], K=1, W=2, B=B, in_shape=(3, hw, hw), classes=10,
                      precision="f32", lr=0.05, momentum=0.0, steps=2), seed=21, T=2, every_step=True, tiny=True)


@pytest.mark.parametrize("precision,c,hw,B", [
    ("bf16", 8, 1, 3), ("bf16", 24, 2, 5), ("bf16", 40, 7, 9), ("bf16", 2056, 3, 2), ("bf16", 16, 2, 700), ("bf16", 72, 4, 1900),
    ("f32", 12, 2, 600), ("f32", 4, 3, 5000)])
def test_global_average_pool_lanes_per_image(precision, c, hw, B):
    # bf16: one pixel, row-lanes that do not fill the workgroup, more chunks than a workgroup, more images than lanes allow a
    # row-lane per pixel; fp32: several images a wave, images past the last
    ops = [{"op": "conv", "cin": 3, "cout": c, "k": 1, "stride": 1, "pad": 0}, {"op": "relu"}, {"op": "gap"},
           {"op": "linear", "cin": c, "cout": 10}, {"op": "softmax_ce"}]
    _compare(Workload(name=f"gap_lanes_{c}", ops=ops, bounds=[0, len(ops)], K=1, W=2, B=B, in_shape=(3, hw, hw), classes=10,
                      precision=precision, lr=0.05, momentum=0.0, steps=2), seed=29, T=2, every_step=True, tiny=precision == "f32")


@pytest.mark.parametrize("W,B", [(2, 7), (3, 8), (2, 31), (5, 32)])
def test_mixing_update_ranges_by_split_count(W, B):
    # 7 / 8 / 31 / 32 splits per data-group: both sides of the lines between 256-, 64- and 32-element ranges
    from test_gpu_gossip import _compare as compare_gossip
    compare_gossip(tiny_resnet(K=2, W=W, B=B, hw=16, c=16, precision="bf16"), seed=22, T=4, mixing=ring_mixing(W, 0.3))


def _two_linear(precision, feat, hidden, W, B):
    ops = [{"op": "linear", "cin": feat, "cout": hidden}, {"op": "relu"}, {"op": "linear", "cin": hidden, "cout": 10},
           {"op": "softmax_ce"}]
    return Workload(name=f"linear_{feat}_{hidden}", ops=ops, bounds=[0, 2, 4], K=2, W=W, B=B, in_shape=(feat, 1, 1),
                    classes=10, precision=precision, lr=0.05, momentum=0.0, steps=4)


@pytest.mark.parametrize("precision,feat,hidden,W,B", [
    ("f32", 12, 8, 1, 1), ("f32", 124, 36, 2, 17), ("f32", 132, 128, 3, 16), ("f32", 1500, 130, 2, 9),
    ("bf16", 24, 16, 1, 15), ("bf16", 248, 136, 2, 31), ("bf16", 264, 40, 2, 33)])
def test_linear_layers_of_few_rows(precision, feat, hidden, W, B):
    # reductions on both sides of eight 64-byte k-steps and with a ragged last one, rows and columns off the
    # 16-element grid, hidden widths beyond one 128-column workgroup
    wl = _two_linear(precision, feat, hidden, W, B)
    _compare(wl, seed=23, T=4, every_step=precision == "f32", tiny=precision == "f32")


@pytest.mark.parametrize("B", [16, 5])
def test_linear_layers_with_weights_per_data_group(B):
    from test_gpu_gossip import _compare as compare_gossip
    compare_gossip(_two_linear("f32", 40, 24, 3, B), seed=24, T=4, mixing=ring_mixing(3, 0.3))


@pytest.mark.parametrize("c,hw,B", [(8, 1, 3), (16, 3, 5), (264, 5, 7), (12, 4, 33)])
def test_batch_norm_row_remainders(c, hw, B):
    # fewer rows than one pass of the workgroup, rows that do not fill the four-row trips, several splits
    from test_gpu_batchnorm import _compare as compare_bn
    ops = [{"op": "conv", "cin": 3, "cout": c, "k": 1, "stride": 1, "pad": 0}, {"op": "bn", "c": c, "eps": 1e-5},
           {"op": "relu"}, {"op": "gap"}, {"op": "linear", "cin": c, "cout": 10}, {"op": "softmax_ce"}]
    compare_bn(Workload(name=f"bn_rows_{c}", ops=ops, bounds=[0, len(ops)], K=1, W=2, B=B, in_shape=(3, hw, hw), classes=10,
                        precision="f32", lr=0.05, momentum=0.0, steps=2), seed=25, T=2, every_step=True, tiny=True)


def _conv_chain(precision, widths, h, w, W, B):
    ops = []
    for cin, cout in zip((3,) + widths[:-1], widths):
        ops += [{"op": "conv", "cin": cin, "cout": cout, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"}]
    ops += [{"op": "gap"}, {"op": "linear", "cin": widths[-1], "cout": 10}, {"op": "softmax_ce"}]
    return Workload(name=f"conv_chain_{h}x{w}", ops=ops, bounds=[0, len(ops)], K=1, W=W, B=B, in_shape=(3, h, w), classes=10,
                    precision=precision, lr=0.05, momentum=0.0, steps=2)


@pytest.mark.parametrize("precision,widths,h,w,W,B", [
    ("bf16", (32, 32, 64), 2, 2, 1, 3), ("bf16", (64, 64, 128), 3, 5, 2, 9), ("bf16", (64, 128, 128), 9, 7, 3, 5),
    ("bf16", (64, 64, 32), 4, 47, 1, 2), ("bf16", (64, 64, 32), 5, 48, 1, 2), ("bf16", (32, 64), 3, 95, 1, 2),
    ("bf16", (64, 192, 256, 200), 4, 4, 2, 5), ("bf16", (32, 64), 3, 96, 1, 2), ("bf16", (64, 128), 2, 160, 1, 2), ("f32", (32, 32, 64), 13, 3, 2, 7),
    ("f32", (16, 48, 32), 6, 10, 2, 3)])
def test_conv3x3_image_sizes(precision, widths, h, w, W, B):
    # images whose rows and planes are no power of two, tiles that hold many images or end inside one; W = 95 / 96: both sides of the
    # longest rows of the 256 x 64 tiles of one 64-byte chunk (the other tiles' limits: test_conv3x3_longest_rows_of_each_tile)
    _compare(_conv_chain(precision, widths, h, w, W, B), seed=26, T=2, every_step=precision == "f32", tiny=precision == "f32")


@pytest.mark.parametrize("B", [4095, 8191])
def test_fp32_conv3x3_tiles_by_pixel_count(B):
    # 256 and 512 tiles of 256 pixels x 128 columns, the last one ragged: 128- and 256-pixel tiles
    _compare(_conv_chain("f32", (32, 96), 4, 4, 1, B), seed=32, T=2, every_step=True, tiny=True)


@pytest.mark.parametrize("widths,h,w,W,B", [
    ((32, 64), 4, 4, 1, 8193),    # 512 x 64 tiles, the last one ragged
    ((64, 192), 8, 8, 1, 513),    # 256 x 128 tiles, ragged columns
    ((64, 80), 8, 8, 1, 133),     # 128 x 128 tiles
    ((64, 80), 8, 8, 3, 11),      # 64 x 64 tiles, ragged columns
    ((64, 64), 3, 191, 1, 1),     # ... the longest rows
    ((64, 64), 3, 192, 1, 1),     # one more: 256 x 64 tiles
    ((16, 48), 5, 7, 2, 9),       # one chunk, 256 x 64 tiles
    ((16, 136), 6, 5, 1, 9),      # ... and 128 x 128 ones
    ((64, 64), 3, 319, 1, 1),     # ... the longest rows
    ((64, 64), 3, 320, 1, 1),     # one more: conv_gather_kernel
    ((48, 96), 3, 359, 1, 1),     # 128 x 128 tiles, the longest rows
    ((48, 96), 3, 360, 1, 1)])    # one more: conv_gather_kernel
def test_fp32_conv3x3_of_split_operands_by_tile(widths, h, w, W, B):
    _compare(_conv_chain("f32", widths, h, w, W, B), seed=61, T=2, every_step=True, tiny=True)


def test_fp32_conv3x3_tiles_stay_within_a_data_group():
    # 65792 pixels a data-group, of 256 x 64 but not of 512 x 64 tiles
    from test_gpu_gossip import _compare as compare_gossip
    compare_gossip(_conv_chain("f32", (32, 64), 4, 4, 2, 4112), seed=62, T=2, mixing=ring_mixing(2, 0.3))


@pytest.mark.parametrize("cin,cout,h,B", [(16, 16, 8, 3), (32, 64, 8, 3), (64, 64, 8, 5), (64, 128, 8, 5), (64, 192, 8, 520), (32, 64, 16, 513)])
def test_fp32_conv3x3_of_values_whose_parts_are_not_finite(cin, cout, h, B):
    # Infinities and values that round to one in bf16: forward sums as fp64 has them (a NaN leaves the epilogue as -infinity), and
    # the weight gradient of a value near the largest. Bound: each of 9 cin terms may add a rounding error of 2^-24 to the sum.
    import paper_2509_05679_amd as P
    import torch.nn.functional as F
    ops = [{"op": "conv", "cin": cin, "cout": cout, "k": 3, "stride": 1, "pad": 1}, {"op": "gap"},
           {"op": "linear", "cin": cout, "cout": 10}, {"op": "softmax_ce"}]
    gen = torch.Generator().manual_seed(63)
    weights = torch.randn((cout, cin, 3, 3), generator=gen) * (2.0 / (9 * cin)) ** 0.5
    head = torch.randn((10, cout), generator=gen) * 0.1
    clean = torch.randn((B, cin, h, h), generator=gen)
    y = torch.randint(10, (B,), generator=gen, dtype=torch.int32)
    for values in ((float("inf"),), (float("-inf"), float("inf")), (3.4e38, 1e-39)):
        x = clean.clone()
        for i, v in enumerate(values):
            x[i, (5 * i) % cin, 3 * i, 1 + i] = v
        wl = Workload(name="not_finite", ops=ops, bounds=[0, 1, len(ops)], K=2, W=1, B=B, in_shape=(cin, h, h), classes=10, precision="f32",
                      lr=1e-37, momentum=0.0, steps=4)
        tr = P.Trainer(P.Spec.from_workload(wl), 1)
        first = np.concatenate([weights.numpy().ravel(), np.zeros(cout, np.float32)])
        tr.dds_set_params(0, first)
        tr.dds_set_params(1, np.concatenate([head.numpy().ravel(), np.zeros(10, np.float32)]))
        for _ in range(3):  # the third updates module 0, with the gradient of the first
            tr.dds_step([x.cuda()], [y.cuda()])
        torch.cuda.synchronize()
        got = torch.from_numpy(tr.dds_debug_read(P.DDS_DBG_OUTPUT, 0, 0).view(np.float32).copy()).reshape(B, h, h, cout).permute(0, 3, 1, 2)
        updated = torch.from_numpy(tr.dds_get_params(0)).double()[:weights.numel()].reshape(weights.shape)
        tr.close()
        wd = weights.double().requires_grad_()
        out = F.conv2d(x.double(), wd, padding=1)
        want = out.detach().float()
        want = torch.where(want.isnan(), torch.full_like(want, float("-inf")), want)
        finite = want.isfinite()
        assert torch.equal(got.isfinite(), finite) and torch.equal(got[~finite], want[~finite])
        small = finite & (want.abs() < 1e3)
        bound = 9 * cin * 2.0 ** -24
        assert (got[small] - want[small]).norm() <= bound * want[small].norm()
        if values[0] == 3.4e38:
            assert (got[finite].double() - out.detach()[finite]).norm() <= bound * out.detach()[finite].norm()
            F.cross_entropy(out.mean((2, 3)) @ head.double().T, y.long()).backward()
            change = wl.lr * wd.grad
            assert change.norm() > 0
            assert ((weights.double() - updated) - change).norm() <= 1e-5 * change.norm() + 2.0 ** -24 * weights.double().norm()


def _stride2_net(c1, c2, k, h, w, W, B, precision="bf16"):
    ops = [{"op": "conv", "cin": 3, "cout": c1, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"},
           {"op": "conv", "cin": c1, "cout": c2, "k": k, "stride": 2, "pad": k // 2}, {"op": "relu"},
           {"op": "conv", "cin": c2, "cout": c2, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"}, {"op": "gap"},
           {"op": "linear", "cin": c2, "cout": 10}, {"op": "softmax_ce"}]
    return Workload(name=f"stride2_k{k}_{h}x{w}", ops=ops, bounds=[0, len(ops)], K=1, W=W, B=B, in_shape=(3, h, w), classes=10,
                    precision=precision, lr=0.05, momentum=0.0, steps=2)


@pytest.mark.parametrize("c1,c2,k,h,w,W,B", [
    (16, 32, 3, 7, 9, 2, 3), (24, 72, 3, 14, 13, 1, 9), (64, 64, 1, 11, 6, 3, 5), (64, 128, 3, 8, 8, 2, 9),
    (32, 64, 3, 28, 30, 1, 3), (72, 136, 3, 3, 2, 2, 65), (96, 160, 3, 5, 4, 2, 3), (128, 256, 1, 4, 4, 1, 7), (8, 8, 1, 1, 5, 2, 30), (16, 16, 3, 2, 178, 1, 1)])
def test_weight_gradients_of_any_image_size(c1, c2, k, h, w, W, B):
    # odd sides, batches that are no whole 128-pixel tiles, channel counts off the 64-channel blocks, a single image
    # row, data-groups of less than a tile, long rows
    _compare(_stride2_net(c1, c2, k, h, w, W, B), seed=27, T=2)


@pytest.mark.parametrize("widths,h,w,W,B", [
    ((8, 16, 16, 32, 32, 8), 1, 1, 1, 1), ((16, 64, 16, 8), 3, 3, 2, 16), ((32, 16, 64, 8), 3, 3, 1, 17), ((64, 32, 32, 16), 15, 15, 3, 5),
    ((32, 32, 32), 2, 378, 1, 2), ((32, 32), 2, 388, 1, 1), ((16, 16, 16), 31, 15, 2, 9), ((20, 12, 24), 5, 4, 2, 7),
    ((32, 32), 16, 16, 1, 1), ((32, 16), 15, 15, 1, 2), ((32, 32), 3, 253, 1, 2), ((32, 32), 3, 254, 1, 2), ((32, 32), 128, 380, 1, 1),
    ((32, 32), 3, 680, 1, 2), ((32, 32), 3, 681, 1, 2)])
def test_weight_gradients_of_narrow_layers(widths, h, w, W, B):
    # 8, 16 and 32 input channels, each with one or two blocks of output rows; one pixel, data-groups of exactly one and of one and a
    # bit 256-pixel tiles (16 x 16 with one and 15 x 15 with two images), the longest rows of two tiles in LDS and of one with 32 channels and
    # the first beyond them, channel counts that fill no row
    _compare(_conv_chain("bf16", widths, h, w, W, B), seed=34, T=2)


@pytest.mark.parametrize("widths,h,w,W,B", [
    ((16, 16), 2, 2, 1, 1), ((16, 16, 12), 5, 7, 3, 4), ((12, 16, 16), 16, 16, 1, 2), ((16, 16), 3, 48, 2, 5), ((32, 16, 16), 8, 6, 2, 3),
    ((64, 16), 4, 16, 1, 3), ((60, 16), 5, 13, 1, 3), ((16, 16), 2, 2000, 1, 1), ((16, 16), 2, 2001, 1, 1),
    ((16, 16), 3, 258, 1, 2), ((16, 16), 3, 259, 2, 2), ((32, 16, 16), 5, 272, 1, 2), ((64, 16), 3, 130, 1, 2), ((60, 16), 4, 131, 1, 2),
    ((64, 16), 3, 144, 1, 2)])
def test_direct_convolutions_of_narrow_layers(widths, h, w, W, B):
    # stems of 16, 32 and 64 output rows, also not filled ones, and 16 -> 16 layers in both directions; rows of 16 pixels and others, less
    # than a run, a ragged last tile; rows on both sides of the line (258 pixels, 130 with 64 outputs) from which a tile's patch is three runs
    _compare(_conv_chain("bf16", widths, h, w, W, B), seed=39, T=2)


@pytest.mark.parametrize("precision", ["f32", "bf16"])
@pytest.mark.parametrize("k,pad,h,w", [(1, 0, 7, 6), (2, 0, 6, 9), (2, 1, 7, 7), (3, 0, 9, 8), (5, 2, 8, 5)])
def test_stride2_input_gradients_by_padding(precision, k, pad, h, w):
    # which parity class of the input gradient has the most taps (and is launched first) depends on the padding
    ops = [{"op": "conv", "cin": 3, "cout": 32, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"},
           {"op": "conv", "cin": 32, "cout": 64, "k": k, "stride": 2, "pad": pad}, {"op": "relu"}, {"op": "gap"},
           {"op": "linear", "cin": 64, "cout": 10}, {"op": "softmax_ce"}]
    _compare(Workload(name=f"stride2_k{k}_pad{pad}", ops=ops, bounds=[0, len(ops)], K=1, W=2, B=37, in_shape=(3, h, w), classes=10,
                      precision=precision, lr=0.05, momentum=0.0, steps=2), seed=33, T=2, every_step=precision == "f32", tiny=precision == "f32")


@pytest.mark.parametrize("c1,c2,k,h,w,W,B", [
    (16, 36, 3, 7, 9, 2, 3), (32, 64, 1, 8, 8, 2, 9), (68, 132, 3, 13, 14, 1, 3), (16, 16, 3, 2, 88, 1, 1),
    (12, 16, 3, 1, 3, 3, 33)])
def test_weight_gradients_of_any_image_size_fp32(c1, c2, k, h, w, W, B):
    # channel counts off the 32-channel panels and 64-channel blocks, partial tiles, rows of more than one tile
    _compare(_stride2_net(c1, c2, k, h, w, W, B, "f32"), seed=28, T=2, every_step=True, tiny=True)


@pytest.mark.parametrize("name,B,steps", [("paper_r20_S1K1", 194, 20), ("paper_r20_S1K1", 7, 40), ("paper_r20_S4K1", 96, 20)])
def test_single_module_beside_its_weight_gradients_is_bit_identical(name, B, steps):
    # one module: weight gradients on a stream of their own where they are long enough (the third case, 1.6 GFLOP on average),
    # against everything on the caller's stream
    from test_gpu_limits import test_run_ahead_across_iterations_is_bit_identical_to_serial_execution as compare
    compare(name, B, steps)


def _middle_linear(precision, feat, hidden, out, W, B, seed):
    # feat -> hidden | hidden -> out -> 10: one step forwards module 0, two steps module 1
    ops = [{"op": "linear", "cin": feat, "cout": hidden}, {"op": "relu"}, {"op": "linear", "cin": hidden, "cout": out}, {"op": "relu"},
           {"op": "linear", "cin": out, "cout": 10}, {"op": "softmax_ce"}]
    wl = Workload(name=f"middle_linear_{hidden}_{out}", ops=ops, bounds=[0, 2, 6], K=2, W=W, B=B, in_shape=(feat, 1, 1), classes=10,
                  precision=precision, lr=0.01, momentum=0.0, steps=4)
    import paper_2509_05679_amd as P
    tr = P.Trainer(P.Spec.from_workload(wl), W)
    for k0, t in enumerate(make_params(wl, seed)):
        tr.dds_set_params(k0, t)
    return tr


@pytest.mark.parametrize("precision,most_us", [("bf16", 60.0), ("f32", 95.0)])
def test_linear_layers_of_many_rows_run_on_the_tiled_kernels(precision, most_us):
    # 512 -> 512 at 4096 rows. Both kernels are right there, but the 16 x 16 tiles take 63 and 73 us where the tiled kernel takes 13
    # and 44. Forward launches of the step (with 64 -> 512 and 512 -> 10): 87 and 120 us with them, 34 and 72 us here
    W, B = 4, 1024
    tr = _middle_linear(precision, 64, 512, 512, W, B, seed=30)
    xs, ys = [torch.zeros((B, 64, 1, 1), device="cuda") for _ in range(W)], [torch.zeros(B, dtype=torch.int32, device="cuda") for _ in range(W)]
    for _ in range(3):
        tr.dds_step(xs, ys)
    times = []
    for _ in range(5):
        tr.dds_profile(2)
        tr.dds_step(xs, ys)
        times.append(1e3 * tr.dds_profile_read()["forward"][0])
    tr.close()
    assert min(times) < most_us, times


def test_profile_classes_of_the_resnet18_launches():
    # 13 of the 21 convolutions and linear layers are 3x3 stride 1; stem, three stride-2 layers, their shortcuts and the head are not
    # (the folded shortcuts and the stem have no input-gradient launch of their own)
    import paper_2509_05679_amd as P
    wl = workload("cfg2_resnet18", B=16)
    tr = P.Trainer(P.Spec.from_workload(wl), wl.W)
    for k0, t in enumerate(make_params(wl, 37)):
        tr.dds_set_params(k0, t)
    xs, ys = [torch.zeros((16, 3, 32, 32), device="cuda") for _ in range(4)], [torch.zeros(16, dtype=torch.int32, device="cuda") for _ in range(4)]
    for _ in range(2 * (wl.K - 1) + 1):
        tr.dds_step(xs, ys)
    tr.dds_profile(2)
    tr.dds_step(xs, ys)
    launches = {k: v[1] for k, v in tr.dds_profile_read().items()}
    tr.close()
    assert launches == {"forward": 8, "dgrad": 4, "wgrad": 1, "forward_dma": 13, "dgrad_dma": 13, "wgrad_dma": 20}


@pytest.mark.parametrize("feat,out,below,above", [(256, 64, 512, 8192), (252, 64, 512, 16384), (2048, 20, 64, 16384)])
def test_fp32_sums_of_a_linear_layer_do_not_depend_on_its_rows(feat, out, below, above):
    # the same rows below and above the line between linear.hip and the tiled kernels (conv_gather_kernel; 252 channels are
    # no whole 64-byte chunks and stay on conv_gemm_kernel): the same sums in the same order, so bit for bit
    import paper_2509_05679_amd as P
    gen = torch.Generator(device="cuda").manual_seed(31)
    x = torch.randn((above, feat, 1, 1), device="cuda", generator=gen)
    y = torch.zeros(above, dtype=torch.int32, device="cuda")
    rows = []
    for n in (below, above):
        tr = _middle_linear("f32", feat, out, 16, 1, n, seed=31)
        tr.dds_step([x[:n].contiguous()], [y[:n].contiguous()])
        stored = tr.dds_debug_read(P.DDS_DBG_OUTPUT, 0, 0).view(np.float32).reshape(n, -1)
        rows.append(stored[:below].copy())
        tr.close()
    assert np.abs(rows[0]).max() > 0 and np.array_equal(rows[0], rows[1])


@pytest.mark.parametrize("widths,h,w,W,B", [
    ((64, 64), 15, 13, 1, 90),    # 17550 pixels: 256 x 64 tiles of 128-byte rows, odd sides, the last tile ragged
    ((64, 64), 5, 47, 1, 70),     # ... the longest rows they fetch
    ((64, 64), 5, 48, 1, 69),     # one more: 256 x 64 tiles of 64-byte rows
    ((64, 128), 3, 159, 1, 1),    # 128 x 128 tiles, the longest rows (160: conv_gather_kernel, above)
    ((128, 128), 3, 75, 1, 2),    # 64 x 64 tiles with a shared reduction, the longest rows
    ((128, 128), 3, 76, 1, 2),    # one more: 128 x 128 tiles
    ((64, 64), 2, 190, 1, 2),     # weight gradient on padded positions, the longest rows
    ((64, 64), 2, 191, 1, 2),     # one more: wgrad_gemm_kernel
])
def test_conv3x3_longest_rows_of_each_tile(widths, h, w, W, B):
    _compare(_conv_chain("bf16", widths, h, w, W, B), seed=34, T=2)


@pytest.mark.parametrize("w", [764, 766])
def test_stride2_weight_gradients_longest_rows(w):
    # 382 and 383 output columns: wgrad_flat_body and wgrad_gemm_kernel
    _compare(_stride2_net(16, 16, 3, 2, w, 1, 2), seed=35, T=2)


@pytest.mark.parametrize("c1,c2,h,w,W,B", [
    (64, 64, 64, 64, 1, 1), (16, 32, 32, 32, 1, 3), (64, 128, 16, 16, 2, 3), (128, 200, 8, 8, 1, 4), (24, 72, 32, 16, 3, 1), (64, 64, 16, 64, 1, 2),
    (40, 64, 4, 302, 1, 2), (40, 64, 4, 303, 1, 2)])
def test_stride2_weight_gradients_by_tile(c1, c2, h, w, W, B):
    # tiles of two rows of 32, four of 16, an image of 8 x 8, four of 4 x 4; data-groups of a single tile; one tile after another down an image; the
    # longest rows whose four planes fit twice and the first that are taken a sub-pixel at a time
    _compare(_stride2_net(c1, c2, 3, h, w, W, B), seed=52, T=2)


def test_shared_reductions_with_weights_per_data_group():
    # four data-groups of 256 or more pixels in one launch of few tiles: both kernels whose 64 x 64 tiles two halves of a workgroup
    # share, forward and input gradients (3x3 at 8 x 8 and 4 x 4, stride 2 with the folded shortcut)
    from test_gpu_gossip import _compare as compare_gossip
    ops = [{"op": "conv", "cin": 3, "cout": 128, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"},
           {"op": "conv", "cin": 128, "cout": 128, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"},
           {"op": "res_begin"}, {"op": "conv", "cin": 128, "cout": 256, "k": 3, "stride": 2, "pad": 1}, {"op": "relu"},
           {"op": "conv", "cin": 256, "cout": 256, "k": 3, "stride": 1, "pad": 1},
           {"op": "res_add", "scale": 1.0, "shortcut": {"cin": 128, "cout": 256, "k": 1, "stride": 2, "pad": 0}}, {"op": "relu"},
           {"op": "gap"}, {"op": "linear", "cin": 256, "cout": 10}, {"op": "softmax_ce"}]
    wl = Workload(name="shared_reductions", ops=ops, bounds=[0, 4, len(ops)], K=2, W=4, B=16, in_shape=(3, 8, 8), classes=10,
                  precision="bf16", lr=0.05, momentum=0.0, steps=4)
    compare_gossip(wl, seed=36, T=4, mixing=ring_mixing(4, 0.3), tiny=False)


@pytest.mark.parametrize("widths,h,w,W,B", [
    ((16,) * 19, 16, 16, 2, 5),                       # more layers of one kind than a launch takes (16)
    ((64, 64, 128, 64, 72, 64), 8, 8, 1, 33),         # whole 128-pixel tiles and others (72 channels in) share a launch
    ((64,) * 5, 32, 32, 1, 700)])                     # launches closed by their work: 5600 tiles a layer, three layers
def test_weight_gradients_that_share_a_launch(widths, h, w, W, B):
    # against every layer in a launch of its own, with the splits that it has in the shared one: the same bits
    import paper_2509_05679_amd as P
    wl = _conv_chain("bf16", widths, h, w, W, B)
    gen = torch.Generator(device="cuda").manual_seed(38)
    xs = [torch.randn((B, 3, h, w), device="cuda", generator=gen) for _ in range(W)]
    ys = [torch.randint(10, (B,), device="cuda", generator=gen, dtype=torch.int32) for _ in range(W)]
    init, runs = make_params(wl, 38), []
    for mode in (0, 3):
        tr = P.Trainer(P.Spec.from_workload(wl), W)
        tr.dds_set_params(0, init[0])
        tr.dds_profile(mode)
        for _ in range(3):
            tr.dds_step(xs, ys)
        runs.append((tr.dds_get_params(0), tr.dds_launches_last_step()))
        tr.close()
    (runs, launches) = zip(*runs)
    assert launches[1] - launches[0] >= 2
    assert np.isfinite(runs[0]).all() and np.array_equal(runs[0], runs[1])
    assert not np.array_equal(runs[0], np.concatenate([p.ravel() for p in init[0]]))


@pytest.mark.parametrize("B", [8, 9, 64, 65])
def test_update_tiles_by_split_count(B):
    # one split per image of 16 x 16 pixels: both sides of the lines between tiles of 1024, 256 and 64 weights; tiles of 8, 16 and 32 input
    # channels, output channels that fill no tile (fp32 nets have one tile size: the other tests)
    _compare(_conv_chain("bf16", (16, 16, 32, 32, 12), 16, 16, 1, B), seed=40, T=2)


@pytest.mark.parametrize("c1,c2,h,w,W,B", [(8, 12, 1, 1, 2, 64), (72, 136, 1, 1, 3, 43), (64, 64, 4, 4, 1, 8), (128, 200, 3, 5, 2, 9), (16, 40, 1, 129, 1, 1)])
def test_weight_gradients_of_pointwise_layers(c1, c2, h, w, W, B):
    # 1x1 convolutions and the head: one whole tile of 128 rows, one row more, less than a tile, channel counts off the 64-channel blocks
    ops = [{"op": "conv", "cin": 3, "cout": c1, "k": 1, "stride": 1, "pad": 0}, {"op": "relu"},
           {"op": "conv", "cin": c1, "cout": c2, "k": 1, "stride": 1, "pad": 0}, {"op": "relu"}, {"op": "gap"},
           {"op": "linear", "cin": c2, "cout": 10}, {"op": "softmax_ce"}]
    _compare(Workload(name=f"pointwise_{c1}_{c2}", ops=ops, bounds=[0, len(ops)], K=1, W=W, B=B, in_shape=(3, h, w), classes=10,
                      precision="bf16", lr=0.05, momentum=0.0, steps=2), seed=41, T=2)


@pytest.mark.parametrize("c,hw,B", [(24, 32, 22), (24, 3, 2), (36, 7, 9), (64, 5, 3), (64, 32, 9), (136, 4, 5)])
def test_batch_norm_sums_shared_by_threads(c, hw, B):
    # four, two and one thread per sum, channel groups that do not divide the workgroup; as many splits as the streaming kernels
    # fold (64 of 24 channels), more than they do (72 of 64), rows too wide for it
    from test_gpu_batchnorm import _compare as compare_bn
    ops = [{"op": "conv", "cin": 3, "cout": c, "k": 1, "stride": 1, "pad": 0}, {"op": "bn", "c": c, "eps": 1e-5},
           {"op": "relu"}, {"op": "gap"}, {"op": "linear", "cin": c, "cout": 10}, {"op": "softmax_ce"}]
    compare_bn(Workload(name=f"bn_sums_{c}", ops=ops, bounds=[0, len(ops)], K=1, W=2, B=B, in_shape=(3, hw, hw), classes=10,
                        precision="f32", lr=0.05, momentum=0.0, steps=2), seed=42, T=2, every_step=True, tiny=True)


def _normalised_block(c, h, w, W, B, cuts=()):
    """A normalised stem, a normalised residual block and one more normalised layer (module boundaries: behind these)."""
    bn = {"op": "bn", "c": c, "eps": 1e-5}
    conv = {"op": "conv", "cin": c, "cout": c, "k": 3, "stride": 1, "pad": 1}
    parts = [[dict(conv, cin=3), bn, {"op": "relu"}],
             [{"op": "res_begin"}, conv, bn, {"op": "relu"}, conv, bn, {"op": "res_add", "scale": 1.0, "shortcut": None}, {"op": "relu"}],
             [conv, bn, {"op": "relu"}, {"op": "gap"}, {"op": "linear", "cin": c, "cout": 10}, {"op": "softmax_ce"}]]
    bounds, ops = [0], []
    for i, part in enumerate(parts):
        ops += part
        if i in cuts or i == 2:
            bounds.append(len(ops))
    return Workload(name=f"normalised_{c}_{h}x{w}", ops=ops, bounds=bounds, K=len(bounds) - 1, W=W, B=B, in_shape=(3, h, w), classes=10,
                    precision="bf16", lr=0.02, momentum=0.0, steps=2)


@pytest.mark.parametrize("c,h,w,W,B,cuts", [
    (16, 32, 32, 2, 3, ()), (16, 9, 5, 3, 2, ()), (16, 8, 8, 2, 520, ()), (16, 33, 32, 1, 3, ()), (32, 16, 16, 1, 5, (1,)), (32, 28, 28, 2, 96, ()), (32, 6, 6, 2, 258, ()),
    (64, 8, 8, 2, 6, (0, 1)), (64, 15, 14, 1, 200, ()), (64, 4, 4, 1, 1024, ()), (64, 10, 10, 1, 257, ())])
def test_normalisations_streamed_by_the_next_layers_launch(c, h, w, W, B, cuts):
    # one to eight runs of 16 pixels a wave, one to eight images a workgroup; with and without a residual or a gradient added; normalisations at a
    # module's end, which nothing follows; one and two workgroups a CU; beyond the largest image of 16 channels (33 x 32), one workgroup too many (257). Held to
    # the oracle that rounds what is stored to bf16: the launches apart are 0.002 to 0.080 of the update away from it (from the exact one
    # 0.12 to 0.22, which is what bf16 storage costs a net of four normalisations)
    from test_gpu_batchnorm import _dead_biases
    wl, T = _normalised_block(c, h, w, W, B, cuts), 2 * len(cuts) + 2
    print(f"[edges] {wl.name} K={wl.K} W={W} B={B} T={T}", flush=True)
    hip, _ = run_hip(wl, 54, T, None, True)
    oracle, _ = run_oracle(wl, 54, T, None, True, q=bf16_round())
    dead = set().union(*[_dead_biases(wl, k0) for k0 in range(wl.K)])
    check_parity(wl, hip, oracle, flat_init(wl, 54), tol=2e-2, update_tol=0.1, label=" rounded", skip=dead)


@pytest.mark.parametrize("c,h,w,W,B", [(16, 9, 5, 3, 4), (64, 8, 8, 2, 5)])
def test_normalisations_streamed_with_weights_per_data_group(c, h, w, W, B):
    # (as above, every data-group's own weights)
    from test_gpu_batchnorm import _dead_biases
    from test_gpu_gossip import _run_hip, _run_oracle
    wl, T = _normalised_block(c, h, w, W, B), 3
    hip, _ = _run_hip(wl, 55, T, ring_mixing(W, 0.3), None)
    oracle, _ = _run_oracle(wl, 55, T, ring_mixing(W, 0.3), None, q=bf16_round())
    for s in range(W):
        check_parity(wl, [hip[t][s] for t in range(T)], [oracle[t][s] for t in range(T)], flat_init(wl, 55), tol=2e-2, update_tol=0.1, skip=_dead_biases(wl, 0))


@pytest.mark.parametrize("cin,cout,h,w,B", [(8, 16, 8, 8, 5), (8, 64, 15, 15, 3), (16, 16, 16, 32, 3), (16, 16, 5, 7, 40), (16, 32, 2, 600, 3),
                                            (32, 32, 32, 32, 3), (32, 32, 3, 300, 3), (32, 16, 2, 600, 2)])
def test_a_pixel_reaches_only_the_taps_that_see_it(cin, cout, h, w, B):
    # a NaN in a corner of the input of a 3x3 layer: its weight gradient is NaN at the four taps that see the corner, and nowhere else
    # (the ReLU behind the layer turns the NaNs of the forward pass into zeros, so nothing else in the net is touched)
    import paper_2509_05679_amd as P
    ops = [{"op": "conv", "cin": cin, "cout": cout, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"}, {"op": "gap"},
           {"op": "linear", "cin": cout, "cout": 10}, {"op": "softmax_ce"}]
    wl = Workload(name=f"corner_{cin}_{cout}", ops=ops, bounds=[0, len(ops)], K=1, W=1, B=B, in_shape=(cin, h, w), classes=10,
                  precision="bf16", lr=0.05, momentum=0.0, steps=1)
    gen = torch.Generator(device="cuda").manual_seed(44)
    for bottom in (0, 1):
        for right in (0, 1):
            x = torch.randn((B, cin, h, w), device="cuda", generator=gen)
            x[B // 2, 1, -bottom, -right] = float("nan")
            tr = P.Trainer(P.Spec.from_workload(wl), 1)
            tr.dds_set_params(0, make_params(wl, 44)[0])
            tr.dds_step([x], [torch.zeros(B, dtype=torch.int32, device="cuda")])
            got = ~np.isfinite(tr.dds_get_params(0))
            tr.close()
            want = np.zeros((cout, cin, 3, 3), bool)
            want[:, 1, bottom:bottom + 2, right:right + 2] = True
            assert np.array_equal(got[:want.size].reshape(want.shape), want) and not got[want.size:].any(), (bottom, right)


def test_direct_convolutions_of_wide_images_copy_three_runs():
    # 16 -> 16 channels, 2^20 pixels in rows of 32 and of 1024: forward and input gradient 41 and 98 us with a patch that holds the pixels
    # between the three image rows too, 49 us with three runs at 1024
    import paper_2509_05679_amd as P

    def best(h, w, B):
        wl = _conv_chain("bf16", (16, 16), h, w, 1, B)
        tr = P.Trainer(P.Spec.from_workload(wl), 1)
        tr.dds_set_params(0, make_params(wl, 45)[0])
        xs, ys = [torch.zeros((B, 3, h, w), device="cuda")], [torch.zeros(B, dtype=torch.int32, device="cuda")]
        times = []
        for _ in range(8):
            tr.dds_profile(2)
            tr.dds_step(xs, ys)
            got = tr.dds_profile_read()
            times.append(got["forward_dma"][0] + got["dgrad_dma"][0])
        tr.close()
        return min(times)

    assert best(256, 1024, 4) < 1.7 * best(32, 32, 1024)


@pytest.mark.parametrize("name", ["cfg2_resnet18", "cfg1_cnn"])
def test_profiling_times_the_launches_of_any_other_step(name):
    import paper_2509_05679_amd as P
    wl = workload(name, B=16)
    tr = P.Trainer(P.Spec.from_workload(wl), wl.W)
    for k0, t in enumerate(make_params(wl, 46)):
        tr.dds_set_params(k0, t)
    xs = [torch.zeros((16, *wl.in_shape), device="cuda") for _ in range(wl.W)]
    ys = [torch.zeros(16, dtype=torch.int32, device="cuda") for _ in range(wl.W)]
    for _ in range(2 * (wl.K - 1) + 1):
        tr.dds_step(xs, ys)
    launches = tr.dds_launches_last_step()
    for mode in (1, 2):
        tr.dds_profile(mode)
        tr.dds_step(xs, ys)
        got = tr.dds_profile_read()
        assert tr.dds_launches_last_step() == launches
        assert sum(v[2] for v in got.values()) == pytest.approx(tr.dds_gemm_flops_per_step(), rel=1e-12)
        assert all(v[0] > 0 for v in got.values() if v[1])
    tr.close()


@pytest.mark.parametrize("c,bn_launches", [(16, 4), (136, 6)])
def test_launches_of_a_normalised_net_are_counted(c, bn_launches):
    # the splits' sums of rows of up to 64 channels are joined by the streaming kernels, those of wider rows by a launch of their own in
    # either direction
    import paper_2509_05679_amd as P
    tail = [{"op": "relu"}, {"op": "gap"}, {"op": "linear", "cin": c, "cout": 10}, {"op": "softmax_ce"}]
    counts = []
    for bn in ([], [{"op": "bn", "c": c, "eps": 1e-5}]):
        ops = [{"op": "conv", "cin": 3, "cout": c, "k": 3, "stride": 1, "pad": 1}] + bn + tail
        wl = Workload(name=f"launches_{c}", ops=ops, bounds=[0, len(ops)], K=1, W=1, B=4, in_shape=(3, 8, 8), classes=10,
                      precision="bf16", lr=0.05, momentum=0.0, steps=1)
        tr = P.Trainer(P.Spec.from_workload(wl), 1)
        tr.dds_set_params(0, make_params(wl, 47)[0])
        tr.dds_step([torch.zeros((4, 3, 8, 8), device="cuda")], [torch.zeros(4, dtype=torch.int32, device="cuda")])
        counts.append(tr.dds_launches_last_step())
        tr.close()
    assert counts[1] - counts[0] == bn_launches


def test_weight_gradients_that_share_no_launch_run_beside_the_input_gradients(monkeypatch):
    # one module of 5x5 layers: 315 us a step with a stream of their own, 358 us (as with DDS_SERIAL) without
    import paper_2509_05679_amd as P
    ops = []
    for cin, cout in ((3, 64), (64, 72), (72, 128), (128, 64)):
        ops += [{"op": "conv", "cin": cin, "cout": cout, "k": 5, "stride": 1, "pad": 2}, {"op": "relu"}]
    ops += [{"op": "gap"}, {"op": "linear", "cin": 64, "cout": 10}, {"op": "softmax_ce"}]
    wl = Workload(name="beside", ops=ops, bounds=[0, len(ops)], K=1, W=4, B=8, in_shape=(3, 14, 14), classes=10, precision="bf16", lr=0.05,
                  momentum=0.0, steps=1)
    xs, ys = [torch.zeros((8, 3, 14, 14), device="cuda") for _ in range(4)], [torch.zeros(8, dtype=torch.int32, device="cuda") for _ in range(4)]

    def best():
        tr = P.Trainer(P.Spec.from_workload(wl), 4)
        tr.dds_set_params(0, make_params(wl, 48)[0])
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(6):
            t0.record()
            for _ in range(20):
                tr.dds_step(xs, ys)
            t1.record()
            t1.synchronize()
            times.append(t0.elapsed_time(t1))
        tr.close()
        return min(times)

    beside = best()
    monkeypatch.setenv("DDS_SERIAL", "1")
    assert beside < 0.95 * best()


def _identity_blocks(c, blocks, h, w, W, B, cuts=()):
    """A stem to c channels and residual blocks of that width; cuts: blocks that a module ends behind. (Nine blocks added at 0.7 each end the first
    step at a loss of 1e9, with every library.)"""
    ops, bounds = [{"op": "conv", "cin": 3, "cout": c, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"}], [0]
    for i in range(blocks):
        ops += [{"op": "res_begin"}, {"op": "conv", "cin": c, "cout": c, "k": 3, "stride": 1, "pad": 1}, {"op": "relu"},
                {"op": "conv", "cin": c, "cout": c, "k": 3, "stride": 1, "pad": 1}, {"op": "res_add", "scale": 0.7 / blocks, "shortcut": None}, {"op": "relu"}]
        if i in cuts:
            bounds.append(len(ops))
    ops += [{"op": "gap"}, {"op": "linear", "cin": c, "cout": 10}, {"op": "softmax_ce"}]
    bounds.append(len(ops))
    return Workload(name=f"identity_blocks_{c}", ops=ops, bounds=bounds, K=len(bounds) - 1, W=W, B=B, in_shape=(3, h, w), classes=10,
                    precision="bf16", lr=0.05, momentum=0.0, steps=2)


@pytest.mark.parametrize("c,blocks,h,w,W,B,cuts", [
    (16, 2, 1, 1, 1, 3, ()), (16, 9, 5, 7, 1, 4, ()), (16, 3, 32, 32, 1, 2, (0,)), (16, 2, 31, 33, 1, 64, ()), (16, 2, 32, 33, 1, 64, ()), (16, 1, 30, 18, 1, 3, ()),
    (32, 2, 2, 3, 1, 300, ()), (32, 2, 16, 16, 1, 3, (0,)), (32, 2, 31, 31, 1, 64, ()), (32, 1, 9, 9, 1, 257, ()), (32, 2, 32, 31, 1, 64, ()),
    (64, 2, 8, 8, 1, 1021, ()), (64, 2, 8, 8, 2, 258, (0,)), (64, 2, 14, 14, 1, 2, ()), (64, 2, 16, 16, 1, 1, ()), (64, 1, 3, 5, 1, 2050, ()), (64, 2, 17, 16, 1, 1, ())])
def test_runs_of_narrow_layers_share_a_launch(c, blocks, h, w, W, B, cuts):
    # one pixel; more layers than a launch takes; a residual added by the first layer of a module's launch; the largest images of each width and
    # the first beyond them (32 x 33 of 16 channels, 32 x 31 of 32, 17 x 16 of 64: a launch each); two and more images a workgroup, the last one short of them
    _compare(_identity_blocks(c, blocks, h, w, W, B, cuts), seed=50, T=2 * len(cuts) + 2)


@pytest.mark.parametrize("c,blocks,h,w,W,B,cuts", [
    (64, 2, 32, 32, 1, 192, ()), (64, 2, 31, 33, 1, 194, (0,)), (64, 1, 32, 32, 1, 461, ()), (64, 3, 17, 16, 1, 256, ()), (64, 1, 20, 21, 2, 100, ()), (64, 2, 1, 250, 1, 193, ()),
    (64, 2, 32, 33, 1, 192, ()), (128, 2, 16, 16, 1, 200, (0,)), (128, 9, 5, 3, 1, 192, ()), (128, 2, 14, 14, 1, 460, ()), (128, 2, 8, 8, 1, 1021, ()), (128, 2, 4, 4, 3, 516, ()),
    (128, 2, 12, 12, 1, 257, ()), (128, 2, 17, 16, 1, 194, ())])
def test_runs_of_wider_layers_share_a_launch(c, blocks, h, w, W, B, cuts):
    # one to eight runs of 16 pixels a wave; more layers than a launch takes; a module's first layer adding a residual; several images a workgroup, the
    # last one short of them; the largest images and the first beyond them (32 x 33 of 64 channels, 17 x 16 of 128); fewest images, two rounds, and
    # counts (257) and lengths (two layers of 461 images) that keep a launch a layer
    _compare(_identity_blocks(c, blocks, h, w, W, B, cuts), seed=53, T=2 * len(cuts) + 2)


@pytest.mark.parametrize("c,h,w,W,B", [(16, 9, 5, 3, 2), (32, 6, 6, 2, 130), (64, 4, 4, 2, 260), (64, 4, 4, 4, 131), (64, 17, 17, 2, 100), (128, 8, 8, 2, 100)])
def test_runs_of_narrow_layers_with_weights_per_data_group(c, h, w, W, B):
    # (64, ..., 131): an odd number of images per data-group, one a workgroup
    from test_gpu_gossip import _compare as compare_gossip
    compare_gossip(_identity_blocks(c, 2, h, w, W, B, (0,)), seed=51, T=4, mixing=ring_mixing(W, 0.3))
