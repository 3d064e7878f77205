"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by
element on the same seeded inputs.  Packing metadata must be bit-exact; outputs
within max relative error 1e-2 (bf16) / 1e-5 (fp32), each layer fed the oracle's
rounded input (teacher forcing), stacks additionally end to end."""
import numpy as np
import pytest

import oracle
from tests import helpers
from tests.helpers import TOL, from_dev, new_dev, pack_layer, rel_err, run_layer_gpu, to_dev
from workloads import configs, dtypes, masks, prng

pytestmark = pytest.mark.gpu

# Stacks end to end: norm-wise bound on the final tensor (max |g - o| / max |o|) plus arg-max agreement.  Element-wise
# 1e-2 cannot hold through several roundings to bf16: a layer's fp32 and the oracle's fp64 sums can land on opposite
# sides of a rounding boundary of an intermediate value, which moves that value by a whole bf16 step (2^-8).
STACK_NORM_TOL = 1e-2


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def layerwise(npas, torch, w, check_meta=True):
    """Teacher-forced layer-by-layer comparison of a workload; returns worst error."""
    rounded, raw = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    shapes = {0: w.x_shape}
    worst = 0.0
    for i, L in enumerate(w.layers):
        in_shape = shapes[L.src]
        shapes[i + 1] = helpers.out_shape(L, in_shape)
        packed = pack_layer(npas, L, w.dtype) if L.kind in ("conv", "fc", "dwconv") else None
        if packed is not None and check_meta and L.kind != "dwconv":
            helpers.check_metadata(oracle, L, packed, w.dtype)
            assert packed.info()["device_ready"] == 1
        xs, _ = dtypes.quantize(rounded[L.src], w.dtype)
        x_dev = to_dev(xs, torch)
        res_dev = None
        if L.res >= 0:
            rs, _ = dtypes.quantize(rounded[L.res], w.dtype)
            res_dev = to_dev(rs, torch)
        bias_dev = helpers.bias_tensors([L], torch)[0]
        y = run_layer_gpu(npas, torch, L, packed, x_dev, in_shape, w.dtype, res_dev, bias_dev)
        got = from_dev(y, w.dtype).reshape(shapes[i + 1])
        err = rel_err(got, rounded[i + 1].reshape(shapes[i + 1]))
        print(f"  layer {i:2d} {L.name or L.kind:12s} in={in_shape} out={shapes[i + 1]} err={err:.3e}", flush=True)
        assert err <= TOL[w.dtype], (i, L.name, err)
        worst = max(worst, err)
    return worst


def test_config1_conv3x3_fp32(npas, torch):
    print("config1 fp32 3x3", flush=True)
    w = configs.config1()
    p = pack_layer(npas, w.layers[0], w.dtype)
    assert npas.conv2d_kernel_name(p, 1, 32, 32, 1, 1) == "conv_wave_f32"      # reductions split over lanes
    layerwise(npas, torch, w)


def test_config1_conv3x3_fp32_one_lane_per_output(npas, torch, force_variant):
    force_variant("valu")
    w = configs.config1()
    p = pack_layer(npas, w.layers[0], w.dtype)
    assert npas.conv2d_kernel_name(p, 1, 32, 32, 1, 1) == "conv_valu_f32"
    layerwise(npas, torch, w)


WAVE_F32 = [
    ("wf_stride2_res_bias_hswish", 2, 9, 9, 8, 12, 3, 3, 2, 1, 4, 4, 2, dtypes.F32, 3, True, True),
    ("wf_wide_group_1x1", 1, 5, 5, 8, 24, 1, 1, 1, 0, 24, 8, 2, dtypes.F32, 0, False, False),
    ("wf_list_not_a_multiple_of_8", 3, 7, 6, 5, 6, 3, 3, 1, 1, 2, 5, 3, dtypes.F32, 1, False, True),
    ("wf_single_filter_groups", 1, 6, 6, 4, 5, 3, 3, 1, 1, 1, 1, 2, dtypes.F32, 2, True, False),
    ("wf_ragged_lanes", 1, 3, 5, 16, 8, 5, 5, 1, 2, 8, 4, 5, dtypes.F32, 0, False, True),
]


@pytest.mark.parametrize("case", WAVE_F32, ids=[c[0] for c in WAVE_F32])
def test_fp32_lane_split_kernel(npas, torch, case):
    _run_edge_case(npas, torch, case, expect_kernel="conv_wave_f32")


def test_config2_pointwise_stack_small(npas, torch):
    print("config2 small batch", flush=True)
    layerwise(npas, torch, configs.config2(batch=2, HW=23))        # 1058 pixels: several tiles + ragged tail


@pytest.mark.parametrize("N,HW,C,F,dtype,res,kernel", [(3, 10, 128, 136, dtypes.F16, True, "conv_smallm_mfma_kernel"), (1, 17, 64, 40, dtypes.BF16, False, "conv_smallm_mfma_kernel"),
                                                       (2, 25, 192, 200, dtypes.BF16, True, "conv_smallm_mfma_kernel"), (13, 29, 128, 136, dtypes.F16, True, "pointwise_ring_kernel"),
                                                       (6, 29, 64, 200, dtypes.F16, False, "pointwise_ring_kernel")])
def test_pointwise_layers_of_few_channels(npas, torch, N, HW, C, F, dtype, res, kernel):
    """1x1 layers on 64 .. 192 channels: split over the waves up to one round of workgroups, the streaming kernel beyond."""
    _run_edge_case(npas, torch, (f"pw_c{C}_f{F}", N, HW, HW, C, F, 1, 1, 1, 0, 8, 4, 2, dtype, 2, res, True), device_kernel=kernel)


def test_config3_fc_block_full(npas, torch):
    print("config3 full", flush=True)
    w = configs.config3()
    p = pack_layer(npas, w.layers[0], w.dtype)
    assert npas.conv2d_kernel_name(p, w.x_shape[0], 1, 1, 1, 0) == "fc_gather_mfma"    # the exact-list kernel
    layerwise(npas, torch, w)


def test_config3_fc_block_full_dense_format_route(npas, torch, force_variant):
    """The same layer through the route that multiplies the dense weight images (what the exact-list kernel replaced)."""
    force_variant("nofcgather")
    w = configs.config3()
    p = pack_layer(npas, w.layers[0], w.dtype)
    assert npas.conv2d_kernel_name(p, w.x_shape[0], 1, 1, 1, 0) != "fc_gather_mfma"
    layerwise(npas, torch, w)


FC_GATHER = [
    # name, B (as N x H x W), C, F, stride, Bf, Bc, rate, dtype, act, use_res, use_bias
    ("fcg_ragged_rows_and_tiles", (37, 1, 1), 192, 88, 1, 16, 32, 5, dtypes.BF16, 1, False, True),
    ("fcg_one_row", (1, 1, 1), 64, 16, 1, 16, 32, 4, dtypes.BF16, 0, False, False),
    ("fcg_8x4_blocks_union_of_two_groups", (3, 9, 11), 256, 136, 1, 8, 4, 5, dtypes.BF16, 3, True, True),
    ("fcg_fp16_long_list", (5, 1, 1), 2048, 40, 1, 16, 32, 2.5, dtypes.F16, 2, False, True),
    ("fcg_strided_1x1", (3, 15, 14), 320, 72, 2, 8, 4, 5, dtypes.BF16, 2, True, False),
    ("fcg_many_tiles_two_rows", (2, 1, 1), 96, 1000, 1, 16, 32, 5, dtypes.BF16, 0, False, True),
]


@pytest.mark.parametrize("case", FC_GATHER, ids=[c[0] for c in FC_GATHER])
def test_fc_gather_kernel(npas, torch, case):
    name, (N, H, W), C, F, stride, Bf, Bc, rate, dtype, act, use_res, use_bias = case
    _run_edge_case(npas, torch, (name, N, H, W, C, F, 1, 1, stride, 0, Bf, Bc, rate, dtype, act, use_res, use_bias),
                   expect_kernel="fc_gather_mfma")


def test_config4_pattern_small(npas, torch):
    print("config4 small", flush=True)
    layerwise(npas, torch, configs.config4(batch=2, HW=28))


def test_config5_residual_stack_reduced(npas, torch):
    print("config5 reduced (64x64 input, width 16)", flush=True)
    layerwise(npas, torch, configs.config5(batch=2, HW=64, width=16))


def test_config5_full_size_batch1_layerwise(npas, torch):
    print("config5 full size, batch 1", flush=True)
    layerwise(npas, torch, configs.config5(batch=1), check_meta=False)


EDGE = [
    # name, N, H, W, C, F, KH, KW, stride, pad, Bf, Bc, rate, dtype, act, use_res, use_bias
    ("ragged_F_and_tail", 3, 9, 11, 16, 40, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, True, True),
    ("stem_like_C3_7x7s2", 2, 29, 31, 3, 24, 7, 7, 2, 3, 8, 4, 2, dtypes.BF16, 1, False, True),
    ("stride2_3x3_two_chunks", 2, 15, 14, 128, 72, 3, 3, 2, 1, 8, 4, 3, dtypes.BF16, 0, False, False),
    ("pointwise_stride2", 2, 15, 14, 320, 72, 1, 1, 2, 0, 8, 4, 5, dtypes.BF16, 2, False, False),
    ("unstructured_1x1_blocks", 1, 8, 8, 16, 16, 3, 3, 1, 1, 1, 1, 3, dtypes.BF16, 0, False, False),
    ("coarse_whole_tensor_block", 1, 8, 8, 16, 32, 3, 3, 1, 1, 32, 16, 2, dtypes.BF16, 0, False, False),
    ("rate1_dense", 1, 6, 7, 8, 16, 3, 3, 1, 1, 8, 4, 1, dtypes.BF16, 0, False, False),
    ("one_pixel_input", 1, 1, 1, 64, 48, 1, 1, 1, 0, 8, 4, 2, dtypes.BF16, 0, False, False),
    ("fp16_storage", 2, 10, 10, 32, 32, 3, 3, 1, 1, 8, 4, 2, dtypes.F16, 1, True, False),
    ("fp32_stride2_res_bias", 2, 9, 9, 8, 12, 3, 3, 2, 1, 4, 4, 2, dtypes.F32, 2, True, True),
    ("fp32_wide_group", 1, 5, 5, 8, 24, 1, 1, 1, 0, 24, 8, 2, dtypes.F32, 0, False, False),
    ("large_C_many_chunks", 1, 7, 7, 600, 130, 1, 1, 1, 0, 8, 4, 2, dtypes.BF16, 1, True, False),
    ("kernel_5x3", 1, 30, 30, 8, 16, 5, 3, 1, 2, 4, 4, 2, dtypes.BF16, 0, False, False),
    # 100 items of 256 x 128 but 196 of 128 x 128: the pointwise ring's half-size tiles, ragged last tile
    ("pointwise_half_size_tiles", 127, 7, 7, 128, 512, 1, 1, 1, 0, 8, 4, 3, dtypes.BF16, 1, True, True),
    # pixel tiles evened out over the workgroups: 196 items of 256 pixels become 252 of 200 (the fourth
    # pixel group of a tile holds 8 pixels), and 100 of 256 become 200 of 128 (two pixel groups empty)
    ("pointwise_tiles_of_200_pixels", 1, 112, 112, 64, 512, 1, 1, 1, 0, 8, 4, 3, dtypes.BF16, 1, True, True),
    ("pointwise_tiles_of_128_pixels", 2, 80, 80, 64, 256, 1, 1, 1, 0, 8, 4, 2, dtypes.BF16, 2, True, False),
    # 50 items of 256 x 128: too few; 392 of 64 x 64 would take two rounds, 98 of 128 x 128 take one
    ("pointwise_medium_tiles_instead_of_small", 32, 14, 14, 256, 256, 1, 1, 1, 0, 8, 4, 3, dtypes.BF16, 1, False, True),
]


def _run_edge_case(npas, torch, case, expect_kernel=None, device_kernel=None, direct_plan=None):
    name, N, H, W, C, F, KH, KW, stride, pad, Bf, Bc, rate, dtype, act, use_res, use_bias = case
    print(f"edge {name}", flush=True)
    xs, xe = dtypes.quantize(prng.normal(7, 1, N * H * W * C).reshape(N, H, W, C), dtype)
    ws, we = dtypes.quantize(prng.normal(7, 2, F * C * KH * KW, 0.2).reshape(F, C, KH, KW), dtype)
    m = masks.block_punched_mask(F, C, KH, KW, Bf, Bc, rate, 99)
    L = configs.Layer("conv", "block_punched", C, F, KH, KW, stride, pad, Bf, Bc, rate, act, w_store=ws, w_exact=we, mask=m)
    oshape = helpers.out_shape(L, (N, H, W, C))
    bias = prng.normal(7, 3, F).astype(np.float32) if use_bias else None
    rs = re = None
    if use_res:
        rs, re = dtypes.quantize(prng.normal(7, 4, int(np.prod(oshape))).reshape(oshape), dtype)
    ref = oracle.round_to(oracle.conv2d_masked(xe, we, m, stride, pad, None if bias is None else bias.astype(np.float64),
                                               re, act), dtype)
    p = pack_layer(npas, L, dtype)
    helpers.check_metadata(oracle, L, p, dtype)
    if expect_kernel is not None:
        assert npas.conv2d_kernel_name(p, N, H, W, stride, pad) == expect_kernel
    if device_kernel is not None:
        assert npas.device_kernel(p, N, H, W, stride, pad) == device_kernel
    if direct_plan is not None:
        layout, _, items = npas.direct_plan(p, N, H, W, stride, pad)
        assert (layout, items) == direct_plan
    y = run_layer_gpu(npas, torch, L, p, to_dev(xs, torch), (N, H, W, C), dtype,
                      None if rs is None else to_dev(rs, torch), None if bias is None else to_dev(bias, torch))
    got = from_dev(y, dtype).reshape(oshape)
    err = rel_err(got, ref)
    print(f"  err={err:.3e}", flush=True)
    assert err <= TOL[dtype]
    # run-to-run determinism: no atomics, one writer per element
    y2 = run_layer_gpu(npas, torch, L, p, to_dev(xs, torch), (N, H, W, C), dtype,
                       None if rs is None else to_dev(rs, torch), None if bias is None else to_dev(bias, torch))
    assert torch.equal(y, y2)


@pytest.mark.parametrize("case", EDGE, ids=[c[0] for c in EDGE])
def test_edge_cases(npas, torch, case):
    _run_edge_case(npas, torch, case)


# k x k, stride 1, whole 64-channel chunks: the direct-weights kernel (forced, so that small
# problems take it too): several images per tile, ragged tiles in every direction, filter
# counts off the 128-filter block, many work items.
SPATIAL = [
    ("sp_7x7_images_per_tile", 11, 7, 7, 64, 136, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, True, True),
    ("sp_14x14_two_chunks", 3, 14, 14, 128, 64, 3, 3, 1, 1, 8, 4, 2, dtypes.BF16, 2, False, True),
    ("sp_ragged_tiles", 2, 30, 29, 64, 260, 3, 3, 1, 1, 4, 4, 2, dtypes.BF16, 0, True, False),
    ("sp_pad0_fp16", 2, 12, 12, 64, 32, 3, 3, 1, 0, 4, 4, 2, dtypes.F16, 1, False, False),
    ("sp_kernel_5x3", 2, 12, 17, 128, 32, 5, 3, 1, 2, 4, 4, 2, dtypes.BF16, 0, False, False),
    ("sp_more_items_than_workgroups", 70, 16, 16, 64, 512, 3, 3, 1, 1, 8, 4, 4, dtypes.BF16, 1, True, True),
]


@pytest.mark.parametrize("case", SPATIAL, ids=[c[0] for c in SPATIAL])
def test_direct_weights_kernel_stride1(npas, torch, case, force_variant):
    force_variant("spatial")
    _run_edge_case(npas, torch, case, expect_kernel="spatial_direct")


RESIDENT = [
    ("res_3x3_64", 3, 20, 23, 64, 64, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, True, True),
    ("res_ragged_filters_fp16", 2, 13, 11, 64, 40, 3, 3, 1, 1, 8, 4, 2, dtypes.F16, 2, False, True),
    ("res_two_chunks_2x2_pad0", 5, 9, 9, 128, 32, 2, 2, 1, 0, 4, 4, 2, dtypes.BF16, 0, True, False),
    ("res_several_images_per_tile", 37, 7, 7, 64, 64, 3, 3, 1, 1, 8, 4, 5, dtypes.BF16, 1, False, False),
    ("res_one_round_16_filters", 20, 56, 56, 64, 16, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, False, True),
]


@pytest.mark.parametrize("case", RESIDENT, ids=[c[0] for c in RESIDENT])
def test_direct_weights_kernel_up_to_64_filters(npas, torch, case, force_variant):
    force_variant("spatial")
    _run_edge_case(npas, torch, case, expect_kernel="spatial_direct")


def test_direct_weights_kernel_chosen_for_a_full_launch(npas, torch):
    """56 x 56, 64 -> 64 at batch 16, chosen by the library itself."""
    _run_edge_case(npas, torch, ("res_full_launch", 16, 56, 56, 64, 64, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, False, True),
                   expect_kernel="spatial_direct")


SPATIAL_STRIDE2 = [
    ("sp2_ragged", 3, 17, 19, 64, 128, 3, 3, 2, 1, 8, 4, 3, dtypes.BF16, 1, True, True),
    ("sp2_two_chunks_fp16", 2, 24, 24, 128, 72, 3, 3, 2, 1, 8, 4, 2, dtypes.F16, 2, False, True),
    ("sp2_several_images_per_tile", 21, 14, 14, 64, 64, 3, 3, 2, 1, 8, 4, 5, dtypes.BF16, 0, True, False),
    ("sp2_even_input_one_row_tiles", 2, 6, 40, 64, 32, 3, 3, 2, 1, 4, 4, 2, dtypes.BF16, 1, False, False),
    ("sp2_more_items_than_workgroups", 70, 32, 32, 64, 512, 3, 3, 2, 1, 8, 4, 4, dtypes.BF16, 1, False, True),
]


@pytest.mark.parametrize("case", SPATIAL_STRIDE2, ids=[c[0] for c in SPATIAL_STRIDE2])
def test_direct_weights_kernel_stride2(npas, torch, case, force_variant):
    force_variant("spatial")
    _run_edge_case(npas, torch, case, expect_kernel="spatial_direct")


def test_direct_weights_kernel_on_7x7_maps(npas, torch):
    """Two 7 x 7 images a tile, 128 filters: one round of 256 items, chosen by the library itself."""
    _run_edge_case(npas, torch, ("sp_7x7_half_tiles", 128, 7, 7, 64, 512, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, True, True),
                   expect_kernel="spatial_direct")


# The direct-weights kernel where its tiles and loops can go wrong: one pixel, four filters, tiles that end with the map or the batch, odd strided maps
# with and without padding, even and long kernels, one and several chunks, more tiles than workgroups.  With the layout of the waves (pixel groups,
# filter halves, shares of the reduction, pixel blocks of a wave) and the number of items that the planner chooses.
DIRECT = [
    (("dir_one_pixel_four_filters", 1, 1, 1, 64, 4, 3, 3, 1, 1, 4, 4, 2, dtypes.BF16, 1, True, True), (1, 2, 2, 3), 1),
    (("dir_stride2_pad0", 2, 30, 29, 192, 68, 3, 3, 2, 0, 4, 4, 3, dtypes.BF16, 2, True, True), (1, 2, 2, 3), 56),
    (("dir_5x5_stride2_fp16", 5, 20, 31, 64, 132, 5, 5, 2, 2, 4, 4, 3, dtypes.F16, 3, False, True), (1, 2, 2, 3), 160),
    (("dir_2x2_pad0", 200, 9, 9, 64, 64, 2, 2, 1, 0, 8, 4, 2, dtypes.BF16, 0, True, False), (2, 1, 2, 3), 200),
    (("dir_7x7", 3, 64, 64, 64, 64, 7, 7, 1, 3, 8, 4, 5, dtypes.BF16, 1, False, False), (2, 1, 2, 3), 144),
    (("dir_two_groups_two_shares", 17, 40, 40, 64, 64, 3, 3, 1, 1, 8, 4, 3, dtypes.F16, 2, True, True), (2, 1, 2, 4), 255),
    (("dir_four_groups", 20, 33, 33, 64, 192, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 3, True, False), (4, 1, 1, 5), 240),
    (("dir_images_past_the_batch", 28, 40, 40, 64, 60, 3, 3, 1, 1, 4, 4, 3, dtypes.BF16, 1, False, True), (4, 1, 1, 3), 250),
    (("dir_two_groups_two_halves", 21, 40, 40, 64, 128, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, True, True), (2, 2, 1, 5), 252),
    (("dir_several_images_two_chunks", 130, 14, 14, 128, 256, 3, 3, 1, 1, 8, 4, 3, dtypes.F16, 1, True, False), (2, 2, 1, 7), 238),
    (("dir_more_tiles_than_workgroups", 64, 28, 28, 64, 320, 3, 3, 2, 1, 8, 4, 3, dtypes.BF16, 0, False, True), (2, 2, 1, 3), 480),
]


@pytest.mark.parametrize("case,layout,items", DIRECT, ids=[c[0][0] for c in DIRECT])
def test_direct_weights_kernel(npas, torch, case, layout, items, force_variant):
    force_variant("spatial")
    _run_edge_case(npas, torch, case, expect_kernel="spatial_direct", direct_plan=(layout, items))


# Every layout that is compiled, in both 16-bit types, with more items than workgroups (a workgroup's second item: the other parity of its tables, the
# exchange of the partial sums used again, the patch and weights asked for across the items): layout, items, N, H, W, C, F, k, stride, pad.  With 256
# channels at stride 1 the first item asks for the next chunks' weights ahead and the second does not.
DIRECT_LAYOUTS = [
    ((1, 2, 2, 3), 510, 102, 30, 30, 64, 64, 5, 2, 2), ((1, 2, 2, 4), 504, 48, 37, 37, 64, 132, 3, 2, 0), ((1, 2, 2, 5), 754, 79, 31, 28, 256, 72, 3, 1, 0),
    ((1, 2, 2, 6), 432, 81, 33, 33, 128, 132, 3, 2, 0), ((1, 2, 2, 7), 510, 104, 17, 16, 256, 196, 3, 1, 1),
    ((2, 1, 2, 3), 500, 115, 39, 38, 64, 4, 2, 2, 1), ((2, 1, 2, 4), 477, 53, 33, 33, 64, 132, 3, 2, 1), ((2, 1, 2, 5), 512, 94, 28, 28, 256, 4, 5, 1, 2),
    ((2, 1, 2, 6), 486, 89, 20, 20, 256, 132, 3, 1, 0), ((2, 1, 2, 7), 495, 87, 35, 34, 256, 4, 2, 1, 1),
    ((2, 2, 1, 3), 490, 91, 28, 26, 64, 132, 2, 2, 1), ((2, 2, 1, 4), 510, 64, 32, 29, 256, 72, 2, 1, 1), ((2, 2, 1, 5), 460, 46, 38, 36, 64, 72, 2, 1, 0),
    ((2, 2, 1, 6), 512, 64, 36, 33, 64, 72, 2, 1, 1), ((2, 2, 1, 7), 486, 90, 37, 34, 256, 72, 2, 1, 0),
    ((4, 1, 1, 3), 507, 65, 39, 37, 64, 4, 3, 1, 1), ((4, 1, 1, 4), 460, 115, 30, 30, 256, 4, 2, 1, 1), ((4, 1, 1, 5), 460, 115, 36, 35, 256, 4, 3, 1, 1),
    ((4, 1, 1, 6), 420, 105, 39, 37, 64, 4, 2, 1, 1), ((4, 1, 1, 7), 444, 111, 40, 40, 64, 4, 5, 1, 2),
]


@pytest.mark.parametrize("dtype,infinite", [(dtypes.BF16, False), (dtypes.F16, True)], ids=["bf16", "fp16_infinite_inputs"])
@pytest.mark.parametrize("case", DIRECT_LAYOUTS, ids=["x".join(map(str, c[0])) for c in DIRECT_LAYOUTS])
def test_direct_weights_kernel_in_every_layout(npas, torch, case, dtype, infinite, force_variant):
    """All images against the split-reduction kernel, the first, the middle and the last one (an item beyond the first 256) against the oracle, with
    infinite inputs over pruned weights there too."""
    layout, items, N, H, W, C, F, k, stride, pad = case
    print(f"direct layout {layout}", flush=True)
    L = configs._bp_conv(61, 0, C, F, k, stride, pad, 4, 4, 3, 0.1, dtype, configs.ACT_RELU6)
    p = pack_layer(npas, L, dtype)
    force_variant("spatial")
    chosen, tile, n_items = npas.direct_plan(p, N, H, W, stride, pad)
    assert (chosen, n_items) == (layout, items) and items > 256
    Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    td = torch.bfloat16 if dtype == dtypes.BF16 else torch.float16
    g = torch.Generator(device="cuda").manual_seed(61)
    x, res = torch.randn(N, H, W, C, generator=g, device="cuda").to(td), torch.randn(N, Ho, Wo, F, generator=g, device="cuda").to(td)
    bias = torch.randn(F, generator=g, device="cuda")
    if infinite:
        for n in (0, N // 2, N - 1):
            for i in range(4):
                x[n, (5 * i) % Ho * stride, (7 * i + 3) % Wo * stride, (37 * i + 11) % C] = float("inf") if i & 1 else -float("inf")

    def run():
        y = torch.full((N, Ho, Wo, F), float("nan"), device="cuda").to(td)
        npas.conv2d_sparse(p, x, y, N, H, W, stride, pad, bias=bias, residual=res, act=L.act)
        torch.cuda.synchronize()
        return y

    y = run()
    assert torch.equal(y.view(torch.int16), run().view(torch.int16))
    force_variant("smallm")
    other = run().double()
    floor = 1e-3 * other.abs().max()
    assert float(((y.double() - other).abs() / other.abs().clamp(min=floor)).max()) <= 2 * TOL[dtype]   # (each of the two within TOL)
    for n in (0, N // 2, N - 1):
        xe, fin = x[n:n + 1].double().cpu().numpy(), torch.isfinite(x[n:n + 1]).cpu().numpy()
        acc = oracle.conv2d_masked(np.where(fin, xe, 0.0), L.w_exact, L.mask, stride, pad, bias.double().cpu().numpy(), res[n:n + 1].double().cpu().numpy(), configs.ACT_NONE)
        inf = oracle.conv2d_masked(np.where(fin, 0.0, np.sign(xe)), np.sign(L.w_exact * L.mask), L.mask, stride, pad, None, None, configs.ACT_NONE)
        assert (inf != 0).any() == infinite
        ref = oracle.round_to(np.clip(np.where(inf > 0, np.inf, np.where(inf < 0, -np.inf, acc)), 0.0, 6.0), dtype)
        err = rel_err(y[n:n + 1].double().cpu().numpy(), ref)
        print(f"  image {n} err={err:.3e}", flush=True)
        assert err <= TOL[dtype]


def test_direct_weights_kernel_beyond_2_gib(npas, torch):
    """Input and output of 3.96 GiB each, just below 2^31 elements: byte offsets beyond 2^31, those of padding beyond the tensors' ends.  200 times the same
    53 images: each group of outputs has to be the first one's, whose images are checked against the oracle."""
    N, HW, C = 10600, 56, 64
    assert 2 ** 31 - 2 ** 25 < N * HW * HW * C < 2 ** 31
    print("direct, 3.96 GiB", flush=True)
    L = configs._bp_conv(62, 0, C, C, 3, 1, 1, 8, 4, 3, 0.1, dtypes.BF16, configs.ACT_NONE)
    p = pack_layer(npas, L, dtypes.BF16)
    assert npas.device_kernel(p, N, HW, HW, 1, 1) == "spatial_direct_kernel"
    g = torch.Generator(device="cuda").manual_seed(62)
    base = torch.randn(53, HW, HW, C, generator=g, device="cuda").to(torch.bfloat16)
    x = base.repeat(200, 1, 1, 1)
    y = torch.full_like(x, float("nan"))
    npas.conv2d_sparse(p, x, y, N, HW, HW, 1, 1)
    torch.cuda.synchronize()
    for n in (0, 52):
        ref = oracle.round_to(oracle.conv2d_masked(base[n:n + 1].double().cpu().numpy(), L.w_exact, L.mask, 1, 1), dtypes.BF16)
        assert rel_err(y[n:n + 1].double().cpu().numpy(), ref) <= TOL[dtypes.BF16]
    groups = y.view(200, -1).view(torch.int16)
    for i in range(1, 200):
        assert torch.equal(groups[i], groups[0]), i
    del x, y, groups
    torch.cuda.empty_cache()


def test_config4_pattern_small_direct_weights_kernel(npas, torch, force_variant):
    force_variant("spatial")
    print("config4 small, direct-weights kernel", flush=True)
    layerwise(npas, torch, configs.config4(batch=3, HW=12))


SWEEP_CASES = [(sch, r) for sch in ("block_punched", "unstructured", "whole_tensor", "pattern", "filter")
               for r in (2.5, 10) if not (sch == "pattern" and r < 2.25)]


@pytest.mark.parametrize("scheme,rate", SWEEP_CASES, ids=["%s_r%s" % c for c in SWEEP_CASES])
def test_rate_sweep_layer_kinds(npas, torch, scheme, rate):
    """The layer kinds of the rate sweep (bench.py --sweep rate), at a size the oracle finishes quickly."""
    from workloads import sweeps
    print(f"sweep {scheme} rate {rate}", flush=True)
    layerwise(npas, torch, sweeps.rate_sweep_layer(scheme, rate, batch=2, HW=11, C=64, F=72))


def test_block_sweep_stack_reduced(npas, torch):
    """The block-size sweep's stack (bench.py --sweep block) at 16x8 blocks, reduced input size."""
    from workloads import sweeps
    print("block sweep 16x8", flush=True)
    layerwise(npas, torch, sweeps.block_sweep_stack(16, 8, batch=1, HW=32), check_meta=False)


DW_CASES = [
    # name, N, H, W, C, stride, dtype, act, use_res, use_bias
    ("dw_bf16_vec", 2, 13, 11, 144, 1, dtypes.BF16, 2, False, True),
    ("dw_bf16_stride2_odd", 3, 15, 14, 24, 2, dtypes.BF16, 2, False, False),
    ("dw_bf16_scalar_channels", 1, 9, 9, 12, 1, dtypes.BF16, 1, True, True),
    ("dw_fp16_res", 2, 8, 10, 32, 1, dtypes.F16, 0, True, False),
    ("dw_fp32", 1, 7, 8, 10, 2, dtypes.F32, 2, True, True),
    ("dw_one_pixel", 1, 1, 1, 16, 1, dtypes.BF16, 0, False, False),
    ("dw_bf16_hardswish", 2, 13, 11, 40, 1, dtypes.BF16, 3, True, True),
    ("dw_fp32_hardswish_scalar", 1, 6, 7, 5, 1, dtypes.F32, 3, False, True),
]


@pytest.mark.parametrize("case", DW_CASES, ids=[c[0] for c in DW_CASES])
def test_depthwise3x3(npas, torch, case):
    name, N, H, W, C, stride, dtype, act, use_res, use_bias = case
    print(f"depthwise {name}", flush=True)
    xs, xe = dtypes.quantize(prng.normal(17, 1, N * H * W * C).reshape(N, H, W, C), dtype)
    ws, we = dtypes.quantize(prng.normal(17, 2, C * 9, 0.3).reshape(C, 3, 3), dtype)
    L = configs.Layer("dwconv", "", C, C, 3, 3, stride, 1, 1, 1, 1.0, act, w_store=ws, w_exact=we)
    oshape = helpers.out_shape(L, (N, H, W, C))
    bias = prng.normal(17, 3, C).astype(np.float32) if use_bias else None
    rs = re = None
    if use_res:
        rs, re = dtypes.quantize(prng.normal(17, 4, int(np.prod(oshape))).reshape(oshape), dtype)
    ref = oracle.round_to(oracle.dwconv3x3(xe, we, stride, None if bias is None else bias.astype(np.float64), re, act), dtype)
    p = pack_layer(npas, L, dtype)
    info = p.info()
    assert info["scheme"] == npas.SCHEME_DEPTHWISE and info["C"] == C and info["device_ready"] == 1
    np.testing.assert_array_equal(p.export()["w_compact"], np.asarray(ws).reshape(C, 9))    # bit-exact round trip
    y = run_layer_gpu(npas, torch, L, p, to_dev(xs, torch), (N, H, W, C), dtype,
                      None if rs is None else to_dev(rs, torch), None if bias is None else to_dev(bias, torch))
    err = rel_err(from_dev(y, dtype).reshape(oshape), ref)
    print(f"  err={err:.3e}", flush=True)
    assert err <= TOL[dtype]


# Edges of the row-block kernel: four rows a thread (launches of more than 196608 output vectors) with one row left over and
# with whole blocks, two columns too (from 360448 one-column threads on: odd, even, two and nine; one, seven stay), one row a thread, stride 2 on odd and even maps, maps narrower than the window, a bias at 4-byte alignment.
@pytest.mark.parametrize("N,H,W,C,stride,dtype", [(5, 201, 199, 8, 1, dtypes.BF16), (13, 64, 60, 32, 1, dtypes.F16), (1, 3, 1, 24, 1, dtypes.BF16),
                                                  (2, 9, 7, 40, 2, dtypes.F16), (3, 32, 2, 16, 2, dtypes.BF16), (9, 151, 149, 16, 2, dtypes.BF16),
                                                  (25, 57, 57, 144, 1, dtypes.BF16), (41, 62, 76, 64, 1, dtypes.F16), (3, 30001, 1, 136, 1, dtypes.BF16),
                                                  (3, 15001, 2, 136, 1, dtypes.BF16), (9, 2225, 9, 64, 1, dtypes.F16), (9, 2861, 7, 64, 1, dtypes.BF16)])
def test_depthwise3x3_row_blocks(npas, torch, N, H, W, C, stride, dtype):
    print(f"depthwise rows N={N} {H}x{W}x{C} stride {stride}", flush=True)
    xs, xe = dtypes.quantize(prng.normal(18, 1, N * H * W * C).reshape(N, H, W, C), dtype)
    ws, we = dtypes.quantize(prng.normal(18, 2, C * 9, 0.3).reshape(C, 3, 3), dtype)
    bias = prng.normal(18, 3, C).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    rs, re = dtypes.quantize(prng.normal(18, 4, N * Ho * Wo * C).reshape(N, Ho, Wo, C), dtype)
    ref = oracle.round_to(oracle.dwconv3x3(xe, we, stride, bias.astype(np.float64), re, configs.ACT_RELU6), dtype)
    p = npas.pack_depthwise3x3(ws, dtype)
    y = new_dev((N, Ho, Wo, C), dtype, torch, fill=0x7FC1)
    b = to_dev(np.concatenate([np.zeros(1, np.float32), bias]), torch)
    npas.depthwise3x3(p, to_dev(xs, torch), y, N, H, W, stride, b.data_ptr() + 4, to_dev(rs, torch), npas.ACT_RELU6)
    torch.cuda.synchronize()
    assert rel_err(from_dev(y, dtype), ref) <= TOL[dtype]


@pytest.mark.parametrize("stride,N,off", [(1, 1, 2), (1, 40, 2), (2, 2, 2), (1, 40, 8), (2, 2, 4)])
def test_depthwise3x3_at_smaller_alignment(npas, torch, stride, N, off):
    """Tensors that start 2, 4 or 8 bytes past an aligned address (input, output and residual): same values as aligned ones."""
    H, W, C = 29, 31, 48
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    ws, _ = dtypes.quantize(prng.normal(20, 2, C * 9, 0.3).reshape(C, 3, 3), dtypes.BF16)
    p = npas.pack_depthwise3x3(ws, dtypes.BF16)
    g = torch.Generator(device="cuda").manual_seed(20)
    x = torch.randn((N, H, W, C), generator=g, device="cuda", dtype=torch.bfloat16)
    r = torch.randn((N, Ho, Wo, C), generator=g, device="cuda", dtype=torch.bfloat16)
    y = torch.empty((N, Ho, Wo, C), dtype=torch.bfloat16, device="cuda")
    npas.depthwise3x3(p, x, y, N, H, W, stride, None, r, npas.ACT_NONE)

    def shifted(t):
        b = torch.zeros(t.numel() + 16, dtype=torch.int16, device="cuda")
        b[off // 2:off // 2 + t.numel()] = t.reshape(-1).view(torch.int16)
        return b

    xo, ro, yo = shifted(x), shifted(r), shifted(torch.zeros_like(y))
    npas.depthwise3x3(p, xo.data_ptr() + off, yo.data_ptr() + off, N, H, W, stride, None, ro.data_ptr() + off, npas.ACT_NONE)
    torch.cuda.synchronize()
    assert torch.equal(yo[off // 2:off // 2 + y.numel()], y.reshape(-1).view(torch.int16))
    assert not yo[:off // 2].any() and not yo[off // 2 + y.numel():].any()


# Inputs past the limits of the row-block kernel's 32-bit forms: 2 GiB and more (buffer range check), and thread counts that its
# reciprocals do not divide (index times divisor 2^32 or more), four rows and one row a thread.
@pytest.mark.parametrize("N,H,W,C,stride", [(65, 256, 256, 256, 1), (65, 257, 257, 256, 2), (2, 92801, 2, 8, 2), (2, 60000, 1, 8, 1),
                                            (5, 4200, 120, 64, 1)],
                         ids=["2gib", "2gib_s2", "index_s2", "index_one_row", "index_four_rows"])
def test_depthwise3x3_past_32_bit_forms(npas, torch, N, H, W, C, stride):
    """All images in one call give the same bits as one call per image (which the 32-bit forms serve): same kernel, same order of
    additions."""
    print(f"depthwise N={N} {H}x{W}x{C} stride {stride}", flush=True)
    ws, _ = dtypes.quantize(prng.normal(19, 2, C * 9, 0.3).reshape(C, 3, 3), dtypes.BF16)
    p = npas.pack_depthwise3x3(ws, dtypes.BF16)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    g = torch.Generator(device="cuda").manual_seed(19)
    x = torch.randn((N, H, W, C), generator=g, device="cuda", dtype=torch.bfloat16)
    b = torch.randn(C, generator=g, device="cuda")
    y = torch.full((N, Ho, Wo, C), float("nan"), dtype=torch.bfloat16, device="cuda")
    npas.depthwise3x3(p, x, y, N, H, W, stride, b, None, npas.ACT_RELU6)
    one = torch.full((Ho, Wo, C), float("nan"), dtype=torch.bfloat16, device="cuda")
    for n in range(N):
        npas.depthwise3x3(p, x[n], one, 1, H, W, stride, b, None, npas.ACT_RELU6)
        torch.cuda.synchronize()
        assert torch.equal(y[n].view(torch.int16), one.view(torch.int16)), f"image {n}"


@pytest.mark.parametrize("stride,bias,act,HW", [(1, False, configs.ACT_RELU6, 13), (2, False, configs.ACT_RELU6, 13),
                                                (1, True, configs.ACT_RELU6, 13), (2, True, configs.ACT_RELU6, 13),
                                                (2, True, configs.ACT_HARDSWISH, 14), (1, True, configs.ACT_HARDSWISH, 9),
                                                (2, False, configs.ACT_RELU6, 31)],
                         ids=["s1", "s2", "s1_bias", "s2_bias", "s2_bias_hswish_even", "s1_bias_hswish", "s2_several_tiles"])
def test_inverted_residual_block_layerwise_and_stack(npas, torch, stride, bias, act, HW):
    """1x1 -> depthwise 3x3 (stride 1 or 2) -> 1x1 (+ input at stride 1), with and without a bias per layer: each layer
    against the oracle, then the stack call end to end, per layer and as one fused launch.  With a bias the padding
    of the depthwise layer must still be zero (not act(bias)): the border pixels are where that shows."""
    from workloads import sweeps
    w = sweeps.inverted_residual_block(batch=2, HW=HW, stride=stride, bias=bias, act=act)
    print(f"inverted residual block, stride {stride} bias {bias} act {act} {HW}x{HW}", flush=True)
    layerwise(npas, torch, w)
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    for flags in (0, 1, 3):          # per layer; pointwise-pair fusion (not applicable); whole-block fusion
        got, st = _run_stack_gpu(npas, torch, w, flags)
        assert st.num_launches() == (1 if flags == 3 else 3)
        norm, worst = helpers.check_stack_output(got, rounded[-1], STACK_NORM_TOL)
        print(f"  run_stack flags={flags} launches={st.num_launches()} norm-wise {norm:.3e} worst element {worst:.3e}", flush=True)
        border = np.concatenate([got[:, 0].ravel(), got[:, -1].ravel(), got[:, :, 0].ravel(), got[:, :, -1].ravel()])
        want = np.concatenate([rounded[-1][:, 0].ravel(), rounded[-1][:, -1].ravel(), rounded[-1][:, :, 0].ravel(), rounded[-1][:, :, -1].ravel()])
        assert rel_err(border, want) <= 0.1, "border pixels (padding of the depthwise layer)"


# The reduction-splitting kernel with 1, 2 and 4 images a workgroup and with 32 pixels x 64 filters: a last block of 1, 15 and 16
# pixels, an odd number of pixel blocks, filters that end inside a 64-filter half and inside an image, fewer steps than waves.
SMALLM_EDGES = [
    ("split_fi1_tail1_f20", 1, 1, 17, 64, 20, 1, 1, 1, 0, 4, 4, 2, dtypes.BF16, 0, True, True),
    ("split_fi1_3x3_s2_f200", 1, 13, 11, 128, 200, 3, 3, 2, 1, 8, 4, 3, dtypes.F16, 3, False, True),
    ("split_fi2_3x3_f128", 3, 15, 17, 64, 128, 3, 3, 1, 1, 8, 4, 2, dtypes.BF16, 1, True, True),
    ("split_fi4_3x3_f68", 1, 37, 41, 64, 68, 3, 3, 1, 1, 4, 4, 2, dtypes.BF16, 2, True, False),
    ("split_fi4_1x1_f64", 1, 53, 51, 256, 64, 1, 1, 1, 0, 8, 4, 2, dtypes.F16, 1, False, True),
    ("split_pb2_odd_blocks_f192", 5, 27, 19, 64, 192, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 2, True, True),
    ("split_pb2_s2_f200", 7, 29, 27, 64, 200, 3, 3, 2, 0, 8, 4, 2, dtypes.F16, 0, True, True),
    ("split_pb2_5x5_f132", 3, 21, 25, 64, 132, 5, 5, 1, 2, 4, 4, 2, dtypes.BF16, 1, False, False),
]


@pytest.mark.parametrize("case", SMALLM_EDGES, ids=[c[0] for c in SMALLM_EDGES])
def test_split_reduction(npas, torch, case):
    npas.set_switches("smallm")      # k x k layers wherever the kernel applies (1x1 layers follow the rule)
    try:
        _run_edge_case(npas, torch, case, expect_kernel="conv_smallm_mfma")
    finally:
        npas.set_switches(None)


# The flat 1x1 kernel: a last block of 1..15 pixels, a last 16-filter tile of 8 and 12 filters, channel counts that end inside a
# 32-deep step, one and several filter groups (with and without 16-byte output segments), stride 2.  (One pixel of a layer at 2x
# takes the exact lists; the dense one, 8 channels, 4-filter tiles and waves of several blocks are in STREAM_FORMS.)
STREAM_EDGES = [
    ("flat_c8_f4_one_pixel", 1, 1, 1, 8, 4, 1, 1, 1, 0, 4, 4, 2, dtypes.BF16, 0, False, True),
    ("flat_c24_f144_tail1", 3, 7, 83, 24, 144, 1, 1, 1, 0, 8, 8, 2, dtypes.BF16, 2, False, False),
    ("flat_c144_f40_tail15_res", 5, 11, 37, 144, 40, 1, 1, 1, 0, 8, 8, 2, dtypes.F16, 3, True, True),
    ("flat_c320m8_f300_groups", 2, 17, 61, 312, 300, 1, 1, 1, 0, 8, 4, 2, dtypes.BF16, 1, True, True),
    ("flat_c280_f200_groups_s2", 5, 41, 39, 280, 200, 1, 1, 2, 0, 8, 8, 2, dtypes.F16, 0, True, False),
    ("flat_c96_f12_many", 9, 61, 59, 96, 12, 1, 1, 1, 0, 4, 8, 2, dtypes.BF16, 2, True, True),
]


@pytest.mark.parametrize("case", STREAM_EDGES, ids=[c[0] for c in STREAM_EDGES])
def test_flat_pointwise(npas, torch, case):
    lists = case[0] == "flat_c8_f4_one_pixel"
    _run_edge_case(npas, torch, case, device_kernel="fc_gather_mfma_kernel" if lists else "pointwise_stream_kernel")


# The same kernel's launch forms: a wave that walks two and three pixel blocks (in one run, in 16- and in 8-byte segments; with one, three
# and five filter groups), a last block of 7 .. 11 pixels met on a later round, groups made because the pixels are few (the last of one
# tile), dense layers of 8 channels, 4 filters and one pixel, and a density that would fit the gather format.
STREAM_FORMS = [
    ("flat_run_two_rounds", 24, 57, 57, 24, 12, 1, 1, 1, 0, 4, 8, 2, dtypes.BF16, 2, True, True),
    ("flat_seg16_two_rounds", 23, 57, 57, 40, 32, 1, 1, 1, 0, 8, 8, 2, dtypes.F16, 3, True, True),
    ("flat_3_groups_three_rounds", 7, 57, 57, 24, 960, 1, 1, 1, 0, 8, 8, 2, dtypes.BF16, 2, True, True),
    ("flat_5_groups_seg8_three_rounds", 5, 53, 51, 40, 1276, 1, 1, 1, 0, 4, 8, 4, dtypes.BF16, 1, False, True),
    ("flat_few_pixels_7_groups", 1, 3, 5, 24, 200, 1, 1, 1, 0, 8, 8, 1, dtypes.BF16, 0, True, True),
    ("flat_few_pixels_seg8_last_4", 1, 9, 9, 16, 36, 1, 1, 1, 0, 4, 8, 1, dtypes.F16, 1, False, True),
    ("flat_dense_c8_f4_one_pixel", 1, 1, 1, 8, 4, 1, 1, 1, 0, 4, 4, 1, dtypes.BF16, 0, False, True),
    ("flat_dense_f20_run", 3, 9, 7, 16, 20, 1, 1, 1, 0, 4, 8, 1, dtypes.BF16, 3, True, False),
    ("flat_low_density", 2, 33, 29, 72, 96, 1, 1, 1, 0, 8, 8, 10, dtypes.BF16, 2, False, True),
]


@pytest.mark.parametrize("case", STREAM_FORMS, ids=[c[0] for c in STREAM_FORMS])
def test_flat_pointwise_launch_forms(npas, torch, case):
    _run_edge_case(npas, torch, case, device_kernel="pointwise_stream_kernel")


@pytest.mark.parametrize("C,F,HW", [(8, 20, 9), (24, 144, 37), (144, 40, 33), (312, 96, 33)])
def test_flat_pointwise_infinite_input_in_the_last_channels(npas, torch, C, F, HW):
    """The matrix steps are 32 channels deep; past the last channel they must meet zeros, not other channels of the pixel: an infinite
    input under kept weights clamps to 0 or 6, as the oracle has it."""
    L = configs._bp_conv(52, 0, C, F, 1, 1, 0, 4, 8, 1, 0.2, dtypes.BF16, configs.ACT_RELU6)
    assert (L.w_exact != 0).all()
    xs, xe = configs._tensor(52, 1, (2, HW, HW, C), 1.0, dtypes.BF16)
    for n, y, x, c, v in ((0, 0, 0, C - 1, np.inf), (0, 5, 7, C - 8, -np.inf), (1, HW - 1, HW - 1, C - 3, np.inf)):
        xe[n, y, x, c] = v
    xs, xe = dtypes.quantize(xe, dtypes.BF16)
    ref = oracle.round_to(oracle.conv2d_masked(xe, L.w_exact, L.mask, 1, 0, None, None, L.act), dtypes.BF16)
    p = pack_layer(npas, L, dtypes.BF16)
    assert npas.device_kernel(p, 2, HW, HW, 1, 0) == "pointwise_stream_kernel"
    y = run_layer_gpu(npas, torch, L, p, to_dev(xs, torch), xe.shape, dtypes.BF16)
    assert rel_err(from_dev(y, dtypes.BF16).reshape(ref.shape), ref) <= TOL[dtypes.BF16]


def _infinite_input_under_pruned_weights(npas, torch, L, N, H, W, dtype, res, kernel):
    """An input that is infinite where a filter's weight is pruned does not reach that filter: outputs against the oracle, which skips
    pruned positions; the infinite inputs clamp to 0 or 6 where the weight is kept."""
    xs, xe = configs._tensor(53, 1, (N, H, W, L.C), 1.0, dtype)
    Ho, Wo = (H + 2 * L.pad - L.KH) // L.stride + 1, (W + 2 * L.pad - L.KW) // L.stride + 1
    for i in range(4):
        xe[i % N, (5 * i) % H // L.stride * L.stride, (7 * i) % W // L.stride * L.stride, (37 * i + 11) % L.C] = np.inf if i & 1 else -np.inf
    xs, xe = dtypes.quantize(xe, dtype)
    rs = re = None
    if res:
        rs, re = configs._tensor(53, 2, (N, Ho, Wo, L.F), 1.0, dtype)
    we = L.w_exact * L.mask
    # the oracle's sum without the pruned terms: finite inputs through the oracle, the infinite ones by their sign
    fin = np.isfinite(xe)
    acc = oracle.conv2d_masked(np.where(fin, xe, 0.0), L.w_exact, L.mask, L.stride, L.pad, None, re, configs.ACT_NONE)
    inf = oracle.conv2d_masked(np.where(fin, 0.0, np.sign(xe)), np.sign(we), L.mask, L.stride, L.pad, None, None, configs.ACT_NONE)
    ref = oracle.round_to(np.clip(np.where(inf > 0, np.inf, np.where(inf < 0, -np.inf, acc)), 0.0, 6.0), dtype)
    assert (inf != 0).any() and (inf == 0).any()
    p = pack_layer(npas, L, dtype)
    assert npas.conv2d_kernel_name(p, N, H, W, L.stride, L.pad) == kernel
    y = run_layer_gpu(npas, torch, L, p, to_dev(xs, torch), xe.shape, dtype, None if rs is None else to_dev(rs, torch))
    assert rel_err(from_dev(y, dtype).reshape(ref.shape), ref) <= TOL[dtype]
    if res:  # the shortcut added in place
        y = to_dev(rs, torch)
        npas.conv2d_sparse(p, to_dev(xs, torch), y, N, H, W, L.stride, L.pad, residual=y, act=L.act)
        torch.cuda.synchronize()
        assert rel_err(from_dev(y, dtype).reshape(ref.shape), ref) <= TOL[dtype]


@pytest.mark.parametrize("C,F,N,HW,k,stride,rate,dtype,res", [(1280, 200, 37, 1, 1, 1, 2, dtypes.BF16, False), (1024, 1000, 300, 1, 1, 1, 2, dtypes.F16, False),
                                                               (256, 128, 3, 11, 1, 2, 3, dtypes.BF16, True), (128, 72, 2, 9, 3, 1, 5, dtypes.F16, True),
                                                               (64, 200, 5, 28, 3, 2, 3, dtypes.BF16, False), (64, 192, 5, 25, 3, 1, 3, dtypes.BF16, True)],
                         ids=["fc", "fc_64_filters", "1x1_s2", "3x3", "3x3_s2", "3x3_two_pixel_blocks"])
def test_split_reduction_infinite_input_under_pruned_weights(npas, torch, C, F, N, HW, k, stride, rate, dtype, res, force_variant):
    force_variant("smallm")
    L = configs._bp_conv(53, 0, C, F, k, stride, k // 2, 4, 4, rate, 0.2, dtype, configs.ACT_RELU6)
    _infinite_input_under_pruned_weights(npas, torch, L, N, HW, HW, dtype, res, "conv_smallm_mfma")


@pytest.mark.parametrize("C,F,N,HW,k,stride,rate,dtype,res", [(128, 72, 2, 9, 3, 1, 5, dtypes.F16, True), (64, 200, 5, 28, 3, 2, 3, dtypes.BF16, False),
                                                               (64, 64, 5, 25, 5, 1, 3, dtypes.BF16, True), (64, 128, 30, 25, 3, 1, 3, dtypes.BF16, True)],
                         ids=["two_shares", "stride2", "5x5", "one_share"])
def test_direct_weights_infinite_input_under_pruned_weights(npas, torch, C, F, N, HW, k, stride, rate, dtype, res, force_variant):
    force_variant("spatial")
    L = configs._bp_conv(53, 0, C, F, k, stride, k // 2, 4, 4, rate, 0.2, dtype, configs.ACT_RELU6)
    _infinite_input_under_pruned_weights(npas, torch, L, N, HW, HW, dtype, res, "spatial_direct")


def test_direct_weights_on_a_map_that_has_overflowed(npas, torch):
    """All outputs of a launch come to the sums over kept weights: about 60 us where all inputs are NaN, 1.4 ms where one channel is infinite (13 ms
    each by loads of 2 bytes and to the end of every sum; 12 us for a finite map).  The bounds leave a factor of three and more."""
    N, HW, C = 32, 28, 128
    ws, _ = dtypes.quantize(prng.normal(33, 1, C * C * 9, 0.1).reshape(C, C, 3, 3), dtypes.BF16)
    p = npas.pack_block_punched(ws, masks.block_punched_mask(C, C, 3, 3, 8, 1, 3, 33), 8, 1, dtypes.BF16)
    assert npas.device_kernel(p, N, HW, HW, 1, 1) == "spatial_direct_kernel"
    y = torch.empty(N, HW, HW, C, dtype=torch.bfloat16, device="cuda")
    plane = torch.ones_like(y)
    plane[..., 3] = float("inf")
    for x, ms in ((torch.full_like(y, float("nan")), 0.5), (plane, 5.0)):
        best = 1e9
        for _ in range(3):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            npas.conv2d_sparse(p, x, y, N, HW, HW, 1, 1)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        print(f"  {best * 1e3:.0f} us", flush=True)
        assert best < ms


@pytest.mark.parametrize("off", [8, 2])
def test_direct_weights_output_at_smaller_alignment(npas, torch, off):
    N, HW, C, F = 20, 28, 64, 72
    ws, _ = dtypes.quantize(prng.normal(31, 1, F * C * 9, 0.1).reshape(F, C, 3, 3), dtypes.BF16)
    p = npas.pack_block_punched(ws, masks.block_punched_mask(F, C, 3, 3, 8, 8, 2, 31), 8, 8, dtypes.BF16)
    xs, _ = dtypes.quantize(prng.normal(31, 2, N * HW * HW * C).reshape(N, HW, HW, C), dtypes.BF16)
    assert npas.device_kernel(p, N, HW, HW, 1, 1) == "spatial_direct_kernel"
    x, n = to_dev(xs, torch), N * HW * HW * F
    y0 = torch.zeros(n, dtype=torch.int16, device="cuda")
    y1 = torch.full((n + 16,), 0x7FC1, dtype=torch.int16, device="cuda")
    npas.conv2d_sparse(p, x, y0, N, HW, HW, 1, 1)
    npas.conv2d_sparse(p, x, y1.data_ptr() + off, N, HW, HW, 1, 1)
    torch.cuda.synchronize()
    assert torch.equal(y1[off // 2:off // 2 + n], y0)
    assert (y1[:off // 2] == 0x7FC1).all() and (y1[off // 2 + n:] == 0x7FC1).all()


@pytest.mark.parametrize("C,F,N,HW,stride,off", [(64, 72, 20, 28, 1, 8), (64, 72, 20, 28, 1, 2), (128, 128, 32, 28, 2, 4), (128, 128, 32, 28, 2, 2),
                                                   (64, 128, 2, 21, 1, 2)],
                         ids=["direct_8_bytes", "direct_2_bytes", "direct_s2_4_bytes", "direct_s2_2_bytes", "split_2_bytes"])
def test_inputs_at_smaller_alignment(npas, torch, C, F, N, HW, stride, off):
    """An input that starts 8, 4 or 2 bytes past an aligned address; at 2 bytes a launch of the direct-weights kernel, whose loads go to LDS, goes to a
    kernel that loads into registers."""
    L = configs._bp_conv(32, 0, C, F, 3, stride, 1, 8, 8, 2, 0.1, dtypes.BF16, configs.ACT_NONE)
    p = pack_layer(npas, L, dtypes.BF16)
    assert npas.device_kernel(p, N, HW, HW, stride, 1) == ("conv_smallm_mfma_kernel" if N == 2 else "spatial_direct_kernel")
    xs, xe = configs._tensor(32, 1, (N, HW, HW, C), 1.0, dtypes.BF16)
    Ho = (HW - 1) // stride + 1
    ref = oracle.round_to(oracle.conv2d_masked(xe[:2], L.w_exact, L.mask, stride, 1), dtypes.BF16)
    flat = np.zeros(xs.size + 16, np.uint16)
    flat[off // 2:off // 2 + xs.size] = xs.reshape(-1)
    y0, y = (new_dev((N, Ho, Ho, F), dtypes.BF16, torch, fill=0x7FC1) for _ in range(2))
    x = to_dev(flat, torch)
    npas.conv2d_sparse(p, x.data_ptr() + off, y, N, HW, HW, stride, 1)
    npas.conv2d_sparse(p, to_dev(xs, torch), y0, N, HW, HW, stride, 1)
    torch.cuda.synchronize()
    got = from_dev(y, dtypes.BF16).reshape(N, Ho, Ho, F)
    assert rel_err(got[:2], ref) <= TOL[dtypes.BF16]
    # against the aligned call: another order of additions moves a value that lies on a rounding boundary by a bf16 step
    assert rel_err(got, from_dev(y0, dtypes.BF16).reshape(got.shape)) <= TOL[dtypes.BF16]


@pytest.mark.parametrize("C,F,N,HW,k,off", [(144, 40, 3, 29, 1, 8), (64, 128, 2, 21, 3, 2), (144, 40, 3, 29, 1, 2), (24, 960, 3, 29, 1, 8),
                                              (24, 960, 3, 29, 1, 2)],
                         ids=["flat_8_bytes", "split_2_bytes", "flat_2_bytes", "flat_groups_8_bytes", "flat_groups_2_bytes"])
def test_outputs_at_smaller_alignment(npas, torch, C, F, N, HW, k, off):
    """An output that starts 8 or 2 bytes past an aligned address: narrower stores, same values."""
    w = prng.normal(31, 1, F * C * k * k, 0.1).reshape(F, C, k, k)
    ws, _ = dtypes.quantize(w, dtypes.BF16)
    m = masks.block_punched_mask(F, C, k, k, 8, 8, 2, 31)
    p = npas.pack_block_punched(ws, m, 8, 8, dtypes.BF16)
    xs, _ = dtypes.quantize(prng.normal(31, 2, N * HW * HW * C).reshape(N, HW, HW, C), dtypes.BF16)
    assert npas.device_kernel(p, N, HW, HW, 1, k // 2) == ("pointwise_stream_kernel" if k == 1 else "conv_smallm_mfma_kernel")
    x, n = to_dev(xs, torch), N * HW * HW * F
    y0 = torch.zeros(n, dtype=torch.int16, device="cuda")
    y1 = torch.full((n + 16,), 0x7FC1, dtype=torch.int16, device="cuda")
    npas.conv2d_sparse(p, x, y0, N, HW, HW, 1, k // 2)
    npas.conv2d_sparse(p, x, y1.data_ptr() + off, N, HW, HW, 1, k // 2)
    torch.cuda.synchronize()
    assert torch.equal(y1[off // 2:off // 2 + n], y0)
    assert (y1[:off // 2] == 0x7FC1).all() and (y1[off // 2 + n:] == 0x7FC1).all()


# Every slot count the fused block is compiled for, partial tiles of 32, 64 and more pixels (the tile follows the number of
# tiles in the batch), filter counts that leave a 16-filter tile partial, dense and pruned projections.
@pytest.mark.parametrize("N,HW,C,t,stride,rate,dtype,bias,act",
                         [(1, 5, 8, 4, 1, 1, dtypes.BF16, True, configs.ACT_RELU6), (2, 9, 16, 4, 2, 1, dtypes.F16, True, configs.ACT_HARDSWISH),
                          (3, 17, 24, 3, 1, 1, dtypes.BF16, False, configs.ACT_RELU), (24, 33, 24, 6, 1, 4, dtypes.BF16, True, configs.ACT_RELU6),
                          (40, 41, 16, 8, 1, 1, dtypes.F16, True, configs.ACT_RELU6), (2, 31, 32, 5, 2, 1, dtypes.BF16, True, configs.ACT_RELU6),
                          (33, 45, 32, 6, 1, 1, dtypes.BF16, True, configs.ACT_HARDSWISH), (70, 31, 24, 8, 2, 1, dtypes.BF16, False, configs.ACT_RELU6),
                          (1, 1, 32, 6, 1, 2, dtypes.F16, True, configs.ACT_RELU6)])
def test_fused_block_slots_and_tiles(npas, torch, N, HW, C, t, stride, rate, dtype, bias, act):
    from workloads import sweeps
    print(f"fused block N={N} {HW}x{HW} {C}->{C * t} stride {stride} rate {rate}", flush=True)
    w = sweeps.inverted_residual_block(batch=N, HW=HW, C=C, t=t, stride=stride, rate=rate, dtype=dtype, bias=bias, act=act)
    ref = oracle.run_stack(w.x_exact, w.layers, w.dtype)[0][-1]
    got, st = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_INVERTED_RESIDUAL)
    assert st.num_launches() == 1
    norm, worst = helpers.check_stack_output(got.reshape(ref.shape), ref, STACK_NORM_TOL)
    print(f"  norm-wise {norm:.3e} worst element {worst:.3e}", flush=True)


# The activations are compiled in: hard-swish, hard-swish, clamp at the slot counts not above, and mixtures with hard-swish.
@pytest.mark.parametrize("C,t,stride,acts,dtype", [(8, 4, 1, (3, 3, 0), dtypes.BF16), (24, 4, 2, (3, 3, 0), dtypes.F16), (16, 8, 1, (3, 3, 1), dtypes.BF16),
                                                   (32, 5, 2, (3, 3, 2), dtypes.BF16), (24, 4, 1, (3, 2, 0), dtypes.BF16),
                                                   (16, 4, 2, (1, 3, 0), dtypes.F16), (32, 6, 1, (2, 0, 3), dtypes.BF16)])
def test_fused_block_activation_mixes(npas, torch, C, t, stride, acts, dtype):
    from workloads import sweeps
    print(f"fused block {C}->{C * t} stride {stride} activations {acts}", flush=True)
    w = sweeps.inverted_residual_block(batch=3, HW=19, C=C, t=t, stride=stride, rate=1, dtype=dtype, bias=True)
    for L, a in zip(w.layers, acts):
        L.act = a
    ref = oracle.run_stack(w.x_exact, w.layers, w.dtype)[0][-1]
    got, st = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_INVERTED_RESIDUAL)
    assert st.num_launches() == 1
    norm, worst = helpers.check_stack_output(got.reshape(ref.shape), ref, STACK_NORM_TOL)
    print(f"  norm-wise {norm:.3e} worst element {worst:.3e}", flush=True)


@pytest.mark.parametrize("C", [8, 24])
def test_fused_block_infinite_input_in_the_last_channels(npas, torch, C):
    """The matrix steps are 32 channels deep; past the last channel they must meet zeros, not other channels of the pixel.  An
    infinite input under kept weights then clamps to 0 or 6 like any other, as the oracle has it."""
    from workloads import sweeps
    w = sweeps.inverted_residual_block(batch=2, HW=11, C=C, t=4, stride=2, rate=1)
    for n, y, x, c, v in ((0, 3, 4, C - 1, np.inf), (1, 0, 0, C - 5, -np.inf), (1, 10, 10, C - 8, np.inf)):
        w.x_exact[n, y, x, c] = v
    w.x_store, _ = dtypes.quantize(w.x_exact, w.dtype)
    assert (w.layers[0].w_exact != 0).all()
    ref = oracle.run_stack(w.x_exact, w.layers, w.dtype)[0][-1]
    assert np.isfinite(ref).all()
    got, st = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_INVERTED_RESIDUAL)
    assert st.num_launches() == 1
    helpers.check_stack_output(got.reshape(ref.shape), ref, STACK_NORM_TOL)


@pytest.mark.parametrize("C,t,stride,acts,HW", [(8, 4, 1, (1, 1, 0), 9), (16, 4, 2, (3, 2, 0), 23), (24, 4, 1, (1, 2, 1), 13), (32, 4, 2, (1, 1, 0), 15),
                                                (32, 5, 1, (3, 2, 3), 21), (32, 6, 1, (1, 1, 0), 17), (32, 6, 2, (3, 1, 0), 17)])
def test_fused_block_expanded_values_that_overflow(npas, torch, C, t, stride, acts, HW):
    """fp16, finite input: two expanded channels overflow to infinity at scattered pixels, and the depthwise layer (negative weights, then
    ReLU or ReLU6) turns them into finite values again.  The other channels of their matrix step must not notice."""
    from workloads import sweeps
    w = sweeps.inverted_residual_block(batch=3, HW=HW, C=C, t=t, stride=stride, rate=1, dtype=dtypes.F16, bias=True)
    mid = C * t
    for L, a in zip(w.layers, acts):
        L.act = a
    for c in (1, mid - 6):
        w.layers[0].w_exact[c] = 0.0
        w.layers[0].w_exact[c, 0, 0, 0] = 32768.0            # times an input above 2: infinite in fp16
        w.layers[0].bias[c] = 0.0
        w.layers[1].w_exact[c] = -np.abs(w.layers[1].w_exact[c]) - 0.0625
        w.layers[1].bias[c] = 0.0
    for L in w.layers[:2]:
        L.w_store, L.w_exact = dtypes.quantize(L.w_exact, w.dtype)
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    assert np.isinf(rounded[1]).any() and np.isfinite(rounded[-1]).all()
    got, st = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_INVERTED_RESIDUAL)
    assert st.num_launches() == 1
    helpers.check_stack_output(got.reshape(rounded[-1].shape), rounded[-1], TOL[dtypes.F16])


def test_run_stack_in_a_hip_graph_replays_like_the_eager_call(npas, torch):
    """npas_run_stack allocates nothing and clears nothing during a run, so a caller may capture it.
    Several replays, with eager work and synchronisations in between, each against the eager result."""
    print("run_stack captured in a HIP graph", flush=True)
    w = configs.config5(batch=2, HW=32, width=16, blocks=(1, 1, 1, 1))
    packed = [pack_layer(npas, L, w.dtype) if L.kind in ("conv", "fc", "dwconv") else None for L in w.layers]
    st = npas.Stack(helpers.stack_descs(npas, w.layers, packed), w.x_shape[1], w.x_shape[2],
                    npas.STACK_FUSE_POINTWISE | npas.STACK_FUSE_INVERTED_RESIDUAL | npas.STACK_FUSE_CONV_MAXPOOL)
    N = w.x_shape[0]
    shapes = {0: w.x_shape}
    for i, L in enumerate(w.layers):
        shapes[i + 1] = helpers.out_shape(L, shapes[L.src])
    wsb = st.workspace_bytes(N)
    ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
    x = to_dev(w.x_store, torch)
    y_eager = new_dev(shapes[len(w.layers)], w.dtype, torch, fill=0x7FC1)
    st.run(x, y_eager, N, ws, wsb)           # also the first call: one-time kernel attributes are set here
    torch.cuda.synchronize()
    y_graph = new_dev(shapes[len(w.layers)], w.dtype, torch, fill=0x7FC1)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        st.run(x, y_graph, N, ws, wsb, torch.cuda.current_stream().cuda_stream)
    for rep in range(3):
        y_graph.fill_(0x7FC1)                # eager work between the replays
        ws.random_(0, 255)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y_graph, y_eager), f"replay {rep} differs from the eager call"


def test_depthwise_handle_is_rejected_by_the_convolution_call(npas, torch):
    ws, _ = dtypes.quantize(prng.normal(18, 1, 16 * 9).reshape(16, 3, 3), dtypes.BF16)
    p = npas.pack_depthwise3x3(ws, dtypes.BF16)
    x = new_dev((1, 4, 4, 16), dtypes.BF16, torch, fill=0)
    y = new_dev((1, 4, 4, 16), dtypes.BF16, torch, fill=0)
    with pytest.raises(npas.NpasError):
        npas.conv2d_sparse(p, x, y, 1, 4, 4, 1, 1)


def test_fc_with_rows_and_columns_pruned_inside_blocks(npas, torch):
    """Block-based FC pruning allows whole rows as well as whole columns of a block to go (section 3)."""
    B, IN, OUT, Br, Bcol = 37, 192, 88, 16, 32
    m = masks.fc_block_mask(OUT, IN, Br, Bcol, 3, 41).copy()
    keys = prng.u64(41, 9, OUT * (IN // Bcol)).reshape(OUT, IN // Bcol)
    rowdrop = (keys % np.uint64(4)) == 0                      # a quarter of the (row, block) pairs lose their row
    m[np.repeat(rowdrop, Bcol, axis=1)] = 0
    assert oracle.validate_fc_block(m, Br, Bcol) == 0
    xs, xe = dtypes.quantize(prng.normal(41, 1, B * IN).reshape(B, IN), dtypes.BF16)
    ws, we = dtypes.quantize(prng.normal(41, 2, OUT * IN, 0.1).reshape(OUT, IN, 1, 1), dtypes.BF16)
    L = configs.Layer("fc", "fc_block", IN, OUT, 1, 1, 1, 0, Br, Bcol, 3.0, 1, w_store=ws, w_exact=we,
                      mask=m.reshape(OUT, IN, 1, 1))
    p = pack_layer(npas, L, dtypes.BF16)
    helpers.check_metadata(oracle, L, p, dtypes.BF16)
    y = run_layer_gpu(npas, torch, L, p, to_dev(xs, torch), (B, IN), dtypes.BF16)
    ref = oracle.round_to(oracle.fc_masked(xe, we, L.mask, None, 1), dtypes.BF16)
    err = rel_err(from_dev(y, dtypes.BF16).reshape(B, OUT), ref)
    print(f"  err={err:.3e}", flush=True)
    assert err <= 1e-2


# Fewer than 8 input channels (an image stem): the whole-reduction kernel.  Ragged tiles, stride 2 with
# padding 3, one to five reduction steps, filter counts below 64, more tiles than workgroups.
SMALLC = [
    ("stem_7x7_s2", 2, 37, 41, 3, 64, 7, 7, 2, 3, 8, 3, 3, dtypes.BF16, 1, False, True),
    ("c1_3x3_f16", 3, 19, 23, 1, 16, 3, 3, 1, 1, 4, 1, 2, dtypes.F16, 1, True, True),
    ("c4_5x5_f36", 2, 20, 18, 4, 36, 5, 5, 1, 2, 4, 4, 2, dtypes.BF16, 2, True, False),
    ("c3_3x3_s2_f8", 1, 9, 9, 3, 8, 3, 3, 2, 1, 8, 3, 2, dtypes.BF16, 0, False, False),
    ("c3_3x3_many_tiles", 13, 128, 128, 3, 8, 3, 3, 1, 1, 8, 3, 2, dtypes.BF16, 1, False, True),
]


@pytest.mark.parametrize("case", SMALLC, ids=[c[0] for c in SMALLC])
def test_small_channel_kernel(npas, torch, case):
    _run_edge_case(npas, torch, case, expect_kernel="conv_smallc_mfma")


def test_small_channel_kernel_on_more_than_65536_tiles_an_image(npas, torch):
    """Tiles times tiles of an image beyond 2^32, where the reciprocal of the tiles of an image is one too high for an image's last tiles."""
    N, HW, F, rows = 2, 5000, 8, 40
    print(f"small channels {N}x{HW}x{HW}x3", flush=True)
    L = configs._bp_conv(63, 0, 3, F, 3, 1, 1, 8, 3, 2, 0.2, dtypes.BF16, configs.ACT_NONE)
    p = pack_layer(npas, L, dtypes.BF16)
    assert npas.device_kernel(p, N, HW, HW, 1, 1) == "conv_smallc_mfma_kernel"
    g = torch.Generator(device="cuda").manual_seed(63)
    x = torch.randn(N, HW, HW, 3, generator=g, device="cuda").to(torch.bfloat16)
    y = torch.full((N, HW, HW, F), float("nan"), dtype=torch.bfloat16, device="cuda")
    npas.conv2d_sparse(p, x, y, N, HW, HW, 1, 1)
    torch.cuda.synchronize()
    assert torch.isfinite(y).all()
    ref = oracle.round_to(oracle.conv2d_masked(x[:, -rows - 1:].double().cpu().numpy(), L.w_exact, L.mask, 1, 1), dtypes.BF16)[:, 1:]
    assert rel_err(y[:, -rows:].double().cpu().numpy(), ref) <= TOL[dtypes.BF16]


# Stride 2 on at most 3 channels and whole 4-byte rows: the kernel by kernel rows.  Partial column blocks and filter quads, one or an odd
# number of conv rows, images smaller than the kernel's reach, both parities of the padding, bands of one pair and of many.
SMALLC_ROWS = [
    ("rows_7x7_s2_ragged", 2, 37, 42, 3, 64, 7, 7, 2, 3, 8, 3, 3, dtypes.BF16, 1, False, True),
    ("rows_7x7_no_pad_res", 3, 29, 46, 3, 36, 7, 7, 2, 0, 4, 3, 2, dtypes.F16, 0, True, False),
    ("rows_5x5_hs_c2", 2, 31, 35, 2, 20, 5, 5, 2, 2, 4, 2, 2, dtypes.BF16, 3, True, True),
    ("rows_3x3_c1_wide_pad", 1, 5, 6, 1, 4, 3, 3, 2, 3, 4, 1, 1, dtypes.F16, 2, False, True),
    ("rows_one_conv_row", 2, 3, 64, 3, 8, 3, 3, 2, 0, 8, 3, 2, dtypes.BF16, 1, False, False),
    ("rows_many_bands", 70, 128, 128, 3, 8, 3, 3, 2, 1, 8, 3, 2, dtypes.BF16, 1, False, True),
]


@pytest.mark.parametrize("case", SMALLC_ROWS, ids=[c[0] for c in SMALLC_ROWS])
def test_small_channel_kernel_by_rows(npas, torch, case):
    _run_edge_case(npas, torch, case, expect_kernel="conv_smallc_mfma", device_kernel="conv_smallc_rows_kernel")


@pytest.mark.parametrize("pool", [False, True])
def test_small_channel_rows_infinite_input_stays_in_its_windows(npas, torch, pool):
    """The slots beside a kernel row's values hold neighbouring pixels: an infinite one must not reach outputs whose window is without it."""
    N, H, W, C, F, k = 1, 32, 36, 3, 16, 7
    layers = [configs._bp_conv(78, 0, C, F, k, 2, 3, 8, C, 2, 0.2, dtypes.BF16, configs.ACT_NONE, 0, -1, "stem")]
    if pool:
        layers.append(configs.Layer("maxpool", src=1, C=F, F=F, KH=3, KW=3, stride=2, pad=1, name="maxpool"))
    xs, xe = configs._tensor(78, 1, (N, H, W, C), 1.0, dtypes.BF16)
    clean, _ = _run_stack_gpu(npas, torch, configs.Workload("clean", dtypes.BF16, xs.shape, xs, xe, layers), npas.STACK_FUSE_CONV_MAXPOOL)
    for iy, ix in ((16, 17), (15, 18), (0, 0), (31, 35)):
        x2 = xs.copy().reshape(N, H, W, C)
        x2[0, iy, ix] = 0x7f80
        got, _ = _run_stack_gpu(npas, torch, configs.Workload("inf", dtypes.BF16, x2.shape, x2, xe, layers), npas.STACK_FUSE_CONV_MAXPOOL)
        oy, ox = np.arange(16)[:, None], np.arange(18)[None, :]
        hit = (np.abs(2 * oy - iy) <= 3) & (np.abs(2 * ox - ix) <= 3)   # conv outputs that see the pixel
        if pool:
            hit = np.array([[hit[max(0, 2 * y - 1):2 * y + 2, max(0, 2 * c - 1):2 * c + 2].any() for c in range(9)] for y in range(8)])
        np.testing.assert_array_equal(got[0][~hit], clean[0][~hit])


# Few output pixels (batch 1, late stages): the kernel that splits the reduction over the waves of a workgroup.
# Stride 2, non-square kernels, filter counts off the 16- and 128-filter grids, ragged pixel tiles, fp16.
SMALLM = [
    ("sm_7x7_512", 1, 7, 7, 512, 512, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, False, True),
    ("sm_stride2_ragged", 3, 15, 14, 128, 72, 3, 3, 2, 1, 8, 4, 3, dtypes.BF16, 0, True, True),
    ("sm_5x3_fp16", 2, 12, 17, 64, 200, 5, 3, 1, 2, 4, 4, 2, dtypes.F16, 2, True, False),
    ("sm_one_step_per_wave", 1, 9, 9, 64, 64, 3, 3, 1, 1, 8, 4, 2, dtypes.BF16, 1, False, False),
    ("sm_more_waves_than_steps", 1, 5, 5, 64, 40, 2, 2, 1, 0, 8, 4, 2, dtypes.BF16, 0, False, False),
    ("sm_many_pixels_little_work", 1, 41, 39, 64, 64, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 1, True, True),
]


@pytest.mark.parametrize("case", SMALLM, ids=[c[0] for c in SMALLM])
def test_small_pixel_count_kernel(npas, torch, case):
    _run_edge_case(npas, torch, case, expect_kernel="conv_smallm_mfma")


def test_block_punched_5x5(npas, torch):
    _run_edge_case(npas, torch, ("kernel_5x5", 2, 17, 19, 16, 24, 5, 5, 1, 2, 8, 4, 3, dtypes.BF16, 1, False, True))
    _run_edge_case(npas, torch, ("kernel_5x5_wide", 2, 12, 12, 64, 72, 5, 5, 1, 2, 8, 4, 2, dtypes.BF16, 0, True, False))


def test_group_with_everything_pruned_gives_bias_only(npas, torch):
    F, C = 32, 16
    m = masks.block_punched_mask(F, C, 3, 3, 8, 4, 2, 5)
    m[8:16] = 0                                  # filter group 1 keeps nothing
    ws, we = dtypes.quantize(prng.normal(8, 2, F * C * 9, 0.2).reshape(F, C, 3, 3), dtypes.BF16)
    xs, xe = dtypes.quantize(prng.normal(8, 1, 6 * 6 * C).reshape(1, 6, 6, C), dtypes.BF16)
    bias = prng.normal(8, 3, F).astype(np.float32)
    L = configs.Layer("conv", "block_punched", C, F, 3, 3, 1, 1, 8, 4, 2, 0, w_store=ws, w_exact=we, mask=m)
    p = pack_layer(npas, L, dtypes.BF16)
    y = from_dev(run_layer_gpu(npas, torch, L, p, to_dev(xs, torch), (1, 6, 6, C), dtypes.BF16, None, to_dev(bias, torch)),
                 dtypes.BF16).reshape(1, 6, 6, F)
    ref = oracle.round_to(oracle.conv2d_masked(xe, we, m, 1, 1, bias.astype(np.float64)), dtypes.BF16)
    np.testing.assert_array_equal(y[..., 8:16], ref[..., 8:16])
    assert rel_err(y, ref) <= 1e-2


def test_garbage_under_the_mask_changes_nothing(npas, torch):
    w = configs.config2(batch=1, HW=9)
    L = w.layers[0]
    junk = L.w_store.copy()
    junk[L.mask == 0] = 0x7F80                    # +inf bit pattern where pruned
    p1 = npas.pack_block_punched(L.w_store, L.mask, L.Bf, L.Bc, w.dtype)
    p2 = npas.pack_block_punched(junk, L.mask, L.Bf, L.Bc, w.dtype)
    x = to_dev(w.x_store, torch)
    y1 = run_layer_gpu(npas, torch, L, p1, x, w.x_shape, w.dtype)
    y2 = run_layer_gpu(npas, torch, L, p2, x, w.x_shape, w.dtype)
    assert torch.equal(y1, y2)


def _run_stack_gpu(npas, torch, w, flags=0):
    packed = [pack_layer(npas, L, w.dtype) if L.kind in ("conv", "fc", "dwconv") else None for L in w.layers]
    biases = helpers.bias_tensors(w.layers, torch)   # alive until the run below has finished
    st = npas.Stack(helpers.stack_descs(npas, w.layers, packed, biases), w.x_shape[1], w.x_shape[2], flags)
    N = w.x_shape[0]
    shape = w.x_shape
    shapes = {0: shape}
    for i, L in enumerate(w.layers):
        shapes[i + 1] = helpers.out_shape(L, shapes[L.src])
    wsb = st.workspace_bytes(N)
    ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
    y = new_dev(shapes[len(w.layers)], w.dtype, torch, fill=(float("nan") if w.dtype == dtypes.F32 else 0x7FC1))
    st.run(to_dev(w.x_store, torch), y, N, ws, wsb)
    torch.cuda.synchronize()
    return from_dev(y, w.dtype).reshape(shapes[len(w.layers)]), st


@pytest.mark.parametrize("flags", [0, 1], ids=["per_layer", "fused_pointwise"])
def test_config2_run_stack_end_to_end(npas, torch, flags):
    print(f"config2 run_stack flags={flags}", flush=True)
    w = configs.config2(batch=2, HW=23)
    got, st = _run_stack_gpu(npas, torch, w, flags)
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    err = rel_err(got, rounded[-1])
    print(f"  launches={st.num_launches()} err={err:.3e}", flush=True)
    assert err <= 1e-2


def test_fp16_storage_through_the_fused_kernels_and_the_pointwise_ring(npas, torch):
    """Every 16-bit kernel is instantiated for fp16 as well as bf16: the fused pair, the fused inverted-residual
    block and the streaming 1x1 kernel on fp16 tensors (fused launches: the stack criterion at the fp16 tolerance)."""
    from workloads import sweeps
    print("fp16: fused pair", flush=True)
    w = configs.config2(batch=2, HW=23, dtype=dtypes.F16)
    got, st = _run_stack_gpu(npas, torch, w, 1)
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    norm, worst = helpers.check_stack_output(got, rounded[-1], TOL[dtypes.F16])
    print(f"  launches={st.num_launches()} norm-wise {norm:.3e} worst element {worst:.3e}", flush=True)
    assert st.num_launches() == 1
    print("fp16: fused inverted-residual block", flush=True)
    w = sweeps.inverted_residual_block(batch=2, HW=13, dtype=dtypes.F16)
    got, st = _run_stack_gpu(npas, torch, w, 3)
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    norm, worst = helpers.check_stack_output(got, rounded[-1], TOL[dtypes.F16])
    print(f"  launches={st.num_launches()} norm-wise {norm:.3e} worst element {worst:.3e}", flush=True)
    assert st.num_launches() == 1
    _run_edge_case(npas, torch, ("fp16_pointwise_ring", 13, 29, 27, 128, 136, 1, 1, 1, 0, 8, 4, 3, dtypes.F16, 2, True, True),
                   expect_kernel="pointwise_ring")
    _run_edge_case(npas, torch, ("fp16_pointwise_split", 3, 9, 11, 128, 136, 1, 1, 1, 0, 8, 4, 3, dtypes.F16, 2, True, True),
                   expect_kernel="conv_smallm_mfma")


def test_config5_run_stack_end_to_end(npas, torch):
    print("config5 reduced run_stack", flush=True)
    w = configs.config5(batch=2, HW=64, width=16)
    got, st = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_CONV_MAXPOOL)
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    ref = rounded[-1]
    norm_err = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"  launches={st.num_launches()} norm-wise err={norm_err:.3e} elementwise={rel_err(got, ref):.3e}", flush=True)
    # 50+ bf16 layers: element-wise 1e-2 cannot hold end to end (roundings compound), the norm-wise bound must
    assert norm_err <= STACK_NORM_TOL
    assert (got.argmax(1) == ref.argmax(1)).all()


STEM_POOL = [
    # name, N, H, W, C, F, k, stride, pad, block channels, act, dtype
    ("stem7x7_ragged", 3, 37, 41, 3, 64, 7, 2, 3, 3, configs.ACT_RELU, dtypes.BF16),
    ("stem7x7_no_activation_fp16", 2, 64, 64, 3, 40, 7, 2, 3, 3, configs.ACT_NONE, dtypes.F16),
    ("conv3x3_stride1_4_channels", 2, 30, 33, 4, 32, 3, 1, 1, 4, configs.ACT_RELU6, dtypes.BF16),
    ("more_tiles_than_workgroups", 9, 224, 224, 3, 64, 7, 2, 3, 3, configs.ACT_RELU, dtypes.BF16),
    ("more_tiles_than_workgroups_odd_width", 12, 224, 223, 3, 64, 7, 2, 3, 3, configs.ACT_RELU, dtypes.BF16),   # 672 tiles of the kernel that is not by rows
    # by kernel rows: partial blocks of 7 pooled columns, odd conv heights and widths, one pooled pixel, hard-swish
    ("rows_7x7_ragged", 3, 39, 58, 3, 64, 7, 2, 3, 3, configs.ACT_RELU, dtypes.BF16),
    ("rows_5x5_hard_swish_fp16", 2, 33, 62, 2, 44, 5, 2, 2, 2, configs.ACT_HARDSWISH, dtypes.F16),
    ("rows_3x3_one_pooled_pixel", 2, 3, 4, 3, 8, 3, 2, 1, 3, configs.ACT_RELU6, dtypes.BF16),
    ("rows_3x3_odd_width", 1, 20, 30, 1, 12, 3, 2, 0, 1, configs.ACT_NONE, dtypes.BF16),
]


@pytest.mark.parametrize("case", STEM_POOL, ids=[c[0] for c in STEM_POOL])
def test_conv_and_maxpool_as_one_kernel(npas, torch, case):
    """A small-channel conv and the 3x3 / stride 2 max pool after it, one launch (NPAS_STACK_FUSE_CONV_MAXPOOL): the
    pooled tensor against the oracle's conv -> round -> max pool, and against the two-launch stack bit for bit."""
    name, N, H, W, C, F, k, stride, pad, Bc, act, dtype = case
    print(f"conv+maxpool {name}", flush=True)
    xs, xe = configs._tensor(77, 1, (N, H, W, C), 1.0, dtype)
    layers = [configs._bp_conv(77, 0, C, F, k, stride, pad, 8, Bc, 2, 0.2, dtype, act, 0, -1, "stem"),
              configs.Layer("maxpool", src=1, C=F, F=F, KH=3, KW=3, stride=2, pad=1, name="maxpool")]
    w = configs.Workload("stem_pool", dtype, (N, H, W, C), xs, xe, layers)
    fused, st = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_CONV_MAXPOOL)
    plain, st0 = _run_stack_gpu(npas, torch, w, 0)
    assert st.num_launches() == 1 and st0.num_launches() == 2
    assert st.workspace_bytes(N) == 0
    np.testing.assert_array_equal(fused, plain)
    if N * H * W <= 64 * 64 * 4:
        rounded, _ = oracle.run_stack(xe, layers, dtype)
        err = rel_err(fused, rounded[-1])
        print(f"  err={err:.3e}", flush=True)
        assert err <= TOL[dtype]


def test_full_size_config2_two_launches_sampled(npas, torch):
    """configs[1] at full size (batch 64, 56x56) through npas_run_stack WITHOUT fusion (two launches of the per-layer
    kernel): sampled pixels against the oracle.  The fused launch is covered by the tests below."""
    print("config2 full size, two launches, sampled", flush=True)
    w = configs.config2()
    got, _ = _run_stack_gpu(npas, torch, w)
    N, H, W, C = w.x_shape
    npx = N * H * W
    idx = (prng.u64(3, 3, 4096) % np.uint64(npx)).astype(np.int64)
    idx[:8] = [0, 1, npx - 1, npx - 2, 127, 128, 129, npx // 2]
    xsub = w.x_exact.reshape(npx, C)[idx].reshape(1, 1, -1, C)
    rounded, _ = oracle.run_stack(xsub, w.layers, w.dtype)
    L2 = w.layers[1]
    err, beyond = helpers.check_two_layer_pointwise(got.reshape(npx, -1)[idx], rounded[-1].reshape(len(idx), -1), rounded[1],
                                                    (L2.w_exact * L2.mask).reshape(L2.F, L2.C))
    print(f"  worst plain err={err:.3e}, share beyond 1e-2: {beyond:.2e}", flush=True)


def _pixel_stack(M, dtype=dtypes.BF16):
    """configs[1]'s two layers on M pixels (a 1 x M image: every pixel of a 1x1 stack is independent)."""
    w = configs.config2(batch=1, HW=1, dtype=dtype)
    xs, xe = configs._tensor(configs.BASE_SEED + 2, 1, (1, 1, M, w.layers[0].C), 1.0, dtype)
    return configs.Workload("cfg2_pixels_%d" % M, dtype, (1, 1, M, w.layers[0].C), xs, xe, w.layers)


# 16-pixel blocks per wave of the fused pair: the kernel is instantiated per count (1..8) and a launch uses two
# neighbouring counts.  M pixels -> ceil(M / 16) blocks over min(ceil(blocks / 4), 512) (or more) workgroups x 4 waves.
FPP_COUNTS = [
    # M, grid, counts in use
    (16 * 5000 - 5, 512, {2, 3}),      # ragged last block
    (16 * 9000 - 10, 512, {4, 5}),
    (64 * 56 * 56, 512, {6, 7}),       # the benchmark's shape
    (16 * 16000 - 7, 512, {7, 8}),
    (16 * 20000, 625, {8}),            # more than 8 blocks per wave at 512 workgroups: the grid grows instead
    (16 * 2048 * 3 + 1, 512, {3, 4}),  # one pixel past a whole number of rounds
]


@pytest.mark.parametrize("M,grid,counts", FPP_COUNTS, ids=["cnt" + "_".join(map(str, sorted(c[2]))) + "_M%d" % c[0] for c in FPP_COUNTS])
def test_fused_pair_every_blocks_per_wave_instantiation(npas, torch, M, grid, counts):
    """Every pixel of the fused 1x1 -> ReLU6 -> 1x1 launch against the oracle, at pixel counts that put 2 .. 8
    blocks on a wave (the host formula for the split is restated here to make sure the case is what it claims)."""
    nblk = -(-M // 16)
    g = max(-(-nblk // 32), min(-(-nblk // 4), 512))
    base, extra = divmod(nblk, 4 * g)
    assert g == grid and ({base, base + 1} if extra else {base}) == counts
    print(f"fused pair M={M} blocks={nblk} grid={g} blocks per wave={sorted(counts)}", flush=True)
    w = _pixel_stack(M)
    got, st = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_POINTWISE)
    assert st.num_launches() == 1 and st.workspace_bytes(1) == 0
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    L2 = w.layers[1]
    err, beyond = helpers.check_two_layer_pointwise(got, rounded[-1], rounded[1], (L2.w_exact * L2.mask).reshape(L2.F, L2.C))
    print(f"  worst plain err={err:.3e}, share beyond 1e-2: {beyond:.2e}", flush=True)


def test_config2_benchmark_configuration_fused(npas, torch):
    """configs[1] exactly as bench.py times it (batch 64, 56 x 56, npas_run_stack with NPAS_STACK_FUSE_POINTWISE, one
    launch, waves of 6 and 7 blocks): every output pixel against the oracle, and the run repeated bit for bit."""
    print("config2 full size, fused, all pixels", flush=True)
    w = configs.config2()
    got, st = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_POINTWISE)
    assert st.num_launches() == 1
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    L2 = w.layers[1]
    err, beyond = helpers.check_two_layer_pointwise(got, rounded[-1], rounded[1], (L2.w_exact * L2.mask).reshape(L2.F, L2.C))
    print(f"  worst plain err={err:.3e}, share beyond 1e-2: {beyond:.2e}", flush=True)
    # first and last block of a few waves, separately (what a wrong block range would hit first)
    npx = got.shape[0] * got.shape[1] * got.shape[2]
    nblk = npx // 16
    base, extra = divmod(nblk, 2048)
    for gw in (0, 1, extra - 1, extra, extra + 1, 2047):
        b0 = gw * base + min(gw, extra)
        cnt = base + (1 if gw < extra else 0)
        for blk in (b0, b0 + cnt - 1):
            sl = slice(16 * blk, 16 * blk + 16)
            assert rel_err(got.reshape(npx, -1)[sl], rounded[-1].reshape(npx, -1)[sl]) <= 3e-2, (gw, blk)
    again, _ = _run_stack_gpu(npas, torch, w, npas.STACK_FUSE_POINTWISE)
    np.testing.assert_array_equal(got, again)


FULL_FLAGS = [0, 7]


@pytest.mark.parametrize("flags", FULL_FLAGS, ids=["per_layer", "all_fusions"])
def test_config5_full_size_run_stack_batch2_logits(npas, torch, flags):
    """The 50-layer stack at full size (224 x 224, all 53 pruned convs + pools + classifier) through npas_run_stack,
    two images, with no fusion and with every fusion flag bench.py sets: the logits against the oracle's
    (norm-wise, the bound stated for stacks end to end, and the arg-max)."""
    print(f"config5 full size run_stack batch 2 flags={flags}", flush=True)
    w = configs.config5(batch=2)
    got, st = _run_stack_gpu(npas, torch, w, flags)
    rounded, _ = oracle.run_stack(w.x_exact, w.layers, w.dtype)
    ref = rounded[-1]
    norm_err = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"  launches={st.num_launches()} norm-wise err={norm_err:.3e} elementwise={rel_err(got, ref):.3e}", flush=True)
    assert st.num_launches() == (len(w.layers) - 1 if flags else len(w.layers))
    assert norm_err <= STACK_NORM_TOL
    assert (got.argmax(1) == ref.argmax(1)).all()


def _run_of_pointwise_layers(npas, torch, N, HW, C0, C, stride, proj_act, G, dtype, bias, act, flags, infinite=(), kernel=None):
    """Stack x -> a (1x1, C), x -> s (1x1, 4C), y = act(W a + s), and with G z = act(W y), between a layer that nothing reads (it takes more workspace than
    the run may ask for) and one that adds y to its product of z (and shows where both lie): y and z on the device, the same from the oracle with the
    projection rounded to storage only where it is a tensor of its own (proj_act is not none), and the first and last layer of each launch of a .. z, counted
    from a.  bias: on all layers, none, or those of these numbers.  kernel: the device function of the layer that adds."""
    A, at = configs, 1 if G else 0      # at: number of layer a

    def pw(idx, Ci, F, act, src, res=-1, st=1):
        L = configs._bp_conv(7, idx, Ci, F, 1, st, 0, 8, 4, 2, (1.0 / Ci) ** 0.5, dtype, act, src, res, name=f"pw{idx}")
        if bias is True or (bias and idx in bias):
            L.bias = prng.normal(8, 300 + idx, F, 0.5).astype(np.float32)
        return L

    first = A.ACT_RELU6 if infinite else A.ACT_RELU # (finite)
    layers = [pw(0, C0, C, first, 0, st=stride), pw(1, C0, 4 * C, proj_act, 0, st=stride), pw(2, C, 4 * C, act, at + 1, at + 2)]
    if G:
        layers = [pw(9, C0, 12 * C, A.ACT_NONE, 0)] + layers + [pw(3, 4 * C, G, act, at + 3), pw(4, G, 4 * C, A.ACT_NONE, at + 4, at + 3)]
    xs, xe = configs._tensor(9, 1, (N, HW, HW, C0), 1.0, dtype)
    for i in infinite:
        xs.reshape(N, HW, HW, C0)[i] = 0x7F80 if dtype == dtypes.BF16 else 0x7C00
    packed = [pack_layer(npas, L, dtype) for L in layers]
    biases = helpers.bias_tensors(layers, torch)
    st = npas.Stack(helpers.stack_descs(npas, layers, packed, biases), HW, HW, flags)
    wsb, Ho = st.workspace_bytes(N), (HW - 1) // stride + 1
    if kernel:
        assert npas.device_kernel(packed[at + 2], N, Ho, Ho, 1, 0) == kernel
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    ws.view(torch.int16).fill_(0x7FC1)
    out = new_dev((N, Ho, Ho, 4 * C), dtype, torch, fill=0x7FC1)
    st.run(to_dev(xs, torch), out, N, ws, wsb)
    torch.cuda.synchronize()
    rows = st.describe(N)
    got = [from_dev(out, dtype).reshape(N, Ho, Ho, -1)]
    if G:
        row = rows[-1]
        assert (row["src"], row["res"]) == (at + 4, at + 3)
        got = [from_dev(ws[row["off_" + k]:row["off_" + k] + row["bytes_" + k]].view(torch.int16), dtype).reshape(N, Ho, Ho, -1) for k in ("res", "src")]
    t = [xe] + [None] * at
    for i, L in enumerate(layers[at:at + (4 if G else 3)]):
        v = oracle.run_layer(L, t, dtype)
        t.append(v if flags and i == 1 and proj_act == A.ACT_NONE else oracle.round_to(v, dtype))
    return got, t[at + 3:], [(r["first"] - at, r["last"] - at) for r in rows if at <= r["first"] < at + 4]


# 16 pixels a wave and block: a last block of 1, 15 and 16 pixels; fewer blocks than waves, more than one round of them; both widths of the
# second layer; the projection (from 4097 or 8193 pixels on, as its layers run on the ring) and the residual (the same, with 128 filters from 24576 on).
@pytest.mark.parametrize("N,HW,proj,G,dtype,bias,act", [
    (1, 111, True, 64, dtypes.BF16, True, configs.ACT_RELU), (3, 47, True, 128, dtypes.F16, False, configs.ACT_RELU6),
    (2, 192, True, 64, dtypes.BF16, False, configs.ACT_RELU), (1, 181, False, 64, dtypes.BF16, True, configs.ACT_RELU6),
    (1, 184, False, 128, dtypes.F16, False, configs.ACT_NONE), (3, 161, False, 128, dtypes.BF16, False, configs.ACT_RELU),
    (1, 193, True, 128, dtypes.F16, True, configs.ACT_RELU6), (3, 113, True, 64, dtypes.BF16, True, configs.ACT_NONE),
    (1, 97, False, 64, dtypes.F16, True, configs.ACT_RELU), (1, 91, True, 64, dtypes.BF16, False, configs.ACT_RELU),
    (1, 111, True, 64, dtypes.BF16, (1,), configs.ACT_RELU), (1, 93, True, 64, dtypes.BF16, (2,), configs.ACT_RELU),
    (1, 93, True, 128, dtypes.F16, (3,), configs.ACT_RELU), (1, 97, False, 64, dtypes.F16, (3,), configs.ACT_RELU)])
def test_end_of_a_bottleneck_block_with_the_next_layer(npas, torch, N, HW, proj, G, dtype, bias, act):
    print(f"bottleneck tail {N}x{HW}x{HW} projection={proj} G={G}", flush=True)
    got, ref, launches = _run_of_pointwise_layers(npas, torch, N, HW, 64, 64, 1, configs.ACT_NONE if proj else configs.ACT_RELU, G, dtype, bias, act,
                                                  npas.STACK_FUSE_POINTWISE)
    assert launches == ([(0, 0), (1, 3)] if proj else [(0, 0), (1, 1), (2, 3)])
    for name, g, r in zip(("sum", "next layer"), got, ref):
        norm, worst = helpers.check_stack_output(g, r, STACK_NORM_TOL if dtype == dtypes.BF16 else STACK_NORM_TOL / 8)
        print(f"  {name}: norm-wise {norm:.3e} worst element {worst:.3e}", flush=True)


@pytest.mark.parametrize("proj,G", [(True, 64), (False, 128)], ids=["projection", "residual"])
def test_end_of_a_bottleneck_block_beyond_2_gib(npas, torch, proj, G):
    """The most pixels one launch takes (sums of 3.8 GiB, byte offsets up to 2^32): 3200 times the same image, whose outputs all have to be the
    first one's; that one is checked against the oracle."""
    A, N, HW, C = configs, 3200, 50, 64
    print(f"bottleneck tail {N}x{HW}x{HW} projection={proj} G={G}", flush=True)
    pw = lambda i, Ci, F, act, src, res=-1: configs._bp_conv(7, i, Ci, F, 1, 1, 0, 8, 4, 2, 0.12, dtypes.BF16, act, src, res)  # noqa: E731
    layers = [pw(0, C, C, A.ACT_RELU, 0), pw(1, C, 4 * C, A.ACT_NONE if proj else A.ACT_RELU, 0), pw(2, C, 4 * C, A.ACT_RELU, 1, 2),
              pw(3, 4 * C, G, A.ACT_RELU, 3)]
    packed = [pack_layer(npas, L, dtypes.BF16) for L in layers]
    st = npas.Stack(helpers.stack_descs(npas, layers, packed), HW, HW, npas.STACK_FUSE_POINTWISE)
    assert [(r["first"], r["last"]) for r in st.describe(N)] == ([(0, 0), (1, 3)] if proj else [(0, 0), (1, 1), (2, 3)])
    assert [(r["first"], r["last"]) for r in st.describe(N + 1)][-1] == (3, 3)      # one image more is too many
    xs, xe = configs._tensor(9, 1, (1, HW, HW, C), 1.0, dtypes.BF16)
    x = to_dev(xs, torch).repeat(N, 1, 1, 1)
    px, wsb = N * HW * HW, st.workspace_bytes(N)
    assert wsb == 2 * px * 9 * C                                                    # a, the shortcut, the sum: all alive in that launch
    ws, z = torch.full((wsb // 2,), 0x7FC1, dtype=torch.int16, device="cuda"), new_dev((N, HW * HW * G), dtypes.BF16, torch, fill=0x7FC1)
    st.run(x, z, N, ws, wsb)
    torch.cuda.synchronize()
    y = ws[5 * C * px:].view(N, -1)
    t = [xe]
    for i, L in enumerate(layers):
        v = oracle.run_layer(L, t, dtypes.BF16)
        t.append(v if proj and i == 1 else oracle.round_to(v, dtypes.BF16))
    for name, got, ref in (("sum", y, t[3]), ("next layer", z, t[4])):
        norm, _ = helpers.check_stack_output(from_dev(got[0], dtypes.BF16).reshape(ref.shape), ref, STACK_NORM_TOL)
        print(f"  {name}: norm-wise {norm:.3e}", flush=True)
        for k in range(0, N, 200):
            assert (got[k:k + 200] == got[0]).all(), (name, k)
    del x, ws, y, z
    torch.cuda.empty_cache()


# The projection as further stages of the layer that adds it: the three tile sizes of the ring, one and two pixel blocks of the split reduction (1, 2 and
# 4 images), layers that have exact lists too, a last tile of few pixels, strides 1 and 2 on odd maps, biases on both, one or none (of both widths of the
# ring's tiles), hard-swish.
RING, SPLIT = "pointwise_ring_kernel", "conv_smallm_mfma_kernel"


@pytest.mark.parametrize("N,HW,C0,C,stride,dtype,bias,act,kernel", [
    (1, 3, 64, 64, 1, dtypes.BF16, True, configs.ACT_RELU, None), (1, 14, 512, 256, 2, dtypes.BF16, True, configs.ACT_RELU, None),
    (3, 15, 128, 128, 2, dtypes.F16, True, configs.ACT_HARDSWISH, None), (1, 28, 256, 128, 1, dtypes.BF16, False, configs.ACT_NONE, None),
    (1, 57, 64, 64, 2, dtypes.BF16, True, configs.ACT_RELU6, SPLIT), (2, 41, 64, 64, 1, dtypes.F16, True, configs.ACT_RELU, RING),
    (9, 27, 128, 128, 2, dtypes.BF16, True, configs.ACT_HARDSWISH, RING), (5, 61, 256, 128, 2, dtypes.F16, False, configs.ACT_RELU, RING),
    (3, 113, 192, 64, 2, dtypes.BF16, True, configs.ACT_RELU6, RING), (7, 63, 64, 192, 1, dtypes.BF16, True, configs.ACT_NONE, RING),
    (1, 14, 512, 256, 2, dtypes.BF16, (1,), configs.ACT_RELU, None), (1, 57, 64, 64, 2, dtypes.BF16, (2,), configs.ACT_RELU6, SPLIT),
    (2, 41, 64, 64, 1, dtypes.F16, (1,), configs.ACT_RELU, RING), (2, 41, 64, 64, 1, dtypes.F16, (2,), configs.ACT_RELU, RING),
    (7, 63, 64, 192, 1, dtypes.BF16, (1,), configs.ACT_NONE, RING), (7, 63, 64, 192, 1, dtypes.BF16, (2,), configs.ACT_NONE, RING)])
def test_projection_shortcut_inside_the_layer_that_adds_it(npas, torch, N, HW, C0, C, stride, dtype, bias, act, kernel):
    print(f"projection joined {N}x{HW}x{HW} {C0} / {stride} + {C} -> {4 * C}", flush=True)
    got, ref, launches = _run_of_pointwise_layers(npas, torch, N, HW, C0, C, stride, configs.ACT_NONE, 0, dtype, bias, act, npas.STACK_FUSE_POINTWISE,
                                                  kernel=kernel)
    assert launches == [(0, 0), (1, 2)]
    norm, worst = helpers.check_stack_output(got[0], ref[0], STACK_NORM_TOL if dtype == dtypes.BF16 else STACK_NORM_TOL / 8)
    print(f"  norm-wise {norm:.3e} worst element {worst:.3e}", flush=True)


# Pixels times pixels of an image beyond 2^32, where the reciprocal of Ho * Wo is one too high for an image's last pixel: strided layers on their own
# (flags 0), and the strided projection inside the layer that adds it.
@pytest.mark.parametrize("flags", [0, 1], ids=["per_layer", "joined"])
@pytest.mark.parametrize("N,HW", [(2, 448), (4, 400)])
def test_strided_pointwise_layers_on_many_pixels(npas, torch, N, HW, flags):
    print(f"strided 1x1 {N}x{HW}x{HW} flags={flags}", flush=True)
    got, ref, launches = _run_of_pointwise_layers(npas, torch, N, HW, 64, 64, 2, configs.ACT_NONE, 0, dtypes.BF16, True, configs.ACT_NONE, flags, kernel=RING)
    assert launches == ([(0, 0), (1, 2)] if flags else [(0, 0), (1, 1), (2, 2)])
    g, r = got[0].reshape(N, -1, 256), ref[0].reshape(N, -1, 256)
    err = np.sqrt(((g - r) ** 2).sum(-1) / (r ** 2).sum(-1))
    print(f"  a pixel's error {err.max():.3e}, last pixels' {err[:, -1].max():.3e}", flush=True)
    assert err.max() <= 5 * 2.0 ** -8      # bf16: two rounded inputs of the sum and its own rounding, half a step (2^-9) each at most; another pixel's sum gives about 1


@pytest.mark.parametrize("N,HW,C0,C,stride,dtype", [(1, 14, 512, 256, 2, dtypes.BF16), (1, 28, 256, 128, 1, dtypes.F16), (1, 3, 64, 64, 1, dtypes.BF16)])
def test_projection_inside_the_adding_layer_with_an_infinite_input(npas, torch, N, HW, C0, C, stride, dtype):
    """Split reduction: an infinite value in the projection's input reaches the filters that keep its channel and no others."""
    print(f"projection joined, infinite input {N}x{HW}x{HW} {C0} / {stride} + {C} -> {4 * C}", flush=True)
    args = (npas, torch, N, HW, C0, C, stride, configs.ACT_NONE, 0, dtype, False, configs.ACT_RELU)
    (apart,), _, one_by_one = _run_of_pointwise_layers(*args, 0, [(0, 0, 0, 1), (0, 2, 2, C0 - 3)])
    (joined,), _, launches = _run_of_pointwise_layers(*args, npas.STACK_FUSE_POINTWISE, [(0, 0, 0, 1), (0, 2, 2, C0 - 3)])
    assert one_by_one == [(0, 0), (1, 1), (2, 2)] and launches == [(0, 0), (1, 2)]
    got = [apart, joined]
    assert np.isinf(got[0]).any() and np.isfinite(got[0]).any()
    for kind in (np.isnan, np.isposinf):
        np.testing.assert_array_equal(kind(got[1]), kind(got[0]))
    finite = np.isfinite(got[0])
    assert np.abs(got[1][finite] - got[0][finite]).max() <= 2e-2 * np.abs(got[0][finite]).max()


def test_run_stack_at_changing_batch_sizes(npas, torch):
    """One stack called at more batch sizes than it keeps placements of, some of them again later: each call gives what a stack of its own gives."""
    w = configs.config5(batch=1, HW=32, width=64, blocks=(1, 2, 1, 1))
    packed = [pack_layer(npas, L, w.dtype) if L.kind in ("conv", "fc") else None for L in w.layers]
    new = lambda: npas.Stack(helpers.stack_descs(npas, w.layers, packed), 32, 32, 7)  # noqa: E731
    one, x = new(), torch.randn(72, 32, 32, 3, generator=torch.Generator(device="cuda").manual_seed(5), device="cuda").to(torch.bfloat16)
    ws = torch.empty(one.workspace_bytes(72), dtype=torch.uint8, device="cuda")
    for N in [3, 1, 3] + list(range(1, 73)) + [2, 72, 1]:
        ys = [torch.full((N, w.layers[-1].F), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        for st, y in zip((one, new()), ys):
            ws.view(torch.int16).fill_(0x7FC1)
            st.run(x[:N], y, N, ws, ws.numel())
        torch.cuda.synchronize()
        assert torch.isfinite(ys[0]).all() and torch.equal(ys[0], ys[1]), N


def test_chained_fused_launches_against_the_oracle(npas, torch):
    """Fused launches whose inputs and outputs are workspace tensors (the placement must keep a fused launch's input
    alive while it writes the output of the last layer it absorbs): three fused 1x1 pairs of unequal widths in a row,
    and two fused inverted-residual blocks without residual, end to end against the oracle and against the
    unfused stack."""
    A = configs

    def pw(seed, idx, C, F, act, src, res=-1):
        return configs._bp_conv(seed, idx, C, F, 1, 1, 0, 8, 8, 2, 0.25, dtypes.BF16, act, src, res, name=f"pw{idx}")

    def dw(seed, idx, C, src):
        ws, we = configs._tensor(seed, 150 + idx, (C, 3, 3), 0.3, dtypes.BF16)
        return configs.Layer("dwconv", "", C, C, 3, 3, 1, 1, 1, 1, 1.0, A.ACT_RELU6, src, -1, ws, we, name=f"dw{idx}")

    chain = [pw(1, 0, 16, 48, A.ACT_RELU6, 0), pw(1, 1, 48, 24, A.ACT_NONE, 1),
             pw(1, 2, 24, 64, A.ACT_RELU6, 2), pw(1, 3, 64, 8, A.ACT_NONE, 3),
             pw(1, 4, 8, 40, A.ACT_HARDSWISH, 4), pw(1, 5, 40, 32, A.ACT_NONE, 5)]
    blocks = [pw(2, 0, 16, 64, A.ACT_RELU6, 0), dw(2, 1, 64, 1), pw(2, 2, 64, 24, A.ACT_NONE, 2),
              pw(2, 3, 24, 96, A.ACT_HARDSWISH, 3), dw(2, 4, 96, 4), pw(2, 5, 96, 32, A.ACT_NONE, 5),
              pw(2, 6, 32, 16, A.ACT_RELU, 6)]
    for name, layers, flag, launches in (("pairs", chain, npas.STACK_FUSE_POINTWISE, 3),
                                         ("blocks", blocks, npas.STACK_FUSE_INVERTED_RESIDUAL, 3)):
        N, HW, C = 5, 37, layers[0].C
        xs, xe = configs._tensor(31, 1, (N, HW, HW, C), 1.0, dtypes.BF16)
        w = configs.Workload("chained_" + name, dtypes.BF16, (N, HW, HW, C), xs, xe, layers)
        rounded, _ = oracle.run_stack(xe, layers, dtypes.BF16)
        fused, st = _run_stack_gpu(npas, torch, w, flag)
        plain, st0 = _run_stack_gpu(npas, torch, w, 0)
        assert st.num_launches() == launches and st0.num_launches() == len(layers)
        assert st.workspace_bytes(N) > 0
        n_f, e_f = helpers.check_stack_output(fused, rounded[-1], STACK_NORM_TOL)
        n_p, e_p = helpers.check_stack_output(plain, rounded[-1], STACK_NORM_TOL)
        print(f"  chained {name}: fused norm-wise {n_f:.3e} worst element {e_f:.3e}; unfused {n_p:.3e} / {e_p:.3e}", flush=True)
        again, _ = _run_stack_gpu(npas, torch, w, flag)
        np.testing.assert_array_equal(fused, again)


HS_CASES = [
    # hard-swish through every epilogue: name, N, H, W, C, F, KH, KW, stride, pad, Bf, Bc, rate, dtype, act, res, bias, variant, kernel
    (("hs_slab", 2, 11, 9, 24, 40, 3, 3, 1, 1, 8, 4, 2, dtypes.BF16, 3, True, True), None, "conv_slab_mfma"),
    (("hs_pointwise_ring", 13, 29, 27, 128, 136, 1, 1, 1, 0, 8, 4, 3, dtypes.BF16, 3, True, True), None, "pointwise_ring"),
    (("hs_pointwise_split", 3, 9, 11, 128, 136, 1, 1, 1, 0, 8, 4, 3, dtypes.BF16, 3, True, True), None, "conv_smallm_mfma"),
    (("hs_spatial", 3, 14, 14, 128, 64, 3, 3, 1, 1, 8, 4, 2, dtypes.BF16, 3, False, True), "spatial", "spatial_direct"),
    (("hs_spatial_f40_fp16", 2, 13, 11, 64, 40, 3, 3, 1, 1, 8, 4, 2, dtypes.F16, 3, True, False), "spatial", "spatial_direct"),
    (("hs_smallm", 1, 7, 7, 128, 72, 3, 3, 1, 1, 8, 4, 3, dtypes.BF16, 3, True, True), None, "conv_smallm_mfma"),
    (("hs_smallc", 2, 21, 23, 3, 32, 5, 5, 2, 2, 8, 3, 2, dtypes.BF16, 3, False, True), None, "conv_smallc_mfma"),
    (("hs_gather", 1, 8, 8, 20, 18, 3, 3, 1, 1, 6, 4, 2, dtypes.BF16, 3, False, True), None, "conv_gather_mfma"),
    (("hs_fp32", 2, 9, 9, 8, 12, 3, 3, 1, 1, 4, 4, 2, dtypes.F32, 3, True, True), None, None),
    # the compiled epilogue variants of the spatial kernels (activation kind x residual), partial filter blocks, stride 2
    (("epi_spatial_hs_res", 3, 14, 14, 128, 128, 3, 3, 1, 1, 8, 4, 2, dtypes.BF16, 3, True, True), "spatial", "spatial_direct"),
    (("epi_spatial_s2_relu_res", 2, 28, 28, 64, 128, 3, 3, 2, 1, 8, 4, 2, dtypes.BF16, 1, True, True), "spatial", "spatial_direct"),
    (("epi_spatial_relu6_res_fp16_f200", 2, 9, 9, 64, 200, 3, 3, 1, 1, 8, 4, 3, dtypes.F16, 2, True, False), "spatial", "spatial_direct"),
    (("epi_spatial_none_nores", 2, 12, 10, 64, 64, 3, 3, 1, 1, 8, 4, 2, dtypes.BF16, 0, False, True), "spatial", "spatial_direct"),
    (("epi_pointwise_hs_nores_partial", 2, 7, 9, 64, 72, 1, 1, 1, 0, 8, 4, 2, dtypes.BF16, 3, False, False), None, None),
]


@pytest.mark.parametrize("case,variant,kernel", HS_CASES, ids=[c[0][0] for c in HS_CASES])
def test_hard_swish_epilogues(npas, torch, case, variant, kernel, force_variant):
    if variant:
        force_variant(variant)
    _run_edge_case(npas, torch, case, expect_kernel=kernel)


def test_full_size_config4_sampled_images(npas, torch):
    print("config4 full size, images 0/17/31", flush=True)
    w = configs.config4()
    L = w.layers[0]
    p = pack_layer(npas, L, w.dtype)
    helpers.check_metadata(oracle, L, p, w.dtype)
    y = from_dev(run_layer_gpu(npas, torch, L, p, to_dev(w.x_store, torch), w.x_shape, w.dtype), w.dtype)
    y = y.reshape(helpers.out_shape(L, w.x_shape))
    for n in (0, 17, 31):
        ref = oracle.round_to(oracle.conv2d_masked(w.x_exact[n:n + 1], L.w_exact, L.mask, 1, 1), w.dtype)
        err = rel_err(y[n:n + 1], ref)
        print(f"  image {n} err={err:.3e}", flush=True)
        assert err <= 1e-2


def test_config5_batch128_sampled_images(npas, torch):
    """The 50-layer stack's layers in the launch configuration the per-layer report times (batch 128: big tiles,
    the streaming pointwise kernel, the direct-weights kernel at both strides, the stem kernel), each on a seeded input of its real shape, checked
    on three of the 128 images (a layer's output for one image depends on that image only)."""
    w = configs.config5(batch=128)
    shapes = {0: w.x_shape}
    for i, L in enumerate(w.layers):
        shapes[i + 1] = helpers.out_shape(L, shapes[L.src])
    want = {"stem7x7": "conv_smallc_mfma", "s0b0_c3": "pointwise_ring", "s1b0_sc": "pointwise_ring", "s1b1_c2": "spatial_direct",
            "s2b1_c3": "pointwise_ring", "s2b0_c2": "spatial_direct", "s3b1_c1": "pointwise_ring", "s3b1_c2": "spatial_direct",
            "s0b1_c2": "spatial_direct"}
    seen = set()
    for i, L in enumerate(w.layers):
        if L.name not in want:
            continue
        seen.add(L.name)
        in_shape, oshape = shapes[L.src], shapes[i + 1]
        N, H, W, C = in_shape
        print(f"config5 batch 128 layer {i} {L.name} in={in_shape}", flush=True)
        xs, xe = dtypes.quantize(prng.normal(500 + i, 1, int(np.prod(in_shape))).reshape(in_shape), w.dtype)
        rs = re = None
        if L.res >= 0:
            rs, re = dtypes.quantize(prng.normal(500 + i, 2, int(np.prod(oshape))).reshape(oshape), w.dtype)
        p = pack_layer(npas, L, w.dtype)
        assert npas.conv2d_kernel_name(p, N, H, W, L.stride, L.pad) == want[L.name]
        y = run_layer_gpu(npas, torch, L, p, to_dev(xs, torch), in_shape, w.dtype, None if rs is None else to_dev(rs, torch))
        got = from_dev(y, w.dtype).reshape(oshape)
        for n in (0, 77, 127):
            ref = oracle.round_to(oracle.conv2d_masked(xe[n:n + 1], L.w_exact, L.mask, L.stride, L.pad, None,
                                                       None if re is None else re[n:n + 1], L.act), w.dtype)
            err = rel_err(got[n:n + 1], ref)
            print(f"  image {n} err={err:.3e}", flush=True)
            assert err <= TOL[w.dtype]
        del xs, xe, rs, re, y, got
        torch.cuda.empty_cache()
    assert seen == set(want)


def test_pools(npas, torch):
    # C = 24 takes the 8-channel vector path for 16-bit storage, C = 5 the scalar one
    for dtype, C in ((dtypes.BF16, 24), (dtypes.F16, 24), (dtypes.BF16, 5), (dtypes.F32, 24)):
        xs, xe = dtypes.quantize(prng.normal(9, 1, 2 * 9 * 11 * C).reshape(2, 9, 11, C), dtype)
        x = to_dev(xs, torch)
        y = new_dev((2, 5, 6, C), dtype, torch)
        npas.maxpool3x3s2(x, y, 2, 9, 11, C, dtype)
        np.testing.assert_array_equal(from_dev(y, dtype).reshape(2, 5, 6, C), oracle.maxpool3x3s2(xe))
        z = new_dev((2, C), dtype, torch)
        npas.global_avgpool(x, z, 2, 9, 11, C, dtype)
        assert rel_err(from_dev(z, dtype).reshape(2, C), oracle.round_to(oracle.global_avgpool(xe), dtype)) <= TOL[dtype]


# Both forms of the vector kernel: fewer pixels than waves, one more than the waves' groups of loads, 64 vectors of four channels and one more, and above
# the numbers of waves (64 vectors each) from which one wave walks all pixels.
@pytest.mark.parametrize("N,H,W,C,dtype", [(3, 1, 1, 24, dtypes.BF16), (1, 1, 3, 260, dtypes.F16), (2, 1, 7, 256, dtypes.BF16), (1, 7, 7, 260, dtypes.F16),
                                           (3, 8, 8, 1028, dtypes.BF16), (513, 2, 2, 256, dtypes.BF16), (512, 2, 2, 256, dtypes.F16),
                                           (1025, 5, 5, 256, dtypes.BF16), (1024, 5, 5, 256, dtypes.BF16), (1030, 1, 1, 260, dtypes.F16)])
def test_global_average_pool_forms(npas, torch, N, H, W, C, dtype):
    print(f"average pool {N}x{H}x{W}x{C}", flush=True)
    xs, xe = dtypes.quantize(prng.normal(9, 2, N * H * W * C).reshape(N, H, W, C) + 1.0, dtype)
    y = new_dev((N, C), dtype, torch, fill=0x7FC1)
    npas.global_avgpool(to_dev(xs, torch), y, N, H, W, C, dtype)
    torch.cuda.synchronize()
    assert rel_err(from_dev(y, dtype).reshape(N, C), oracle.round_to(oracle.global_avgpool(xe), dtype)) <= TOL[dtype]
