"""CPU-side tests of the HIP library: it loads, exports what include/npas.h
declares, packs (host logic) bit-identically to the oracle's packer, rejects
illegal masks, and fails loudly instead of computing without a GPU."""
import ctypes
import os
import re
import shutil
import subprocess
import time

import numpy as np
import pytest

import oracle
import paper_2012_00596_amd as npas
from tests import helpers
from workloads import configs, dtypes, masks, prng

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "npas.h")).read()
    declared = set(re.findall(r"\b(npas_[a-z0-9_]+)\s*\(", header))
    declared -= {"npas_packed", "npas_stack"}
    assert declared == set(npas.binding.EXPORTS)
    L = npas.lib()
    for name in declared:
        assert hasattr(L, name), name


@pytest.mark.parametrize("builder,kw", [
    (configs.config1, {}),
    (configs.config2, dict(batch=1, HW=4)),
    (configs.config3, dict(batch=2)),
    (configs.config4, dict(batch=1, HW=4)),
    (configs.config5, dict(batch=1, HW=32, width=16, blocks=(1, 1, 1, 1))),
])
def test_packing_metadata_bit_exact_vs_oracle(builder, kw):
    w = builder(**kw)
    for L in w.layers:
        if L.kind not in ("conv", "fc"):
            continue
        p = helpers.pack_layer(npas, L, w.dtype)
        helpers.check_metadata(oracle, L, p, w.dtype)
        info = p.info()
        assert info["F"] == L.F and info["C"] == L.C and info["dtype"] == w.dtype


@pytest.mark.parametrize("dtype", [dtypes.F32, dtypes.BF16, dtypes.F16])
@pytest.mark.parametrize("F,C,k,Bf,Bc,rate", [(10, 7, 3, 4, 4, 2), (5, 3, 7, 8, 4, 5), (16, 16, 1, 1, 1, 3),
                                               (12, 8, 3, 12, 8, 2), (9, 40, 1, 16, 32, 5)])
def test_packing_edge_blocks_and_degenerate_sizes(dtype, F, C, k, Bf, Bc, rate):
    m = masks.block_punched_mask(F, C, k, k, Bf, Bc, rate, 31)
    store, exact = dtypes.quantize(prng.normal(5, 3, F * C * k * k).reshape(F, C, k, k), dtype)
    p = npas.pack_block_punched(store, m, Bf, Bc, dtype)
    L = configs.Layer("conv", "block_punched", C, F, k, k, 1, 0, Bf, Bc, rate, w_store=store, w_exact=exact, mask=m)
    helpers.check_metadata(oracle, L, p, dtype)
    # garbage under the mask must not leak into the compact form
    junk = store.copy()
    junk[m == 0] = 0x7FC0 if dtype != dtypes.F32 else np.nan
    e1, e2 = p.export(), npas.pack_block_punched(junk, m, Bf, Bc, dtype).export()
    for key in e1:
        np.testing.assert_array_equal(e1[key].view(np.uint8), e2[key].view(np.uint8))


def test_fc_rows_and_columns():
    OUT, IN = 40, 70
    m = masks.fc_block_mask(OUT, IN, 16, 32, 4, 9)
    m[3, :32] = 0            # a pruned row inside a block
    store, exact = dtypes.quantize(prng.normal(6, 3, OUT * IN).reshape(OUT, IN), dtypes.BF16)
    p = npas.pack_fc_block(store, m, 16, 32, dtypes.BF16)
    L = configs.Layer("fc", "fc_block", IN, OUT, 1, 1, 1, 0, 16, 32, 4, w_store=store.reshape(OUT, IN, 1, 1),
                      w_exact=exact.reshape(OUT, IN, 1, 1), mask=m.reshape(OUT, IN, 1, 1))
    helpers.check_metadata(oracle, L, p, dtypes.BF16)


def test_illegal_masks_are_rejected_not_repaired():
    F, C = 8, 8
    w = np.zeros((F, C, 3, 3), dtype=np.float32)
    m = masks.block_punched_mask(F, C, 3, 3, 4, 4, 2, 16)
    bad = m.copy()
    bad[1, 2, 1, 1] ^= 1
    with pytest.raises(npas.NpasError) as e:
        npas.pack_block_punched(w, bad, 4, 4, dtypes.F32)
    assert e.value.code == npas.E_MASK_NOT_BLOCK_UNIFORM and "filter 1" in str(e.value)
    bad = m.copy()
    bad[0, 0, 0, 0] = 3
    with pytest.raises(npas.NpasError) as e:
        npas.pack_block_punched(w, bad, 4, 4, dtypes.F32)
    assert e.value.code == npas.E_MASK_VALUE
    mf = masks.fc_block_mask(32, 64, 16, 32, 4, 17)
    hole = mf.copy()
    hole[5, int(np.flatnonzero(mf[5])[0])] = 0
    with pytest.raises(npas.NpasError) as e:
        npas.pack_fc_block(np.zeros((32, 64), np.float32), hole, 16, 32, dtypes.F32)
    assert e.value.code == npas.E_MASK_NOT_BLOCK_UNIFORM
    lib = masks.pattern_library(8, 5)
    mp, _ = masks.pattern_mask(6, 6, lib, 0.3, 18)
    badp = mp.copy()
    k = np.argwhere(mp.reshape(36, 9).sum(1) == 4)[0, 0]
    badp.reshape(36, 9)[k, 4] = 0
    with pytest.raises(npas.NpasError) as e:
        npas.pack_pattern(np.zeros((6, 6, 3, 3), np.float32), badp, lib, dtypes.F32)
    assert e.value.code == npas.E_MASK_NOT_IN_LIBRARY
    with pytest.raises(npas.NpasError) as e:
        npas.pack_block_punched(w, m, 4, 4, 7)
    assert e.value.code == npas.E_DTYPE
    with pytest.raises(npas.NpasError) as e:
        npas.pack_block_punched(w, m, 0, 4, dtypes.F32)
    assert e.value.code == npas.E_SHAPE
    h = ctypes.c_void_p()
    assert npas.lib().npas_pack_block_punched(None, None, 1, 1, 1, 1, 1, 1, 0, None, ctypes.byref(h)) == npas.E_NULL


def test_run_calls_validate_arguments_before_touching_the_gpu():
    w = np.ones((4, 4, 3, 3), dtype=np.float32)
    p = npas.pack_block_punched(w, np.ones_like(w, dtype=np.uint8), 2, 2, dtypes.F32)
    L = npas.lib()
    assert L.npas_conv2d_sparse(p.handle, None, None, 1, 4, 4, 1, 1, None, None, 0, None) == npas.E_NULL
    assert L.npas_conv2d_sparse(p.handle, 256, 256, 0, 4, 4, 1, 1, None, None, 0, None) == npas.E_SHAPE
    assert L.npas_conv2d_sparse(p.handle, 256, 256, 1, 1, 1, 1, 0, None, None, 0, None) == npas.E_SHAPE   # empty output
    assert L.npas_fc_sparse(p.handle, 256, 256, 1, None, 0, None) == npas.E_SHAPE                          # 3x3 is no FC
    assert L.npas_maxpool3x3s2(None, None, 1, 4, 4, 4, 0, None) == npas.E_NULL
    assert L.npas_global_avgpool(256, 256, 1, 4, 4, 4, 9, None) == npas.E_DTYPE
    if not p.info()["device_ready"]:
        # no GPU here: the product path must fail loudly, never compute on the CPU
        assert L.npas_conv2d_sparse(p.handle, 256, 256, 1, 4, 4, 1, 1, None, None, 0, None) == npas.E_HIP
        assert "no device copy" in npas.last_error()


def test_stack_wiring_checks_and_workspace():
    w = configs.config5(batch=1, HW=32, width=16, blocks=(1, 1, 1, 1))
    packed = [helpers.pack_layer(npas, L, w.dtype) if L.kind in ("conv", "fc") else None for L in w.layers]
    descs = helpers.stack_descs(npas, w.layers, packed)
    st = npas.Stack(descs, 32, 32)
    assert st.num_launches() <= len(w.layers)
    ws1, ws4 = st.workspace_bytes(1), st.workspace_bytes(4)
    assert 0 < ws1 and ws1 % 256 == 0 and 3 * ws1 < ws4 <= 4 * ws1 + 256 * len(descs)
    # the workspace must at least hold the largest layer's live set: stem output + pooled output
    assert ws1 >= (16 * 16 * 16 + 8 * 8 * 16) * 2
    bad = [dict(d) for d in descs]
    bad[3]["src"] = 7                        # reads a tensor that does not exist yet
    with pytest.raises(npas.NpasError) as e:
        npas.Stack(bad, 32, 32)
    assert e.value.code == npas.E_SHAPE
    bad = [dict(d) for d in descs]
    bad[2]["res"] = 1                        # residual of the wrong shape
    with pytest.raises(npas.NpasError):
        npas.Stack(bad, 32, 32)
    assert npas.lib().npas_run_stack(st.handle, 256, 256, 1, None, 0, None) == npas.E_WORKSPACE


def _bp_layer(C, F, k, seed, rate=3):
    m = masks.block_punched_mask(F, C, k, k, 8, 4 if C % 4 == 0 else C, rate, seed)
    store, _ = dtypes.quantize(prng.normal(seed, 1, F * C * k * k, 0.1).reshape(F, C, k, k), dtypes.BF16)
    return npas.pack_block_punched(store, m, 8, 4 if C % 4 == 0 else C, dtypes.BF16)


def test_kernel_choice_follows_layer_and_launch_shape():
    """Host logic only: which kernel a layer gets depends on its shape and on how many tiles the launch has."""
    name = npas.conv2d_kernel_name
    p = _bp_layer(64, 64, 3, 41)                       # k x k on whole 64-channel chunks
    assert name(p, 128, 56, 56, 1, 1) == "spatial_direct"
    assert name(p, 8, 56, 56, 1, 1) == "spatial_direct"          # more than one round of the split reduction
    assert name(p, 1, 56, 56, 1, 1) == "conv_smallm_mfma"        # little work in all: reduction split over the waves
    p = _bp_layer(128, 128, 3, 42)
    assert name(p, 128, 28, 28, 1, 1) == "spatial_direct"
    assert name(p, 8, 28, 28, 1, 1) == "spatial_direct"
    assert name(p, 128, 56, 56, 2, 1) == "spatial_direct"        # stride 2, with any padding
    assert name(p, 128, 56, 56, 2, 0) == "spatial_direct"
    assert name(p, 128, 56, 56, 3, 1) == "conv_slab_mfma"        # ... but no more
    assert name(p, 1, 28, 28, 1, 1) == "conv_smallm_mfma"
    p = _bp_layer(64, 256, 1, 43)
    assert name(p, 128, 56, 56, 1, 0) == "pointwise_ring"
    assert name(p, 1, 14, 14, 1, 0) == "conv_smallm_mfma"        # up to 256 output pixels
    assert name(p, 1, 28, 28, 1, 0) == "conv_smallm_mfma"        # 4 x 49 workgroups: still one round
    assert name(p, 1, 56, 56, 1, 0) == "pointwise_ring"
    p = _bp_layer(1024, 256, 1, 46)
    assert name(p, 8, 7, 7, 1, 0) == "conv_smallm_mfma"          # long reduction, 7 x 16 workgroups: one round
    assert name(p, 32, 14, 14, 1, 0) == "pointwise_ring"
    p = _bp_layer(3, 64, 7, 44)
    assert name(p, 2, 224, 224, 2, 3) == "conv_smallc_mfma"      # fewer than 8 input channels
    p = _bp_layer(24, 144, 1, 45, rate=4)
    assert name(p, 64, 56, 56, 1, 0) == "conv_slab_mfma"         # channels not a multiple of 64


def test_device_kernel_tells_the_stem_kernels_apart():
    """By kernel rows: stride 2, at most 3 channels, rows of whole 4-byte words; everything else stays with the whole-reduction kernel."""
    p = _bp_layer(3, 64, 7, 44)
    assert npas.device_kernel(p, 2, 224, 224, 2, 3) == "conv_smallc_rows_kernel"
    assert npas.device_kernel(p, 128, 224, 224, 2, 0) == "conv_smallc_rows_kernel"
    for W, stride in ((225, 2), (224, 1)):
        assert npas.device_kernel(p, 2, 224, W, stride, 3) == "conv_smallc_mfma_kernel"
    assert npas.device_kernel(_bp_layer(4, 64, 5, 47), 2, 64, 64, 2, 2) == "conv_smallc_mfma_kernel"


def test_device_kernel_tells_the_forms_of_the_slab_route_apart():
    """1x1 layers on at most 320 channels, no multiple of 64, take the flat kernel in either list format; with padding, wider layers
    and k x k layers the kernel of their format."""
    name, kernel = npas.conv2d_kernel_name, npas.device_kernel
    p = _bp_layer(24, 144, 1, 45, rate=4)
    assert (name(p, 64, 56, 56, 1, 0), kernel(p, 64, 56, 56, 1, 0)) == ("conv_slab_mfma", "pointwise_stream_kernel")
    assert kernel(p, 64, 56, 56, 1, 1) == "conv_slab_mfma_kernel"
    p = _bp_layer(144, 64, 1, 45, rate=20)
    assert kernel(p, 64, 56, 56, 1, 0) == "pointwise_stream_kernel" and kernel(p, 64, 56, 56, 1, 1) == "conv_gather_mfma_kernel"
    p = _bp_layer(328, 64, 1, 45, rate=2)
    assert kernel(p, 64, 56, 56, 1, 0) == "conv_slab_mfma_kernel"
    p = _bp_layer(64, 64, 3, 41)
    assert kernel(p, 8, 56, 56, 1, 1) == "spatial_direct_kernel" and kernel(p, 1, 56, 56, 1, 1) == "conv_smallm_mfma_kernel"
    assert kernel(p, 64, 56, 56, 3, 1) == "conv_slab_mfma_kernel"


# ---- workspace placement of fused stacks (host logic: works without a GPU) -----------------------------------

def _pw(seed, idx, C, F, act, src, res=-1):
    return configs._bp_conv(seed, idx, C, F, 1, 1, 0, 8, 8, 2, 0.2, dtypes.BF16, act, src, res, name=f"pw{idx}")


def _dw(seed, idx, C, src, stride=1):
    ws, we = configs._tensor(seed, 150 + idx, (C, 3, 3), 0.3, dtypes.BF16)
    return configs.Layer("dwconv", "", C, C, 3, 3, stride, 1, 1, 1, 1.0, configs.ACT_RELU6, src, -1, ws, we, name=f"dw{idx}")


def _stack(layers, HW, flags):
    packed = [helpers.pack_layer(npas, L, dtypes.BF16) if L.kind in ("conv", "fc", "dwconv") else None for L in layers]
    return npas.Stack(helpers.stack_descs(npas, layers, packed), HW, HW, flags)


def _assert_placement_is_safe(st, N):
    """No launch may write over bytes that it, or a later launch, still has to read: tensors whose lifetimes
    (launch that writes them .. last launch that reads them) intersect must not share workspace bytes."""
    rows = st.describe(N)
    assert len(rows) == st.num_launches(N) <= st.num_launches()
    assert [r["first"] for r in rows] == [0] + [r["last"] + 1 for r in rows[:-1]]     # every layer in one launch
    born, last_read, where = {}, {}, {}
    for r, row in enumerate(rows):
        for t in range(row["first"] + 1, row["last"] + 2):      # also the sum that a launch stores in front of its last layer
            born[t] = r
        for key in ("src", "res"):
            t = row[key]
            if t >= 0:
                last_read[t] = r
                if row["off_" + key] >= 0:
                    assert where.setdefault(t, (row["off_" + key], row["bytes_" + key])) == (row["off_" + key], row["bytes_" + key])
        t = row["out"]
        assert t == row["last"] + 1
        if row["off_out"] >= 0:
            where[t] = (row["off_out"], row["bytes_out"])
    for off, size in where.values():
        assert off % 256 == 0 and off + size <= st.workspace_bytes(N)
    ts = sorted(where)
    for i, a in enumerate(ts):
        for b in ts[i + 1:]:
            la, lb = (born.get(a, -1), last_read.get(a, born.get(a, -1))), (born.get(b, -1), last_read.get(b, born.get(b, -1)))
            if la[0] <= lb[1] and lb[0] <= la[1]:               # alive during a common launch
                (oa, sa), (ob, sb) = where[a], where[b]
                assert oa + sa <= ob or ob + sb <= oa, f"tensors {a} and {b} overlap in the workspace while both are alive"
    return rows


def test_fused_launches_never_write_over_their_own_inputs():
    A = configs
    # three fused 1x1 pairs in a row, of unequal widths (before the fix tensor 4 was placed over tensor 2)
    chain = [_pw(1, 0, 16, 48, A.ACT_RELU6, 0), _pw(1, 1, 48, 24, A.ACT_NONE, 1),
             _pw(1, 2, 24, 64, A.ACT_RELU6, 2), _pw(1, 3, 64, 8, A.ACT_NONE, 3),
             _pw(1, 4, 8, 40, A.ACT_RELU6, 4), _pw(1, 5, 40, 32, A.ACT_NONE, 5)]
    st = _stack(chain, 12, npas.STACK_FUSE_POINTWISE)
    rows = _assert_placement_is_safe(st, 3)
    assert [(r["first"], r["last"]) for r in rows] == [(0, 1), (2, 3), (4, 5)]
    assert rows[1]["off_src"] >= 0 and rows[1]["off_out"] >= 0
    # two inverted-residual blocks without residual, then a plain layer
    blocks = [_pw(2, 0, 16, 64, A.ACT_RELU6, 0), _dw(2, 1, 64, 1), _pw(2, 2, 64, 24, A.ACT_NONE, 2),
              _pw(2, 3, 24, 96, A.ACT_RELU6, 3), _dw(2, 4, 96, 4), _pw(2, 5, 96, 32, A.ACT_NONE, 5),
              _pw(2, 6, 32, 16, A.ACT_RELU, 6)]
    st = _stack(blocks, 10, npas.STACK_FUSE_INVERTED_RESIDUAL)
    rows = _assert_placement_is_safe(st, 2)
    assert [(r["first"], r["last"]) for r in rows] == [(0, 2), (3, 5), (6, 6)]
    # with a residual the fused block reads its input again at its last layer
    res = [_pw(3, 0, 24, 24, A.ACT_RELU, 0), _pw(3, 1, 24, 96, A.ACT_RELU6, 1), _dw(3, 2, 96, 2),
           _pw(3, 3, 96, 24, A.ACT_NONE, 3, res=1), _pw(3, 4, 24, 16, A.ACT_NONE, 4)]
    st = _stack(res, 9, npas.STACK_FUSE_INVERTED_RESIDUAL)
    rows = _assert_placement_is_safe(st, 2)
    assert (rows[1]["first"], rows[1]["last"], rows[1]["src"], rows[1]["res"]) == (1, 3, 1, 1)
    # the same stacks without fusion, and a residual stack with every fusion allowed
    for layers, hw in ((chain, 12), (blocks, 10), (res, 9)):
        _assert_placement_is_safe(_stack(layers, hw, 0), 2)
    w = configs.config5(batch=1, HW=32, width=16, blocks=(1, 2, 1, 1))
    for flags in (0, npas.STACK_FUSE_POINTWISE | npas.STACK_FUSE_INVERTED_RESIDUAL | npas.STACK_FUSE_CONV_MAXPOOL):
        st = _stack(w.layers, 32, flags)
        rows = _assert_placement_is_safe(st, 3)
        assert rows[-1]["off_out"] == -2 and rows[0]["off_src"] == -1


@pytest.mark.parametrize("N,HW,tails,joined", [(1, 64, 0, 4), (3, 96, 0, 4), (8, 224, 2, 3), (7, 224, 1, 3)])
def test_runs_of_pointwise_layers_never_write_over_their_inputs(N, HW, tails, joined):
    """A projection, the layer that adds it and the next layer may run as one launch: what the first two read is still there when the last one
    writes, the workspace is no larger than without, and the launches listed are those that are made."""
    w = configs.config5(batch=1, HW=32, width=64, blocks=(2, 1, 1, 1))
    plain, st = _stack(w.layers, HW, 0), _stack(w.layers, HW, npas.STACK_FUSE_POINTWISE)
    assert st.workspace_bytes(N) <= plain.workspace_bytes(N)
    rows, names = _assert_placement_is_safe(st, N), [L.name for L in w.layers]
    assert [(r["first"], r["last"]) for r in _assert_placement_is_safe(plain, N)] == [(i, i) for i in range(len(names))]
    runs = [[names[i] for i in range(r["first"], r["last"] + 1)] for r in rows if r["last"] > r["first"]]
    joins = [[f"s{s}b0_sc", f"s{s}b0_c3"] for s in range(joined)]    # (of 7 and 8 images the last stage's two layers take different kernels)
    if tails:
        joins[0].append("s0b1_c1")
    if tails == 2:                          # 128 filters: from 24576 pixels on
        joins.insert(1, ["s0b1_c3", "s1b0_c1"])
    assert runs == joins
    for r in rows:
        if r["first"] in [names.index(j[0]) for j in joins if j[0].endswith("_sc")]:
            add, proj = w.layers[r["first"] + 1], w.layers[r["first"]]
            assert (r["src"], r["res"]) == (add.src, proj.src)


def test_benchmark_floor_counts_what_the_launches_move():
    """bench.stack_floor_us: layer by layer without fusion; a projection inside the layer that adds it moves no bytes, a sum handed to the next layer is
    written and not read again."""
    import bench
    w = configs.config5(batch=1, HW=32, width=64, blocks=(2, 1, 1, 1))
    w.x_shape = (8, 224, 224, 3)
    packed = [helpers.pack_layer(npas, L, dtypes.BF16) if L.kind in ("conv", "fc") else None for L in w.layers]
    rows = bench.layer_costs(w, packed, helpers)
    descs, names, px = helpers.stack_descs(npas, w.layers, packed), [L.name for L in w.layers], 8 * 56 * 56
    plain = npas.Stack(descs, 224, 224, 0).describe(8)
    assert bench.stack_floor_us(rows, plain) == pytest.approx(sum(r["floor_us"] for r in rows))
    launches = npas.Stack(descs, 224, 224, npas.STACK_FUSE_POINTWISE).describe(8)
    for first, last, channels in (("s0b0_sc", "s0b1_c1", 64 + 64 + 256 + 64), ("s0b1_c3", "s1b0_c1", 64 + 256 + 256 + 128)):
        span = range(names.index(first), names.index(last) + 1)
        l = [l for l in launches if (l["first"], l["last"]) == (span[0], span[-1])]
        us = 2 * px * channels + sum(rows[i]["wbytes"] for i in span)
        assert bench.stack_floor_us(rows, l) == pytest.approx(us / (bench.HBM_PEAK_GBS * 1e3))


def test_a_layer_joins_one_fused_launch_only():
    """A 1x1 layer in front of a fused inverted-residual block must not swallow the block's first layer as the
    second half of a fused pair (the block would then never run)."""
    A = configs
    layers = [_pw(4, 0, 16, 24, A.ACT_RELU6, 0),
              _pw(4, 1, 24, 32, A.ACT_RELU6, 1), _dw(4, 2, 32, 2), _pw(4, 3, 32, 16, A.ACT_NONE, 3)]
    st = _stack(layers, 8, npas.STACK_FUSE_POINTWISE | npas.STACK_FUSE_INVERTED_RESIDUAL)
    rows = _assert_placement_is_safe(st, 2)
    assert [(r["first"], r["last"]) for r in rows] == [(0, 0), (1, 3)]
    assert {r["out"] for r in rows} == {1, 4}


def test_device_functions_have_names_of_their_own():
    """A profile or device_kernel() names a kernel: no two sources define the same one, and each name the dispatch gives is defined."""
    defined = []
    for src in npas.binding.SOURCES:
        text = open(os.path.join(npas.binding._CSRC, src)).read()
        defined += set(re.findall(r"__global__[^;{]*?\b(\w+_kernel)\(", text))
    assert len(defined) == len(set(defined)), sorted(n for n in defined if defined.count(n) > 1)
    api = open(os.path.join(npas.binding._CSRC, "api.cpp")).read()
    assert set(re.findall(r'"(\w+_kernel)"', api)) <= set(defined)


def test_switches_are_read_once_and_can_be_replaced():
    p = _bp_layer(128, 128, 3, 42)
    assert npas.conv2d_kernel_name(p, 2, 14, 14, 1, 1) == "conv_smallm_mfma"
    npas.set_switches("spatial")
    try:
        assert npas.conv2d_kernel_name(p, 2, 14, 14, 1, 1) == "spatial_direct"
    finally:
        npas.set_switches(None)
    assert npas.conv2d_kernel_name(p, 2, 14, 14, 1, 1) == "conv_smallm_mfma"


def test_direct_weights_kernel_is_planned_within_its_limits():
    """Launches beyond 2^24 input pixels take it too (byte offsets are 32-bit, tensors below 4 GiB); a patch of a 64-channel chunk has to fit in LDS
    twice, so the largest kernels go elsewhere, and strides beyond 2 do."""
    p = _bp_layer(64, 128, 3, 43)
    assert 42700 * 28 * 28 * 64 <= 2 ** 31 - 1 and 42700 * 28 * 28 >= 1 << 24
    for N, pad in ((128, 1), (42700, 0)):
        layout, tile, items = npas.direct_plan(p, N, 28, 28, 1, pad)
        Ho = 26 + 2 * pad
        assert layout[0] * layout[1] * layout[2] == 4 and np.prod(tile) <= 16 * layout[3] * layout[0]
        assert items == -(-N // tile[0]) * -(-Ho // tile[1]) * -(-Ho // tile[2]) * (2 // layout[1])
    with pytest.raises(npas.NpasError):
        npas.direct_plan(p, 128, 56, 56, 3, 1)
    npas.set_switches("spatial")
    try:
        assert npas.conv2d_kernel_name(_bp_layer(64, 8, 23, 44), 64, 56, 56, 1, 11) == "spatial_direct"
        assert npas.conv2d_kernel_name(_bp_layer(64, 8, 25, 44), 64, 56, 56, 1, 12) != "spatial_direct"   # one pixel's patch: 79 KB
    finally:
        npas.set_switches(None)


def test_planning_a_new_shape_is_quick():
    """A batch size or map that a program has not run before is planned in its first call, on the caller's time: 40-70 us here (400-700 without
    passing over sizes that cannot win)."""
    p = _bp_layer(128, 128, 3, 45)
    us = []
    for N in range(33, 97):
        t = time.perf_counter()
        npas.conv2d_kernel_name(p, N, 28, 28, 1, 1)
        us.append((time.perf_counter() - t) * 1e6)
    assert sorted(us)[len(us) // 2] < 250


def test_a_stem_layer_is_planned_within_each_call():
    """The bands of the kernel by rows are chosen in every run call: 2.5 us for 16384 rows (23 with every number of bands looked at)."""
    p, best = _bp_layer(3, 64, 7, 44), 1.0
    for _ in range(300):
        t = time.perf_counter()
        npas.device_kernel(p, 1, 16384, 64, 2, 3)
        best = min(best, time.perf_counter() - t)
    assert best < 12e-6


def test_run_calls_marshal_like_the_c_abi():
    """The Python run calls: tensors, addresses and None as pointers, integers of any kind as sizes; library errors come back with
    their code, wrong types are refused before the library is called."""
    torch = pytest.importorskip("torch")
    p = _bp_layer(64, 64, 1, 47)
    x = torch.zeros((1, 8, 8, 64), dtype=torch.bfloat16)
    # the library's own checks, in the order of its arguments: a missing output, an empty output, an unknown activation
    for args, code in (((p, x, None, 1, 8, 8, 1, 0), npas.E_NULL), ((p, x, x, 1, np.int64(0), 8, 1, 0), npas.E_SHAPE),
                       ((p, 256, 256, 1, 0, 0, 1, 0), npas.E_SHAPE)):
        with pytest.raises(npas.NpasError) as e:
            npas.conv2d_sparse(*args)
        assert e.value.code == code and "libnpas error" in str(e.value)
    with pytest.raises(npas.NpasError) as e:
        npas.fc_sparse(p, x, x, B=-1, bias=None, act=npas.ACT_RELU)
    assert e.value.code == npas.E_SHAPE
    with pytest.raises(npas.NpasError) as e:
        npas.depthwise3x3(p, x, x, 1, 8, 8, stride=1)          # not a depthwise handle
    assert e.value.code == npas.E_SHAPE
    with pytest.raises(AssertionError):
        npas.conv2d_sparse(p, x.permute(0, 3, 1, 2), x, 1, 8, 8, 1, 0)
    with pytest.raises(TypeError):
        npas.conv2d_sparse(p, x, x, 1.0, 8, 8, 1, 0)
    with pytest.raises(AttributeError):
        npas.conv2d_sparse(p, "x", x, 1, 8, 8, 1, 0)
    with pytest.raises(AttributeError):
        npas.fc_sparse(None, x, x, 1)


def test_run_calls_take_ctypes_values_and_stream_objects():
    """What ctypes accepts as a stream or a size, the run calls accept: a c_void_p, an object with `_as_parameter_` (torch's
    stream objects), a c_int; a tensor is no stream."""
    torch = pytest.importorskip("torch")
    p, x = _bp_layer(64, 64, 1, 48), torch.zeros(64, dtype=torch.bfloat16)
    dw = npas.pack_depthwise3x3(np.zeros((8, 3, 3), np.uint16), dtypes.BF16)
    st = npas.Stack(helpers.stack_descs(npas, [_pw(6, 0, 16, 16, configs.ACT_NONE, 0)],
                                        [helpers.pack_layer(npas, _pw(6, 0, 16, 16, configs.ACT_NONE, 0), dtypes.BF16)]), 4, 4)

    class Stream:
        def __init__(self, value):
            self._as_parameter_ = value

    for s in (ctypes.c_void_p(), ctypes.c_void_p(64), Stream(ctypes.c_void_p(64)), Stream(0), np.int64(0), None, 0):
        N = ctypes.c_int(0) if not isinstance(s, np.int64) else 0    # refused by the library, on its own shape check
        calls = [lambda: npas.conv2d_sparse(p, x, x, N, 1, 1, 1, 0, stream=s), lambda: npas.fc_sparse(p, x, x, N, stream=s),
                 lambda: npas.depthwise3x3(dw, x, x, N, 1, 1, 1, stream=s), lambda: st.run(x, x, N, None, 0, s)]
        for call in calls:
            if isinstance(s, np.int64):                                  # ctypes takes no NumPy number as an address
                with pytest.raises(ctypes.ArgumentError):
                    call()
                continue
            with pytest.raises(npas.NpasError) as e:
                call()
            assert e.value.code == npas.E_SHAPE
    for s in (x, 1.5, object()):
        with pytest.raises(ctypes.ArgumentError):
            npas.conv2d_sparse(p, x, x, 0, 1, 1, 1, 0, stream=s)
        with pytest.raises(ctypes.ArgumentError):
            st.run(x, x, 0, None, 0, s)


@pytest.mark.parametrize("C,F,rate,B,dense", [(1280, 1000, 2, 256, True), (1280, 1000, 5, 256, False), (2048, 1000, 5, 64, True),
                                              (256, 1000, 3, 64, False), (256, 1000, 3, 128, True), (2048, 1000, 3, 512, False),
                                              (2048, 1000, 2, 512, True), (1280, 4096, 5, 128, False), (4096, 100, 5, 512, False),
                                              (4096, 1000, 5, 512, True)])
def test_fc_layers_take_their_lists_or_the_dense_images(C, F, rate, B, dense):
    """The lists of an FC layer or its dense images: the shapes on both sides of each line of the rule (host logic; the times
    on both sides, and where the lines no longer lie right, stand at the rule)."""
    m = masks.fc_block_mask(F, C, 16, 32, rate, 49)
    p = npas.pack_fc_block(np.zeros((F, C), np.uint16), m, 16, 32, dtypes.BF16)
    assert npas.conv2d_kernel_name(p, B, 1, 1, 1, 0) == ("conv_smallm_mfma" if dense else "fc_gather_mfma")


@pytest.mark.parametrize("C,F,N,HW,kernel", [(256, 256, 64, 7, "spatial_direct"), (256, 256, 16, 14, "spatial_direct"), (320, 320, 64, 7, "spatial_direct"),
                                             (512, 512, 32, 7, "spatial_direct"), (256, 256, 16, 7, "conv_smallm_mfma")])
def test_low_density_3x3_layers_take_the_kernels_of_the_denser_ones(C, F, N, HW, kernel):
    """3x3 layers at 10x in the gather format: the split-reduction kernel in one round of workgroups, the direct-weights kernel beyond, as at other
    densities above an eighth (host logic; the times stand at the rule)."""
    p = _bp_layer(C, F, 3, 50, rate=10)
    assert npas.conv2d_kernel_name(p, N, HW, HW, 1, 1) == kernel


def _sgprs(text):
    return {n for a, b, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text) for n in (range(int(a), int(b) + 1) if a else (int(one),))}


def test_scalar_operands_of_vector_memory_instructions_keep_their_wait_states(tmp_path):
    """The ISA's manually inserted wait states around vector memory instructions, in every kernel of the built library: one between a scalar write of M0
    and a load to LDS, five between a vector instruction's write of a scalar register and a vector memory instruction that reads it.  The
    compiler keeps them for its own instructions only, not within or around inline assembly."""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    shutil.copy(npas.binding._LIB, tmp_path)
    subprocess.run([objdump, "--offloading", "libnpas.so"], cwd=tmp_path, check=True, capture_output=True)
    loads = 0
    for code in sorted(tmp_path.glob("*gfx950")):
        asm = subprocess.run([objdump, "-d", "--no-show-raw-insn", code], check=True, capture_output=True, text=True).stdout
        kernel, before = "", []  # (op, operands, wait states it stands for)
        for line in asm.splitlines():
            label = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if label:
                kernel, before = label.group(1), []
                continue
            op, _, args = line.split("//")[0].strip().partition(" ")
            if not op:
                continue
            if re.match(r"(buffer|global|flat|scratch)_", op):
                if op.startswith("global_load_lds") or (op.startswith("buffer_load") and re.search(r"\blds\b", args)):
                    loads += 1
                    assert not (before and before[-1][0].startswith("s_") and before[-1][1].split(",")[0].strip() == "m0"), (kernel, before[-3:], line)
                read, states = _sgprs(args), 0
                for o, a, n in reversed(before[-5:]):
                    if states >= 5:
                        break
                    if o.startswith("v_"):
                        written = a.split(",")[:2 if re.match(r"v_(add|sub|subrev)c?_co|v_mad_[ui]64|v_div_scale", o) else 1]
                        assert not _sgprs(",".join(written)) & read, (kernel, before[-6:], line)
                    states += n
            before = before[-7:] + [(op, args, int(args, 0) + 1 if op == "s_nop" else 1)]
    assert loads > 500  # (direct loads are in the library, and the scan has seen them)
