"""GPU parity at the edges of the projection's and block GEMMs' tiles: row
counts around the first tile's 256 (128) output rows and the later ones' 253
(125), and d_model from one K-step of 64 up to past the ring's depth, where the
main loop runs its shortened prologue and tails.  A grid whose 128 x 128 tiles
fit the card at once takes those; more heads and layers force the 256 x 256
ones.  Bounds as in the other parity tests: every product rounds its operands
once to bf16, 5e-3 per slab."""
import pytest

import workloads as W
from gpu_harness import TOL_BF16, TOL_F32, check_pairs, log, run, upload
from test_gpu_group import _check_group, _run
from workloads.device import upload_group
from workloads.group import make_group

pytestmark = pytest.mark.gpu

LENGTHS = {125: [122, 3], 128: [128], 129: [127, 2], 253: [1, 252], 256: [256], 257: [255, 2], 509: [250, 3, 256],
           510: [253, 253, 4], 763: [1, 508, 254]}


def _check(rows, d_model, d, weights, k_heads, v_heads, layers):
    shape = W.Shape(d_model, k_heads, v_heads, d, d, weight_dtype=weights)
    wl = W.make_workload("tile", shape, LENGTHS[rows], n_layers=layers, seed=rows + d_model)
    log(f"tile edges: T={wl.t_total}, D={d_model}, d={d}, {weights}, {layers} layers")
    dev = upload(wl)
    run(dev)
    check_pairs(dev, [(li, b) for li in (0, layers - 1) for b in range(len(wl.seg_lens))], TOL_BF16)


@pytest.mark.parametrize("weights", [W.BF16, W.FP8])
@pytest.mark.parametrize("rows,d_model,d", [(125, 64, 128), (128, 128, 64), (129, 192, 32), (253, 256, 128),
                                            (257, 320, 64), (510, 384, 128)])
def test_projection_small_tile_edges(rows, d_model, d, weights):
    _check(rows, d_model, d, weights, 2, 4, 2)


@pytest.mark.parametrize("weights", [W.BF16, W.FP8])
@pytest.mark.parametrize("rows,d_model,d,k_heads,v_heads,layers",
                         [(256, 64, 128, 8, 48, 4), (257, 128, 64, 16, 96, 4), (509, 192, 32, 128, 128, 2),
                          (510, 256, 128, 8, 48, 2), (763, 320, 64, 16, 96, 2), (257, 384, 128, 8, 48, 4)])
def test_projection_big_tile_edges(rows, d_model, d, k_heads, v_heads, layers, weights):
    _check(rows, d_model, d, weights, k_heads, v_heads, layers)


def test_states_do_not_depend_on_the_tile_shape():
    """A segment replayed alone (small tiles) and inside a batch of big ones
    gives the same bits: the products accumulate along K in one order and the
    key norm's sum is one tree in both."""
    import torch
    shape = W.Shape(256, 8, 48, 128, 128)
    wl = W.make_workload("shape", shape, [100, 201, 300, 162], n_layers=2, seed=7)
    dev = upload(wl)
    run(dev)
    cu = wl.cu_seqlens
    for b in range(4):
        one = W.make_workload("one", shape, [wl.seg_lens[b]], n_layers=1, seed=7)
        one.layers[0] = wl.layers[0]
        part = upload(one)
        part.layers[0].anchors = dev.layers[0].anchors[cu[b]:cu[b + 1]].contiguous()
        run(part)
        assert torch.equal(part.layers[0].state_out[0], dev.layers[0].state_out[b]), b
        assert torch.equal(part.layers[0].tail_out[0], dev.layers[0].tail_out[b]), b


def _f32_shape(d_model, heads, d):
    return W.Shape(d_model, heads, heads, d, d, anchor_dtype=W.F32, weight_dtype=W.F32, conv_dtype=W.F32,
                   tail_dtype=W.F32)


# fp32 scan: lengths around its 64-row chunks, where two teams take turns at the
# state (none, one, an odd and an even number of chunks), and enough units for
# one team each.  With the many heads the conv takes its 64-row blocks, with the
# few 16-row ones; the tail's blocks ride behind both.
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("heads,layers,lens", [(2, 1, [1, 64, 65, 128, 129, 200]), (2, 1, [3, 0, 192]), (2, 2, [2]),
                                               (64, 1, [1, 64, 65, 128, 129, 200, 66])])
def test_f32_scan_and_conv_edges(heads, layers, lens, d):
    wl = W.make_workload("f32", _f32_shape(64, heads, d), lens, n_layers=layers, seed=d + heads)
    log(f"fp32 edges: {lens}, {heads} heads of {d}, {layers} layers")
    dev = upload(wl)
    run(dev)
    check_pairs(dev, [(li, b) for li in range(layers) for b in range(len(lens))], TOL_F32)


@pytest.mark.parametrize("rows,d_ff", [(256, 128), (257, 192 + 64), (510, 384)])
def test_block_gemm_tile_edges(rows, d_ff):
    shape = W.Shape(256, 2, 4, 64, 64)
    gw = make_group("tile", shape, LENGTHS[rows], n_layers=2, d_ff=d_ff, seed=rows)
    dg = upload_group(gw)
    _run(dg)
    log(f"block GEMM tile edges: T={gw.t_total}, d_ff={d_ff}: {_check_group(dg)}")
