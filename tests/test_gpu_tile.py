"""GPU parity at the edges of the projection's and block GEMMs' tiles: row
counts around the first tile's 256 (128) output rows and the later ones' 253
(125), and d_model from one K-step of 64 up to past the ring's depth, where the
main loop runs its shortened prologue and tails.  A grid whose 128 x 128 tiles
fit the card at once takes those; more heads and layers force the 256 x 256
ones, and each case asserts the tile it is meant for from the rule as it stands
in the source.  Bounds as in the other parity tests: every product rounds its
operands once to bf16, 5e-3 per slab."""
import os
import re

import pytest
import torch

import workloads as W
from gpu_harness import TOL_BF16, TOL_F32, check_pairs, log, run, upload
from test_gpu_group import _check_group, _run
from workloads.device import upload_group
from workloads.group import make_group

pytestmark = pytest.mark.gpu

LENGTHS = {125: [122, 3], 128: [128], 129: [127, 2], 253: [1, 252], 256: [256], 257: [255, 2], 509: [250, 3, 256],
           510: [253, 253, 4], 763: [1, 508, 254]}
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_33477_amd", "csrc")


def _takes_small_tiles(shape, rows, layers):
    """Whether a call's first projection launch (up to 4 layers) takes the 128
    x 128 tiles: the condition of proj_conv_kernel.hpp's run(), read from it."""
    with open(os.path.join(CSRC, "proj_conv_kernel.hpp")) as f:
        src = f.read()
    halo = int(re.search(r"constexpr int HALO = (\d+);", src).group(1))
    rule = re.search(r"if \((.*)\)\s*return run_tile<TileSmall", src).group(1)
    rect = shape.d_k != shape.d_v
    cols = (shape.n_k_heads * (128 if rect else shape.d_k) + shape.n_v_heads * (shape.d_v + 2))

    def tiles(edge):
        tm = 1 + -(-max(rows - edge, 0) // (edge - halo))
        return min(layers, 4) * tm * -(-cols // edge)

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    names = {"small": tiles(128), "big": tiles(256), "cus": cus, "rounds": -(-tiles(256) // cus)}
    return bool(eval(rule.replace("||", " or ").replace("&&", " and "), {"__builtins__": {}}, names))


def _check(rows, d_model, d, weights, k_heads, v_heads, layers, small, lens=None, slots=None, with_q=True, **kw):
    dk, dv = d if isinstance(d, tuple) else (d, d)
    shape = W.Shape(d_model, k_heads, v_heads, dk, dv, weight_dtype=weights, **kw)
    wl = W.make_workload("tile", shape, lens or LENGTHS[rows], n_layers=layers, seed=rows + d_model, slot_ids=slots,
                         n_slots=slots and len(slots))
    assert wl.t_total == rows and _takes_small_tiles(shape, rows, layers) == small
    log(f"tile edges: T={wl.t_total}, D={d_model}, d={d}, {weights}, {layers} layers, {kw}")
    dev = upload(wl, with_q=with_q)
    run(dev)
    live = [b for b, s in enumerate(wl.slot_ids) if s >= 0]
    check_pairs(dev, [(li, b) for li in (0, layers - 1) for b in live if wl.seg_lens[b]], TOL_BF16)
    for ns in dev.layers:
        for b in live:
            if wl.seg_lens[b] == 0:
                assert torch.all(ns.state_out[wl.slot_ids[b]] == 0) and torch.all(ns.tail_out[wl.slot_ids[b]] == 0)
        for slot in set(range(wl.n_slots)) - set(wl.slot_ids):
            assert torch.all(torch.isnan(ns.state_out[slot])) and torch.all(torch.isnan(ns.tail_out[slot]))


@pytest.mark.parametrize("weights", [W.BF16, W.FP8])
@pytest.mark.parametrize("rows,d_model,d", [(125, 64, 128), (128, 128, 64), (129, 192, 32), (253, 256, 128),
                                            (257, 320, 64), (510, 384, 128)])
def test_projection_small_tile_edges(rows, d_model, d, weights):
    _check(rows, d_model, d, weights, 2, 4, 2, small=True)


@pytest.mark.parametrize("weights", [W.BF16, W.FP8])
@pytest.mark.parametrize("rows,d_model,d,k_heads,v_heads,layers",
                         [(256, 64, 128, 8, 48, 4), (257, 128, 64, 16, 96, 4), (509, 192, 32, 128, 128, 2),
                          (510, 256, 128, 8, 48, 2), (763, 320, 64, 16, 96, 2), (257, 384, 128, 8, 48, 4)])
def test_projection_big_tile_edges(rows, d_model, d, k_heads, v_heads, layers, weights):
    _check(rows, d_model, d, weights, k_heads, v_heads, layers, small=False)


# 96 x 192 heads: few take the small tiles, OLMo-Hybrid's 30 the big ones
@pytest.mark.parametrize("weights", [W.BF16, W.FP8])
@pytest.mark.parametrize("rows,d_model,heads,layers", [(128, 64, 2, 2), (253, 128, 2, 2), (256, 64, 30, 4),
                                                       (257, 128, 30, 3), (509, 64, 30, 2), (763, 192, 30, 1)])
def test_projection_rect_head_edges(rows, d_model, heads, layers, weights):
    _check(rows, d_model, (96, 192), weights, heads, heads, layers, small=heads == 2)


# The big tile's masked rows and its three ways to load the taps: conv widths
# below 4, fp32 taps and tails, a sentinel and an empty segment, no q channels.
@pytest.mark.parametrize("weights,d,k_heads,v_heads,kw", [
    (W.BF16, 128, 8, 48, dict(conv_width=3)),
    (W.FP8, 128, 8, 48, dict(conv_width=2, with_q=False)),
    (W.BF16, 128, 8, 48, dict(conv_dtype=W.F32, tail_dtype=W.F32)),
    (W.FP8, 64, 16, 96, dict(conv_dtype=W.F32)),
    (W.BF16, 32, 128, 128, dict(conv_width=3, conv_dtype=W.F32, with_q=False)),
    (W.BF16, (96, 192), 30, 30, dict(conv_width=2, tail_dtype=W.F32)),
    (W.FP8, (96, 192), 30, 30, dict(conv_dtype=W.F32))])
def test_projection_big_tile_forms(weights, d, k_heads, v_heads, kw):
    _check(510, 128, d, weights, k_heads, v_heads, 2, small=False, lens=[200, 0, 250, 2, 58],
           slots=[3, 1, -1, 4, 0], **kw)


@pytest.mark.parametrize("weights,d,k_heads,v_heads,layers", [(W.BF16, 128, 8, 48, 2), (W.FP8, 128, 8, 48, 2),
                                                             (W.BF16, 64, 16, 96, 2), (W.FP8, 32, 96, 96, 2),
                                                             (W.BF16, (96, 192), 30, 30, 1)])
def test_states_do_not_depend_on_the_tile_shape(weights, d, k_heads, v_heads, layers):
    """A segment replayed alone (small tiles; square heads: two workgroups per
    unit in the scan) and inside a batch of big ones (one per unit) gives the
    same bits: the products accumulate along K in one order, the key norm's sum
    is one tree in both and a state column's steps are the same."""
    dk, dv = d if isinstance(d, tuple) else (d, d)
    shape = W.Shape(256, k_heads, v_heads, dk, dv, weight_dtype=weights)
    wl = W.make_workload("shape", shape, [100, 201, 300, 162], n_layers=layers, seed=7)
    assert not _takes_small_tiles(shape, wl.t_total, layers)
    dev = upload(wl)
    run(dev)
    cu = wl.cu_seqlens
    for b in range(4):
        one = W.make_workload("one", shape, [wl.seg_lens[b]], n_layers=1, seed=7)
        assert _takes_small_tiles(shape, wl.seg_lens[b], 1)
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


def test_f32_tail_too_large_to_ride_behind_the_conv():
    """Hundreds of segments with next to no rows: more (segment, 4 channels)
    tail blocks than fit behind the conv's one row block, so the tail keeps a
    launch of its own; empty segments get zero states and tails."""
    lens = [0] * 200
    lens[3], lens[77], lens[199] = 1, 40, 2
    heads, d = 16, 32
    assert len(lens) * (3 * heads * d // 4) > 60000      # tail_rides_conv's bound for up to 64 rows
    wl = W.make_workload("f32_tail", _f32_shape(64, heads, d), lens, seed=9)
    dev = upload(wl)
    run(dev)
    check_pairs(dev, [(0, 3), (0, 77), (0, 199)], TOL_F32)
    empty = [b for b, n in enumerate(lens) if n == 0]
    assert torch.all(dev.layers[0].state_out[empty] == 0) and torch.all(dev.layers[0].tail_out[empty] == 0)


@pytest.mark.parametrize("rows,d_ff", [(256, 128), (257, 192 + 64), (510, 384)])
def test_block_gemm_tile_edges(rows, d_ff):
    shape = W.Shape(256, 2, 4, 64, 64)
    gw = make_group("tile", shape, LENGTHS[rows], n_layers=2, d_ff=d_ff, seed=rows)
    dg = upload_group(gw)
    _run(dg)
    log(f"block GEMM tile edges: T={gw.t_total}, d_ff={d_ff}: {_check_group(dg)}")


@pytest.mark.parametrize("rows", [257, 510])
@pytest.mark.parametrize("v_heads", [1, 3])
def test_block_gemm_short_rings(v_heads, rows):
    """The output projection's K is the value width: 64 and 192 are one and
    three K-steps, where the prologue refetches its last step and the tail
    refills B alone."""
    gw = make_group("rings", W.Shape(256, 1, v_heads, 64, 64), LENGTHS[rows], n_layers=2, d_ff=128,
                    seed=rows + v_heads)
    dg = upload_group(gw)
    _run(dg)
    log(f"block GEMM, K = {64 * v_heads}: T={gw.t_total}: {_check_group(dg)}")
