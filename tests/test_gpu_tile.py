"""GPU parity at the edges of the 256 x 256 tile (projection and block GEMMs):
row counts around the first tile's 256 output rows and the later ones' 253,
and d_model from one K-step of 64 up to past the ring's depth, where the main
loop runs its shortened prologue and tails.  Bounds as in the other parity
tests: every product rounds its operands once to bf16, 5e-3 per slab."""
import pytest

import workloads as W
from gpu_harness import TOL_BF16, check_pairs, log, run, upload
from test_gpu_group import _check_group, _run
from workloads.device import upload_group
from workloads.group import make_group

pytestmark = pytest.mark.gpu

LENGTHS = {256: [256], 257: [255, 2], 509: [250, 3, 256], 510: [253, 253, 4], 763: [1, 508, 254]}


@pytest.mark.parametrize("weights", [W.BF16, W.FP8])
@pytest.mark.parametrize("rows,d_model,d", [(256, 64, 128), (257, 128, 64), (509, 192, 32), (510, 256, 128),
                                            (763, 320, 64), (257, 384, 128)])
def test_projection_tile_edges(rows, d_model, d, weights):
    shape = W.Shape(d_model, 2, 4, d, d, weight_dtype=weights)
    wl = W.make_workload("tile", shape, LENGTHS[rows], n_layers=2, seed=rows + d_model)
    log(f"tile edges: T={wl.t_total}, D={d_model}, d={d}, {weights}")
    dev = upload(wl)
    run(dev)
    check_pairs(dev, [(li, b) for li in range(2) for b in range(len(wl.seg_lens))], TOL_BF16)


@pytest.mark.parametrize("rows,d_ff", [(256, 128), (257, 192 + 64), (510, 384)])
def test_block_gemm_tile_edges(rows, d_ff):
    shape = W.Shape(256, 2, 4, 64, 64)
    gw = make_group("tile", shape, LENGTHS[rows], n_layers=2, d_ff=d_ff, seed=rows)
    dg = upload_group(gw)
    _run(dg)
    log(f"block GEMM tile edges: T={gw.t_total}, d_ff={d_ff}: {_check_group(dg)}")
