"""GPU parity of the bf16 scan on both sides of the rule that splits a unit (a
segment of one value head) over two workgroups: with few units each workgroup
runs half of one unit's state columns; with more, a workgroup runs whole units
one after the other.  Each side at every head width, with an initial state, no
decay, a sentinel slot and an empty segment among the units, against the fp64
oracle; an empty segment's state is the initial one, bit for bit."""
import os
import re

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_harness import TOL_BF16, check_slab, log, run, upload

pytestmark = pytest.mark.gpu

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_33477_amd", "csrc",
                      "gdn_scan_bf16.hip")


def _splits_units(units):
    """The condition of the scan's run(), read from its source."""
    with open(SOURCE) as f:
        src = f.read()
    halves, rule = re.search(r"int64_t halves = (.*);\s*if \((halves .*)\) {", src).groups()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    env = {"__builtins__": {}, "units": units, "device_cus": lambda: cus}
    return bool(eval(rule, {**env, "halves": eval(halves.replace("/", "//"), env)}))


@pytest.mark.parametrize("form", ["zero", "state_in", "no_decay"])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("k_heads,v_heads,split", [(2, 4, True), (8, 96, False)])
def test_units_of_every_kind(k_heads, v_heads, split, d, form):
    shape = W.Shape(64, k_heads, v_heads, d, d)
    lens, slots = [70, 0, 33, 129, 1], [2, 0, -1, 1, 4]
    assert _splits_units(len(lens) * v_heads) == split
    wl = W.make_workload("units", shape, lens, seed=d + v_heads, slot_ids=slots, n_slots=5)
    L = wl.layers[0]
    S0 = None
    if form != "zero":
        S0 = np.random.default_rng(d).standard_normal((5, v_heads, d, d)).astype(np.float32) * np.float32(0.5)
    if form == "no_decay":
        L.a_log[:] = -40.0
    log(f"scan units: {v_heads} heads of {d}, {form}")
    dev = upload(wl, state_in=None if S0 is None else [S0])
    run(dev)
    out, tail = dev.layers[0].state_out.cpu().numpy(), dev.layers[0].tail_out.float().cpu().numpy()
    cu = wl.cu_seqlens
    for b, slot in enumerate(slots):
        if slot < 0:
            continue
        init = np.zeros((v_heads, d, d), np.float32) if S0 is None else S0[slot]
        if lens[b] == 0:
            assert np.array_equal(out[slot], init) and not tail[slot].any()
            continue
        ref = oracle.replay_segment(shape, L, L.anchors[cu[b]:cu[b + 1]], S0=init.astype(np.float64))
        check_slab(wl, 0, b, out[slot], tail[slot], TOL_BF16, ref=ref)
    assert np.isnan(out[3]).all() and np.isnan(tail[3]).all()      # no segment has slot 3
