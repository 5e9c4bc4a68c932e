"""Performance cases: the calls a serving system makes of this library.

A case is one call of a public entry point (or, for the sidecar, the calls of
one serving step) on inputs that already sit on the GPU, as they do in a
serving process: anchors, weights, tables, output slots and a workspace.

Three kinds:
  replay   sr_replay_state: the states and conv tails of `layers` independent
           linear-attention layers rebuilt for a packed batch of hits
  group    sr_replay_group: a group of blocks rebuilt from its entry anchors
  sidecar  one serving step of the anchor pool: the prefill's sampled rows
           compacted and written into their blocks, then the last anchors of
           the hits gathered into a packed batch

Hit lengths are drawn from [lo, hi] with the case's own `lens` seed, so they
belong to the case; `page` > 1 rounds them up to whole pages.
"""
import math
import random

import numpy as np
import torch

import paper_2609_33477_amd as sr

DEVICE = "cuda"
TORCH_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
PAGE, PER_PAGE = 64, 4
L2_EPS = NORM_EPS = 1e-6


def _replay(name, **kw):
    case = {"name": name, "kind": "replay", "dtype": "bf16", "weights": "bf16", "recurrence": "gdn",
            "d_model": 2560, "k_heads": 16, "v_heads": 32, "d_k": 128, "d_v": 128, "conv_width": 4,
            "layers": 1, "hits": 1, "lo": 128, "hi": 128, "page": 1, "lens": 0, "sentinels": 0,
            "dt_bias": 0.0, "q_tail": True, "state_in": False}
    case.update(kw)
    return case


def listed():
    return [
        # The smallest call there is: one short fp32 replay of a toy layer, as
        # an integration check or a float32 model makes it.  Launches count.
        _replay("tiny_f32", dtype="f32", weights="f32", d_model=128, k_heads=2, v_heads=2, d_k=32, d_v=32,
                lo=256, hi=256),
        # One interactive session hits the cache: 128 anchors through one
        # 3-layer group of the Qwen3.5-4B linear layers.  Pure latency.
        _replay("hit_4b", layers=3),
        # A mixed batch: hits of any length from a few rows up, two of them
        # padding segments with the sentinel slot.
        _replay("ragged_4b", layers=3, hits=11, lo=1, hi=700, sentinels=2, lens=3),
        # A serving step's hits, 8 x 128 anchors, through all 24 linear layers.
        _replay("serve_4b_24l", layers=24, hits=8),
        # One long suffix through one small square-headed layer.
        _replay("gdn_single", d_model=2048, v_heads=16, lo=2048, hi=2048),
        # The 16-request varlen batch of the headline benchmark.
        _replay("varlen16", hits=16, lo=512, hi=4096, page=64, lens=16),
        # Throughput with long suffixes and slow decay.
        _replay("stress64", d_model=4096, k_heads=32, hits=64, lo=1024, hi=8192, page=64, lens=64,
                dt_bias=-7.494),
        # Twelve layers of the 27B shape with fp8 weights in one call.
        _replay("multilayer12_fp8", weights="fp8", d_model=5120, v_heads=48, layers=12, hits=4, lo=4096, hi=4096),
        # The per-head-decay recurrence on the same batch as varlen16.
        _replay("varlen16_decay", recurrence="decay", hits=16, lo=512, hi=4096, page=64, lens=16),
        # OLMo-Hybrid-7B's rectangular heads.
        _replay("olmo_varlen", d_model=3840, k_heads=30, v_heads=30, d_k=96, d_v=192, hits=16, lo=512, hi=4096,
                page=64, lens=6),
        # Group replay: 8 hits of the replay cap through a 3-layer group.
        {"name": "group_4b", "kind": "group", "d_model": 2560, "k_heads": 16, "v_heads": 32, "d_k": 128,
         "d_v": 128, "conv_width": 4, "d_ff": 9728, "layers": 3, "hits": 8, "lo": 512, "hi": 512, "page": 1,
         "lens": 0, "sentinels": 0, "dt_bias": 0.0},
        # One step of the anchor pool: 16 prefills of 4096 tokens written, 8
        # hits at the replay cap read back, 7 anchored layers.
        {"name": "sidecar_step", "kind": "sidecar", "anchored": 7, "d_model": 2560, "prefills": 16,
         "prefill_lo": 4096, "prefill_hi": 4096, "hits": 8, "lo": 512, "hi": 512, "page": 1, "lens": 0},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# A drawn case does at most this much multiply-add work (stress64, the largest
# listed case, does 2.1e13) and moves at most this many bytes.
DRAW_FLOPS, DRAW_BYTES = 1.0e13, 4.0e9


def _draw(rng):
    kind = rng.choice(["replay"] * 7 + ["group", "sidecar"])
    if kind == "sidecar":
        lo = _log_int(rng, 1, 1024)
        pre = _log_int(rng, 1, 4096)
        return {"kind": kind, "anchored": rng.randint(1, 12), "d_model": 64 * _log_int(rng, 2, 80),
                "prefills": _log_int(rng, 1, 32), "prefill_lo": max(1, pre // 4), "prefill_hi": pre,
                "hits": _log_int(rng, 1, 32), "lo": max(1, lo // 8), "hi": lo, "page": 1,
                "lens": rng.randint(0, 1 << 20)}
    hits = _log_int(rng, 1, 64)
    hi = _log_int(rng, 4, 8192)
    base = {"hits": hits, "lo": max(1, hi // rng.choice([1, 2, 8, 64])), "hi": hi, "page": rng.choice([1, 1, 64]),
            "lens": rng.randint(0, 1 << 20), "sentinels": rng.choice([0, 0, min(2, hits - 1)]),
            "conv_width": rng.choice([4, 4, 4, 3, 2])}
    if kind == "group":
        k_heads = rng.choice([2, 4, 8, 16])
        d = rng.choice([64, 128, 128])
        return {"kind": kind, "d_model": 256 * rng.randint(1, 16), "k_heads": k_heads,
                "v_heads": k_heads * rng.choice([1, 2, 3]), "d_k": d, "d_v": d, "d_ff": 128 * _log_int(rng, 4, 96),
                "layers": rng.randint(1, 4), "dt_bias": rng.choice([0.0, -7.494]), **base}
    form = rng.choice(["f32", "bf16", "bf16", "bf16", "fp8", "decay", "rect"])
    k_heads = _log_int(rng, 1, 32)
    v_heads = k_heads * rng.choice([1, 2, 3]) if k_heads <= 16 else k_heads
    d = rng.choice([32, 64, 128, 128, 128, 128])
    case = _replay("", d_model=64 * _log_int(rng, 2, 80), k_heads=k_heads, v_heads=v_heads, d_k=d, d_v=d,
                   layers=_log_int(rng, 1, 24), dt_bias=rng.choice([0.0, -7.494]), q_tail=rng.random() < 0.8,
                   state_in=rng.random() < 0.2, **base)
    if form == "f32":
        case.update(dtype="f32", weights="f32", hi=min(case["hi"], 1024), lo=min(case["lo"], 1024),
                    layers=min(case["layers"], 3), hits=min(case["hits"], 8))
        case["sentinels"] = min(case["sentinels"], case["hits"] - 1)
    elif form == "fp8":
        case["weights"] = "fp8"
    elif form == "decay":
        case["recurrence"] = "decay"
    elif form == "rect":
        k_heads = 2 * rng.randint(1, 15)
        case.update(d_k=96, d_v=192, k_heads=k_heads, v_heads=k_heads)
    del case["name"]
    return case


def draw(rng):
    while True:
        case = _draw(rng)
        w = work(case)
        if w["flops"] <= DRAW_FLOPS * (0.02 if case.get("dtype") == "f32" else 1) and w["bytes"] <= DRAW_BYTES:
            return case


# ------------------------------------------------------------------ shapes
class _Shape:
    """The fields of sr_shape."""

    def __init__(self, case):
        self.d_model, self.n_k_heads, self.n_v_heads = case["d_model"], case["k_heads"], case["v_heads"]
        self.d_k, self.d_v, self.conv_width, self.l2_eps = case["d_k"], case["d_v"], case["conv_width"], L2_EPS
        self.anchor_dtype = case.get("dtype", "bf16")
        self.weight_dtype = {"fp8": "fp8_e4m3"}.get(case.get("weights", "bf16"), case.get("weights", "bf16"))
        self.conv_dtype = self.tail_dtype = self.anchor_dtype
        self.recurrence = case.get("recurrence", "gdn")


def _lengths(case, lo="lo", hi="hi", n="hits"):
    rng = random.Random(1000 * case["lens"] + case[n])
    return [-(-rng.randint(case[lo], case[hi]) // case["page"]) * case["page"] for _ in range(case[n])]


def _slots(case):
    """Slot of each hit: live hits in a fixed permutation, the last hits of
    the batch padding segments."""
    live = list(range(case["hits"] - case["sentinels"]))
    random.Random(case["lens"]).shuffle(live)
    return live + [-1] * case["sentinels"]


def _widths(case):
    return case["k_heads"] * case["d_k"], case["v_heads"] * case["d_v"]


def work(case):
    if case["kind"] == "sidecar":
        row = case["d_model"] * 2
        written = sum(_sampled(n) for n in _lengths(case, "prefill_lo", "prefill_hi", "prefills"))
        tokens = sum(_lengths(case, "prefill_lo", "prefill_hi", "prefills"))
        read = sum(_lengths(case))
        return {"bytes": 2 * case["anchored"] * row * (written + read) + 4 * (tokens + 3 * written + read),
                "flops": 0}
    rows = sum(L for L, s in zip(_lengths(case), _slots(case)) if s >= 0)
    live = case["hits"] - case["sentinels"]
    D, hv = case["d_model"], case["v_heads"]
    ck, cv = _widths(case)
    act = 4 if case.get("dtype") == "f32" else 2
    wb = {"f32": 4, "bf16": 2, "fp8": 1}[case.get("weights", "bf16")]
    state = live * hv * case["d_k"] * case["d_v"] * 4
    tail = live * (2 * ck + cv) * (case["conv_width"] - 1) * act
    scan = 4 * hv * case["d_k"] * case["d_v"]
    if case["kind"] == "replay":
        proj = ck + cv + 2 * hv
        q = ck if case["q_tail"] else 0
        tail_rows = sum(min(L, case["conv_width"] - 1) for L, s in zip(_lengths(case), _slots(case)) if s >= 0)
        states = state * (2 if case["state_in"] else 1)
        per_layer = rows * D * act + (proj + q) * D * wb + states + tail
        return {"bytes": case["layers"] * per_layer,
                "flops": case["layers"] * (2 * rows * D * proj + rows * scan + 2 * tail_rows * D * q)}
    n, ff = case["layers"], case["d_ff"]
    full = 2 * rows * D * (2 * ck + 2 * cv + 2 * hv) + 2 * rows * D * cv + 6 * rows * D * ff + rows * scan * 3 // 2
    last = 2 * rows * D * (ck + cv + 2 * hv) + rows * scan
    weights = ((2 * ck + 2 * cv + 2 * hv) * D * n + (cv * D + 3 * D * ff) * (n - 1)) * 2
    return {"bytes": rows * D * 2 + weights + n * (state + tail), "flops": (n - 1) * full + last}


# Relative 2-norm between two correct implementations at the same precision.
# Measured against `exact`: fp32 1e-6 or less, bf16 and fp8 2.5e-3 to 3.5e-3
# (each operand of a product rounded once), the chained group 3.5e-3 in its
# first layer to 6e-3 in its third.
def tolerance(case):
    if case["kind"] == "sidecar":
        return "exact"
    if case["kind"] == "group":
        return {"rel": 2e-2}
    return {"rel": 5e-6 if case["dtype"] == "f32" else 1.2e-2}


# ------------------------------------------------------------------ inputs
def _randn(gen, *shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
    x = torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32)
    return x.mul_(std).add_(mean).to(dtype)


def _quantise(w):
    """Per-output-channel fp8: w ~ q * s with s = bf16(max|row| / 448)."""
    s = (w.abs().amax(dim=1) / 448.0).clamp_min(2.0 ** -30).to(torch.bfloat16)
    return (w / s.float()[:, None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn), s


def _tables(case):
    lens = _lengths(case)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=DEVICE)
    return lens, cu, torch.tensor(_slots(case), dtype=torch.int32, device=DEVICE)


def _gates(gen, case):
    hv = case["v_heads"]
    a_log = torch.rand(hv, generator=gen, device=DEVICE) * math.log(16.0)
    return a_log, _randn(gen, hv, std=0.5, mean=case["dt_bias"], dtype=torch.float32)


def _weights(gen, case, names):
    ck, cv = _widths(case)
    rows = {"q": ck, "k": ck, "v": cv, "z": cv, "a": case["v_heads"], "b": case["v_heads"]}
    out = {}
    for n in names:
        w = _randn(gen, rows[n], case["d_model"], std=0.02, dtype=torch.float32)
        if case.get("weights") == "fp8":
            out["w_" + n], out["s_" + n] = _quantise(w)
        else:
            out["w_" + n] = w.to(TORCH_DTYPES[case.get("dtype", "bf16")])
    return out


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    return {"replay": _prepare_replay, "group": _prepare_group, "sidecar": _prepare_sidecar}[case["kind"]](case, gen)


def _prepare_replay(case, gen):
    lens, cu, slots = _tables(case)
    rows, live = sum(lens), case["hits"] - case["sentinels"]
    ck, cv = _widths(case)
    act = TORCH_DTYPES[case["dtype"]]
    layers = []
    for _ in range(case["layers"]):
        t = _weights(gen, case, ["k", "v", "a", "b"] + (["q"] if case["q_tail"] else []))
        t["anchors"] = _randn(gen, rows, case["d_model"], dtype=act)
        t["conv_w"] = _randn(gen, ck + cv, case["conv_width"], std=0.02, dtype=act)
        t["a_log"], t["dt_bias"] = _gates(gen, case)
        shape = (live, case["v_heads"], case["d_k"], case["d_v"])
        if case["state_in"]:
            t["state_in"] = _randn(gen, *shape, std=0.1, dtype=torch.float32)
        t["state_out"] = torch.zeros(shape, dtype=torch.float32, device=DEVICE)
        c_tail = ck + cv + (ck if case["q_tail"] else 0)
        t["tail_out"] = torch.zeros(live, c_tail, case["conv_width"] - 1, dtype=act, device=DEVICE)
        layers.append(sr.LayerTensors(**t))
    shape = _Shape(case)
    ws = torch.empty(max(256, sr.replay_workspace_size(shape, len(layers), rows)), dtype=torch.uint8, device=DEVICE)
    return {"kind": "replay", "case": case, "shape": shape, "layers": layers, "lens": lens, "rows": rows, "cu": cu,
            "slots": slots, "n_slots": live, "workspace": ws}


def _prepare_group(case, gen):
    lens, cu, slots = _tables(case)
    rows, live, D, ff = sum(lens), case["hits"] - case["sentinels"], case["d_model"], case["d_ff"]
    ck, cv = _widths(case)
    anchors = _randn(gen, rows, D)
    blocks = []
    for _ in range(case["layers"]):
        t = _weights(gen, case, "qkvzab")
        t["conv_w"] = _randn(gen, 2 * ck + cv, case["conv_width"], std=0.02)
        t["a_log"], t["dt_bias"] = _gates(gen, case)
        for n, size in (("norm_o", case["d_v"]), ("ln_in", D), ("ln_post", D)):
            t[n] = _randn(gen, size, std=0.1, mean=1.0)
        for n, r, c in (("w_o", D, cv), ("w_gate", ff, D), ("w_up", ff, D), ("w_down", D, ff)):
            t[n] = _randn(gen, r, c, std=0.02)
        t["state_out"] = torch.zeros(live, case["v_heads"], case["d_k"], case["d_v"], dtype=torch.float32,
                                     device=DEVICE)
        t["tail_out"] = torch.zeros(live, 2 * ck + cv, case["conv_width"] - 1, dtype=torch.bfloat16, device=DEVICE)
        blocks.append(sr.BlockTensors(**t))
    shape = _Shape(case)
    ws = torch.empty(max(256, sr.group_workspace_size(shape, ff, rows)), dtype=torch.uint8, device=DEVICE)
    return {"kind": "group", "case": case, "shape": shape, "d_ff": ff, "blocks": blocks, "anchors": anchors,
            "lens": lens, "rows": rows, "cu": cu, "slots": slots, "n_slots": live, "workspace": ws}


def _sampled(n):
    """Anchors of an n-token prefill: the last PER_PAGE positions of each page."""
    return n // PAGE * PER_PAGE + max(0, n % PAGE - (PAGE - PER_PAGE))


def _prepare_sidecar(case, gen):
    A, d = case["anchored"], case["d_model"]
    host = np.random.default_rng(case["lens"])
    pre, hits = _lengths(case, "prefill_lo", "prefill_hi", "prefills"), _lengths(case)
    extra = [int(x) for x in host.integers(0, 2 * PER_PAGE + 2, len(hits))]
    pre_pages = [-(-n // PAGE) for n in pre]
    hit_pages = [-(-(n + e) // PER_PAGE) for n, e in zip(hits, extra)]
    n_pre, n_hit = sum(pre_pages), sum(hit_pages)
    blocks = host.permutation(n_pre + n_hit).astype(np.int32)      # as a paged allocator hands them out

    def cu(x):
        return np.concatenate([[0], np.cumsum(x)]).astype(np.int32)

    def dev(x):
        return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to(DEVICE)

    positions = np.concatenate([np.arange(n) for n in pre])
    request = np.concatenate([np.full(n, r) for r, n in enumerate(pre)])
    dest = dev(sr.anchor_dest_table(positions, request, blocks[:n_pre], cu(pre_pages), PAGE, PER_PAGE))
    pool = _randn(gen, (n_pre + n_hit) * A * PER_PAGE, d)
    tokens = len(positions)
    return {"kind": "sidecar", "case": case, "sidecar": sr.make_sidecar(pool, A, PER_PAGE, d), "pool": pool,
            "hidden": [_randn(gen, tokens, d) for _ in range(A)], "dest": dest,
            "sel": torch.zeros(tokens, dtype=torch.int32, device=DEVICE),
            "n_sel": torch.zeros(1, dtype=torch.int32, device=DEVICE),
            "block_table": dev(blocks[n_pre:]), "block_cu": dev(cu(hit_pages)), "first": dev(extra),
            "n_anchors": dev(hits),
            "out": [torch.zeros(sum(hits), d, dtype=torch.bfloat16, device=DEVICE) for _ in range(A)],
            "cu": torch.zeros(len(hits) + 1, dtype=torch.int32, device=DEVICE)}


# ------------------------------------------------------------------ the call
def run(s):
    if s["kind"] == "replay":
        sr.replay_state(s["shape"], s["layers"], len(s["lens"]), s["rows"], s["cu"], s["slots"], s["workspace"],
                        n_slots=s["n_slots"])
        return [t for L in s["layers"] for t in (L.state_out, L.tail_out)]
    if s["kind"] == "group":
        sr.replay_group(s["shape"], s["d_ff"], NORM_EPS, s["blocks"], s["anchors"], len(s["lens"]), s["rows"],
                        s["cu"], s["slots"], s["workspace"], n_slots=s["n_slots"])
        return [t for b in s["blocks"] for t in (b.state_out, b.tail_out)]
    sr.anchor_compact(s["dest"], s["sel"], s["n_sel"])
    sr.anchor_write(s["sidecar"], s["hidden"], s["dest"], s["sel"], s["n_sel"])
    sr.anchor_gather(s["sidecar"], s["block_table"], s["block_cu"], s["first"], s["n_anchors"],
                     range(s["case"]["anchored"]), s["out"], s["cu"])
    return [s["pool"], s["cu"], s["n_sel"]] + s["out"]


# ------------------------------------------------------- the result in 64 bits
def _conv_silu(p, taps, lens):
    """SiLU of the causal depthwise conv, zero history before each segment."""
    y = torch.empty_like(p)
    w, at = taps.shape[1], 0
    for L in lens:
        x = p[at:at + L]
        acc = x * taps[:, w - 1]
        for lag in range(1, min(w, L)):
            acc[lag:] += x[:-lag] * taps[:, w - 1 - lag]
        y[at:at + L] = acc * torch.sigmoid(acc)
        at += L
    return y


def _unit(x, heads):
    x = x.view(x.shape[0], heads, -1)
    return x / torch.sqrt((x * x).sum(-1, keepdim=True) + L2_EPS)


def _weight64(t, n):
    w = getattr(t, "w_" + n).double()
    s = getattr(t, "s_" + n, None)
    return w if s is None else w * s.double()[:, None]


def _recur(case, k, v, g, beta, lens, M, q=None):
    """Token by token over all segments at once; g = alpha.  Rows past a
    segment's end leave its state unchanged.  Returns (M, o or None)."""
    rep = case["v_heads"] // case["k_heads"]
    n, H, dk, dv = len(lens), case["v_heads"], case["d_k"], case["d_v"]
    start = torch.tensor([0] + lens[:-1], device=DEVICE).cumsum(0)
    length = torch.tensor(lens, device=DEVICE)
    o = None if q is None else torch.zeros_like(v)
    M = M.reshape(n * H, dk, dv)
    for t in range(max(lens)):
        live = (t < length)
        row = (start + t).clamp_(max=v.shape[0] - 1)
        kt = k[row].repeat_interleave(rep, 1).reshape(n * H, dk, 1)
        a = torch.where(live[:, None], g[row], torch.ones_like(g[row])).reshape(n * H, 1, 1)
        b = (beta[row] * live[:, None]).reshape(n * H, 1, 1)
        write = b * v[row].reshape(n * H, 1, dv)
        if case.get("recurrence", "gdn") == "gdn":
            write = write - a * b * torch.bmm(kt.transpose(1, 2).contiguous(), M)
        M.mul_(a).baddbmm_(kt, write)
        if q is not None:
            qt = q[row].repeat_interleave(rep, 1).reshape(n * H, 1, dk)
            o[row[live]] = torch.bmm(qt, M).reshape(n, H, dv)[live]
    return M.view(n, H, dk, dv), o


def _tail64(p, lens, w):
    out = torch.zeros(len(lens), p.shape[1], w - 1, dtype=torch.float64, device=DEVICE)
    at = 0
    for i, L in enumerate(lens):
        m = min(L, w - 1)
        if m:
            out[i, :, w - 1 - m:] = p[at + L - m:at + L].T
        at += L
    return out


def _place(x, slots, n_slots):
    out = torch.zeros((n_slots,) + tuple(x.shape[1:]), dtype=torch.float64, device=DEVICE)
    live = [i for i, s in enumerate(slots) if s >= 0]
    out[torch.tensor([slots[i] for i in live], device=DEVICE)] = x[torch.tensor(live, device=DEVICE)]
    return out


def _mixer64(case, t, x, taps, lens, slots, n_slots, state_in=None, outputs=False):
    """(state, raw k | v projections, o) of one layer on its input rows x."""
    ck, _ = _widths(case)
    hv = case["v_heads"]
    p = torch.cat([x @ _weight64(t, "k").T, x @ _weight64(t, "v").T], 1)
    act = _conv_silu(p, taps[-p.shape[1]:], lens)
    k = _unit(act[:, :ck], case["k_heads"])
    v = act[:, ck:].reshape(len(x), hv, case["d_v"])
    a, b = x @ _weight64(t, "a").T, x @ _weight64(t, "b").T
    g = torch.exp(-torch.exp(t.a_log.double()) * torch.nn.functional.softplus(a + t.dt_bias.double()))
    M = torch.zeros(len(lens), hv, case["d_k"], case["d_v"], dtype=torch.float64, device=DEVICE)
    if state_in is not None:
        for i, s in enumerate(slots):
            if s >= 0:
                M[i] = state_in[s].double()
    q = pq = None
    if outputs:
        pq = x @ _weight64(t, "q").T
        q = _unit(_conv_silu(pq, taps[:ck], lens), case["k_heads"]) / math.sqrt(case["d_k"])
    M, o = _recur(case, k, v, g, torch.sigmoid(b), lens, M, q)
    return _place(M, slots, n_slots), p, pq, o


def exact(case, seed):
    if case["kind"] == "sidecar":
        return None                        # rows are copied, nothing is computed
    lens, slots = _lengths(case), _slots(case)
    # one step per row of the longest hit, its launches and its passes over the
    # fp64 states: seconds on this card
    states = len(lens) * case["v_heads"] * case["d_k"] * case["d_v"]
    cost = case["layers"] * max(lens) * (2e-4 + 1.6e-11 * states)
    if cost > 15:
        return None
    s = prepare(case, seed)
    w, n_slots = case["conv_width"], s["n_slots"]
    ck, cv = _widths(case)
    out = []
    if case["kind"] == "replay":
        for t in s["layers"]:
            x = t.anchors.double()
            state, p, _, _ = _mixer64(case, t, x, t.conv_w.double(), lens, slots, n_slots, t.state_in)
            if case["q_tail"]:
                p = torch.cat([x @ _weight64(t, "q").T, p], 1)
            out += [state, _place(_tail64(p, lens, w), slots, n_slots)]
        return out

    def rms(x, weight):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + NORM_EPS) * weight.double()

    def silu(x):
        return x * torch.sigmoid(x)

    h = s["anchors"].double()
    for j, t in enumerate(s["blocks"]):
        x = rms(h, t.ln_in)
        last = j + 1 == len(s["blocks"])
        state, p, pq, o = _mixer64(case, t, x, t.conv_w.double(), lens, slots, n_slots, outputs=not last)
        pq = x @ _weight64(t, "q").T if last else pq
        out += [state, _place(_tail64(torch.cat([pq, p], 1), lens, w), slots, n_slots)]
        if not last:
            z = (x @ _weight64(t, "z").T).view(len(x), case["v_heads"], case["d_v"])
            h = h + (rms(o, t.norm_o) * silu(z)).reshape(len(x), cv) @ t.w_o.double().T
            u = rms(h, t.ln_post)
            h = h + (silu(u @ t.w_gate.double().T) * (u @ t.w_up.double().T)) @ t.w_down.double().T
    return out
