"""The workloads whose speed this repository tracks, through its public binding.

Each case is one call path a user of ``paper_2606_23419_amd.grinqh`` runs in
earnest, at sizes of this repository's own workloads (Llama3-8B- and
Qwen3-8B-shaped linears, group 128, the paper's level sets and budgets):

* ``decode``: one token step (or B tokens) through whole decoder layers, the
  merged qkv, o, merged gate|up and down projections of each.  The step is
  captured once as a HIP graph over a fixed activation buffer and one output
  arena, as a serving loop keeps it, and a pass is one replay.  Levels are
  graded from thresholds inside the VMM, or by an exact top-k assignment
  launch per projection input.  Several layers, so that weights come from HBM.
* ``lut``: the same step over non-uniform (look-up-table) weights.
* ``single``: one eager VMM call, the smallest thing a program asks for.
* ``prefill``: one decoder layer's four projections on M prompt tokens, eager.
* ``pack``: quantise + nest + pack of one fp16 weight matrix (model loading).
* ``calibrate``: thresholds from calibration activations (offline).

Weights, activations and thresholds are drawn on the GPU from the seed: codes
of Gaussian weights, Student-t(3) activations with 1% outlier channels (x20),
SiLU(g)*u into the down projection.
"""
from __future__ import annotations

import zlib

import torch

from paper_2606_23419_amd import grinqh as g

GROUP = 128

# average-bit budgets as precision distributions in basis points, per level set
BUDGETS = {
    "0,2,4,8": {2: (3000, 5000, 1500, 500), 3: (2000, 4000, 2500, 1500),
                4: (2000, 2000, 3000, 3000), 8: (0, 0, 0, 10000)},
    "0,2,4,6,8": {2: (3000, 4500, 2000, 500, 0), 3: (2500, 2200, 3100, 2200, 0),
                  4: (2000, 800, 2400, 4800, 0), 6: (2000, 0, 0, 2000, 6000),
                  8: (0, 0, 0, 0, 10000)},
    "0,2,3,4,8": {2: (3000, 4000, 2000, 500, 500), 3: (2000, 3000, 2000, 1500, 1500),
                  4: (2000, 1000, 2000, 2000, 3000)},
    "0,2,4,6": {3: (2500, 2200, 3100, 2200), 4: (2000, 800, 2400, 4800), 6: (0, 0, 0, 10000)},
    "0,2,4": {2: (3500, 2500, 4000), 3: (2500, 100, 7400), 4: (0, 0, 10000)},
}


def listed():
    llama = {"hidden": 4096, "kv": 1024, "inter": 14336}
    return [
        # one small linear, called by itself: launch and call overhead
        {"name": "single_1024", "path": "single", "K": 1024, "N": 1024, "B": 1,
         "levels": "0,2,4,8", "bits": 4},
        # the flagship: batch-1 decode of a Llama3-8B-shaped model at 4 average bits
        {"name": "decode_b1_4bit", "path": "decode", "mode": "threshold", "B": 1, "layers": 4,
         "levels": "0,2,4,6,8", "bits": 4, **llama},
        # the same at the paper's lowest budget
        {"name": "decode_b1_2bit", "path": "decode", "mode": "threshold", "B": 1, "layers": 4,
         "levels": "0,2,4,6,8", "bits": 2, **llama},
        # four sequences decoded together
        {"name": "decode_b4_4bit", "path": "decode", "mode": "threshold", "B": 4, "layers": 4,
         "levels": "0,2,4,6,8", "bits": 4, **llama},
        # exact per-token budgets: top-k assignment launches before the VMMs
        {"name": "decode_topk_b1_3bit", "path": "decode", "mode": "topk", "B": 1, "layers": 4,
         "levels": "0,2,4,6,8", "bits": 3, **llama},
        # Qwen3-8B-shaped layers with an odd level width (1-bit planes)
        {"name": "decode_qwen_b1_4bit", "path": "decode", "mode": "threshold", "B": 1, "layers": 4,
         "levels": "0,2,3,4,8", "bits": 4, "hidden": 4096, "kv": 1024, "inter": 12288},
        # 4-bit stored weights, two sequences
        {"name": "decode_bmax4_b2_3bit", "path": "decode", "mode": "threshold", "B": 2, "layers": 6,
         "levels": "0,2,4", "bits": 3, **llama},
        # decode over non-uniform nested weights
        {"name": "lut_b1_4bit", "path": "lut", "B": 1, "layers": 3, "levels": "0,2,4,6,8",
         "bits": 4, **llama},
        # a long prompt through one layer
        {"name": "prefill_2048", "path": "prefill", "M": 2048, "levels": "0,2,4,6,8", **llama},
        # a short prompt of odd length
        {"name": "prefill_77", "path": "prefill", "M": 77, "levels": "0,2,4,6,8", **llama},
        # loading one MLP matrix: RTN and packing from fp16
        {"name": "pack_28672x4096", "path": "pack", "K": 4096, "N": 28672, "levels": "0,2,4,6,8"},
        # thresholds of one input from 256 calibration tokens
        {"name": "calibrate_256x4096", "path": "calibrate", "K": 4096, "S": 256,
         "levels": "0,2,4,6,8", "bits": 4},
    ]


def _log(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], spread over the logarithm."""
    v = lo * (hi / lo) ** rng.random()
    return int(min(hi, max(lo, round(v / step) * step)))


def draw(rng):
    path = rng.choice(["single", "decode", "decode", "decode", "decode", "lut", "prefill",
                       "prefill", "pack", "calibrate"])
    levels = rng.choice(sorted(BUDGETS))
    bits = rng.choice(sorted(BUDGETS[levels]))
    # outputs come in tiles of 256 (2-bit planes) or 512 (1-bit planes)
    nstep = 512 if "3" in levels else 256
    if path == "single":
        return {"path": path, "K": _log(rng, 128, 4096, 128), "N": _log(rng, nstep, 4096, nstep),
                "B": rng.randint(1, 4), "levels": levels, "bits": bits}
    if path == "pack":
        return {"path": path, "K": _log(rng, 256, 8192, 128), "N": _log(rng, 1024, 14336, nstep),
                "levels": levels}
    if path == "calibrate":
        return {"path": path, "K": _log(rng, 512, 14336, 128), "S": int(_log(rng, 4, 256, 1)),
                "levels": levels, "bits": bits}
    dims = {"hidden": _log(rng, 1024, 5120, nstep), "kv": nstep * rng.randint(1, 2),
            "inter": _log(rng, 2048, 14336, nstep)}
    per_layer = _layer_weights(dims)
    if path == "prefill":
        # no more products than 2048 tokens through the listed layer
        most = int(2048 * 218103808 / per_layer)
        return {"path": path, "M": _log(rng, 5, min(2048, most), 1), "levels": levels, **dims}
    layers = max(1, min(4, int(4 * 218103808 / per_layer)))
    if path == "lut":
        return {"path": path, "B": rng.randint(1, 2), "layers": 1 if per_layer > 1 << 26 else 2,
                "levels": levels, "bits": bits, **dims}
    return {"path": path, "mode": rng.choice(["threshold", "threshold", "topk"]),
            "B": rng.randint(1, 4), "layers": layers, "levels": levels, "bits": bits, **dims}


# ------------------------------------------------------------------ inputs --
def _layer_weights(c):
    return sum(K * N for _, K, N in _projections(c))


def _projections(c):
    h, kv, inter = c["hidden"], c["kv"], c["inter"]
    return [("qkv", h, h + 2 * kv), ("o", h, h), ("gate_up", h, 2 * inter), ("down", inter, h)]


def _levels(c):
    return tuple(int(b) for b in c["levels"].split(","))


def _gen(seed, *tag):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(zlib.crc32(repr((int(seed),) + tag).encode()))
    return gen


def _codes(seed, tag, K, N, b_max):
    """Codes (uint8 [N, K]) and scales (fp16 [N, K/128]) of Gaussian weights:
    the group's largest weight, about 2.7 standard deviations, fills the range."""
    gen = _gen(seed, tag, "codes")
    half = 1 << (b_max - 1)
    q = torch.randn((N, K), generator=gen, device="cuda", dtype=torch.float32)
    q = q.mul_((half - 1) / 2.7).round_().clamp_(-half, half - 1).add_(half).to(torch.uint8)
    s = torch.rand((N, K // GROUP), generator=gen, device="cuda").mul_(2e-4).add_(3e-4).half()
    return q, s


def _acts(seed, tag, role, tokens, K, swiglu):
    """fp16 [tokens, K] activations; the outlier channels belong to `tag`
    alone, so calibration and run tokens share them."""
    gen = _gen(seed, tag, role)
    if swiglu:
        a = torch.randn((tokens, K), generator=gen, device="cuda")
        u = torch.randn((tokens, K), generator=gen, device="cuda")
        return (torch.nn.functional.silu(a) * u).half()
    z = torch.randn((tokens, K), generator=gen, device="cuda")
    chi = torch.randn((3, tokens, K), generator=gen, device="cuda").square_().sum(0).div_(3.0)
    x = z / chi.sqrt()
    out = torch.randperm(K, generator=_gen(seed, tag, "outliers"), device="cuda")[: round(0.01 * K)]
    x[:, out] *= 20.0
    return x.clamp_(-60000.0, 60000.0).half()


def _theta(samples, p_bp):
    """Thresholds theta_1..theta_n: the mean over samples of the linear
    quantile of |x| at the cumulative fractions (float64), rounded to fp32."""
    a = samples.abs().double().sort(dim=1).values
    K = a.shape[1]
    out, U = [], 0
    for p in p_bp[:-1]:
        U += p
        lo, num = (K - 1) * U // 10000, (K - 1) * U % 10000
        hi = min(lo + 1, K - 1)
        out.append((a[:, lo] + (num / 10000.0) * (a[:, hi] - a[:, lo])).mean().float().item())
    return out


def _thresholds(c, seed, tag, K, swiglu):
    return _theta(_acts(seed, tag, "calib", 16, K, swiglu), BUDGETS[c["levels"]][c["bits"]])


def _tables(seed, tag, N, levels):
    """Nested centroid tables {b: fp16 [N, 2^b]} of Gaussian rows."""
    b_max = levels[-1]
    top = torch.randn((N, 1 << b_max), generator=_gen(seed, tag, "luts"), device="cuda").mul_(0.02)
    top = top.sort(dim=1).values
    return {b: top.view(N, 1 << b, -1).mean(dim=2).half() for b in levels[1:]}


def _weights(seed, tag, K, N):
    return torch.randn((N, K), generator=_gen(seed, tag, "w"), device="cuda").mul_(0.02).half()


def _captured(step):
    """`step` as a replayable HIP graph (one eager pass first loads the kernels)."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    return graph


def _prepare_step(c, seed):
    """A decode step (uniform or LUT weights) over `layers` decoder layers."""
    lut = c["path"] == "lut"
    lv, B = _levels(c), c["B"]
    width = sum(N for _, _, N in _projections(c))
    arena = torch.zeros(c["layers"] * B * width, dtype=torch.float32, device="cuda")
    calls, ys, maps, at = [], [], [], 0
    for layer in range(c["layers"]):
        for name, K, N in _projections(c):
            tag = "%s%d" % (name, layer)
            desc = g.grinqh_resolve_desc(g.make_desc(K, N, lv))
            q, s = _codes(seed, tag, K, N, lv[-1])
            pc, ps = g.grinqh_pack(desc, codes=q, scales=None if lut else s.contiguous())
            del q, s
            x = _acts(seed, tag, "x", B, K, name == "down")
            y = arena[at: at + B * N].view(B, N)
            at += B * N
            ys.append(y)
            if lut:
                tab = g.lut_table_array(desc, _tables(seed, tag, N, lv))
                th = _thresholds(c, seed, tag, K, name == "down")
                calls.append((g.grinqh_vmm_lut_threshold, (desc, pc, tab, x, th), {"y": y, "accumulate": True}))
            elif c["mode"] == "topk":
                counts = g.grinqh_topk_counts(K, BUDGETS[c["levels"]][c["bits"]])
                lm = torch.zeros((B, K), dtype=torch.uint8, device="cuda")
                maps.append(lm)
                calls.append((g.grinqh_assign, (desc, x, g.GRINQH_ASSIGN_TOPK), {"counts": counts, "out": lm}))
                calls.append((g.grinqh_vmm, (desc, pc, ps, x, lm), {"y": y, "accumulate": True}))
            else:
                th = _thresholds(c, seed, tag, K, name == "down")
                calls.append((g.grinqh_vmm_threshold, (desc, pc, ps, x, th), {"y": y, "accumulate": True}))

    def step():
        arena.zero_()
        for f, args, kw in calls:
            f(*args, **kw)

    out = {"y": ys}
    if maps:
        out["levels"] = maps
    return {"graph": _captured(step), "calls": calls, "out": out}


def prepare(case, seed):
    c, path = case, case["path"]
    if path in ("decode", "lut"):
        return {"path": path, **_prepare_step(c, seed)}
    lv = _levels(c)
    if path == "single":
        desc = g.grinqh_resolve_desc(g.make_desc(c["K"], c["N"], lv))
        q, s = _codes(seed, "w", c["K"], c["N"], lv[-1])
        pc, ps = g.grinqh_pack(desc, codes=q, scales=s)
        return {"path": path, "args": (desc, pc, ps, _acts(seed, "w", "x", c["B"], c["K"], False),
                                       _thresholds(c, seed, "w", c["K"], False))}
    if path == "prefill":
        calls = []
        for name, K, N in _projections(c):
            desc = g.grinqh_resolve_desc(g.make_desc(K, N, lv))
            q, s = _codes(seed, name, K, N, lv[-1])
            pc, ps = g.grinqh_pack(desc, codes=q, scales=s)
            del q, s
            calls.append((desc, pc, ps, _acts(seed, name, "x", c["M"], K, name == "down")))
        return {"path": path, "calls": calls}
    if path == "pack":
        desc = g.grinqh_resolve_desc(g.make_desc(c["K"], c["N"], lv))
        return {"path": path, "desc": desc, "W": _weights(seed, "w", c["K"], c["N"])}
    desc = g.grinqh_resolve_desc(g.make_desc(c["K"], 1024, lv))
    return {"path": path, "desc": desc, "x": _acts(seed, "w", "calib", c["S"], c["K"], False),
            "p": BUDGETS[c["levels"]][c["bits"]]}


def run(state):
    path = state["path"]
    if path in ("decode", "lut"):
        state["graph"].replay()
        return state["out"]
    if path == "single":
        desc, pc, ps, x, th = state["args"]
        return g.grinqh_vmm_threshold(desc, pc, ps, x, th)
    if path == "prefill":
        return [g.grinqh_prefill(desc, pc, ps, x) for desc, pc, ps, x in state["calls"]]
    if path == "pack":
        return g.grinqh_pack(state["desc"], W=state["W"])
    return g.grinqh_calibrate(state["desc"], state["x"], state["p"])


# -------------------------------------------------------------------- work --
def _read_bits(c):
    """Expected bits of a weight row read: the deepest of B tokens' levels."""
    lv, p, B = _levels(c), BUDGETS[c["levels"]][c["bits"]], c["B"]
    cum, prev, out = 0.0, 0.0, 0.0
    for b, bp in zip(lv, p):
        cum += bp / 10000.0
        out += b * (cum ** B - prev ** B)
        prev = cum
    return out


def _vmm_work(c, K, N):
    p, B = BUDGETS[c["levels"]][c["bits"]], c["B"]
    active = 1.0 - p[0] / 10000.0
    lut = c["path"] == "lut"
    # codes, scales (or the tables of the levels in use), x, y
    side = N * 2 * sum(1 << b for b, bp in zip(_levels(c)[1:], p[1:]) if bp) if lut else K // GROUP * N * 2
    return K * N * _read_bits(c) / 8 + side + 2 * B * K + 4 * B * N, 2.0 * B * active * K * N


def work(case):
    c, path = case, case["path"]
    if path in ("decode", "lut"):
        w = [_vmm_work(c, K, N) for _, K, N in _projections(c)] * c["layers"]
    elif path == "single":
        w = [_vmm_work(c, c["K"], c["N"])]
    elif path == "prefill":
        b, M = _levels(c)[-1], c["M"]
        w = [(K * N * b / 8 + K // GROUP * N * 2 + 2 * M * K + 4 * M * N, 2.0 * M * K * N)
             for _, K, N in _projections(c)]
    elif path == "pack":
        K, N, b = c["K"], c["N"], _levels(c)[-1]
        w = [(2 * K * N + K * N * b / 8 + K // GROUP * N * 2, 0)]
    else:
        w = [(2 * c["S"] * c["K"] + 4 * (len(_levels(c)) - 1), 0)]
    return {"bytes": float(sum(b for b, _ in w)), "flops": float(sum(f for _, f in w))}


def tolerance(case):
    path = case["path"]
    if path in ("pack", "calibrate"):
        return "exact"   # bytes, and thresholds in a fixed order of float64 operations
    if path == "prefill":
        # weights rounded once to fp16: 2^-11 at most per weight, about 2e-4 in the sum
        return {"rel": 8e-4}
    if path == "lut":
        # fp32 sums of exact products in any order: 1.3e-7 seen
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}
    # the same sums, with the codes' offsets taken out at the end of a group:
    # up to 1.8e-5 from float64 seen (1-bit planes, B = 4)
    return {"rel": 6e-5, "max": 5e-4, "differ": 0.0}


# ------------------------------------------------------------------- exact --
def _assign_topk(x, counts):
    """Level per channel: |x| descending, ties to the lower channel."""
    order = x.abs().double().sort(dim=1, descending=True, stable=True).indices
    lv = torch.cat([torch.full((n,), j, dtype=torch.uint8, device=x.device)
                    for j, n in reversed(list(enumerate(counts)))])
    out = torch.empty(x.shape, dtype=torch.uint8, device=x.device)
    for t in range(x.shape[0]):
        out[t, order[t]] = lv
    return out


def _counts(K, p_bp):
    C = [(sum(p_bp[j:]) * K + 5000) // 10000 for j in range(len(p_bp))] + [0]
    return [C[j] - C[j + 1] for j in range(len(p_bp))]


def _grade(x, th):
    a = x.abs().float()
    return sum((a >= t).to(torch.uint8) for t in torch.tensor(th, dtype=torch.float32, device=x.device))


def _exact_vmm(c, seed, tag, K, N, swiglu, topk, lut):
    lv = _levels(c)
    b_max = lv[-1]
    half = 1 << (b_max - 1)
    q, s = _codes(seed, tag, K, N, b_max)
    x = _acts(seed, tag, "x", c["B"], K, swiglu)
    if topk:
        lm = _assign_topk(x, _counts(K, BUDGETS[c["levels"]][c["bits"]]))
    else:
        lm = _grade(x, _thresholds(c, seed, tag, K, swiglu))
    tabs = _tables(seed, tag, N, lv) if lut else None
    y = torch.zeros((x.shape[0], N), dtype=torch.float64, device=x.device)
    for t in range(x.shape[0]):
        for l, b in enumerate(lv):
            cols = (lm[t] == l).nonzero().view(-1)
            if b == 0 or cols.numel() == 0:
                continue
            xb = x[t, cols].double()
            qb = q[:, cols] >> (b_max - b)
            if lut:
                w = tabs[b].double().gather(1, qb.long())
            else:
                w = qb.double().mul_(1 << (b_max - b)).add_(-half + (2.0 ** (b_max - b - 1) if b < b_max else 0.0))
                w = w.mul_(s[:, cols // GROUP].double())
            y[t] += w @ xb
    return y, lm


def exact(case, seed):
    c, path = case, case["path"]
    if path in ("decode", "lut"):
        topk = c.get("mode") == "topk"
        got = [_exact_vmm(c, seed, "%s%d" % (name, layer), K, N, name == "down", topk, path == "lut")
               for layer in range(c["layers"]) for name, K, N in _projections(c)]
        out = {"y": [y for y, _ in got]}
        if topk:
            out["levels"] = [lm for _, lm in got]
        return out
    if path == "single":
        return _exact_vmm(c, seed, "w", c["K"], c["N"], False, False, False)[0]
    if path == "prefill":
        b_max = _levels(c)[-1]
        out = []
        for name, K, N in _projections(c):
            q, s = _codes(seed, name, K, N, b_max)
            x = _acts(seed, name, "x", c["M"], K, name == "down").double()
            w = q.double().sub_(1 << (b_max - 1)).view(N, K // GROUP, GROUP).mul_(s.double().unsqueeze(2))
            out.append(x @ w.view(N, K).t().contiguous())
        return out
    if path == "pack":
        return None   # bytes: compared as they are
    samples = _acts(seed, "w", "calib", c["S"], c["K"], False)
    a = samples.abs().double().sort(dim=1).values
    K, out, U = c["K"], [], 0
    for p in BUDGETS[c["levels"]][c["bits"]][:-1]:
        U += p
        lo, num = (K - 1) * U // 10000, (K - 1) * U % 10000
        hi = min(lo + 1, K - 1)
        out.append((a[:, lo] + (num / 10000.0) * (a[:, hi] - a[:, lo])).mean())
    return torch.stack(out)
