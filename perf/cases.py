"""The work that users of this framework run, as measurable cases: whole layer shares from one-batch decode to the
bottleneck GPU of a prefill, two colocated models, the preemptive send layout, and the host planner.

A layer share is route -> traffic -> dispatch -> expert FFN over the rows that arrive -> (shared experts) -> combine,
called the way bench.py and a serving loop call it: arguments bound once, device memory kept between the calls.  The
two all-to-alls are not the framework's; the rows they bring (`recv`, `ret`) are prepared, N(0, 1) like every activation.
Shapes come from workloads/configs.py and the tests or are generic.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2410_17043_amd as P

DEV = "cuda"
SILU, GELU, SWIGLU = P.ACT_SILU_MLP, P.ACT_GELU_MLP, P.ACT_SWIGLU

# H, F, E, k, G, activation, renormalised weights, capacity factor, Zipf exponent of the expert popularity
SHAPES = {
    "tiny": dict(H=64, F=128, E=8, k=2, G=4, act=SILU, renorm=0, cap=0.0, zipf=0.0),
    "mixtral": dict(H=4096, F=14336, E=8, k=2, G=8, act=SWIGLU, renorm=1, cap=0.0, zipf=1.0),
    "switch": dict(H=1024, F=4096, E=64, k=1, G=16, act=GELU, renorm=0, cap=1.25, zipf=1.2),
    "small_moe": dict(H=2048, F=5632, E=16, k=2, G=8, act=SWIGLU, renorm=1, cap=0.0, zipf=0.0),
    "finegrained": dict(H=2048, F=1408, E=64, k=6, G=16, act=SWIGLU, renorm=0, cap=0.0, zipf=1.1),
    "odd": dict(H=1152, F=2304, E=24, k=3, G=6, act=SILU, renorm=0, cap=0.0, zipf=0.7),
    "fp32": dict(H=1024, F=2816, E=16, k=4, G=8, act=SWIGLU, renorm=1, cap=0.0, zipf=1.0),
}


def _layer(name, shape, T, R, dtype="bf16", shared=0, noalloc=False, graph=False):
    """T local tokens; R rows received by this GPU's E / G experts from G sources."""
    c = dict(name=name, kind="layer", T=T, R=R, dtype=dtype, shared=shared, noalloc=noalloc, graph=graph)
    c.update(SHAPES[shape])
    return c


def _pair(a, b):
    """Two layer shares on one GPU as one flat case."""
    return dict({"a_" + k: v for k, v in a.items() if k != "name"}, kind="pair", **{"b_" + k: v for k, v in b.items() if k != "name"})


def _half(c, which):
    return {k[2:]: v for k, v in c.items() if k.startswith(which + "_")}


def listed():
    finegrained = SHAPES["finegrained"]
    return [
        # the smallest call: a tiny fp32 share (the configuration that everything is first checked on); all launches
        _layer("tiny_fp32", "tiny", 256, 517, dtype="fp32"),
        # one decode step of a batch of 16 per GPU: every expert weight is read for a handful of rows; dispatch by the
        # entry point for loops that cannot allocate
        _layer("decode_mixtral", "mixtral", 16, 37, noalloc=True),
        # one decode step of 64 sequences per GPU, many small experts: four local experts, up to 64 segments of a few
        # rows, replayed as a HIP graph as decode loops are
        _layer("decode_finegrained", "finegrained", 64, 403, shared=2, graph=True),
        # a prompt chunk between decode and prefill
        _layer("chunk_mixtral", "mixtral", 256, 701),
        # nothing is a power of two: 24 experts top-3 over 6 GPUs, ragged rows, a plain MLP
        _layer("ragged_odd", "odd", 1013, 2741),
        # an ordinary fp32 share
        _layer("layer_fp32", "fp32", 1024, 3001, dtype="fp32"),
        # prefill of a top-1 layer with a capacity limit: short K, GELU, 64 experts, dropped tokens
        _layer("prefill_switch", "switch", 8192, 10199),
        # two models on one GPU, each on its stream
        dict(_pair(_layer("", "mixtral", 2048, 4147), _layer("", "small_moe", 4096, 8267)), name="colocated"),
        # prefill on the GPU with the most popular expert: the headline workload
        _layer("prefill_mixtral", "mixtral", 4096, 20571),
        # the same for many small experts with two shared ones: the largest
        _layer("prefill_finegrained", "finegrained", 16384, 612329, shared=2),
        # send buffer in the layout of the preemptive plan, and back: no FFN, all data movement
        dict(name="send_chunks", kind="chunks", T=16384, dtype="bf16", **finegrained),
        # the planner itself: transmission order of one all-to-all on unequal links
        dict(name="plan_order", kind="plan", G=16, E=64, T=16384, k=6, zipf=1.1, hetero=True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_layer(rng, dtype=None):
    dtype = dtype or ("fp32" if rng.random() < 0.15 else "bf16")
    shape = dict(SHAPES[rng.choice(sorted(SHAPES))])
    if dtype == "bf16" and shape["H"] < 128:
        shape["H"] = 256                                    # the bf16 FFN needs multiples of 128
    if rng.random() < 0.4:                                   # widths of no particular shape
        shape["H"], shape["F"] = 128 * rng.randint(2, 32), 128 * rng.randint(2, 56)
    if dtype == "fp32":
        shape["H"], shape["F"] = min(shape["H"], 1024), min(shape["F"], 2816)
    shape["act"] = rng.choice([shape["act"], SILU, GELU, SWIGLU])
    c = dict(kind="layer", dtype=dtype, shared=0, noalloc=rng.random() < 0.25, graph=rng.random() < 0.25, **shape)
    largest = 2 * 3 * 2048 * 1408 * 600000 if dtype == "bf16" else 5e10
    row_flops = 2 * (3 if c["act"] == SWIGLU else 2) * c["H"] * c["F"]
    c["T"] = _log_int(rng, 1, min(16384, (380 << 20) // (c["k"] * c["H"] * (2 if dtype == "bf16" else 4))))
    # what a GPU receives goes with its batch: from a quarter of the even share to several times it
    even = max(1, c["T"] * c["k"])
    c["R"] = max(1, min(int(even * math.exp(rng.uniform(math.log(0.25), math.log(6.0)))), int(largest / row_flops)))
    if c["k"] == 6 and rng.random() < 0.5:
        c["shared"] = 2
    return c


def draw(rng):
    kind = rng.choice(["layer"] * 7 + ["pair", "chunks", "plan"])
    if kind == "pair":
        a, b = _draw_layer(rng, "bf16"), _draw_layer(rng, "bf16")
        for c in (a, b):
            c.update(graph=False, noalloc=False, R=max(1, c["R"] // 2))
        return _pair(a, b)
    if kind == "chunks":
        c = _draw_layer(rng, "bf16")
        return {k: v for k, v in dict(c, kind="chunks").items() if k not in ("F", "act", "R", "shared", "noalloc", "graph")}
    if kind == "plan":
        G = rng.randint(3, 16)
        return dict(kind="plan", G=G, E=G * rng.randint(1, 8), T=_log_int(rng, 64, 16384), k=rng.randint(1, 4), zipf=rng.uniform(0.0, 1.2),
                    hetero=rng.random() < 0.5)
    return _draw_layer(rng)


# ------------------------------------------------------------------------------------------ preparation
def _tdtype(c):
    return P.TORCH_DTYPE[c["dtype"]]


def _normal(gen, rows, cols, dtype, sigma=1.0):
    out = torch.empty((rows, cols), dtype=dtype, device=DEV)
    step = max(1, (1 << 26) // cols)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        out[r:r + n] = torch.randn((n, cols), generator=gen, device=DEV) * sigma
    return out


def _popularity(c):
    p = np.arange(1, c["E"] + 1, dtype=np.float64) ** -c["zipf"]
    return p / p.sum()


def _i32(n):
    return torch.zeros(n, dtype=torch.int32, device=DEV)


def _weights(gen, H, F, act, dtype):
    return {"w1": _normal(gen, F, H, dtype, 0.02), "w_up": _normal(gen, F, H, dtype, 0.02) if act == SWIGLU else None,
            "w_down": _normal(gen, H, F, dtype, 0.02)}


def _ffn(c, recv, seg_off, seg_exp, experts, F, out):
    """Bound expert FFN and everything it needs alive."""
    table = P.expert_table(experts)
    so, se = torch.tensor(seg_off, dtype=torch.int32, device=DEV), torch.tensor(seg_exp, dtype=torch.int32, device=DEV)
    R = recv.shape[0]
    ws = torch.empty(P.moe_ffn_workspace_bytes(R, c["H"], F, c["act"], c["dtype"]), dtype=torch.uint8, device=DEV)
    return P.bind_expert_ffn(recv, R, so, se, len(seg_exp), table, c["H"], F, c["act"], c["dtype"], out, ws), (experts, table, so, se, ws)


def _capacity(c):
    return int(math.ceil(c["cap"] * c["T"] * c["k"] / c["E"])) if c["cap"] > 0 else 0


def _gate(c, gen, rng):
    """What the gate and the send buffer of a share need; a dict of tensors and handles."""
    T, H, E, k, G, dt = c["T"], c["H"], c["E"], c["k"], c["G"], _tdtype(c)
    s = {"ctx": P.MoeCtx(T, H, E, k, G, c["dtype"], c["renorm"], _capacity(c)), "x": _normal(gen, T, H, dt),
         "wg": _normal(gen, E, H, dt, 0.02), "bias": None, "e2g": (np.arange(E) // (E // G)).astype(np.int32),
         "idx": torch.zeros((T, k), dtype=torch.int32, device=DEV), "w": torch.zeros((T, k), device=DEV),
         "expert_count": _i32(E), "dest_count": _i32(G), "n_dropped": _i32(1), "order": rng.permutation(G).astype(np.int32),
         "send_buf": torch.zeros((T * k, H), dtype=dt, device=DEV), "s2r": _i32(T * k), "r2s": _i32(T * k),
         "ret": _normal(gen, T * k, H, dt), "y": torch.zeros((T, H), dtype=dt, device=DEV), "shared_out": None}
    if c["zipf"] > 0:
        s["bias"] = torch.tensor(np.log(_popularity(c)), dtype=torch.float32, device=DEV)
    s["ctx"].set_rank_reuse(True)                            # the dispatch directly follows the traffic call
    s["b_route"] = P.bind_route(s["ctx"], s["x"], s["wg"], s["bias"], s["idx"], s["w"])
    s["b_traffic"] = P.bind_traffic(s["ctx"], s["idx"], s["e2g"], s["expert_count"], s["dest_count"], s["n_dropped"])
    return s


def _share(c, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    s = _gate(c, gen, rng)
    H, F, E, G, dt = c["H"], c["F"], c["E"], c["G"], _tdtype(c)
    n_local = E // G
    s["seg_offset"], s["seg_expert"] = _i32(E + 1), _i32(E)
    if not c["noalloc"]:
        s["b_dispatch"] = P.bind_dispatch(s["ctx"], s["x"], s["idx"], s["e2g"], s["order"], s["send_buf"], s["s2r"], s["r2s"], s["seg_offset"],
                                          s["seg_expert"])
    # the received rows: source by source, expert by expert inside a source, as popular as the first GPU's experts
    pop = np.tile(_popularity(c)[:n_local], G)
    rows = rng.multinomial(c["R"], pop / pop.sum())
    keep = np.nonzero(rows)[0]
    seg_off = np.concatenate([[0], np.cumsum(rows[keep])])
    s["recv"] = _normal(gen, c["R"], H, dt)
    s["ffn_out"] = torch.zeros((c["R"], H), dtype=dt, device=DEV)
    s["b_ffn"], s["keep"] = _ffn(c, s["recv"], seg_off, keep % n_local, [_weights(gen, H, F, c["act"], dt) for _ in range(n_local)], F, s["ffn_out"])
    if c["shared"]:                                          # shared experts: one expert of their widths together, over the local tokens
        Fs = F * c["shared"]
        s["shared_out"] = torch.zeros((c["T"], H), dtype=dt, device=DEV)
        s["b_shared"], s["keep_shared"] = _ffn(c, s["x"], [0, c["T"]], [0], [_weights(gen, H, Fs, c["act"], dt)], Fs, s["shared_out"])
    s["b_combine"] = P.bind_combine(s["ctx"], s["ret"], s["s2r"], s["w"], s["shared_out"], s["y"])
    s["case"] = c
    s["outputs"] = {n: s[n] for n in ("idx", "w", "expert_count", "dest_count", "n_dropped", "send_buf", "s2r", "r2s", "seg_offset", "seg_expert",
                                      "ffn_out", "y")}
    if c["shared"]:
        s["outputs"]["shared_out"] = s["shared_out"]
    return s


def _chunks(c, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    s = _gate(c, gen, rng)
    D, B = _plan_inputs(dict(c, hetero=True), 0)             # statistics of earlier batches: the same plan whatever arrives
    plan = P.aurora_chunks(D, B, 0)
    s["plan"] = P.MoeChunkPlan(s["ctx"], s["e2g"], plan)
    nc = len(plan) + c["G"]
    s["chunk_offset"], s["piece_offset"], s["piece_expert"], s["n_pieces"] = _i32(nc + 1), _i32(nc + c["E"] + 1), _i32(nc + c["E"]), _i32(1)
    s["b_dispatch"] = P.bind_dispatch_chunks(s["ctx"], s["plan"], s["x"], s["idx"], s["send_buf"], s["s2r"], s["r2s"], s["chunk_offset"],
                                             s["piece_offset"], s["piece_expert"], s["n_pieces"])
    s["b_combine"] = P.bind_combine(s["ctx"], s["ret"], s["s2r"], s["w"], None, s["y"])
    s["case"] = c
    s["outputs"] = {n: s[n] for n in ("idx", "w", "expert_count", "dest_count", "n_dropped", "send_buf", "s2r", "r2s", "chunk_offset",
                                      "piece_offset", "piece_expert", "n_pieces", "y")}
    return s


def _plan_inputs(c, seed):
    rng = np.random.default_rng(seed + 1)
    G = c["G"]
    per_gpu = _popularity(c).reshape(G, -1).sum(axis=1)
    D = rng.multinomial(c["T"] * c["k"], per_gpu, size=G).astype(np.int64)
    return D, (rng.uniform(0.5, 1.0, size=G) if c["hetero"] else None)


def prepare(case, seed):
    if case["kind"] == "plan":
        D, B = _plan_inputs(case, seed)
        return {"case": case, "D": D, "B": B}
    if case["kind"] == "pair":
        return {"case": case, "a": _share(_half(case, "a"), seed), "b": _share(_half(case, "b"), seed + 1), "side": torch.cuda.Stream()}
    if case["kind"] == "chunks":
        return _chunks(case, seed)
    s = _share(case, seed)
    if case["graph"]:                                        # captured once, replayed every step
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _launch(s)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"], stream=side):
            _launch(s)
    return s


# ------------------------------------------------------------------------------------------ one pass
def _launch(s):
    c = s["case"]
    st = torch.cuda.current_stream().cuda_stream
    s["b_route"](st)
    s["b_traffic"](st)
    if c.get("noalloc"):
        P.moe_dispatch_noalloc((c["T"], c["H"], c["E"], c["k"], c["G"], c["dtype"], c["renorm"], _capacity(c)), s["x"], s["idx"], s["e2g"],
                               s["order"], s["send_buf"], s["s2r"], s["r2s"], s["seg_offset"], s["seg_expert"])
    else:
        s["b_dispatch"](st)
    if "b_ffn" in s:
        s["b_ffn"](st)
    if "b_shared" in s:
        s["b_shared"](st)
    s["b_combine"](st)


def run(state):
    c = state["case"]
    if c["kind"] == "plan":
        p = P.aurora_order(state["D"], state["B"])
        spare = c["G"] * c["G"] - p["n_rounds"]              # at most G^2 - 2 G + 2 rounds, as many as the traffic needs: one shape for all
        p["duration"] = np.pad(p["duration"], (0, spare))
        p["dst"] = np.pad(p["dst"], ((0, spare), (0, 0)), constant_values=-1)
        return {k: v for k, v in p.items() if isinstance(v, np.ndarray) or k in ("bmax", "port_bound", "order_time", "makespan_order", "order_source")}
    if c["kind"] == "pair":
        main, side = torch.cuda.current_stream(), state["side"]
        side.wait_stream(main)
        _launch(state["a"])
        with torch.cuda.stream(side):
            _launch(state["b"])
        main.wait_stream(side)
        return {"a": state["a"]["outputs"], "b": state["b"]["outputs"]}
    if "graph" in state:
        state["graph"].replay()
    else:
        _launch(state)
    return state["outputs"]


# ------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    if c["kind"] == "plan":
        return {"bytes": 8 * c["G"] * c["G"] + 4 * 2 * c["G"] * c["G"], "flops": 0}
    if c["kind"] == "pair":
        a, b = work(_half(c, "a")), work(_half(c, "b"))
        return {k: a[k] + b[k] for k in a}
    T, H, E, k, b = c["T"], c["H"], c["E"], c["k"], 2 if c["dtype"] == "bf16" else 4
    nbytes = T * H * b + E * H * b + 2 * T * k * H * b + T * H * b + T * k * (4 + 4 + 4 + 4)   # x, Wg, send_buf, ret, y, the index arrays
    flops = 2 * T * H * E + 2 * T * k * H
    if c["kind"] == "layer":
        mats = 3 if c["act"] == SWIGLU else 2
        n_local = min(E // c["G"], c["R"])
        nbytes += 2 * c["R"] * H * b + n_local * mats * H * c["F"] * b
        flops += 2 * mats * H * c["F"] * c["R"]
        if c["shared"]:
            nbytes += T * H * b + mats * H * c["F"] * c["shared"] * b
            flops += 2 * mats * H * c["F"] * c["shared"] * T
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what the path shows against the same in 64 bits: bf16 rounds the intermediate and the output once each (2.4e-3,
    largest 1e-2 on the FFN output); fp32 sums of up to 2816 products in order (1.3e-6, largest 8e-6)."""
    if case["kind"] == "plan":
        return {"rel": 1e-9, "differ": 0.0}                  # the order and the rounds are whole numbers: none may differ
    c = _half(case, "a") if case["kind"] == "pair" else case
    if c["dtype"] == "fp32":
        return {"rel": 5e-6, "max": 3.2e-5, "differ": 0.0}
    return {"rel": 9.5e-3, "max": 4e-2, "differ": 0.0}
