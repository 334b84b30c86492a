"""Parity of the HIP path (through the C ABI) with the CPU oracle on the same seeded inputs.

Integer results (indices, counts, permutation, copied rows) must be bit-exact.  Floating
point: fp32 within 1e-5, bf16 within 2e-2, both as max|diff| / max|ref| per tensor.
"""
import dataclasses
import itertools

import numpy as np
import pytest
import torch

import workloads as W
from oracle import moe_layer as O

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "bf16": 2e-2}


@pytest.fixture(scope="module")
def H():
    from tests import harness
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return harness


def small(name, **kw):
    return W.scaled(W.get_config(name), **kw)


# reduced shapes the oracle finishes in seconds; several tiles and ragged tails everywhere
ROUTE_CASES = [
    W.get_config("c1_tiny_fp32"),
    small("c1_tiny_fp32", T=3, H=4, E=2, k=1, G=2),
    small("c1_tiny_fp32", T=37, H=100, E=5, k=3, G=5),
    small("c2_mixtral", T=203, H=1032),
    small("c2_mixtral", T=64, H=4096),
    small("c3_switch", T=517, H=256),
    small("c4b_coloc", T=130, H=512),
    small("c5_finegrained", T=301, H=512),
    small("c5_finegrained", T=65, H=264, E=160, k=9, G=16),
    small("c1_tiny_fp32", T=50, H=36, E=200, k=16, G=8),
    small("c2_mixtral", T=33, H=64, E=24, k=4, G=8),
    small("c2_mixtral", T=17, H=8, E=17, k=2, G=1),              # one 16-byte chunk per row, one expert past a tile
    small("c5_finegrained", T=100, H=520, E=65, k=6, G=5),       # second pass of 64 experts holds a single expert
    small("c3_switch", T=40, H=1024, E=256, k=16, G=64),         # the limits of E, k and G
    # both sides of where two token tiles share a block; k = E; more choices than lanes of the four-lane selection
    small("c2_mixtral", T=4096, H=96, E=24, k=4, G=8),
    small("c2_mixtral", T=4097, H=96, E=24, k=4, G=8),
    small("c3_switch", T=4113, H=64, E=33, k=1, G=3),
    small("c5_finegrained", T=20, H=64, E=33, k=16, G=3),
    small("c2_mixtral", T=12801, H=32, E=18, k=16, G=6),
    small("c2_mixtral", T=12801, H=32, E=40, k=9, G=8),
    # more than 64 experts: one, two and four waves per block
    small("c2_mixtral", T=33, H=32, E=256, k=2, G=8),
    small("c2_mixtral", T=18, H=96, E=65, k=4, G=5),
    small("c2_mixtral", T=18, H=160, E=128, k=1, G=8),
    # ... and in fp64: a wave per token while there is one for each, then 16 lanes
    small("c1_tiny_fp32", T=1, H=100, E=65, k=16, G=5),
    small("c1_tiny_fp32", T=8, H=512, E=256, k=7, G=8),
    small("c1_tiny_fp32", T=9, H=512, E=256, k=7, G=8),
    small("c1_tiny_fp32", T=18, H=512, E=130, k=2, G=2),
]


def route_inputs(cfg):
    inp = W.make_layer_inputs(cfg)
    if inp["gate_bias"] is None and cfg.index % 2 == 1:
        inp["gate_bias"] = np.linspace(-0.5, 0.5, cfg.E).astype(np.float32)
    return inp


@pytest.mark.parametrize("cfg", ROUTE_CASES, ids=lambda c: "%s-T%d-H%d-E%d-k%d" % (c.name, c.T, c.H, c.E, c.k))
def test_route(H, cfg):
    inp = route_inputs(cfg)
    idx_ref, w_ref, z = O.route(inp["x"], inp["w_gate"], inp["gate_bias"], cfg.k, cfg.renorm)
    margin = O.route_margin(z, cfg.k).min()
    assert margin > 1e-9, "seed gives a near tie; bit-exact indices would not be meaningful"
    sh = H.Share(cfg)
    x, wg = H.dev(inp["x"], cfg.dtype), H.dev(inp["w_gate"], cfg.dtype)
    bias = None if inp["gate_bias"] is None else torch.from_numpy(inp["gate_bias"]).to(H.DEV)
    sh.route(x, wg, bias)
    torch.cuda.synchronize()
    assert np.array_equal(H.host(sh.idx), idx_ref)
    assert H.rel_err(H.host(sh.w), w_ref) < 1e-5
    assert np.max(np.abs(H.host(sh.w) / w_ref - 1.0)) < 1e-5


def lane_tree(v):
    """fp32 sum along the last axis (up to 16 values) in the order of 16 lanes that exchange at distances 8, 4, 2, 1."""
    v = np.concatenate([v, np.zeros(v.shape[:-1] + (16 - v.shape[-1],), np.float32)], axis=-1)
    while v.shape[-1] > 1:
        h = v.shape[-1] // 2
        v = v[..., :h] + v[..., h:]
    return v


@pytest.mark.parametrize("T", [333, 3])
@pytest.mark.parametrize("E,k,dtype,H_", [(16, 4, "fp32", 64), (5, 5, "fp32", 36), (64, 16, "fp32", 100), (200, 9, "fp32", 36), (24, 3, "bf16", 40)])
def test_renormalised_weights_of_the_fp32_gate_are_quotients_rounded_once(H, T, E, k, dtype, H_):
    """With the probabilities p (renorm = 0) of the same inputs: w = fl(p / sum p), to the bit."""
    cfg = small("c1_tiny_fp32", T=T, H=H_, E=E, k=k, G=1)
    cfg = dataclasses.replace(cfg, dtype=dtype, renorm=0)
    r = np.random.default_rng(E)
    x, wg = H.dev(r.standard_normal((cfg.T, H_)), dtype), H.dev(0.2 * r.standard_normal((E, H_)), dtype)
    got = {}
    for renorm in (0, 1):
        sh = H.Share(dataclasses.replace(cfg, renorm=renorm))
        sh.route(x, wg, None)
        torch.cuda.synchronize()
        got[renorm] = H.host(sh.w)
    assert np.array_equal(got[1], got[0] / lane_tree(got[0]))


@pytest.mark.parametrize("cfg", [small("c2_mixtral", T=203, H=1024), small("c5_finegrained", T=301, H=512),
                                 small("c3_switch", T=40, H=1024, E=256, k=16, G=64), small("c1_tiny_fp32", T=37, H=100, E=5, k=3, G=5)],
                         ids=lambda c: "%s-T%d-E%d-k%d" % (c.name, c.T, c.E, c.k))
def test_route_phases_diag_gives_the_results_of_moe_route_and_ordered_marks(H, cfg):
    """The timed instantiation of the gate kernel is the gate kernel: same indices and weights; its clock marks
    do not go backwards within a wave; a shape that takes the fp64 kernel reports no marks."""
    inp = route_inputs(cfg)
    sh = H.Share(cfg)
    x, wg = H.dev(inp["x"], cfg.dtype), H.dev(inp["w_gate"], cfg.dtype)
    bias = None if inp["gate_bias"] is None else torch.from_numpy(inp["gate_bias"]).to(H.DEV)
    sh.route(x, wg, bias)
    idx2, w2 = torch.full_like(sh.idx, -7), torch.full_like(sh.w, float("nan"))
    marks = torch.zeros((cfg.T // 16 + 1) * 128, dtype=torch.int64, device=H.DEV)
    tpb = H.P.moe_diag_route_phases(sh.ctx, x, wg, bias, idx2, w2, marks)
    torch.cuda.synchronize()
    assert torch.equal(idx2, sh.idx) and torch.equal(w2, sh.w)
    if cfg.dtype == "fp32" or cfg.H % 32:
        assert tpb == 0 and int(marks.abs().sum()) == 0
        return
    assert tpb in (16, 32, 64)
    nb = (cfg.T + tpb - 1) // tpb
    a = marks[:nb * 128].cpu().numpy().reshape(nb, 16, 8)
    assert int(np.abs(marks[nb * 128:].cpu().numpy()).sum()) == 0
    live = a[:, :, 0] > 0
    assert live[:, 0].all()
    t = a[:, :, :5]
    assert (np.diff(t, axis=2)[live] >= 0).all()
    ends = a[:, :, 5]
    assert ((ends == 0) | (ends >= a[:, :, 4]))[live].all()
    with pytest.raises(H.P.MoeError):
        H.P.moe_diag_route_phases(sh.ctx, x, wg, bias, idx2, w2, marks[:16])


def test_route_ties_pick_lower_index(H):
    cfg = small("c2_mixtral", T=96, H=256, E=8, k=3)
    inp = W.make_layer_inputs(cfg)
    wg = inp["w_gate"].copy()
    wg[5] = wg[1]; wg[6] = wg[1]; wg[7] = wg[2]            # duplicated gate rows: exact ties
    idx_ref, w_ref, _ = O.route(inp["x"], wg, None, cfg.k, cfg.renorm)
    sh = H.Share(cfg)
    sh.route(H.dev(inp["x"], cfg.dtype), H.dev(wg, cfg.dtype), None)
    torch.cuda.synchronize()
    assert np.array_equal(H.host(sh.idx), idx_ref)
    assert H.rel_err(H.host(sh.w), w_ref) < 1e-5


@pytest.mark.parametrize("E,k,H_", [(8, 2, 1024), (65, 6, 520), (160, 9, 264)])
def test_route_near_ties_take_the_exact_path(H, E, k, H_):
    """Gate rows that differ from one another in a single element by one bf16 step: every gap
    between logits is far below what fp32 accumulation resolves, yet far above fp64 rounding,
    so the indices are well defined and any kernel that decides them from approximate logits
    must fall back to exact ones for (nearly) every token."""
    cfg = small("c2_mixtral", T=150, H=H_, E=E, k=k, G=1)
    inp = W.make_layer_inputs(cfg)
    base = inp["w_gate"][0].astype(np.float32)
    wg = np.tile(base, (E, 1))
    for e in range(1, E):
        j = (7 * e) % H_
        bits = wg[e, j:j + 1].view(np.uint32)
        bits += np.uint32((1 + e // H_) << 16)               # next bf16 value(s) away from zero
    idx_ref, w_ref, z = O.route(inp["x"], wg, None, cfg.k, cfg.renorm)
    margin = O.route_margin(z, cfg.k)
    assert margin.max() < 1e-2
    ok = margin > 1e-9          # bf16 values have few bits, so some products coincide exactly: those tokens are skipped
    assert ok.mean() > 0.5
    sh = H.Share(cfg)
    sh.route(H.dev(inp["x"], cfg.dtype), H.dev(wg, cfg.dtype), None)
    torch.cuda.synchronize()
    assert np.array_equal(H.host(sh.idx)[ok], idx_ref[ok])
    assert H.rel_err(H.host(sh.w)[ok], w_ref[ok]) < 1e-5


DISPATCH_CASES = [
    (W.get_config("c1_tiny_fp32"), 0),
    (small("c1_tiny_fp32", T=1, H=4, E=2, k=1, G=2), 0),
    (small("c2_mixtral", T=1500, H=520), 0),
    (small("c3_switch", T=3000, H=128), None),             # config's own capacity (scaled with T)
    (small("c3_switch", T=2100, H=64), 7),
    (small("c5_finegrained", T=1111, H=136), 0),
    (small("c5_finegrained", T=700, H=64, E=160, k=9, G=16), 30),
    # more than 8192 slots: many blocks count
    (small("c5_finegrained", T=3100, H=64), 0),
    (small("c3_switch", T=20011, H=32), None),
    (small("c2_mixtral", T=8193, H=64), 0),               # 16386 slots, the last block of 1024 nearly empty
    (small("c2_mixtral", T=8192, H=64), 0),               # 16384 slots, the last one full
    (small("c2_mixtral", T=4097, H=64), 0),               # 8194 slots, just over the single-block limit
    (small("c2_mixtral", T=4096, H=64), 0),               # 8192 slots, the single-block limit itself
    # row lengths that pick the other copy geometries: several short rows per wave (1, 2, 4 KB rows; a ragged
    # last wave), rows longer than a wave's 8 KB cut into pieces (a whole number of pieces and a ragged one)
    (small("c2_mixtral", T=203, H=512), 0),               # 1 KB rows: 8 tokens per wave
    (small("c3_switch", T=517, H=1024), 9),               # 2 KB rows, k = 1: 4 tokens per wave, dropped slots
    (small("c5_finegrained", T=131, H=512), 0),           # 1 KB rows to 6 slots: 2 tokens per wave
    (small("c4b_coloc", T=99, H=2048), 0),                # 4 KB rows: 2 tokens per wave
    (small("c2_mixtral", T=77, H=8192), 0),               # 16 KB rows: two pieces
    (small("c1_tiny_fp32", T=50, H=2304, E=5, k=3, G=5), 0),   # 9 KB rows: a full piece and a 1 KB one
]


@pytest.mark.parametrize("cfg,cap", DISPATCH_CASES, ids=lambda v: getattr(v, "name", str(v)))
def test_traffic_and_dispatch(H, cfg, cap):
    if cap is not None:
        cfg = dataclasses.replace(cfg, capacity_factor=0.0)
    capacity = cfg.capacity if cap is None else cap
    inp = W.make_layer_inputs(cfg)
    idx_ref, _, _ = O.route(inp["x"], inp["w_gate"], inp["gate_bias"], cfg.k, cfg.renorm)
    e2g = inp["expert_to_gpu"]
    r = np.random.default_rng(cfg.seed_base)
    orders = [list(range(cfg.G)), list(r.permutation(cfg.G))]
    if cfg.name == "c1_tiny_fp32" and cfg.G == 4:
        orders = list(itertools.permutations(range(4)))     # all 24 transmission orders
    sh = H.Share(cfg)
    sh.ctx.close()
    sh.ctx = H.P.MoeCtx(cfg.T, cfg.H, cfg.E, cfg.k, cfg.G, cfg.dtype, cfg.renorm, capacity)
    x = H.dev(inp["x"], cfg.dtype)
    sh.idx.copy_(torch.from_numpy(idx_ref))
    ec, dc, nd, _ = O.traffic(idx_ref, e2g, cfg.G, capacity)
    sh.traffic(e2g)
    torch.cuda.synchronize()
    assert np.array_equal(H.host(sh.expert_count), ec)
    assert np.array_equal(H.host(sh.dest_count), dc)
    assert int(sh.n_dropped.item()) == nd
    if capacity:
        assert nd > 0
    for order in orders:
        ref = O.dispatch(inp["x"], idx_ref, e2g, order, capacity)
        sh.slot_to_row.fill_(-7); sh.row_to_slot.fill_(-7); sh.send_buf.zero_()
        sh.dispatch(x, e2g, order)
        torch.cuda.synchronize()
        n = ref["n_rows"]
        assert np.array_equal(H.host(sh.slot_to_row), ref["slot_to_row"])
        assert np.array_equal(H.host(sh.row_to_slot)[:n], ref["row_to_slot"])
        assert np.all(H.host(sh.row_to_slot)[n:] == -7)                    # nothing written past the kept rows
        assert np.array_equal(H.host(sh.seg_offset), ref["seg_offset"])
        assert np.array_equal(H.host(sh.seg_expert), ref["seg_expert"])
        assert np.array_equal(H.host(sh.send_buf)[:n], ref["send_buf"])    # bitwise row copies
        assert not H.host(sh.send_buf)[n:].any()
    # determinism: a second run gives the same bytes
    a = sh.slot_to_row.clone()
    sh.dispatch(x, e2g, orders[-1])
    torch.cuda.synchronize()
    assert torch.equal(a, sh.slot_to_row)


@pytest.mark.parametrize("cfg", [small("c2_mixtral", T=700, H=264), small("c5_finegrained", T=3000, H=64)],
                         ids=lambda c: c.name)
def test_dispatch_alone_and_after_in_place_index_rewrite(H, cfg):
    """moe_dispatch never depends on an earlier call unless rank reuse was switched on; with reuse on, the
    ranks of a moe_traffic serve exactly one directly following dispatch on the same index array."""
    inp = W.make_layer_inputs(cfg)
    e2g = inp["expert_to_gpu"]
    order = list(np.random.default_rng(3).permutation(cfg.G))
    idx_a, _, _ = O.route(inp["x"], inp["w_gate"], inp["gate_bias"], cfg.k, cfg.renorm)
    idx_b = np.ascontiguousarray(idx_a[::-1])                      # a different, still valid, routing
    x = H.dev(inp["x"], cfg.dtype)
    sh = H.Share(cfg)

    def check(idx_ref):
        ref = O.dispatch(inp["x"], idx_ref, e2g, order, cfg.capacity)
        torch.cuda.synchronize()
        assert np.array_equal(H.host(sh.slot_to_row), ref["slot_to_row"])
        assert np.array_equal(H.host(sh.seg_offset), ref["seg_offset"])
        assert np.array_equal(H.host(sh.send_buf)[:ref["n_rows"]], ref["send_buf"])

    sh.idx.copy_(torch.from_numpy(idx_a))
    sh.dispatch(x, e2g, order)                                     # fresh context: ranks computed inside
    check(idx_a)
    # default (no reuse): indices rewritten in place behind the library's back, no invalidate: still right
    sh.traffic(e2g)
    sh.idx.copy_(torch.from_numpy(idx_b))
    sh.dispatch(x, e2g, order)
    check(idx_b)
    # reuse on: traffic then dispatch (one kernel) is right ...
    sh.ctx.set_rank_reuse(True)
    sh.traffic(e2g)
    sh.dispatch(x, e2g, order)
    check(idx_b)
    # ... the ranks are used once: a rewrite after that dispatch cannot reach a stale rank
    sh.idx.copy_(torch.from_numpy(idx_a))
    sh.dispatch(x, e2g, order)
    check(idx_a)
    # ... a rewrite between traffic and dispatch is the caller's to announce
    sh.traffic(e2g)
    sh.idx.copy_(torch.from_numpy(idx_b))
    sh.ctx.invalidate()
    sh.dispatch(x, e2g, order)
    check(idx_b)
    # ... and ranks made for another pointer are never used
    sh.traffic(e2g)
    other = sh.idx.clone()
    other.copy_(torch.from_numpy(idx_a))
    H.P.moe_dispatch(sh.ctx, x, other, e2g, order, sh.send_buf, sh.slot_to_row, sh.row_to_slot, sh.seg_offset,
                     sh.seg_expert)
    check(idx_a)
    # ... nor after a moe_route on the context (it rewrites the indices)
    sh.idx.copy_(torch.from_numpy(idx_b))
    sh.traffic(e2g)
    sh.route(x, H.dev(inp["w_gate"], cfg.dtype), None if inp["gate_bias"] is None else torch.from_numpy(inp["gate_bias"]).float().to(H.DEV))
    sh.dispatch(x, e2g, order)
    check(idx_a)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("E,k,masked", [(8, 2, 3), (8, 2, 6), (24, 3, 20), (64, 6, 58), (200, 9, 150)])
@pytest.mark.parametrize("T", [37, 13000])
def test_route_leaves_out_experts_with_a_bias_of_minus_infinity(H, T, E, k, masked, dtype):
    """Masked experts are as good as absent, also where exactly k are left; so is a bias that sets logits 1e-9 of themselves apart
    (closer than fp32 numbers are): the same choice as that of fp64 logits of the experts that are left."""
    P = H.P
    Hd = 64 if T > 1000 else 96
    r = np.random.default_rng(E + k)
    x = W.round_to_dtype(r.standard_normal((T, Hd)).astype(np.float32), dtype)
    wg = W.round_to_dtype((r.standard_normal((E, Hd)) * 0.02).astype(np.float32), dtype)
    left = np.sort(r.permutation(E)[masked:])
    wg[left[1::2]] = wg[left[0:2 * (len(left) // 2):2]]         # pairs of equal rows: only the bias tells them apart
    bias = np.full(E, -np.inf, np.float32)
    bias[left] = np.float32(1e-9) * r.permutation(len(left))
    z = x.astype(np.float64) @ wg[left].astype(np.float64).T + bias[left].astype(np.float64)
    idx_ref = left[np.argsort(-z, axis=1, kind="stable")[:, :k]]
    zk = -np.sort(-z, axis=1)
    clear = np.min(zk[:, :-1] - zk[:, 1:], axis=1) > 1e-12 if len(left) > 1 else np.ones(T, bool)
    assert clear.mean() > 0.99
    ctx = P.MoeCtx(T, Hd, E, k, 1, dtype, 0, 0)
    idx = torch.zeros((T, k), dtype=torch.int32, device=H.DEV)
    w = torch.zeros((T, k), device=H.DEV)
    P.moe_route(ctx, H.dev(x, dtype), H.dev(wg, dtype), torch.from_numpy(bias).to(H.DEV), idx, w)
    torch.cuda.synchronize()
    assert np.array_equal(H.host(idx)[clear], idx_ref[clear])
    p = np.exp(z - z.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    assert H.rel_err(H.host(w), -np.sort(-p, axis=1)[:, :k]) < 1e-5
    ctx.close()


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,E,k", [(300, 8, 4), (300, 16, 5), (300, 24, 4), (5000, 24, 5), (14000, 30, 4), (300, 64, 6), (5000, 64, 6), (14000, 64, 4), (300, 160, 6)])
@pytest.mark.parametrize("what", ["common bias", "too few left", "too few above the lowest"])
def test_route_orders_logits_that_rounding_cannot_tell_apart(H, T, E, k, what, dtype):
    """Pairs of logits that are 2^-26 apart, which the sum of 32 products next to 1 loses: all logits on one fp32 number by a common
    bias, or fewer experts than choices left by the bias (the others follow by index).  Every logit is exact in fp64."""
    P = H.P
    r = np.random.default_rng(E * k)
    x, wg = np.zeros((T, 128), np.float32), np.zeros((E, 128), np.float32)
    x[:, 0] = x[:, 32] = 1.0
    x[:, 1] = 2.0 ** -13
    x[np.arange(T), 33 + r.integers(0, 95, size=T)] = r.choice([1.0, -1.0, 0.5], size=T)
    wg[:, 0], wg[:, 32] = 1.0, -1.0
    for h in range(33, 128):                                     # up to 2^-5: less than half a spacing of 2^20
        wg[:, h] = 2.0 ** -13 * r.permutation(np.arange(E) // 2 * (256 // E) + 1)
    wg[r.permutation(E)[:E // 2], 1] = 2.0 ** -13
    wg[1], wg[0, 33:] = wg[E - 1], 2.0 ** -5
    wg[1, 1], wg[E - 1, 1] = 0.0, 2.0 ** -13
    bias = np.full(E, {"common bias": (-1) ** k * 2.0 ** 20, "too few left": -np.inf, "too few above the lowest": np.finfo(np.float32).min}[what], np.float32)
    if what != "common bias":
        bias[np.concatenate([[0, 1, E - 1], 2 + r.permutation(E - 3)])[:k - 1]] = 0.0
    z = x.astype(np.float64) @ wg.astype(np.float64).T + bias.astype(np.float64)
    idx_ref = np.argsort(-z, axis=1, kind="stable")[:, :k]
    p = np.exp(z - z.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    ctx = P.MoeCtx(T, 128, E, k, 1, dtype, 0, 0)
    idx = torch.zeros((T, k), dtype=torch.int32, device=H.DEV)
    w = torch.zeros((T, k), device=H.DEV)
    P.moe_route(ctx, H.dev(x, dtype), H.dev(wg, dtype), torch.from_numpy(bias).to(H.DEV), idx, w)
    torch.cuda.synchronize()
    assert np.array_equal(H.host(idx), idx_ref)
    assert H.rel_err(H.host(w), np.take_along_axis(p, idx_ref, axis=1)) < 1e-5
    ctx.close()


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,E,k", [(40, 8, 2), (300, 24, 4), (5000, 64, 6), (14000, 30, 3), (14000, 64, 6), (40, 160, 6)])
def test_route_rows_with_nan_or_infinities_change_no_other(H, T, E, k, dtype):
    """A few tokens whose logits are no numbers, among tokens of zeros (all logits equal: the first k experts) and ordinary ones."""
    r = np.random.default_rng(T + E)
    x, wg = W.round_to_dtype(r.standard_normal((T, 96)).astype(np.float32), dtype), W.round_to_dtype(r.standard_normal((E, 96)).astype(np.float32), dtype)
    kind = r.integers(0, 6, size=T)
    x[kind == 0] = 0.0
    odd = x.copy()
    odd[kind == 1, 3], odd[kind == 2, 50], odd[kind == 3, 7] = np.nan, np.inf, -np.inf
    got = []
    for rows in (x, odd):
        ctx = H.P.MoeCtx(T, 96, E, k, 1, dtype, 1, 0)
        idx, w = torch.full((T, k), -7, dtype=torch.int32, device=H.DEV), torch.full((T, k), -7.0, device=H.DEV)
        H.P.moe_route(ctx, H.dev(rows, dtype), H.dev(wg, dtype), None, idx, w)
        torch.cuda.synchronize()
        got.append((H.host(idx), H.host(w)))
        ctx.close()
    same = (kind == 0) | (kind > 3)
    assert np.array_equal(got[0][0][same], got[1][0][same]) and np.array_equal(got[0][1][same], got[1][1][same])
    assert np.array_equal(got[1][0][kind == 0], np.tile(np.arange(k), (int((kind == 0).sum()), 1)))
    z = x.astype(np.float64) @ wg.astype(np.float64).T
    assert np.array_equal(got[0][0], np.argsort(-z, axis=1, kind="stable")[:, :k])


@pytest.mark.parametrize("T,k,E,cap", [
    (1, 1, 2, 0), (64, 1, 64, 1), (65, 3, 17, 9), (256, 2, 64, 0), (512, 1, 3, 100),        # lists that every wave of the scatter counts
    (171, 3, 16, 0), (100, 2, 65, 0),                                                         # one slot or one expert too many for that
    (1025, 1, 2, 0), (2048, 2, 3, 700), (4097, 1, 4, 0), (4096, 2, 3, 0), (10240, 1, 4, 0), (10241, 1, 4, 0),   # a ballot per expert, and not
    (6144, 2, 3, 0), (12289, 1, 3, 0), (8193, 2, 2, 9000), (16384, 1, 2, 0),
    (16385, 1, 16, 900), (8200, 2, 17, 0), (8193, 2, 64, 0), (16400, 1, 65, 0),               # counts added up by every block of the rank kernel, or not
    (131072, 2, 64, 0), (131073, 2, 64, 5000),
    (131072, 2, 65, 0), (131073, 2, 65, 0), (131072, 2, 256, 1000), (131073, 2, 256, 1000),   # 256 blocks, and one more: three launches
    (524288, 2, 16, 0), (1048577, 1, 16, 70000), (1048577, 1, 3, 0)])                         # 1024, and one more
def test_ranks_of_dispatch_alone_after_traffic_and_without_allocation(H, T, k, E, cap):
    """All three ways to a send buffer against a stable sort on the host; some indices name no expert and have no row."""
    P = H.P
    cfg = small("c1_tiny_fp32", T=T, H=4, E=E, k=k, G=1)
    r = np.random.default_rng(T + E)
    pop = 1.0 / np.arange(1, E + 1)
    idx = r.choice(E, size=T * k, p=pop / pop.sum()).astype(np.int32)
    idx[r.integers(0, T * k, size=T * k // 10)] = -1
    idx[r.integers(0, T * k, size=T * k // 10)] = E
    e2g = (np.arange(E) * 2 // E).astype(np.int32) if E > 1 else np.zeros(1, np.int32)
    send_order = np.concatenate([np.nonzero(e2g == d)[0] for d in (1, 0)])
    place = np.full(E, -1)
    place[send_order] = np.arange(E)
    ok = (idx >= 0) & (idx < E)
    by_place = np.argsort(np.where(ok, place[np.clip(idx, 0, E - 1)], E), kind="stable")[:ok.sum()]   # experts in send order, slots ascending
    counts = np.bincount(idx[ok], minlength=E)
    kept = np.minimum(counts, cap) if cap else counts
    start, off = np.cumsum(counts[send_order]) - counts[send_order], np.concatenate([[0], np.cumsum(kept[send_order])])
    slot_to_row = np.full(T * k, -1)
    for p in range(E):
        rows = by_place[start[p]:start[p] + kept[send_order[p]]]
        slot_to_row[rows] = off[p] + np.arange(len(rows))
    shape = (T, 4, E, k, 2, "fp32", 0, cap)
    x = torch.arange(T * 4, dtype=torch.float32, device=H.DEV).reshape(T, 4)
    di = torch.from_numpy(idx.reshape(T, k)).to(H.DEV)
    i32 = lambda n: torch.full((n,), -7, dtype=torch.int32, device=H.DEV)
    for way in ("alone", "traffic", "noalloc"):
        if way == "noalloc" and T * k > 1 << 20:                 # more than it has room for
            continue
        out = [torch.zeros((T * k, 4), device=H.DEV), i32(T * k), i32(T * k), i32(E + 1), i32(E)]
        with_ctx = P.MoeCtx(*shape)
        if way == "noalloc":
            P.moe_dispatch_noalloc(shape, x, di, e2g, [1, 0], *out)
        else:
            if way == "traffic":
                with_ctx.set_rank_reuse(True)
                ec, dc, nd = i32(E), i32(2), i32(1)
                P.moe_traffic(with_ctx, di, e2g, ec, dc, nd)
            P.moe_dispatch(with_ctx, x, di, e2g, [1, 0], *out)
        torch.cuda.synchronize()
        if way == "traffic":
            assert np.array_equal(H.host(ec), kept) and int(nd.item()) == counts.sum() - kept.sum()
            assert np.array_equal(H.host(dc), [kept[e2g == d].sum() for d in (0, 1)])
        send_buf, s2r, r2s, seg_off, seg_exp = [H.host(t) for t in out]
        assert np.array_equal(seg_off, off) and np.array_equal(seg_exp, send_order), way
        assert np.array_equal(s2r, slot_to_row), way
        has = np.nonzero(slot_to_row >= 0)[0]
        assert np.array_equal(r2s[slot_to_row[has]], has) and np.all(r2s[off[-1]:] == -7), way
        assert np.array_equal(send_buf[slot_to_row[has], 0], 4.0 * (has // k)), way
        with_ctx.close()


CHUNK_CASES = [small("c2_mixtral", T=300, H=264), small("c3_switch", T=700, H=128), small("c5_finegrained", T=260, H=64),
               small("c3_switch", T=40, H=64),                 # most experts get no token at all
               small("c1_tiny_fp32", T=37, H=100, E=5, k=3, G=5), small("c5_finegrained", T=3000, H=64, E=160, k=9, G=16),
               small("c2_mixtral", T=203, H=512), small("c3_switch", T=517, H=1024),      # several short rows per wave
               small("c2_mixtral", T=77, H=8192)]                                          # long rows in pieces


@pytest.mark.parametrize("cfg", CHUNK_CASES, ids=lambda c: "%s-T%d-E%d-k%d-G%d" % (c.name, c.T, c.E, c.k, c.G))
def test_dispatch_chunks(H, cfg):
    """Send buffer in the layout of a preemptive plan: bit-exact against the oracle for plans that
    cover too little, too much, nothing, name no GPU, and for the plan of the Appendix A rounds."""
    P = H.P
    inp = W.make_layer_inputs(cfg)
    idx_ref, _, _ = O.route(inp["x"], inp["w_gate"], inp["gate_bias"], cfg.k, cfg.renorm)
    e2g = inp["expert_to_gpu"]
    _, dc, _, _ = O.traffic(idx_ref, e2g, cfg.G, cfg.capacity)
    r = np.random.default_rng(cfg.seed_base + 9)
    plans = [[], [(g, 10 ** 9) for g in r.permutation(cfg.G)]]
    plans.append([(int(r.integers(-1, cfg.G + 1)), int(r.integers(-2, max(2, 2 * dc.max() // 3)))) for _ in range(40)])
    plans.append([(int(r.integers(0, cfg.G)), int(r.integers(0, 9))) for _ in range(4096)])     # the largest plan allowed
    # the traffic matrix of the workload with this GPU's measured row, planned by the library
    g = 0
    D = np.array(W.make_traffic_matrix(cfg)["D"], dtype=np.int64)
    D[g] = dc
    plans.append(P.aurora_chunks(D, None, g))
    sh = H.Share(cfg)
    x = H.dev(inp["x"], cfg.dtype)
    sh.idx.copy_(torch.from_numpy(idx_ref))
    for chunks in plans:
        ref = O.dispatch_chunks(inp["x"], idx_ref, e2g, chunks, cfg.capacity)
        nc = len(chunks) + cfg.G
        plan = P.MoeChunkPlan(sh.ctx, e2g, chunks)
        co = torch.full((nc + 1,), -7, dtype=torch.int32, device=H.DEV)
        po = torch.full((nc + cfg.E + 1,), -7, dtype=torch.int32, device=H.DEV)
        pe = torch.full((nc + cfg.E,), -7, dtype=torch.int32, device=H.DEV)
        npieces = torch.zeros(1, dtype=torch.int32, device=H.DEV)
        sh.send_buf.zero_()
        sh.slot_to_row.fill_(-9)
        sh.row_to_slot.fill_(-9)
        P.moe_dispatch_chunks(sh.ctx, plan, x, sh.idx, sh.send_buf, sh.slot_to_row, sh.row_to_slot, co, po, pe, npieces)
        torch.cuda.synchronize()
        n = ref["n_rows"]
        assert np.array_equal(H.host(sh.slot_to_row), ref["slot_to_row"])
        assert np.array_equal(H.host(sh.row_to_slot)[:n], ref["row_to_slot"])
        assert np.array_equal(H.host(sh.send_buf)[:n], ref["send_buf"])                     # bitwise row copies
        assert np.array_equal(H.host(co), ref["chunk_offset"])
        m = int(npieces.item())
        assert m == len(ref["piece_expert"])
        assert np.array_equal(H.host(po)[:m + 1], ref["piece_offset"])
        assert np.array_equal(H.host(pe)[:m], ref["piece_expert"])
        plan.close()


def make_segments(r, R, nseg, n_local):
    cuts = np.sort(r.integers(0, R + 1, size=nseg - 1))
    off = [0] + [int(c) for c in cuts] + [R]
    exp = [int(v) for v in r.integers(0, n_local, size=nseg)]
    return off, exp


FFN_CASES = [
    # dtype, act, R, H, F, n_local, nseg
    ("fp32", 0, 300, 64, 128, 2, 5),
    ("fp32", 1, 77, 36, 52, 3, 4),
    ("fp32", 2, 130, 64, 128, 2, 6),
    # several turns of the fp32 ring of k-tiles, with and without a partial last one; K shorter than the ring
    ("fp32", 2, 131, 164, 228, 2, 6),
    ("fp32", 0, 65, 160, 96, 1, 1),
    ("fp32", 1, 64, 8, 40, 2, 3),
    ("bf16", 2, 700, 256, 384, 2, 5),
    ("bf16", 2, 1, 128, 128, 1, 1),
    ("bf16", 1, 523, 256, 512, 3, 7),
    ("bf16", 0, 300, 128, 256, 2, 3),
    ("bf16", 2, 1029, 512, 1408, 4, 9),
    # few tiles and a long K: the tiles of the last, mostly empty round are cut along K into pieces
    ("bf16", 2, 300, 2048, 2048, 1, 1),
    ("bf16", 1, 700, 2048, 2304, 3, 6),
    ("bf16", 0, 257, 3072, 2048, 2, 2),
    # a last round that is between a quarter and half full: two and three pieces of 64 k-tiles
    ("bf16", 2, 700, 4096, 4608, 1, 1),
    ("bf16", 2, 500, 6144, 5120, 1, 1),
    # many short segments with the experts interleaved (several sources, several local experts): tiles
    # gather rows from all segments of an expert
    ("bf16", 1, 2000, 256, 512, 4, 64),
    ("bf16", 2, 1500, 384, 256, 3, 200),
    ("bf16", 0, 900, 2048, 2304, 2, 31),                   # with pieces along K as well
    ("bf16", 2, 200, 256, 2048, 3, 1024),                  # more segments than rows, pieces along K
    ("bf16", 0, 60, 256, 2048, 3, 1024),
    ("bf16", 2, 3000, 256, 256, 64, 1024),                 # the limits: 64 local experts, 1024 segments (many of them empty)
    ("bf16", 1, 5000, 128, 256, 32, 300),
    # experts that are too large for the kernel of both GEMMs: as a small one of the same kind, on the tiles
    ("fp32", 0, 300, 64, 320, 2, 5),
    ("fp32", 2, 130, 64, 192, 2, 6),
    ("bf16", 0, 300, 128, 512, 2, 3),
    # shares of at most 64 rows: the weight-streaming kernels (64-row tiles, tiles cut along K when they are few)
    ("bf16", 2, 16, 2048, 2048, 1, 1),
    ("bf16", 2, 64, 1024, 1408, 2, 3),
    ("bf16", 1, 33, 512, 768, 1, 1),                       # GELU, one row past a 32-row MFMA tile
    ("bf16", 0, 64, 2048, 2304, 3, 9),                     # gathered tiles
    ("bf16", 2, 60, 4096, 1536, 4, 40),                    # more segments than rows in most tiles
    ("bf16", 2, 64, 256, 128, 64, 64),                     # one row per segment, 64 local experts: 64 tiles of one row
    ("bf16", 1, 50, 128, 12800, 2, 2),                     # 100 stages of K in the second GEMM, many pieces
    # just past that path
    ("bf16", 1, 65, 512, 768, 1, 1),
    ("bf16", 2, 250, 256, 128, 64, 250),
]


def takes_small(R, n_local, nseg, Hd, F, act, dtype):
    """Whether a share runs both GEMMs in one kernel."""
    from paper_2410_17043_amd import _lib
    got = _lib.load().moe_selfcheck_small(R, min(n_local, nseg, R), nseg, Hd, F, act, 1 if dtype == "bf16" else 0, 256)
    assert got in (0, 1)
    return got == 1


@pytest.mark.parametrize("dtype,act,R,Hd,F,n_local,nseg", FFN_CASES)
def test_expert_ffn(H, dtype, act, R, Hd, F, n_local, nseg):
    case = (dtype, act, R, Hd, F, n_local, nseg)
    assert takes_small(R, n_local, nseg, Hd, F, act, dtype) == (case in (("fp32", 0, 300, 64, 128, 2, 5), ("fp32", 2, 130, 64, 128, 2, 6), ("bf16", 0, 300, 128, 256, 2, 3)))
    cfg = small("c2_mixtral" if dtype == "bf16" else "c1_tiny_fp32", H=Hd, F=F, act=act, dtype=dtype)
    r = np.random.default_rng(R * 7 + F)
    recv = W.round_to_dtype(r.standard_normal((R, Hd)).astype(np.float32), dtype)
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off, exp = make_segments(r, R, nseg, n_local)
    ref = O.expert_ffn(recv, off, exp, experts, act)
    out = H.run_ffn(H.dev(recv, dtype), off, exp, [H.weights_to_dev(w, dtype) for w in experts], Hd, F, act, dtype)
    got = H.host(out)
    assert np.isfinite(got).all()
    H.assert_close(got, ref, dtype)


@pytest.mark.parametrize("which", [1, 2])
def test_ffn_phases_diag_gives_the_results_of_moe_expert_ffn_and_ordered_marks(H, which):
    """The timed instantiation of the GEMM kernel is the GEMM kernel: bitwise the same output; its clock marks do
    not go backwards; blocks that found no tile stop after the first mark; a share of the streaming kernels is refused."""
    Hd, F, R, act = 512, 1408, 700, 2
    cfg = small("c2_mixtral", H=Hd, F=F)
    r = np.random.default_rng(3)
    recv = W.round_to_dtype(r.standard_normal((R, Hd)).astype(np.float32), "bf16")
    experts = [H.weights_to_dev(W.make_expert_weights(cfg, e), "bf16") for e in range(2)]
    off, exp = make_segments(r, R, 5, 2)
    x = H.dev(recv, "bf16")
    ref = H.run_ffn(x, off, exp, experts, Hd, F, act, "bf16")
    i32 = dict(dtype=torch.int32, device=H.DEV)
    so, se = torch.tensor(off, **i32), torch.tensor(exp, **i32)
    ws = torch.empty(H.P.moe_ffn_workspace_bytes(R, Hd, F, act, "bf16"), dtype=torch.uint8, device=H.DEV)
    out = torch.full_like(ref, float("nan"))
    marks = torch.zeros(H.P.ffn_phase_marks_len(R, len(exp), Hd, F, act, which), dtype=torch.int64, device=H.DEV)
    H.P.moe_diag_ffn_phases(x, R, so, se, len(exp), experts, Hd, F, act, "bf16", out, ws, which, marks)
    torch.cuda.synchronize()
    rows = np.zeros(R, dtype=bool)
    for a, b in zip(off[:-1], off[1:]):
        rows[a:b] = True
    assert torch.equal(out[torch.from_numpy(rows).to(H.DEV)], ref[torch.from_numpy(rows).to(H.DEV)])
    a = marks.cpu().numpy().reshape(-1, 4, 4)
    ran = a[:, 0, 3] > 0                                           # blocks that had a tile (the others stop after mark 0)
    assert ran.sum() >= 3                                          # a few tiles at least
    assert (np.diff(a[ran], axis=2) >= 0).all()
    assert (a[~ran][:, :, 1:] == 0).all()
    with pytest.raises(H.P.MoeError):
        H.P.moe_diag_ffn_phases(x, R, so, se, len(exp), experts, Hd, F, act, "bf16", out, ws, which, marks[:64])
    with pytest.raises(H.P.MoeError):
        H.P.moe_diag_ffn_phases(x, 40, torch.tensor([0, 40], **i32), torch.tensor([0], **i32), 1, experts, Hd, F, act, "bf16", out, ws,
                                which, marks)


@pytest.mark.parametrize("R,Hd,F,act,which,rows", [(1000, 256, 3712, 2, 1, 128), (8000, 256, 4736, 0, 1, 128), (2217, 512, 5248, 2, 2, 192)])
def test_ffn_phases_diag_marks_every_tile(H, R, Hd, F, act, which, rows):
    """Every tile has marks: of the height that moe_expert_ffn takes with marks of ffn_phase_marks_len elements, of 256
    rows with as few as that height needs."""
    import ctypes as C
    from paper_2410_17043_amd import _lib
    got = (C.c_int32 * 2)()
    assert _lib.load().moe_selfcheck_tile_shapes(R, 1, 1, Hd, F, act, 256, got) == 0 and got[which - 1] == rows
    cfg = small("c2_mixtral", H=Hd, F=F, act=act)
    experts = [H.weights_to_dev(W.make_expert_weights(cfg, 0), "bf16")]
    x = H.dev(W.round_to_dtype(np.random.default_rng(R).standard_normal((R, Hd)).astype(np.float32), "bf16"), "bf16")
    ref = H.run_ffn(x, [0, R], [0], experts, Hd, F, act, "bf16")
    i32 = dict(dtype=torch.int32, device=H.DEV)
    so, se = torch.tensor([0, R], **i32), torch.tensor([0], **i32)
    ws = torch.empty(H.P.moe_ffn_workspace_bytes(R, Hd, F, act, "bf16"), dtype=torch.uint8, device=H.DEV)
    N, halved = (F, act == 2) if which == 1 else (Hd, False)
    for bm in (rows, 256):
        cols = (128 if bm == 128 else 256) // (2 if halved else 1)
        tiles = -(-R // bm) * -(-N // cols)
        n = H.P.ffn_phase_marks_len(R, 1, Hd, F, act, which) if bm == rows else ((-(-R // 256) + 1) * -(-N // cols) + 256) * 16
        marks, out = torch.zeros(n, dtype=torch.int64, device=H.DEV), torch.full_like(ref, float("nan"))
        H.P.moe_diag_ffn_phases(x, R, so, se, 1, experts, Hd, F, act, "bf16", out, ws, which, marks)
        torch.cuda.synchronize()
        a = marks.cpu().numpy().reshape(-1, 4, 4)
        done = int((a[:, :, 3] > 0).all(axis=1).sum())
        assert done >= tiles and (a[:tiles, :, 3] > 0).all()        # as many items as tiles, or more where some are cut
        assert torch.equal(out, ref) if bm == rows else H.rel_err(H.host(out), H.host(ref)) < 2 ** -7
    with pytest.raises(H.P.MoeError):
        H.P.moe_diag_ffn_phases(x, R, so, se, 1, experts, Hd, F, act, "bf16", out, ws, which, marks[:((-(-R // 256)) * -(-N // cols) + 100) * 16])


@pytest.mark.parametrize("F,one_kernel", [(256, True), (384, False)])
def test_expert_ffn_leaves_rows_outside_segments_untouched(H, F, one_kernel):
    assert takes_small(400, 1, 2, 128, F, 2, "bf16") == one_kernel
    cfg = small("c2_mixtral", H=128, F=F)
    r = np.random.default_rng(5)
    recv = W.to_bf16_grid(r.standard_normal((400, 128)).astype(np.float32))
    experts = [W.make_expert_weights(cfg, 0)]
    out = H.run_ffn(H.dev(recv, "bf16"), [10, 10, 300], [0, 0], [H.weights_to_dev(experts[0], "bf16")], 128, F, 2, "bf16")
    got = H.host(out)
    assert np.isnan(got[:10]).all() and np.isnan(got[300:]).all() and np.isfinite(got[10:300]).all()
    ref = O.expert_ffn(recv[10:300], [0, 290], [0], experts, 2)
    H.assert_close(got[10:300], ref, "bf16")


def test_expert_ffn_rows_beyond_the_32_bit_offsets_of_a_gathered_tile(H):
    """R * F * 2 bytes above 4 GiB: tiles may no longer gather rows from distant segments (their row offsets
    are 32-bit byte offsets), so only adjacent segments of an expert share tiles.  Sampled rows against the
    oracle, plus: no row outside the segments is written."""
    Hd, F, R, n_local = 128, 16384, 140000, 2
    assert R * F * 2 > 2 ** 32
    cfg = small("c2_mixtral", H=Hd, F=F)
    r = np.random.default_rng(99)
    recv = W.round_to_dtype(r.standard_normal((R, Hd)).astype(np.float32), "bf16")
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off = [0, 300, 300, 20000, 20100, 60000, 60001, 99000, 99000, 120000, 139000]     # the last 1000 rows: no segment
    exp = [0, 1, 1, 0, 1, 0, 1, 1, 0, 0]
    out = H.run_ffn(H.dev(recv, "bf16"), off, exp, [H.weights_to_dev(w, "bf16") for w in experts], Hd, F, 2, "bf16")
    assert torch.isnan(out[139000:]).all().item() and torch.isfinite(out[:139000]).all().item()
    rows = np.unique(np.concatenate([r.integers(0, 139000, size=150), np.array(off[:-1]), np.array(off[1:]) - 1]))
    rows = rows[(rows >= 0) & (rows < 139000)]
    seg = np.searchsorted(np.array(off), rows, side="right") - 1
    got = H.host(out[torch.from_numpy(rows).to(H.DEV)])
    ref = np.stack([O.ffn(recv[i:i + 1], experts[exp[g]]["w1"], experts[exp[g]]["w_up"], experts[exp[g]]["w_down"], 2)[0]
                    for i, g in zip(rows, seg)])
    H.assert_close(got, ref, "bf16")


@pytest.mark.parametrize("run", [1, 2])
def test_mfma_run_sum_stays_inside_the_error_model_of_the_gate(H, run):
    """The gate certifies indices with the bound |run sum - exact| <= run * 1.05 * 2^-18 * sum |x_i w_i| on what
    v_mfma_f32_16x16x32_bf16 returns.  The instruction is fed random and adversarial operands (wide exponent
    spread, one huge term among many just too small to register, cancelling giants) and held to that bound;
    the exact sums come from rationals-free fp64 (products of bf16 are exact, 64 of them add exactly enough)."""
    r = np.random.default_rng(17 + run)
    K = 32 * run
    fam = []
    a = r.standard_normal((512, 16, K)); b = 0.02 * r.standard_normal((512, 16, K)); fam.append((a, b))
    a = r.standard_normal((512, 16, K)) * 2.0 ** r.integers(-12, 13, size=(512, 16, K))
    b = r.standard_normal((512, 16, K)) * 2.0 ** r.integers(-12, 13, size=(512, 16, K)); fam.append((a, b))
    for q in range(16, 34):                                # one term 2^q, the others a hair below each power of two near its last place
        for small in (1.0, 1.9921875, 3.984375, 7.96875, 15.9375):
            a = np.full((1, 16, K), small); b = np.ones((1, 16, K))
            pos = int(r.integers(0, K))
            a[:, :, pos] = 2.0 ** (q // 2); b[:, :, pos] = 2.0 ** (q - q // 2)
            fam.append((a, b))
            a2, b2 = a.copy(), b.copy()                    # and with a cancelling partner
            a2[:, :, (pos + 5) % K] = -2.0 ** (q // 2); b2[:, :, (pos + 5) % K] = 2.0 ** (q - q // 2)
            fam.append((a2, b2))
    worst = 0.0
    for a, b in fam:
        a, b = W.to_bf16_grid(a.astype(np.float32)), W.to_bf16_grid(b.astype(np.float32))
        d = torch.empty((a.shape[0], 16, 16), dtype=torch.float32, device=H.DEV)
        H.P.moe_diag_mfma_run_sum(H.dev(a, "bf16"), H.dev(b, "bf16"), d)
        torch.cuda.synchronize()
        a64, b64 = a.astype(np.float64), b.astype(np.float64)
        exact = np.einsum("tik,tjk->tij", a64, b64)
        mass = np.einsum("tik,tjk->tij", np.abs(a64), np.abs(b64))
        worst = max(worst, float(np.max(np.abs(H.host(d).astype(np.float64) - exact) / mass)))
    print("worst |error| / sum|x w| for a chain of %d: %.3e = %.3f * 2^-18" % (run, worst, worst * 2.0 ** 18))
    assert worst <= run * 1.05 * 2.0 ** -18


COMBINE_CASES = [W.get_config("c1_tiny_fp32"), small("c2_mixtral", T=333, H=520), small("c3_switch", T=1000, H=64),
                 small("c5_finegrained", T=257, H=264),
                 # k outside 1, 2, 6: the loop kernel (a whole number of groups of four rows, a ragged one, the limit)
                 small("c2_mixtral", T=211, H=520, E=24, k=4), small("c1_tiny_fp32", T=37, H=100, E=5, k=3, G=5),
                 small("c5_finegrained", T=65, H=264, E=160, k=9, G=16), small("c3_switch", T=40, H=1024, E=256, k=16, G=64)]


@pytest.mark.parametrize("cfg", COMBINE_CASES, ids=lambda c: "%s-T%d-H%d-k%d" % (c.name, c.T, c.H, c.k))
@pytest.mark.parametrize("with_shared", [False, True])
def test_combine(H, cfg, with_shared):
    inp = W.make_layer_inputs(cfg)
    idx_ref, w_ref, _ = O.route(inp["x"], inp["w_gate"], inp["gate_bias"], cfg.k, cfg.renorm)
    cap = cfg.capacity
    d = O.dispatch(inp["x"], idx_ref, inp["expert_to_gpu"], list(range(cfg.G)), cap)
    r = np.random.default_rng(11)
    S = cfg.T * cfg.k
    ret = W.round_to_dtype(r.standard_normal((S, cfg.H)).astype(np.float32), cfg.dtype)
    shared = W.round_to_dtype(r.standard_normal((cfg.T, cfg.H)).astype(np.float32), cfg.dtype) if with_shared else None
    w32 = w_ref.astype(np.float32)
    ref = O.combine(ret[:d["n_rows"]], d["slot_to_row"], w32, shared)
    sh = H.Share(cfg)
    sh.slot_to_row.copy_(torch.from_numpy(d["slot_to_row"]))
    sh.w.copy_(torch.from_numpy(w32))
    sh.combine(H.dev(ret, cfg.dtype), None if shared is None else H.dev(shared, cfg.dtype))
    torch.cuda.synchronize()
    assert H.rel_err(H.host(sh.y), ref) < (1e-6 if cfg.dtype == "fp32" else 2 ** -8)


@pytest.mark.parametrize("k", [1, 2, 6])
@pytest.mark.parametrize("dtype,Hd", [("bf16", 4104), ("fp32", 2052)])
def test_combine_of_few_and_of_many_tokens_gives_the_same_bits(H, dtype, Hd, k):
    """1024 tokens (a wave per piece of a row) against the first 1024 of 1030 (a wave per token), rows that end inside a
    piece, dropped slots, one token with all of them dropped; and both against a plain sum."""
    P, T = H.P, 1030
    r = np.random.default_rng(k)
    ret = H.dev(W.round_to_dtype(r.standard_normal((T * k, Hd)).astype(np.float32), dtype), dtype)
    shared = H.dev(W.round_to_dtype(r.standard_normal((T, Hd)).astype(np.float32), dtype), dtype)
    rows = np.where(r.random(T * k) < 0.1, -1, r.integers(0, 1024 * k, size=T * k)).astype(np.int32)
    rows[5 * k:6 * k] = -1
    s2r, w = torch.from_numpy(rows).to(H.DEV), torch.from_numpy(r.random((T, k)).astype(np.float32)).to(H.DEV)
    got = []
    for n in (1024, T):
        ctx, y = P.MoeCtx(n, Hd, 8, k, 8, dtype, 0, 0), torch.full((n, Hd), float("nan"), dtype=ret.dtype, device=H.DEV)
        P.moe_combine(ctx, ret, s2r[:n * k], w[:n], shared[:n], y)
        got.append(H.host(y))
    assert np.array_equal(got[0], got[1][:1024])
    ref = H.host(shared).astype(np.float64)
    for j in range(k):
        sl = rows.reshape(T, k)[:, j]
        ref += np.where(sl[:, None] >= 0, H.host(w)[:, j:j + 1].astype(np.float64) * H.host(ret)[np.maximum(sl, 0)], 0.0)
    assert H.rel_err(got[1], ref) < (1e-6 if dtype == "fp32" else 2 ** -8)


# The tile heights (first GEMM, second GEMM) a share takes, with rows just past a tile edge, gathered tiles, two maps in
# one workspace, and too many segments for two maps (then both GEMMs take the first one's height).
TILE_SHAPE_CASES = [(129, 256, 1408, 1, 1, 2, (128, 128)), (385, 128, 9216, 1, 2, 2, (192, 128)), (513, 128, 9216, 2, 9, 2, (256, 128)),
                    (2000, 1024, 4608, 2, 7, 0, (192, 192)), (1151, 2048, 4608, 1, 3, 1, (128, 192)), (2500, 1024, 4608, 3, 40, 0, (256, 192)),
                    (2500, 1024, 4608, 3, 600, 0, (256, 192))]


@pytest.mark.parametrize("R,Hd,F,n_local,nseg,act,rows", TILE_SHAPE_CASES)
def test_expert_ffn_tile_heights(H, R, Hd, F, n_local, nseg, act, rows):
    from paper_2410_17043_amd import _lib
    shape_of = _lib.load().moe_selfcheck_tile_shape
    assert (shape_of(R, n_local, F, Hd, act, 256), shape_of(R, n_local, Hd, F, -1, 256)) == rows
    cfg = small("c2_mixtral", H=Hd, F=F, act=act)
    r = np.random.default_rng(R + nseg)
    recv = W.to_bf16_grid(r.standard_normal((R, Hd)).astype(np.float32))
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off, exp = make_segments(r, R, nseg, n_local)
    out = H.run_ffn(H.dev(recv, "bf16"), off, exp, [H.weights_to_dev(w, "bf16") for w in experts], Hd, F, act, "bf16")
    H.assert_close(H.host(out), O.expert_ffn(recv, off, exp, experts, act), "bf16")


# Several tiles per block: the pipeline runs from one tile into the next.  K of four k-tiles (the first trip of a tile is
# the one before its last), gathered rows and ragged last tiles in every position, N of half a tile, pieces behind whole tiles.
@pytest.mark.parametrize("R,Hd,F,n_local,nseg,act,rows", [(9001, 128, 3200, 3, 40, 2, (192, 128)), (17000, 1152, 128, 5, 20, 0, (128, 192)),
                                                          (70000, 128, 256, 2, 9, 1, (192, 128)), (2217, 512, 5248, 2, 7, 2, (256, 128)),
                                                          (5623, 512, 2176, 2, 2, 2, (256, 128))])
def test_expert_ffn_blocks_walk_through_tiles(H, R, Hd, F, n_local, nseg, act, rows):
    test_expert_ffn_tile_heights(H, R, Hd, F, n_local, nseg, act, rows)


# fp32 tiles of 64 x 64: one row past a tile, a K that is no multiple of the 32-wide k-tile, gathered tiles, N below a tile
@pytest.mark.parametrize("act,R,Hd,F,n_local,nseg", [(2, 65, 100, 68, 1, 1), (0, 129, 36, 260, 2, 9), (1, 64, 4, 4, 1, 1), (2, 300, 128, 96, 3, 64),
                                                     (0, 14900, 64, 320, 3, 64)])     # the last by a tile map, for its many tiles
def test_expert_ffn_fp32_tiles(H, act, R, Hd, F, n_local, nseg):
    cfg = small("c1_tiny_fp32", H=Hd, F=F, act=act)
    r = np.random.default_rng(R + F)
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off, exp = make_segments(r, R, nseg, n_local)
    out = H.run_ffn(H.dev(recv, "fp32"), off, exp, [H.weights_to_dev(w, "fp32") for w in experts], Hd, F, act, "fp32")
    H.assert_close(H.host(out), O.expert_ffn(recv, off, exp, experts, act), "fp32")


@pytest.mark.parametrize("nseg", [1, 63, 64, 65])
def test_expert_ffn_fp32_tiles_from_the_segment_list(H, nseg):
    """Gathered tiles, empty segments, segments of no local expert and rows outside all segments, on both sides of the
    segment count up to which the blocks work out their tiles themselves."""
    R, Hd, F, n_local = 300, 64, 96, 3
    cfg = small("c1_tiny_fp32", H=Hd, F=F, act=2)
    r = np.random.default_rng(nseg)
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off = np.sort(r.integers(3, R - 4, size=nseg + 1))
    exp = r.integers(-1, n_local + 1, size=nseg) if nseg > 1 else np.array([2])
    assert f32_rows(R, min(n_local, nseg), nseg, Hd, F, 2) == [64, 64]
    out = H.host(H.run_ffn(H.dev(recv, "fp32"), off, exp, [H.weights_to_dev(w, "fp32") for w in experts], Hd, F, 2, "fp32"))
    done, ref = np.zeros(R, dtype=bool), np.zeros((R, Hd))
    for i in range(nseg):
        if 0 <= exp[i] < n_local and off[i + 1] > off[i]:
            w = experts[exp[i]]
            done[off[i]:off[i + 1]] = True
            ref[off[i]:off[i + 1]] = O.ffn(recv[off[i]:off[i + 1]], w["w1"], w["w_up"], w["w_down"], 2)
    assert np.isnan(out[~done]).all()
    H.assert_close(out[done], ref[done], "fp32")


# Narrow tiles: every form in both GEMMs and every activation, one k-tile less than the ring and many more, tiles of one row,
# gathered tiles, beside the weight-streaming kernels, and a map of more than 64 segments
@pytest.mark.parametrize("R,Hd,F,n_local,nseg,act,forms", [
    (6, 128, 1536, 7, 16, 1, [0, 11]), (6, 1536, 128, 7, 64, 0, [11, 0]), (45, 128, 512, 1, 4, 1, [21, 11]), (45, 512, 128, 1, 1, 2, [11, 21]), (77, 128, 1280, 6, 64, 1, [21, 11]), (65, 1152, 512, 8, 64, 1, [11, 12]),
    (278, 1280, 640, 4, 13, 2, [12, 12]), (226, 640, 384, 7, 64, 2, [21, 21]), (232, 1280, 512, 8, 16, 2, [21, 22]), (298, 896, 1152, 4, 16, 2, [42, 21]),
    (360, 1408, 640, 3, 65, 2, [22, 22]), (418, 1536, 896, 6, 64, 0, [12, 42]), (906, 768, 256, 8, 65, 2, [22, 42]), (403, 2048, 1408, 4, 64, 2, [42, 42]), (65, 2048, 2816, 1, 2, 0, None), (1, 1152, 256, 1, 1, 2, [11, 11])])
def test_expert_ffn_narrow_tiles(H, R, Hd, F, n_local, nseg, act, forms):
    import ctypes as C
    from paper_2410_17043_amd import _lib
    got = (C.c_int32 * 2)()
    assert _lib.load().moe_selfcheck_narrow(R, min(n_local, nseg, R), nseg, Hd, F, act, 256, got) == 0
    assert forms is None or list(got) == forms
    cfg = small("c2_mixtral", H=Hd, F=F, act=act)
    r = np.random.default_rng(R + nseg)
    recv = W.to_bf16_grid(r.standard_normal((R, Hd)).astype(np.float32))
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off, exp = make_segments(r, R, nseg, n_local)
    out = H.host(H.run_ffn(H.dev(recv, "bf16"), off, exp, [H.weights_to_dev(w, "bf16") for w in experts], Hd, F, act, "bf16"))
    H.assert_close(out[off[0]:off[-1]], O.expert_ffn(recv, off, exp, experts, act)[off[0]:off[-1]], "bf16")


@pytest.mark.parametrize("R,lo,hi,expert", [(60, 5, 70, 0), (60, -3, 33, 0), (60, 0, 60, 1), (60, 0, 60, -1), (60, 40, 40, 0), (100, 1, 100, 0), (1, 0, 1, 0)])
def test_expert_ffn_narrow_tiles_of_one_segment(H, R, lo, hi, expert):
    """A list of one segment, whose tiles come from its offsets: clipped to the rows that there are, nothing of an unknown
    expert, no other row is written."""
    import ctypes as C
    from paper_2410_17043_amd import _lib
    got = (C.c_int32 * 2)()
    assert _lib.load().moe_selfcheck_narrow(R, 1, 1, 512, 128, 2, 256, got) == 0 and got[0] and got[1]
    cfg = small("c2_mixtral", H=512, F=128, act=2)
    recv = W.to_bf16_grid(np.random.default_rng(R).standard_normal((R, 512)).astype(np.float32))
    w = W.make_expert_weights(cfg, 0)
    out = H.host(H.run_ffn(H.dev(recv, "bf16"), [lo, hi], [expert], [H.weights_to_dev(w, "bf16")], 512, 128, 2, "bf16"))
    lo, hi = max(lo, 0), min(hi, R) if expert == 0 else max(lo, 0)
    assert np.isnan(out[:lo]).all() and np.isnan(out[hi:]).all()
    if hi > lo:
        H.assert_close(out[lo:hi], O.ffn(recv[lo:hi], w["w1"], w["w_up"], w["w_down"], 2), "bf16")


# Grids that are numbered in strips (192 to 3000 tiles, no thicker bands of N, K of 640 and more; the first two have a K of 128 and stay in bands): the numbers come from either map kernel, for one GEMM, the
# other or both, with one height and with two; strips of two widths, a last round that is cut along K behind whole tiles.
@pytest.mark.parametrize("R,Hd,F,n_local,nseg,act,strips", [(3300, 128, 1024, 3, 12, 0, (0, 0)), (3300, 1024, 128, 3, 100, 1, (0, 0)), (3300, 640, 1024, 3, 12, 0, (1, 0)),
                                                            (3300, 1024, 768, 3, 100, 1, (0, 1)), (4000, 1152, 1408, 4, 9, 2, (1, 1)), (2741, 1152, 2304, 4, 24, 0, (1, 1)),
                                                            (8500, 2048, 768, 2, 5, 0, (1, 1))])
def test_expert_ffn_grids_in_strips(H, R, Hd, F, n_local, nseg, act, strips):
    import ctypes as C
    from paper_2410_17043_amd import _lib
    got = (C.c_int32 * 2)()
    assert _lib.load().moe_selfcheck_tile_shapes(R, n_local, nseg, Hd, F, act, 256, got) == 0
    grids = [(-(-R // got[0]), -(-F // ((64 if got[0] == 128 else 128) if act == 2 else (128 if got[0] == 128 else 256)))), (-(-R // got[1]), -(-Hd // (128 if got[1] == 128 else 256)))]
    assert any(192 <= m * n <= 3000 and not (m // 8 < 4 and n // 8 > m // 8) for m, n in grids), grids
    numbered = (C.c_int32 * 2)()
    assert _lib.load().moe_selfcheck_strips(R, n_local, Hd, F, act, got, numbered) == 0
    assert tuple(numbered) == strips
    cfg = small("c2_mixtral", H=Hd, F=F, act=act)
    r = np.random.default_rng(R + nseg)
    recv = W.to_bf16_grid(r.standard_normal((R, Hd)).astype(np.float32))
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off, exp = make_segments(r, R, nseg, n_local)
    out = H.host(H.run_ffn(H.dev(recv, "bf16"), off, exp, [H.weights_to_dev(w, "bf16") for w in experts], Hd, F, act, "bf16"))
    H.assert_close(out, O.expert_ffn(recv, off, exp, experts, act), "bf16")


# 128 x 128 tiles by the two orders of their loads: the shortest loops (four and six k-tiles), the last K of the spread loads beside the first of the
# early ones, more tiles than run at a time (a block goes on to another tile behind a loop of four and of eight k-tiles), gathered tiles.
@pytest.mark.parametrize("R,Hd,F,n_local,nseg,act,early", [(300, 128, 512, 1, 1, 0, (0, 0)), (700, 256, 384, 2, 100, 2, (0, 0)), (500, 1024, 1152, 1, 3, 1, (0, 1)),
                                                           (500, 1152, 1024, 2, 80, 2, (1, 0)), (2907, 128, 1792, 5, 90, 2, (0, 1)), (2907, 256, 1792, 5, 30, 2, (0, 1))])
def test_expert_ffn_128_row_tiles_of_short_and_long_loops(H, R, Hd, F, n_local, nseg, act, early):
    import ctypes as C
    from paper_2410_17043_amd import _lib
    lib, rows, forms = _lib.load(), (C.c_int32 * 2)(), (C.c_int32 * 2)()
    assert lib.moe_selfcheck_tile_shapes(R, n_local, nseg, Hd, F, act, 256, rows) == 0 and lib.moe_selfcheck_narrow(R, n_local, nseg, Hd, F, act, 256, forms) == 0
    assert not takes_small(R, n_local, nseg, Hd, F, act, "bf16") and not any(forms) and 128 in rows
    assert [lib.moe_selfcheck_early_loads(128, K) for K in (Hd, F)] == list(early)
    cfg = small("c2_mixtral", H=Hd, F=F, act=act)
    r = np.random.default_rng(R + nseg)
    recv = W.to_bf16_grid(r.standard_normal((R, Hd)).astype(np.float32))
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off, exp = make_segments(r, R, nseg, n_local)
    out = H.host(H.run_ffn(H.dev(recv, "bf16"), off, exp, [H.weights_to_dev(w, "bf16") for w in experts], Hd, F, act, "bf16"))
    H.assert_close(out, O.expert_ffn(recv, off, exp, experts, act), "bf16")


# Both GEMMs in one kernel (32-row tiles): one row, a row less and more than a tile, several tiles; one column tile per wave and
# several, in either GEMM; rows from all over, experts in falling order (more runs than experts), segments without rows, of unknown
# experts and outside the rows.  Against the oracle, against the GEMMs by themselves (of
# the same list with empty segments behind it, more than that kernel takes), and against moe_expert_ffn_timed, which runs and times it.
@pytest.mark.parametrize("dtype,act,R,Hd,F,n_local,off,exp", [
    ("fp32", 0, 517, 64, 128, 2, None, 8), ("fp32", 2, 33, 64, 64, 1, [0, 33], [0]), ("fp32", 1, 31, 256, 64, 3, None, 5), ("fp32", 0, 1, 128, 128, 1, [0, 1], [0]),
    ("fp32", 2, 700, 64, 128, 2, [0, 90, 90, 200, 333, 700], [1, 0, 0, 1, 0]), ("fp32", 0, 300, 64, 192, 4, None, 64),
    ("bf16", 2, 300, 256, 128, 2, None, 8), ("bf16", 1, 32, 128, 128, 1, [0, 32], [0]), ("bf16", 0, 1029, 128, 256, 4, None, 64), ("bf16", 2, 8000, 128, 256, 2, None, 3),
    ("bf16", 0, 260, 256, 128, 3, [5, 60, 70, 130, 130, 300], [2, -1, 0, 1, 2]), ("bf16", 2, 65, 128, 128, 2, [0, 1, 33, 65], [1, 5, 0]),
    ("bf16", 1, 1, 128, 128, 1, [0, 1], [0]),
    # overlapping segments: more runs of one expert than experts, and more tiles than rows
    ("fp32", 0, 64, 64, 64, 1, [0, 64, 10, 64, 20, 64, 30], [0, 0, 0, 0, 0, 0])])
def test_expert_ffn_small(H, dtype, act, R, Hd, F, n_local, off, exp):
    from paper_2410_17043_amd import _lib
    r = np.random.default_rng(R + Hd)
    if off is None:
        off, exp = make_segments(r, R, exp, n_local)
    assert _lib.load().moe_selfcheck_small(R, min(n_local, len(exp), R), len(exp), Hd, F, act, 1 if dtype == "bf16" else 0, 256) == 1
    cfg = small("c2_mixtral", H=Hd, F=F, act=act)
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    if dtype == "bf16":
        recv = W.to_bf16_grid(recv)
    dev = [H.weights_to_dev(w, dtype) for w in experts]
    x = H.dev(recv, dtype)
    out = H.host(H.run_ffn(x, off, exp, dev, Hd, F, act, dtype))
    apart = torch.full((R, Hd), float("nan"), dtype=H.P.TORCH_DTYPE[dtype], device="cuda")
    ws = torch.empty(H.P.moe_ffn_workspace_bytes(R, Hd, F, act, dtype), dtype=torch.uint8, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    timed = torch.full_like(apart, float("nan"))
    ms = H.P.moe_expert_ffn_timed(x, R, torch.tensor(off, **i32), torch.tensor(exp, **i32), len(exp), dev, Hd, F, act, dtype, timed, ws)
    assert ms[0] == 0.0 and ms[1] > 0.0 and ms[2] == 0.0
    assert np.array_equal(H.host(timed), out, equal_nan=True)
    more = 65 - len(exp)
    assert _lib.load().moe_selfcheck_small(R, min(n_local, 65, R), 65, Hd, F, act, 1 if dtype == "bf16" else 0, 256) == 0
    H.P.moe_expert_ffn(x, R, torch.tensor(list(off) + [off[-1]] * more, **i32), torch.tensor(list(exp) + [0] * more, **i32), 65, dev, Hd, F, act, dtype, apart, ws)
    apart = H.host(apart)
    written = np.zeros(R, dtype=bool)
    for i, e in enumerate(exp):
        if 0 <= e < n_local:
            written[max(off[i], 0):max(min(off[i + 1], R), 0)] = True
    assert np.isnan(out[~written]).all() and np.isnan(apart[~written]).all()
    H.assert_close(out[written], apart[written], dtype)
    ref = np.full((R, Hd), np.nan)
    for i, e in enumerate(exp):
        lo, hi = max(off[i], 0), min(off[i + 1], R)
        if 0 <= e < n_local and hi > lo:
            ref[lo:hi] = O.ffn(recv[lo:hi], experts[e]["w1"], experts[e]["w_up"], experts[e]["w_down"], act)
    H.assert_close(out[written], ref[written], dtype)


# The outputs may lie over the received rows, in place or some rows further: each output still comes from the rows as they were.
@pytest.mark.parametrize("dtype,Hd,F,act", [("fp32", 64, 128, 0), ("bf16", 256, 128, 2)])
@pytest.mark.parametrize("shift", [0, 1, 40, -40, -1])
def test_expert_ffn_small_experts_over_their_own_rows(H, dtype, Hd, F, act, shift):
    from paper_2410_17043_amd import _lib
    R, n_local, nseg = 700, 2, 9
    assert _lib.load().moe_selfcheck_small(R, n_local, nseg, Hd, F, act, 1 if dtype == "bf16" else 0, 256) == 1
    r = np.random.default_rng(shift + 50)
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    if dtype == "bf16":
        recv = W.to_bf16_grid(recv)
    off, exp = make_segments(r, R, nseg, n_local)
    experts = [W.make_expert_weights(small("c2_mixtral", H=Hd, F=F, act=act), e) for e in range(n_local)]
    both = torch.zeros((R + 40, Hd), dtype=H.P.TORCH_DTYPE[dtype], device=H.DEV)
    x = both[max(-shift, 0):][:R]
    out = both[max(shift, 0):][:R]
    x.copy_(H.dev(recv, dtype))
    i32 = dict(dtype=torch.int32, device=H.DEV)
    ws = torch.empty(H.P.moe_ffn_workspace_bytes(R, Hd, F, act, dtype), dtype=torch.uint8, device=H.DEV)
    H.P.moe_expert_ffn(x, R, torch.tensor(off, **i32), torch.tensor(exp, **i32), nseg, [H.weights_to_dev(w, dtype) for w in experts], Hd, F, act, dtype, out, ws)
    H.assert_close(H.host(out), O.expert_ffn(recv, off, exp, experts, act), dtype)


# fp32 GEMMs on three bf16 parts (128-row tiles): a K that ends inside a k-tile and an odd number of them, gathered and
# ragged tiles, N of no whole tile, several tiles per block, one kernel of each kind with a map of its own, K of the least four k-tiles
@pytest.mark.parametrize("act,R,Hd,F,n_local,nseg,rows", [(1, 1800, 1156, 1164, 2, 9, [128, 128]), (2, 3000, 292, 1156, 3, 40, [128, 64]),
                                                          (0, 40000, 260, 356, 1, 1, [128, 128]), (0, 12000, 516, 772, 2, 700, [128, 128]),
                                                          (0, 20000, 128, 356, 1, 1, [128, 128])])
def test_expert_ffn_fp32_in_parts(H, act, R, Hd, F, n_local, nseg, rows):
    assert f32_rows(R, n_local, nseg, Hd, F, act) == rows
    test_expert_ffn_fp32_tiles(H, act, R, Hd, F, n_local, nseg)


def f32_rows(R, n_local, nseg, Hd, F, act):
    import ctypes
    from paper_2410_17043_amd import _lib
    got = (ctypes.c_int32 * 2)()
    assert _lib.load().moe_selfcheck_f32_kernels(R, n_local, nseg, Hd, F, act, 256, got) == 0
    return list(got)


@pytest.mark.parametrize("R,Hd,F,n_local,nseg,act,cut", [
    (8355, 512, 2048, 1, 1, 0, [2, 8]), (6600, 640, 1300, 1, 1, 1, [0, 5]), (3071, 1024, 2816, 1, 1, 2, [4, 0]),
    # several experts in ragged runs (rows of a cut tile from all over), both map kernels, and one that may cut but has nothing to
    (6619, 952, 296, 4, 9, 2, [3, 0]), (8499, 512, 1012, 2, 9, 0, [2, 4]), (8301, 452, 1016, 2, 90, 1, [2, 4]), (8142, 984, 472, 4, 65, 2, [4, 2]),
    (6238, 476, 656, 2, 9, 2, [1, 0])])
def test_expert_ffn_fp32_in_parts_tiles_cut_along_k(H, R, Hd, F, n_local, nseg, act, cut):
    """Tiles of a last round in pieces, against the same tiles whole (a workspace without room for pieces) and the oracle: also for
    rows of huge, tiny and infinite elements, NaN and zeros, whose sums no piece may judge alone."""
    import ctypes as C
    from paper_2410_17043_amd import _lib
    P, lib = H.P, _lib.load()
    r = np.random.default_rng(R + nseg)
    off, exp = make_segments(r, R, nseg, n_local)
    c_off, c_exp, parts2 = (C.c_int32 * (nseg + 1))(*off), (C.c_int32 * nseg)(*exp), (C.c_int32 * 2)()
    tiles_m = lib.moe_selfcheck_tile_map(c_off, c_exp, nseg, R, 128, n_local, 1)
    assert tiles_m > 0 and lib.moe_selfcheck_f32_cuts(R, min(n_local, nseg), nseg, Hd, F, act, 256, tiles_m, parts2) == 0
    assert list(parts2) == cut                                   # pieces of a tile in either GEMM; 1: none, but it could
    cfg = small("c1_tiny_fp32", H=Hd, F=F, act=act, dtype="fp32")
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    special = np.sort(r.permutation(R)[:12])
    plain = np.setdiff1d(np.arange(R), special)
    ref = O.expert_ffn(recv, off, exp, experts, act)[plain]
    recv[special[0], 5] = np.inf
    recv[special[1], 7] = np.nan
    recv[special[2:4]] = 0.0
    recv[special[4:6]] *= np.float32(2.0 ** -110)
    recv[special[6:8], ::9] *= np.float32(2.0 ** 40)
    recv[special[8]] *= np.float32(2.0 ** -140)
    recv[special[9]] *= np.float32(2.0 ** 90)
    x, dw = H.dev(recv, "fp32"), [H.weights_to_dev(w, "fp32") for w in experts]
    so, se = torch.tensor(off, dtype=torch.int32, device=H.DEV), torch.tensor(exp, dtype=torch.int32, device=H.DEV)
    full = P.moe_ffn_workspace_bytes(R, Hd, F, act, "fp32")
    out = []
    for room in (full, full, full - 1):
        out.append(torch.full((R, Hd), -7.0, device=H.DEV))
        P.moe_expert_ffn(x, R, so, se, nseg, dw, Hd, F, act, "fp32", out[-1], torch.empty(room, dtype=torch.uint8, device=H.DEV))
    torch.cuda.synchronize()
    assert torch.equal(out[0].view(torch.int32), out[1].view(torch.int32))       # the same bits on every run
    a, b = H.host(out[0]), H.host(out[2])
    assert np.array_equal(np.isfinite(a), np.isfinite(b)) and np.array_equal(np.isnan(a), np.isnan(b))
    H.assert_close(a[plain], ref, "fp32")
    assert H.rms_rel_err(a[plain], b[plain]) < 1e-6
    assert (max(cut) > 1) != np.array_equal(a[plain], b[plain])                 # sums in another order, or the same
    for row in special:                                          # each row on its own scale (sums of up to F products in two orders)
        fin = np.isfinite(a[row])
        if fin.any() and np.abs(b[row][fin]).max() > 0:
            assert H.rel_err(a[row][fin], b[row][fin]) < 1e-5, row


def test_expert_ffn_fp32_in_parts_takes_every_value(H):
    """Rows and weight rows of any scale, zeros in front, elements far apart, infinities, NaN."""
    R, Hd, F, n_local, nseg = 6000, 356, 1012, 2, 40
    assert f32_rows(R, n_local, nseg, Hd, F, 0) == [128, 128]
    cfg = small("c1_tiny_fp32", H=Hd, F=F, act=0)
    r = np.random.default_rng(5)
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    scale = 10.0 ** r.integers(-30, 20, size=R)
    recv *= scale[:, None].astype(np.float32)
    recv[100:103] = 0.0
    recv[200, :64] = 0.0
    recv[300, :32] *= np.float32(1e-9)
    recv[301, 5] *= np.float32(1e6)
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    experts[0]["w1"][7] *= np.float32(1e-25)
    experts[1]["w_down"][3, :40] = 0.0
    bad = [1000, 2500, 2501]
    recv[bad[0], 350], recv[bad[1], 0], recv[bad[2], 40] = np.inf, np.nan, -np.inf
    off, exp = make_segments(r, R, nseg, n_local)
    out = H.host(H.run_ffn(H.dev(recv, "fp32"), off, exp, [H.weights_to_dev(w, "fp32") for w in experts], Hd, F, 0, "fp32"))
    fine = np.ones(R, dtype=bool)
    fine[bad] = False
    with np.errstate(all="ignore"):
        ref = O.expert_ffn(np.where(fine[:, None], recv, 0.0), off, exp, experts, 0)
    assert (~np.isfinite(out[~fine])).any(axis=1).all()
    assert np.isfinite(out[fine]).all() and (out[100:103] == 0).all()
    # per row: two sums of up to 1012 terms, each within sqrt(K) 2^-24 of the norms of its factors, and their rounding;
    # what lies below the normal range of fp32 (rows of 1e-30, squared by silu) rounds to multiples of 2^-149
    err = np.linalg.norm(out - ref, axis=1)[fine]
    assert (err <= 4e-6 * np.linalg.norm(ref, axis=1)[fine] + np.sqrt(Hd) * 1012 * 2.0 ** -149).all()


def test_expert_ffn_fp32_in_parts_rows_of_zeros_change_no_other(H):
    """Rows and weight rows of zeros change no bit of the others (a tile formed again would), and rows of tiny elements
    keep their precision."""
    R, Hd, F = 6000, 356, 1012
    assert f32_rows(R, 1, 1, Hd, F, 0) == [128, 128]
    r = np.random.default_rng(6)
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    tiny = np.arange(50, R, 500)
    recv[tiny] *= np.float32(2.0 ** -117)
    w = W.make_expert_weights(small("c1_tiny_fp32", H=Hd, F=F, act=0), 0)
    whole = H.host(H.run_ffn(H.dev(recv, "fp32"), [0, R], [0], [H.weights_to_dev(w, "fp32")], Hd, F, 0, "fp32"))
    rows, cols = np.arange(3, R, 90), np.arange(1, Hd, 60)
    recv[rows], w["w_down"][cols] = 0.0, 0.0
    out = H.host(H.run_ffn(H.dev(recv, "fp32"), [0, R], [0], [H.weights_to_dev(w, "fp32")], Hd, F, 0, "fp32"))
    assert (out[rows] == 0).all() and (out[:, cols] == 0).all()
    assert np.array_equal(np.delete(np.delete(out, rows, 0), cols, 1), np.delete(np.delete(whole, rows, 0), cols, 1))
    ref = O.ffn(recv[tiny], w["w1"], w["w_up"], w["w_down"], 0)         # the bound of the test above
    err = np.linalg.norm(out[tiny] - ref, axis=1)
    assert (err <= 4e-6 * np.linalg.norm(ref, axis=1) + np.sqrt(Hd) * 1012 * 2.0 ** -149).all()


@pytest.mark.parametrize("operand", ["rows", "weights"])
@pytest.mark.parametrize("p", [13, 24, 30, 40, 100])
def test_expert_ffn_fp32_in_parts_large_elements_hide_no_other(H, operand, p):
    """An element of 2^p that meets weights of zero (or the other way round) leaves the sum to the others, which keep their
    precision: the bound of the tests above, from operands without that column."""
    R, Hd, F = 6000, 356, 1012
    assert f32_rows(R, 1, 1, Hd, F, 0) == [128, 128]
    r = np.random.default_rng(7)
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    w = W.make_expert_weights(small("c1_tiny_fp32", H=Hd, F=F, act=0), 0)
    recv[:, 5], w["w1"][:, 5] = 0.0, 0.0
    ref = O.ffn(recv, w["w1"], w["w_up"], w["w_down"], 0)
    if operand == "rows":
        recv[:, 5] = 2.0 ** p
    else:
        w["w1"][:, 5] = 2.0 ** p
    out = H.host(H.run_ffn(H.dev(recv, "fp32"), [0, R], [0], [H.weights_to_dev(w, "fp32")], Hd, F, 0, "fp32"))
    err = np.linalg.norm(out - ref, axis=1)
    assert (err <= 4e-6 * np.linalg.norm(ref, axis=1)).all(), (err / np.linalg.norm(ref, axis=1)).max()


def test_expert_ffn_fp32_in_parts_single_products_are_rounded_as_in_fp32(H):
    """Rows with one nonzero element, whose products with the weights are large enough that silu is the identity (20 and
    above: off by 2e-9), and a w_down with one per row.  A product of parts leaves out up to 2^-24 of it, its small
    products are rounded below 2^-31 of it and the sum once, 2^-24: 4 x 2^-24 for both GEMMs, and what silu and those add."""
    R, Hd, F = 6000, 356, 1012
    assert f32_rows(R, 1, 1, Hd, F, 0) == [128, 128]
    r = np.random.default_rng(8)
    recv = np.zeros((R, Hd), dtype=np.float32)
    recv[np.arange(R), r.integers(0, Hd, size=R)] = r.uniform(20, 40, size=R)
    w = {"w1": r.uniform(1, 2, size=(F, Hd)).astype(np.float32), "w_up": None, "w_down": np.zeros((Hd, F), dtype=np.float32)}
    w["w_down"][np.arange(Hd), r.integers(0, F, size=Hd)] = r.uniform(-2, 2, size=Hd)
    out = H.host(H.run_ffn(H.dev(recv, "fp32"), [0, R], [0], [H.weights_to_dev(w, "fp32")], Hd, F, 0, "fp32"))
    ref = (recv.astype(np.float64) @ w["w1"].T.astype(np.float64)) @ w["w_down"].T.astype(np.float64)
    assert np.abs(out / ref - 1).max() <= 4.1 * 2.0 ** -24


def test_expert_ffn_fp32_in_parts_no_row_depends_on_its_neighbours(H):
    """Infinities, NaN, the largest floats, zeros in front and rows of tiny elements in every tile change no bit of the other rows."""
    R, Hd, F = 6000, 356, 1012
    assert f32_rows(R, 1, 1, Hd, F, 0) == [128, 128]
    r = np.random.default_rng(9)
    recv = r.standard_normal((R, Hd)).astype(np.float32)
    dw = H.weights_to_dev(W.make_expert_weights(small("c1_tiny_fp32", H=Hd, F=F, act=0), 0), "fp32")
    whole = H.host(H.run_ffn(H.dev(recv, "fp32"), [0, R], [0], [dw], Hd, F, 0, "fp32"))
    odd = np.arange(R) % 37 == 5
    which = np.nonzero(odd)[0]
    for i, row in enumerate(which):
        if i % 5 == 0: recv[row, i % Hd] = np.inf
        elif i % 5 == 1: recv[row, i % Hd] = np.nan
        elif i % 5 == 2: recv[row, i % Hd] = np.float32(3.4e38)
        elif i % 5 == 3: recv[row, :32] = 0.0
        else: recv[row] *= np.float32(1e-35)
    out = H.host(H.run_ffn(H.dev(recv, "fp32"), [0, R], [0], [dw], Hd, F, 0, "fp32"))
    assert np.array_equal(out[~odd], whole[~odd])
    assert (~np.isfinite(out[which[0::5]])).any(axis=1).all() and np.isnan(out[which[1::5]]).all()


@pytest.mark.parametrize("R,nseg,F,one_kernel", [(60, 5, 384, False), (300, 63, 384, False), (300, 64, 384, False), (300, 65, 384, False), (1000, 64, 384, False),
                                                 (60, 5, 256, False), (300, 63, 256, False), (300, 64, 256, False), (300, 65, 256, False), (500, 64, 256, True), (1000, 64, 256, True)])
def test_expert_ffn_tile_map_skips_what_it_must(H, R, nseg, F, one_kernel):
    """Empty segments, segments of no local expert, rows before the first and after the last segment, on both sides of
    the segment count where the map kernel changes, and in the kernel that works its tiles out without a map."""
    Hd, n_local = 128, 3
    assert takes_small(R, n_local, nseg, Hd, F, 2, "bf16") == one_kernel
    cfg = small("c2_mixtral", H=Hd, F=F)
    r = np.random.default_rng(nseg)
    recv = W.to_bf16_grid(r.standard_normal((R, Hd)).astype(np.float32))
    experts = [W.make_expert_weights(cfg, e) for e in range(n_local)]
    off = np.sort(r.integers(3, R - 4, size=nseg + 1))
    off[1] = off[0]                                                   # an empty one for certain
    exp = r.integers(-1, n_local + 1, size=nseg)
    out = H.host(H.run_ffn(H.dev(recv, "bf16"), off, exp, [H.weights_to_dev(w, "bf16") for w in experts], Hd, F, 2, "bf16"))
    done = np.zeros(R, dtype=bool)
    ref = np.zeros((R, Hd))
    for i in range(nseg):
        if 0 <= exp[i] < n_local and off[i + 1] > off[i]:
            w = experts[exp[i]]
            done[off[i]:off[i + 1]] = True
            ref[off[i]:off[i + 1]] = O.ffn(recv[off[i]:off[i + 1]], w["w1"], w["w_up"], w["w_down"], 2)
    assert np.isnan(out[~done]).all()
    H.assert_close(out[done], ref[done], "bf16")
