"""GPU parity of the simulated run time of sampled placements (gdp_evaluate,
in-order list scheduling with transfer costs and the per-device memory cap)
against the oracle: makespans, validity and run times bit for bit."""
import numpy as np
import pytest

from oracle import gdp_oracle as O
from paper_1910_01578_amd import workloads as W
from tests.parity import workload

pytestmark = pytest.mark.gpu

ALL = W.CONFIG_ORDER


def _log(*a):
    print(*a, flush=True)


def _check(g, costs, pl_np, D, ev, time_unit=1e-6):
    import torch
    pl = torch.from_numpy(np.ascontiguousarray(pl_np, np.int32)).cuda()
    mk, valid, rt = ev.evaluate(pl, time_unit)
    torch.cuda.synchronize()
    ref = O.simulate_placements(g.graph_ptr, g.row_ptr, g.col_idx, pl_np, D, costs.op_cost, costs.out_xfer,
                                costs.op_mem, costs.mem_cap)
    got_mk = mk.cpu().numpy()
    assert np.array_equal(got_mk, ref["makespan"]), np.argwhere(got_mk != ref["makespan"])[:5]
    assert np.array_equal(valid.cpu().numpy().astype(bool), ref["valid"])
    want_rt = (ref["makespan"].astype(np.float64) * time_unit).astype(np.float32)
    assert np.array_equal(rt.cpu().numpy(), want_rt)
    return ref


def _far_edges(g, dist):
    src = np.repeat(np.arange(g.n_nodes), np.diff(g.row_ptr))
    return int((g.col_idx - src > dist).sum())


@pytest.mark.parametrize("name", ALL)
def test_evaluate_sampled_placements(name):
    """The workloads' own sampled placements, straight from gdp_sample."""
    from paper_1910_01578_amd import gdp
    cfg, g, w = workload(name)
    costs = W.make_costs(cfg, g)
    dg = gdp.DeviceGraph(g, cfg.dtype)
    r = gdp.Runner(dg, gdp.DevicePolicy(cfg, w), cfg.k_samples)
    r.forward(cfg.sample_seed)
    ev = gdp.Evaluator(dg, cfg.n_devices, cfg.k_samples, costs)
    pl = r.placements.cpu().numpy()
    ref = _check(g, costs, pl, cfg.n_devices, ev)
    _log(f"evaluate {name}: K={cfg.k_samples} edges beyond 256 ids {_far_edges(g, 256)}  makespan "
         f"[{ref['makespan'].min()}, {ref['makespan'].max()}]  valid {ref['valid'].mean():.3f}")


def test_evaluate_random_and_concentrated_placements_two_sample_blocks():
    """K = 100 (two blocks of 64 samples, the second ragged), placements from
    uniform to all-on-one-device, so both validity outcomes occur."""
    from paper_1910_01578_amd import gdp
    cfg, g, w = workload("recurrent_12000")
    assert _far_edges(g, 256) > 0
    costs = W.make_costs(cfg, g)
    rng = np.random.default_rng(7)
    K, D, N = 100, cfg.n_devices, g.n_nodes
    bias = np.linspace(0.0, 1.0, K)[:, None]
    pl = np.where(rng.random((K, N)) < bias, 0, rng.integers(0, D, (K, N))).astype(np.int32)
    ev = gdp.Evaluator(gdp.DeviceGraph(g, cfg.dtype), D, K, costs)
    ref = _check(g, costs, pl, D, ev, time_unit=2.5e-7)
    assert ref["valid"].any() and (~ref["valid"]).any()


@pytest.mark.parametrize("case", ["single_node", "no_edges", "many_devices", "ragged_128_graphs", "zero_costs"])
def test_evaluate_edge_cases(case):
    from paper_1910_01578_amd import gdp
    base = W.get_config("tiny_layered_256")
    rng = np.random.default_rng(3)
    D, K = 4, 9
    if case == "single_node":
        g = W.graph_from_arrays(base, [0, 1], [0, 0], np.array([], np.int32), W.make_features(base, 1, rng))
    elif case == "no_edges":
        g = W.graph_from_arrays(base, [0, 300], [0] * 301, np.array([], np.int32), W.make_features(base, 300, rng))
    elif case == "ragged_128_graphs":
        sizes = tuple(int(s) for s in rng.integers(1, 60, 128))
        c = base.replace(graph_sizes=sizes)
        g = W.make_graph(c)
    else:
        g = W.make_graph(base)
    if case == "many_devices":
        D, K = 64, 70
    costs = W.make_costs(base.replace(n_devices=D), g)
    if case == "zero_costs":
        costs = W.OpCosts(np.zeros_like(costs.op_cost), costs.out_xfer, costs.op_mem, costs.mem_cap)
    pl = rng.integers(0, D, (K, g.n_nodes)).astype(np.int32)
    ev = gdp.Evaluator(gdp.DeviceGraph(g, base.dtype), D, K, costs)
    _check(g, costs, pl, D, ev)
    _log("evaluate edge", case, "ok")


@pytest.mark.parametrize("cost", [2 ** 20, 2 ** 31 - 1])
def test_evaluate_time_range_marks_the_graph(cost):
    """Finish times that reach 2^26 units in one graph (2^20 per op: past the
    packed word's range, inside 32 bits; 2^31 - 1: past 32 bits as well) give
    -1 for that graph only."""
    import torch

    from paper_1910_01578_amd import gdp
    c = W.get_config("tiny_layered_256").replace(graph_sizes=(100, 50))
    g = W.make_graph(c)
    costs = W.make_costs(c, g)
    big = costs.op_cost.copy()
    big[:100] = cost                           # one device runs the first graph's 100 ops one after another
    costs = W.OpCosts(big, costs.out_xfer, costs.op_mem, costs.mem_cap)
    K, D = 3, c.n_devices
    pl = np.zeros((K, g.n_nodes), np.int32)
    ev = gdp.Evaluator(gdp.DeviceGraph(g, c.dtype), D, K, costs)
    mk, _, _ = ev.evaluate(torch.from_numpy(pl).cuda())
    torch.cuda.synchronize()
    ref = O.simulate_placements(g.graph_ptr, g.row_ptr, g.col_idx, pl, D, costs.op_cost, costs.out_xfer, costs.op_mem,
                                costs.mem_cap)
    got = mk.cpu().numpy()
    assert np.all(got[0] == -1) and ref["makespan"][0].min() >= 2 ** 26
    assert np.array_equal(got[1], ref["makespan"][1])


@pytest.mark.parametrize("xfer", [2 ** 26 - 1, 2 ** 26, 2 ** 31 - 1])
@pytest.mark.parametrize("v,preds,lanes", [
    (100, range(90, 98), False),     # in the op's own window of 64, more than its slots hold
    (100, range(40, 48), False),     # in the window before it, likewise
    (200, range(10, 18), False),     # further back
    (200, (10, 17, 130, 150, 190, 191, 192, 193), True),
])
def test_evaluate_transfer_range(v, preds, lanes, xfer):
    """A transfer of 2^26 units and more gives -1 where its edge crosses devices and
    nowhere else, wherever the predecessor lies; one of 2^26 - 1 is exact.  Sample i
    has the i-th of eight such predecessors away from op v's device, the last none."""
    import torch

    from paper_1910_01578_amd import gdp
    n, D, preds = 256, 4, list(preds)
    base = W.get_config("tiny_layered_256").replace(graph_sizes=(n,))
    rows = [[v] if u in preds else [] for u in range(n)]
    row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    rng = np.random.default_rng(v)
    g = W.graph_from_arrays(base, [0, n], row_ptr, np.concatenate(rows).astype(np.int64), W.make_features(base, n, rng))
    out = rng.integers(0, 90, n).astype(np.int32)
    out[preds] = xfer
    costs = W.OpCosts(np.zeros(n, np.int32), out, rng.integers(1, 200, n).astype(np.int32), np.array([10 ** 6], np.int64))
    kinds = len(preds) + 1
    pl = np.tile(rng.integers(1, D, n).astype(np.int32), (kinds, 1))
    pl[:, v] = pl[:, preds] = 0
    for i, u in enumerate(preds):
        pl[i, u] = 1 + i % (D - 1)
    K = 16384 if lanes else kinds                # a lane a sample takes many samples
    ref = O.simulate_placements(g.graph_ptr, g.row_ptr, g.col_idx, pl, D, costs.op_cost, costs.out_xfer, costs.op_mem,
                                costs.mem_cap)["makespan"][0]
    assert np.all(ref[:-1] == xfer) and ref[-1] == 0
    pl = pl[np.arange(K) % kinds]
    ev = gdp.Evaluator(gdp.DeviceGraph(g, base.dtype), D, K, costs)
    mk, _, _ = ev.evaluate(torch.from_numpy(pl).cuda())
    torch.cuda.synchronize()
    want = np.where(ref >= 2 ** 26, -1, ref)[np.arange(K) % kinds]
    assert np.array_equal(mk.cpu().numpy()[0], want)
    _log("evaluate transfer", v, xfer, "ok")


def test_evaluate_feeds_advantages():
    """run_time from gdp_evaluate and its validity go straight into gdp_advantages."""
    import torch

    from paper_1910_01578_amd import gdp
    cfg, g, w = workload("superposition_4x")
    costs = W.make_costs(cfg, g)
    dg = gdp.DeviceGraph(g, cfg.dtype)
    r = gdp.Runner(dg, gdp.DevicePolicy(cfg, w), cfg.k_samples)
    r.forward(cfg.sample_seed)
    ev = gdp.Evaluator(dg, cfg.n_devices, cfg.k_samples, costs)
    mk, valid, rt = ev.evaluate(r.placements)
    base = gdp.RewardBaseline(g.n_graphs)
    reward, adv = base.advantages(rt, valid)
    torch.cuda.synchronize()
    ref = O.rewards_advantages(rt.cpu().numpy(), valid.cpu().numpy(), np.zeros(g.n_graphs), np.zeros(g.n_graphs, np.int64))
    np.testing.assert_allclose(reward.cpu().numpy(), ref["reward"], rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(adv.cpu().numpy(), ref["advantage"], rtol=0, atol=1e-5)


def _dag(n, rng, dense, far, far_span):
    """A DAG of n ops: every op reads its predecessor; inside every second run of
    64 ops each op reads every dense-th op of the 100 before it, and `far` ops
    read one op at least far_span ids back."""
    src, dst = [np.arange(n - 1)], [np.arange(1, n)]
    for v in range(1, n):
        if dense and (v // 64) % 2:
            u = np.arange(max(0, v - 100), v - 1, dense)
            src.append(u)
            dst.append(np.full(u.size, v))
    if far:
        v = rng.integers(far_span + 1, n, far)
        u = (rng.random(far) * (v - far_span)).astype(np.int64)
        src.append(u)
        dst.append(v)
    key = np.unique(np.concatenate(src) * np.int64(n) + np.concatenate(dst))
    s, d = key // n, key % n
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(s, minlength=n))])
    return row_ptr, d


@pytest.mark.parametrize("n,K,D,dense,far,far_span", [
    (200, 3, 5, 1, 0, 0),            # up to 99 predecessors, beyond the slots, in and before the window
    (1000, 2, 64, 7, 50, 300),       # some beyond the slots, old ones among them
    (33000, 2, 8, 0, 3000, 32700),   # 32,768 finish times on chip: read-backs at their edge
    (17000, 260, 3, 0, 900, 16300),  # 16,384 on chip
    (8300, 515, 2, 0, 900, 8100),    # 8,192
    (8300, 768, 2, 0, 900, 8100),    # 8,192 for the last time
    (8300, 769, 2, 0, 900, 8100),    # 4,096 for the first time
    (4200, 1030, 8, 0, 900, 4000),   # 4,096
])
def test_evaluate_windows_and_rings(n, K, D, dense, far, far_span):
    """Edges beyond the per-op slots, and every length of the on-chip ring of
    finish times with predecessors on both sides of its edge."""
    from paper_1910_01578_amd import gdp
    base = W.get_config("tiny_layered_256")
    rng = np.random.default_rng(n)
    row_ptr, col = _dag(n, rng, dense, far, far_span)
    g = W.graph_from_arrays(base, [0, n], row_ptr, col, W.make_features(base, n, rng))
    cap = np.array([100 * n // D], np.int64)
    costs = W.OpCosts(rng.integers(0, 50, n).astype(np.int32), rng.integers(0, 90, n).astype(np.int32),
                      rng.integers(1, 200, n).astype(np.int32), cap)
    skew = rng.random((K, 1))
    pl = np.where(rng.random((K, n)) < skew, rng.integers(0, D, (K, 1)), rng.integers(0, D, (K, n))).astype(np.int32)
    _check(g, costs, pl, D, gdp.Evaluator(gdp.DeviceGraph(g, base.dtype), D, K, costs))
    _log("evaluate windows", n, K, "ok")


@pytest.mark.parametrize("sizes,K,D", [
    ((256,) + (1, 2, 63, 64, 65, 129, 255) * 18 + (3,), 128, 8),   # 256 waves, up to 256 ops
    ((90, 130), 8200, 64),                                         # the last block of samples 8 of 64
    ((500, 300) * 8, 2100, 3),                                     # past the ring of 256 nodes
])
def test_evaluate_a_lane_a_sample(sizes, K, D):
    """Many short graphs and samples, one lane a sample: ragged sizes and blocks of
    samples, predecessors behind the ring, one graph past the time range."""
    import torch

    from paper_1910_01578_amd import gdp
    c = W.get_config("tiny_layered_256").replace(graph_sizes=sizes)
    parts = [_dag(n, np.random.default_rng(n), 0, n // 4, n // 2) if n > 8 else _dag(n, None, 0, 0, 0) for n in sizes]
    starts = np.concatenate([[0], np.cumsum(sizes)])
    edges = np.concatenate([[0], np.cumsum([p[1].size for p in parts])])
    row_ptr = np.concatenate([[0]] + [p[0][1:] + e for p, e in zip(parts, edges)])
    col = np.concatenate([p[1] + s for p, s in zip(parts, starts)])
    rng = np.random.default_rng(K)
    n = int(starts[-1])
    g = W.graph_from_arrays(c, starts, row_ptr, col, W.make_features(c, n, rng))
    cost = rng.integers(0, 50, n).astype(np.int32)
    cost[0] = 2 ** 26
    cap = np.array([100 * s // D for s in sizes], np.int64)
    costs = W.OpCosts(cost, rng.integers(0, 90, n).astype(np.int32), rng.integers(1, 200, n).astype(np.int32), cap)
    pl = rng.integers(0, D, (K, n)).astype(np.int32)
    ev = gdp.Evaluator(gdp.DeviceGraph(g, c.dtype), D, K, costs)
    mk, valid, _ = ev.evaluate(torch.from_numpy(pl).cuda())
    torch.cuda.synchronize()
    keep = np.concatenate([np.arange(min(K, 130)), np.arange(max(0, K - 130), K)]) if K > 260 else np.arange(K)
    ref = O.simulate_placements(g.graph_ptr, g.row_ptr, g.col_idx, pl[keep], D, costs.op_cost, costs.out_xfer,
                                costs.op_mem, costs.mem_cap)
    got = mk.cpu().numpy()[:, keep]
    assert np.all(got[0] == -1) and ref["makespan"][0].min() >= 2 ** 26
    assert np.array_equal(got[1:], ref["makespan"][1:])
    assert np.array_equal(valid.cpu().numpy()[:, keep].astype(bool), ref["valid"])
    _log("evaluate by lanes", len(sizes), K, "ok")
