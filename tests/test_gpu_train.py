"""GPU parity of the update step (training forward with every intermediate
kept, backward pass, log-probs of given placements, Adam) against the oracle
(oracle/policy_grad.py): every weight gradient of the GNN, the placer and the
head, on the five workloads and edge cases, plus a directional derivative of
the whole loss at the largest size on the GPU's own forward."""
import numpy as np
import pytest

from oracle import gdp_oracle as O
from oracle import policy_grad as PG
from paper_1910_01578_amd import workloads as W
from tests.parity import rel_err_rows, to_np, workload

pytestmark = pytest.mark.gpu

ALL = W.CONFIG_ORDER
# The training path computes in fp32 for both element types (bf16 weights and
# features are widened on load), so both are held to the fp32 bar.
TOL = {"f32": 1e-4, "bf16": 1e-4}


def _log(*a):
    print(*a, flush=True)


def _trainer(cfg, g, w, **pol):
    from paper_1910_01578_amd import gdp
    dg = gdp.DeviceGraph(g, cfg.dtype)
    pol = gdp.DevicePolicy(cfg, w, **pol)
    return gdp.Trainer(dg, pol, cfg.k_samples)


def _tensor_err(got, ref):
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    e = float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-30))
    return e if e == e else float("inf")       # (a NaN would lose every comparison of max())


def _compare_grads(t, ref, cfg, attention=True, film=True, tol=None):
    tol = TOL[cfg.dtype] if tol is None else tol
    worst = (0.0, "")
    for l, lg in enumerate(t.grad_gnn):
        for k, v in lg.items():
            e = _tensor_err(to_np(v), ref["gnn"][l][k])
            worst = max(worst, (e, f"gnn[{l}].{k}"))
    for l, lg in enumerate(t.grad_placer):
        for k, v in lg.items():
            if (not film and k.startswith("film")) or (not attention and k in ("w_qkv", "b_qkv", "w_o", "b_o",
                                                                               "ln1_g", "ln1_b")):
                continue
            e = _tensor_err(to_np(v), ref["placer"][l][k])
            worst = max(worst, (e, f"placer[{l}].{k}"))
    for k, v in t.grad_head.items():
        e = _tensor_err(to_np(v), ref["head"][k])
        worst = max(worst, (e, f"head.{k}"))
    _log(f"  worst gradient error {worst[0]:.3e} ({worst[1]})")
    assert worst[0] <= tol, worst


def _run(cfg, g, w, seed=0, attention=None, film=None, make=_trainer):
    import torch
    t = make(cfg, g, w, attention=attention, film=film)
    logits, _ = t.forward()
    dl = np.random.default_rng(seed).normal(size=(g.n_nodes, cfg.n_devices)) / np.sqrt(g.n_nodes)
    t.backward(torch.from_numpy(dl.astype(np.float32)).cuda())
    torch.cuda.synchronize()
    gnn, pl, hd = w.f64()
    att = cfg.attention if attention is None else attention
    fl = cfg.film if film is None else film
    # the ReLU signs and max-pool winners are taken as the GPU's fp32 forward took
    # them (a pre-activation within rounding of zero may fall either way)
    ref = PG.policy_backward(g.graph_ptr, g.row_ptr, g.col_idx, g.x, gnn, pl, hd["w_out"], hd["b_out"],
                             dl.astype(np.float32).astype(np.float64), fanout=cfg.fanout, nb_seed=cfg.nb_seed,
                             n_heads=cfg.heads, seg_len=cfg.seg_len, mem_len=cfg.mem_len, film=fl, attention=att,
                             decisions=t.decisions())
    err_l = rel_err_rows(to_np(logits), ref["logits"])
    _log(f"  train-forward logits err {err_l:.3e}")
    assert err_l <= TOL[cfg.dtype]
    return t, ref, att, fl


@pytest.mark.parametrize("name", ALL)
def test_backward_parity_workloads(name):
    cfg, g, w = workload(name)
    _log("backward", name)
    t, ref, att, fl = _run(cfg, g, w)
    _compare_grads(t, ref, cfg, att, fl)


EDGE = [
    ("no_attention", dict(), dict(attention=False)),
    ("film_off", dict(), dict(film=False)),
    ("mem0_ragged", dict(seg_len=48, mem_len=0), {}),
    ("mem_gt_seg", dict(seg_len=32, mem_len=80), {}),
    ("dh64_many_devices", dict(heads=1, n_devices=64), {}),
    ("ragged_graphs", dict(graph_sizes=(6, 37, 200, 63)), {}),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("label,over,pol", EDGE, ids=[e[0] for e in EDGE])
def test_backward_parity_edge_cases(label, over, pol, dtype):
    width = dict(hidden=128, heads=8, d_ff=512) if dtype == "bf16" else {}
    if "heads" in over and dtype == "bf16":
        width["heads"] = 2
        over = {k: v for k, v in over.items() if k != "heads"}
    cfg = W.get_config("tiny_layered_256").replace(dtype=dtype, **{**width, **over})
    g, w = W.make_graph(cfg), W.make_weights(cfg)
    _log("backward edge", label, dtype)
    t, ref, att, fl = _run(cfg, g, w, seed=1, **pol)
    _compare_grads(t, ref, cfg, att, fl)


def test_single_node_graph():
    cfg = W.get_config("tiny_layered_256")
    rng = np.random.default_rng(2)
    g = W.graph_from_arrays(cfg, [0, 1], [0, 0], np.array([], np.int32), W.make_features(cfg, 1, rng))
    w = W.make_weights(cfg)
    _log("backward single node")
    t, ref, att, fl = _run(cfg, g, w, seed=2)
    _compare_grads(t, ref, cfg, att, fl)


def test_backward_is_deterministic():
    import torch
    cfg, g, w = workload("superposition_4x")
    t = _trainer(cfg, g, w)
    t.forward()
    dl = torch.from_numpy(np.random.default_rng(3).normal(size=(g.n_nodes, cfg.n_devices)).astype(np.float32)).cuda()
    outs = []
    for _ in range(2):
        t.backward(dl)
        torch.cuda.synchronize()
        outs.append([v.clone().cpu().numpy().tobytes() for l in t.grad_placer + t.grad_gnn for v in l.values()])
    assert outs[0] == outs[1]


def test_log_prob_and_ppo_chain():
    """log-probs of given placements against the oracle, and PPO's logit gradient
    fed through the backward against the oracle chain."""
    import torch
    cfg, g, w = workload("inception_2500")
    t = _trainer(cfg, g, w)
    logits, lse = t.forward()
    rng = np.random.default_rng(4)
    K = cfg.k_samples
    pl = rng.integers(0, cfg.n_devices, (K, g.n_nodes)).astype(np.int32)
    plt = torch.from_numpy(pl).cuda()
    logp = t.log_prob(plt)
    torch.cuda.synchronize()
    lg = to_np(logits).astype(np.float64)
    own = O.log_prob_of(lg, O.logsumexp_rows(lg), g.graph_ptr, pl)
    assert float(np.abs(to_np(logp) - own).max() / np.abs(own).max()) <= 1e-5
    logp_old = logp + torch.from_numpy(rng.normal(scale=0.3, size=logp.shape).astype(np.float32)).cuda()
    adv = torch.from_numpy(rng.normal(size=logp.shape).astype(np.float32)).cuda()
    loss, dl = t.ppo_grad(plt, logp, logp_old, adv, 0.2)
    t.backward(dl)
    torch.cuda.synchronize()
    gnn, plw, hd = w.f64()
    ref = PG.policy_backward(g.graph_ptr, g.row_ptr, g.col_idx, g.x, gnn, plw, hd["w_out"], hd["b_out"],
                             to_np(dl).astype(np.float64), fanout=cfg.fanout, nb_seed=cfg.nb_seed, n_heads=cfg.heads,
                             seg_len=cfg.seg_len, mem_len=cfg.mem_len, film=cfg.film, decisions=t.decisions())
    _compare_grads(t, ref, cfg)


def test_adam_step_against_oracle():
    import torch
    cfg = W.get_config("tiny_layered_256").replace(dtype="bf16", hidden=128, heads=8, d_ff=512)
    g, w = W.make_graph(cfg), W.make_weights(cfg)
    t = _trainer(cfg, g, w)
    rng = np.random.default_rng(5)
    states = []
    for prm, master, grd, m, v in t._adam:
        grd.copy_(torch.from_numpy(rng.normal(size=tuple(grd.shape)).astype(np.float32)))
        states.append((master.cpu().numpy().astype(np.float64), np.zeros(tuple(grd.shape)), np.zeros(tuple(grd.shape))))
    for step in (1, 2):
        t.adam(lr=1e-2)
        torch.cuda.synchronize()
        for i, (prm, master, grd, m, v) in enumerate(t._adam):
            p0, m0, v0 = states[i]
            # the ABI takes the hyper-parameters as fp32: the oracle gets the same values
            hp = [float(np.float32(x)) for x in (1e-2, 0.9, 0.999, 1e-8)]
            p1, m1, v1 = PG.adam_step(p0, grd.cpu().numpy(), m0, v0, step, *hp)
            np.testing.assert_allclose(master.cpu().numpy(), p1, rtol=1e-5, atol=1e-6)
            np.testing.assert_allclose(m.cpu().numpy(), m1, rtol=1e-5, atol=1e-7)
            np.testing.assert_allclose(v.cpu().numpy(), v1, rtol=1e-5, atol=1e-9)
            # the dtype copy is the master rounded to bf16 (nearest even)
            want = W.bf16_to_f64(W.bf16_bits(master.cpu().numpy()))
            assert np.array_equal(prm.float().cpu().numpy().astype(np.float64), want)
            states[i] = (master.cpu().numpy().astype(np.float64), m1, v1)


def test_directional_derivative_full_size_fp32():
    """At 52,000 nodes in fp32: the change of sum(dl * logits) along the gradient
    direction equals the gradient's norm (central difference on the GPU's own
    training forward).  Without memory (mem_len = 0): with memory the gradient
    leaves out, by the paper's stop-gradient, the path through the cached rows,
    which a difference of the forward does include (the oracle's pins check that
    part against a difference with the memory frozen)."""
    import torch
    cfg = W.get_config("gnmt8_52000").replace(dtype="f32", mem_len=0)
    g, w = W.make_graph(cfg), W.make_weights(cfg)
    t = _trainer(cfg, g, w)
    dl = torch.from_numpy((np.random.default_rng(6).normal(size=(g.n_nodes, cfg.n_devices))
                           / np.sqrt(g.n_nodes)).astype(np.float32)).cuda()
    t.forward()
    t.backward(dl)
    torch.cuda.synchronize()
    pairs = []
    for lw, lg in zip(t.policy.gnn_t, t.grad_gnn):
        pairs += [(lw[k], lg[k]) for k in lw]
    for lw, lg in zip(t.policy.placer_t, t.grad_placer):
        pairs += [(lw[k], lg[k]) for k in lw]
    pairs += [(t.policy.head_t[k], t.grad_head[k]) for k in t.policy.head_t]
    gnorm = float(np.sqrt(sum(float((gr.double() ** 2).sum()) for _, gr in pairs)))
    base = [p.clone() for p, _ in pairs]

    def loss(step):
        for (p, gr), b in zip(pairs, base):
            p.copy_(b + step * gr)
        logits, _ = t.forward()
        torch.cuda.synchronize()
        return float((logits.double() * dl.double()).sum())
    # steps of parameter-space length 2e-3, 5e-4, 1.25e-4: the difference must
    # converge to |g|^2 (the ReLU and max-pool kinks a longer step crosses bias it)
    fds = []
    for length in (2e-3, 5e-4, 1.25e-4):
        eps = length / gnorm
        fds.append((loss(eps) - loss(-eps)) / (2 * eps))
    for (p, _), b in zip(pairs, base):
        p.copy_(b)
    _log(f"directional derivative: central differences {[f'{f:.6e}' for f in fds]}  |g|^2 {gnorm ** 2:.6e}")
    assert abs(fds[-1] - gnorm ** 2) <= 0.02 * gnorm ** 2


# One graph size or head layout a branch of the products' and the attention's
# dispatch with aligned arrays: rows one past a tile, products of many rows with a
# ragged last tile (d_ff = 1,024: 8 column tiles, so 8,193 rows take the
# direct-to-register kernel), an odd number of devices in the head, head sizes of 16
# and 32 with one and two columns a lane and 64 with one, memories longer than and
# unaligned to the segments.
KERNEL_PATHS = [
    ("tile_plus_1_odd_devices", "bf16", dict(graph_sizes=(129,), hidden=128, heads=4, n_devices=7)),
    ("many_rows_ragged", "bf16", dict(graph_sizes=(8193,), hidden=128, heads=4, d_ff=1024, seg_len=512, mem_len=100)),
    ("many_rows_f32", "f32", dict(graph_sizes=(8193,), hidden=128, heads=8, d_ff=1024, seg_len=128, mem_len=128)),
    ("dh16_two_columns", "f32", dict(graph_sizes=(700, 65, 1, 127), hidden=64, heads=4, seg_len=128, mem_len=200)),
    ("dh16_one_column", "bf16", dict(graph_sizes=(300, 64), hidden=128, heads=8, seg_len=72, mem_len=33)),
    ("dh32_two_columns", "bf16", dict(graph_sizes=(1100, 3), hidden=128, heads=4, seg_len=520, mem_len=600)),
    ("dh64_ragged", "f32", dict(graph_sizes=(333, 65), hidden=256, heads=4, seg_len=128, mem_len=128)),
]


@pytest.mark.parametrize("label,dtype,over", KERNEL_PATHS, ids=[k[0] for k in KERNEL_PATHS])
def test_backward_parity_kernel_paths(label, dtype, over):
    cfg = W.get_config("tiny_layered_256").replace(dtype=dtype, **over)
    g, w = W.make_graph(cfg), W.make_weights(cfg)
    _log("backward kernel path", label)
    t, ref, att, fl = _run(cfg, g, w, seed=3)
    _compare_grads(t, ref, cfg, att, fl)


def _unaligned_trainer(cfg, g, w, **pol):
    """A Trainer whose features, GNN weights and gradients lie one element past a
    16-byte boundary, each between guard elements (t.guards)."""
    import torch

    from paper_1910_01578_amd import gdp
    t = _trainer(cfg, g, w, **pol)
    t.guards = []

    def move(a):
        buf = torch.full((a.numel() + 18,), 7.0, dtype=a.dtype, device=a.device)
        v = buf[1:a.numel() + 1].view(a.shape)
        v.copy_(a)
        assert v.data_ptr() % 16 == a.element_size()
        t.guards.append((buf, a.numel()))
        return v
    t.graph.x = move(t.graph.x)
    t.graph.c.x = t.graph.x.data_ptr()
    t.policy.gnn_t = [{k: move(a) for k, a in l.items()} for l in t.policy.gnn_t]
    t.grad_gnn = [{k: move(a) for k, a in l.items()} for l in t.grad_gnn]
    t.grad_placer = [{k: move(a) for k, a in l.items()} for l in t.grad_placer]
    t.grad_head = {k: move(a) for k, a in t.grad_head.items()}
    order = ("w_pool", "b_pool", "w_self", "w_neigh", "b_upd")
    for l in range(cfg.gnn_layers):
        t.policy._gl[l] = gdp.GdpGnnLayer(*[t.policy.gnn_t[l][k].data_ptr() for k in order])
        t._gg[l] = gdp.GdpGnnLayerGrad(*[t.grad_gnn[l][k].data_ptr() for k in order])
    for l in range(cfg.placer_layers):
        t._gp[l] = gdp.GdpPlacerLayerGrad(*[t.grad_placer[l][k].data_ptr() for k in gdp.PLACER_LAYER_FIELDS])
    t.grads.w_out, t.grads.b_out = t.grad_head["w_out"].data_ptr(), t.grad_head["b_out"].data_ptr()
    return t


@pytest.mark.parametrize("dtype,over", [
    ("f32", dict(graph_sizes=(65,))),                                 # one piece of k, one past a 64-row tile
    ("bf16", dict(graph_sizes=(65,))),
    ("f32", dict(graph_sizes=(700, 1))),                              # two pieces, added by elements
    ("bf16", dict(graph_sizes=(1030, 3), hidden=128, heads=8, d_ff=512)),
])
def test_backward_parity_unaligned_arrays(dtype, over):
    """The products' scalar loads and stores, which arrays off a 16-byte boundary take
    (placer weights have to be aligned; the calls accept any other array as it is):
    one and several pieces of k, bias sums, both types, nothing written beside."""
    cfg = W.get_config("tiny_layered_256").replace(dtype=dtype, **over)
    g, w = W.make_graph(cfg), W.make_weights(cfg)
    _log("backward unaligned", dtype, g.n_nodes)
    t, ref, att, fl = _run(cfg, g, w, seed=4, make=_unaligned_trainer)
    _compare_grads(t, ref, cfg, att, fl)
    for buf, n in t.guards:
        assert bool((buf[:1] == 7).all()) and bool((buf[n + 1:] == 7).all())


def _gradients(t, dl):
    import torch
    t.backward(torch.from_numpy(dl).cuda())
    torch.cuda.synchronize()
    d = t.policy.cfg.hidden
    out = {}
    for part, layers in (("gnn", t.grad_gnn), ("placer", t.grad_placer), ("head", [t.grad_head])):
        for l, lg in enumerate(layers):
            for k, v in lg.items():
                if k.endswith("_qkv"):
                    out.update({f"{part}[{l}].{k[0]}_{q}": to_np(v[i * d:(i + 1) * d]) for i, q in enumerate("qkv")})
                else:
                    out[f"{part}[{l}].{k}"] = to_np(v)
    return out


def _opposed(dtype, **over):
    """Two copies of one graph with gradients dL/dlogits of opposite sign.  Every
    row of one copy is then the other's negative, and every weight's gradient
    their sum: 0 where each operation rounds both ways alike.  The norms of those
    gradients, by the norms under independent gradients of the same size."""
    cfg = W.get_config("tiny_layered_256").replace(dtype=dtype, **over)
    one, w = W.make_graph(cfg), W.make_weights(cfg)
    n, e = one.n_nodes, one.n_edges
    g = W.graph_from_arrays(cfg, [0, n, 2 * n], np.concatenate([one.row_ptr, one.row_ptr[1:] + e]),
                            np.concatenate([one.col_idx, one.col_idx + n]), np.concatenate([one.x, one.x]))
    t = _trainer(cfg, g, w)
    logits, _ = t.forward()
    assert bool((logits[:n] == logits[n:]).all())
    dl = (np.random.default_rng(8).normal(size=(2 * n, cfg.n_devices)) / np.sqrt(n)).astype(np.float32)
    free = _gradients(t, dl)
    opposed = _gradients(t, np.concatenate([dl[:n], -dl[:n]]))
    return {k: float(np.linalg.norm(opposed[k].astype(np.float64)) / np.linalg.norm(free[k].astype(np.float64)))
            for k in free}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_products_round_both_ways_alike(dtype):
    """The last layer's gradients behind the head: dH = dR W_2 and dZ = dH W_1 over
    16,386 rows in 128 x 128 tiles.  A result that leans by r of its root mean
    square appears as r sqrt(16,386) = 128 r: 4e-7 to 1e-6 for the 3e-9 to 8e-9 of
    products with all planes on one sum, against the rounding of the sums over
    rows, 3e-8 for columns and 1e-7 for w_1 (16 rows an instruction)."""
    err = _opposed(dtype, graph_sizes=(8193,), hidden=128, heads=4, d_ff=1024, seg_len=128, mem_len=128)
    got = {k: err[f"placer[1].{k}"] for k in ("b_o", "ln1_g", "ln1_b", "w_1", "b_1", "b_2", "ln2_g", "ln2_b")}
    _log("  opposed gradients", {k: f"{v:.1e}" for k, v in got.items()})
    assert max(got.values()) <= 2e-7, got


@pytest.mark.parametrize("heads,seg", [(8, 128), (4, 128), (4, 96), (2, 128)])
def test_attention_rounds_both_ways_alike(heads, seg):
    """The gradients of W_q and W_k, differences of sums far larger than they are:
    4e-7 to 9e-7 with fp32 instructions (each result rounded to either side), 3e-6
    to 2e-5 where every row's dO . v, dQ and dK lean by 6e-9 of their size, as with
    all plane pairs on one sum."""
    err = _opposed("bf16" if heads == 4 else "f32", graph_sizes=(8193,), hidden=128, heads=heads, d_ff=256, seg_len=seg,
                   mem_len=seg - 28)
    got = {k: v for k, v in err.items() if k.startswith("placer") and k.split(".")[1] in ("w_q", "w_k", "w_v", "b_v")}
    _log("  opposed gradients", {k: f"{v:.1e}" for k, v in got.items()})
    assert max(got.values()) <= 1.5e-6, got


def _extreme(case, dtype, n, hidden, **over):
    """A policy and a graph whose products meet operands that a bf16 cannot hold,
    every result of the forward finite."""
    cfg = W.get_config("tiny_layered_256").replace(**{**dict(dtype=dtype, graph_sizes=(n,), hidden=hidden,
                                                             heads=hidden // 32, placer_layers=1, film=False), **over})
    g, w = W.make_graph(cfg), W.make_weights(cfg)
    x = g.x.copy()
    rows = [0, n // 2, n - 1]

    def put(layer, name, change):
        a = layer[name][0].copy()
        change(a)
        layer[name] = W._finish(cfg, a)

    def negative(*cols):
        def change(a):
            a[:, cols] = -0.01
        return change
    if case in ("huge", "infinite"):           # features in column 3
        x[rows, 3] = 3.4e38 if case == "huge" else np.inf
        put(w.gnn[0], "w_self", negative(3))   # the rows' ReLU is 0, their sigmoids 0 or 1
        if case == "huge":
            put(w.gnn[0], "w_pool", negative(3))
    elif case == "huge_hidden":                # layer 0's output 3.399e38 in column 5, from features bf16 can hold
        x[rows, 3], x[rows, 4] = 2.0 ** 127, 1.5 * 2.0 ** 119
        put(w.gnn[0], "w_pool", negative(3, 4))

        def one_large(a):
            a[:, [3, 4]] = -0.01
            a[5, [3, 4]] = 255 / 128, 1.0
        put(w.gnn[0], "w_self", one_large)
        put(w.gnn[1], "w_self", negative(5))
        put(w.gnn[1], "w_pool", negative(5))
    elif case == "huge_keys":                  # keys of 3.4e38 in column 0 for some rows: no weight, no gradient
        x[:, 3] = 0.0
        x[rows, 3] = 1.0                       # the rows' column 5 is 1, the others' 0
        for layer, col in zip(w.gnn, (3, 5)):
            def carry(a, col=col):
                a[5] = 0.0
                a[5, col] = 1.0
            put(layer, "w_self", carry)
            put(layer, "w_neigh", lambda a: a[5].fill(0.0))
            put(layer, "b_upd", lambda a: a[5:6].fill(0.0))

        def keys(a):
            a[[0, hidden]] = 0.0
            a[hidden, 5] = 3.4e38

        def biases(a):
            a[0], a[hidden] = -1.0, 0.0
        put(w.placer[0], "w_qkv", keys)
        put(w.placer[0], "b_qkv", biases)
    else:                                      # keys of minus infinity for part of the rows: no weight
        def keys(a):
            a[0] = 0.0                         # query column 0: -1, from its bias
            a[hidden] = 0.0
            a[hidden, :2] = 3e38
        put(w.placer[0], "w_qkv", keys)

        def query(a):
            a[0] = -1.0
        put(w.placer[0], "b_qkv", query)
    return cfg, W.graph_from_arrays(cfg, [0, n], g.row_ptr, g.col_idx, x), w


@pytest.mark.parametrize("case,dtype,n,hidden", [
    ("huge", "f32", 300, 64), ("huge", "f32", 32800, 256), ("huge_hidden", "f32", 300, 128),
    ("huge_hidden", "bf16", 300, 64), ("huge_hidden", "bf16", 32800, 256), ("infinite", "f32", 300, 64),
    ("infinite", "f32", 32800, 256), ("infinite_keys", "f32", 300, 64), ("infinite_keys", "bf16", 300, 128)])
def test_operands_beyond_bf16(case, dtype, n, hidden):
    """Infinite operands and finite ones that round to a bf16 infinity (3.396e38 to
    3.403e38), in 64 x 64 and 128 x 128 tiles and in the bf16 weights' kernel: what
    fp32 products give, an infinity only where one of them is."""
    import torch
    cfg, g, w = _extreme(case, dtype, n, hidden)
    _log("operands beyond bf16", case, dtype, n)
    t = _trainer(cfg, g, w)
    logits, _ = t.forward()
    dl = (np.random.default_rng(9).normal(size=(n, cfg.n_devices)) / np.sqrt(n)).astype(np.float32)
    t.backward(torch.from_numpy(dl).cuda())
    torch.cuda.synchronize()
    gnn, pl, hd = w.f64()
    x = np.where(np.isinf(g.x), 1e30, g.x)     # in the oracle as good as infinite (its masks are products)
    ref = PG.policy_backward(g.graph_ptr, g.row_ptr, g.col_idx, x, gnn, pl, hd["w_out"], hd["b_out"],
                             dl.astype(np.float64), fanout=cfg.fanout, nb_seed=cfg.nb_seed, n_heads=cfg.heads,
                             seg_len=cfg.seg_len, mem_len=cfg.mem_len, film=False, decisions=t.decisions())
    # the oracle's own decisions: the GPU's ReLU turns a NaN into 0, which pinned ones would follow
    own = O.policy_forward(g.graph_ptr, g.row_ptr, g.col_idx, x, gnn, pl, hd["w_out"], hd["b_out"], fanout=cfg.fanout,
                           nb_seed=cfg.nb_seed, n_heads=cfg.heads, seg_len=cfg.seg_len, mem_len=cfg.mem_len,
                           k_samples=1, sample_seed=0, film=False)["logits"]
    assert np.isfinite(own).all()
    assert rel_err_rows(to_np(logits), own) <= TOL[dtype]
    if case == "infinite_keys":
        return                                 # a gradient through them is 0 * infinity
    if case == "infinite":                     # and so is that of the infinite features' weights
        for k in ("w_self", "w_pool"):
            assert np.isnan(to_np(t.grad_gnn[0][k][:, 3])).all()
            ref["gnn"][0][k][:, 3] = 0.0
            t.grad_gnn[0][k][:, 3] = 0.0
    _compare_grads(t, ref, cfg, film=False)


@pytest.mark.parametrize("heads,hidden,seg", [(4, 64, 64), (4, 64, 128), (2, 64, 64), (4, 128, 128), (2, 128, 64)])
def test_gradients_of_keys_beyond_bf16(heads, hidden, seg):
    """Finite keys that round to a bf16 infinity, without weight in any query: the
    gradients of every query and key are those of fp32 products, in each form of
    the attention's backward (head sizes of 16, 32 and 64, one and two columns)."""
    import torch
    n = 300
    cfg, g, w = _extreme("huge_keys", "f32", n, hidden, heads=heads, seg_len=seg, mem_len=50)
    _log("keys beyond bf16", heads, hidden, seg)
    t = _trainer(cfg, g, w)
    logits, _ = t.forward()
    dl = (np.random.default_rng(9).normal(size=(n, cfg.n_devices)) / np.sqrt(n)).astype(np.float32)
    t.backward(torch.from_numpy(dl).cuda())
    torch.cuda.synchronize()
    gnn, pl, hd = w.f64()
    ref = PG.policy_backward(g.graph_ptr, g.row_ptr, g.col_idx, g.x, gnn, pl, hd["w_out"], hd["b_out"],
                             dl.astype(np.float64), fanout=cfg.fanout, nb_seed=cfg.nb_seed, n_heads=cfg.heads,
                             seg_len=cfg.seg_len, mem_len=cfg.mem_len, film=False, decisions=t.decisions())
    assert np.isfinite(ref["logits"]).all()
    assert rel_err_rows(to_np(logits), ref["logits"]) <= TOL["f32"]
    _compare_grads(t, ref, cfg, film=False)


@pytest.mark.parametrize("seg,mem", [(2 ** 31 - 1, 0), (2 ** 31 - 64, 2 ** 31 - 1), (2 ** 30 + 1, 7)])
def test_segments_longer_than_any_graph(seg, mem):
    """Up to the largest int: the same bits as segments that just hold every graph,
    in the placement network and in both passes of the update step."""
    import torch

    from paper_1910_01578_amd import gdp
    dl, got = None, []
    for s in (640, seg):
        cfg = W.get_config("tiny_layered_256").replace(graph_sizes=(300, 129), seg_len=s, mem_len=mem)
        g, w = W.make_graph(cfg), W.make_weights(cfg)
        t = _trainer(cfg, g, w)
        logits, _ = t.forward()
        dl = dl if dl is not None else torch.randn(g.n_nodes, cfg.n_devices, device="cuda")
        out = {"logits": to_np(logits), **_gradients(t, dl.cpu().numpy())}
        r = gdp.Runner(t.graph, t.policy, cfg.k_samples)
        r.forward(cfg.sample_seed)
        out["place"] = to_np(r.logits)
        got.append(out)
    torch.cuda.synchronize()
    _log("long segments", seg, mem)
    assert all(np.array_equal(got[0][k], got[1][k]) for k in got[0])
    assert all(np.isfinite(v).all() for v in got[0].values())
