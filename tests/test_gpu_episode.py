"""GPU parity of the on-device MDP transition and episode loop (Section 2.1) against the
float64 oracle (oracle/episode.py + the forward oracle), through the C ABI.

The sampled action is an integer decided by floating point: the kernel decides in fp32 on its
own logits, the oracle in float64 on the same logits; they may differ only where the uniform
number lies within MARGIN of a boundary of the cumulative distribution, and then only by
picking the neighbouring device.  Everything the transition writes is compared bit for bit
given the action; each step's logits are compared with the oracle's forward pass on the same
state (the oracle replays the device's actions)."""
import numpy as np
import pytest

import oracle
from oracle import episode as ep
from workloads import make_workload, make_episode

from gpu_common import assert_logits_close

pytestmark = pytest.mark.gpu
MARGIN = 1e-5


def check_action(logits_row, u, a_gpu, what):
    a_ref = ep.sample_action(logits_row.astype(np.float64), float(u))
    if a_gpu == a_ref:
        return
    assert ep.decision_margin(logits_row.astype(np.float64), float(u)) < MARGIN and abs(a_gpu - a_ref) == 1, \
        f"{what}: action {a_gpu}, oracle {a_ref}, u {u}, logits {logits_row}"


def test_single_transition_on_synthetic_logits():
    import torch
    import paper_1906_08879_amd as pl
    dev = torch.device("cuda:0")
    w = make_workload("layered200", B=40)
    D = w.D
    rng = np.random.default_rng(77)
    order, _, _ = make_episode(w, 1)
    t = 3
    logits = (rng.normal(size=(w.B, D)) * 2).astype(np.float32)
    logits[0] = 0.0                                   # uniform
    logits[1] = [0.0, 60.0, 0.0, -5.0]                # saturated
    logits[2] = [1e6, 1e6 - 1.0, 1e6 - 2.0, -1e6]     # large scale, as the raw features give
    u = rng.random(w.B, dtype=np.float32)
    u[0], u[3], u[4] = 0.25, 0.0, np.float32(1.0 - 2.0 ** -24)
    placement = rng.integers(0, D, size=w.n_tot).astype(np.int32)
    feats = np.array(w.node_feats, dtype=np.float32)
    feats[:, 2] = 0.0
    cur = np.array([order[w.node_off[b] + t] for b in range(w.B)], dtype=np.int32)
    cur[5] = -1                                       # an episode that is over
    cur[6] = int(w.n_nodes[6])                        # outside the graph
    g = pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst)
    t_l, t_u, t_o = (torch.from_numpy(x).to(dev) for x in (logits, u, order))
    t_f, t_p, t_c = (torch.from_numpy(x.copy()).to(dev) for x in (feats, placement, cur))
    act = torch.full((w.B,), 99, dtype=torch.int32, device=dev)
    logp = torch.full((w.B,), float("nan"), dtype=torch.float32, device=dev)
    pl.episode_step(g, D, t_l, t_u, t_o, t, t_f, t_p, t_c, act, logp)
    torch.cuda.synchronize()
    act, logp = act.cpu().numpy(), logp.cpu().numpy()
    new_f, new_p, new_c = t_f.cpu().numpy(), t_p.cpu().numpy(), t_c.cpu().numpy()
    exp_p, exp_f = placement.copy(), feats.copy()
    for b in range(w.B):
        n0, n_b = int(w.node_off[b]), int(w.n_nodes[b])
        if b in (5, 6):
            assert act[b] == -1 and logp[b] == 0.0 and new_c[b] == -1
            continue
        check_action(logits[b], u[b], int(act[b]), f"graph {b}")
        assert abs(logp[b] - ep.log_prob(logits[b].astype(np.float64), int(act[b]))) <= 1e-5 * max(1.0, abs(logp[b]))
        vis = exp_f[n0:n0 + n_b, 2].astype(np.float64)
        nxt = ep.transition(exp_p[n0:n0 + n_b], vis, order[n0:n0 + n_b], t, int(cur[b]), int(act[b]))
        exp_f[n0:n0 + n_b, 2] = vis
        assert new_c[b] == nxt
    np.testing.assert_array_equal(new_p, exp_p)
    np.testing.assert_array_equal(new_f, exp_f)
    assert act[0] == 1 and act[1] == 1 and act[3] == ep.sample_action(logits[3].astype(np.float64), 0.0)
    g.close()


def replay(w, b, order, uniforms, placement0, actions):
    """The oracle's episode of graph b with the device's actions forced."""
    n0, n1 = int(w.node_off[b]), int(w.node_off[b + 1])
    e0, e1 = int(w.edge_off[b]), int(w.edge_off[b + 1])
    blob = oracle.weights_as_stored(w.weights, w.D, w.H, w.n_layers, w.group_by_device, w.weight_dtype)
    base = np.array(w.node_feats[n0:n1], dtype=np.float64)

    def fwd(placement, visited, cur):
        feats = base.copy()
        feats[:, 2] = visited
        return oracle.forward_graph(n1 - n0, w.edge_src[e0:e1], w.edge_dst[e0:e1], feats, placement, cur,
                                    blob, w.D, w.H, w.n_layers, w.k_sweeps, w.group_by_device)["logits"]

    return ep.run_episode(fwd, n1 - n0, placement0[n0:n1], order[n0:n1], uniforms[:, b], actions=actions)


def run_device_episode(w, n_steps, order, uniforms, placement0):
    import torch
    import paper_1906_08879_amd as pl
    dev = torch.device("cuda:0")
    g = pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst)
    wt = pl.Weights(w.weights, w.D, w.H, w.n_layers, w.k_sweeps, w.group_by_device, w.weight_dtype)
    feats = np.array(w.node_feats, dtype=np.float32)
    feats[:, 2] = 0.0
    cur = np.array([order[w.node_off[b]] for b in range(w.B)], dtype=np.int32)
    t_f, t_p, t_c, t_o, t_u = (torch.from_numpy(np.ascontiguousarray(x)).to(dev)
                               for x in (feats, placement0, cur, order, uniforms))
    logits = torch.full((n_steps, w.B, w.D), float("nan"), dtype=torch.float32, device=dev)
    act = torch.full((n_steps, w.B), 99, dtype=torch.int32, device=dev)
    logp = torch.full((n_steps, w.B), float("nan"), dtype=torch.float32, device=dev)
    pl.episode_run(g, wt, t_f, t_p, t_c, t_o, t_u, 0, n_steps, logits, True, act, logp)
    torch.cuda.synchronize()
    out = dict(logits=logits.cpu().numpy(), actions=act.cpu().numpy(), logp=logp.cpu().numpy(),
               placement=t_p.cpu().numpy(), visited=t_f.cpu().numpy()[:, 2], cur=t_c.cpu().numpy())
    g.close()
    wt.close()
    return out


def check_against_replay(w, b, n_steps, order, uniforms, placement0, dev_out, complete):
    n0, n1 = int(w.node_off[b]), int(w.node_off[b + 1])
    T = min(n_steps, n1 - n0)
    r = replay(w, b, order, uniforms[:T], placement0, dev_out["actions"][:T, b])
    assert_logits_close(dev_out["logits"][:T, b], r["logits"], f"{w.name} graph {b}: logits of every step", 0.1)
    for t in range(T):
        check_action(dev_out["logits"][t, b], uniforms[t, b], int(dev_out["actions"][t, b]), f"graph {b} step {t}")
        lp = ep.log_prob(dev_out["logits"][t, b].astype(np.float64), int(dev_out["actions"][t, b]))
        assert abs(dev_out["logp"][t, b] - lp) <= 1e-5 * max(1.0, abs(lp)), (b, t)
    np.testing.assert_array_equal(dev_out["placement"][n0:n1], r["placement"])
    np.testing.assert_array_equal(dev_out["visited"][n0:n1], r["visited"].astype(np.float32))
    assert dev_out["cur"][b] == r["cur"]
    if complete:                                      # Section 2.1: |V| steps visit every node once
        assert r["cur"] == -1 and r["visited"].sum() == n1 - n0
        assert (dev_out["actions"][T:, b] == -1).all() and (dev_out["logp"][T:, b] == 0).all()


@pytest.mark.parametrize("name,B", [("random32", 1), ("layered200", 6)])
def test_whole_episode_matches_oracle_replay(name, B):
    w = make_workload(name, B=B)
    n_steps = int(w.n_nodes.max()) + 2                # two steps past the end: nothing may change
    order, uniforms, placement0 = make_episode(w, n_steps)
    out = run_device_episode(w, n_steps, order, uniforms, placement0)
    for b in range(w.B):
        check_against_replay(w, b, n_steps, order, uniforms, placement0, out, complete=True)


def test_episode_segment_at_full_size():
    # the batch and launch configuration that the benchmark times; two graphs are replayed
    w = make_workload("nasnet")
    n_steps = 6
    order, uniforms, placement0 = make_episode(w, n_steps)
    out = run_device_episode(w, n_steps, order, uniforms, placement0)
    assert np.isfinite(out["logits"]).all()
    assert ((out["actions"] >= 0) & (out["actions"] < w.D)).all()
    for b in (0, w.B - 1):
        check_against_replay(w, b, n_steps, order, uniforms, placement0, out, complete=False)
    # every graph: exactly n_steps nodes visited, those of its order, placed where the actions say
    for b in range(w.B):
        n0 = int(w.node_off[b])
        first = order[n0:n0 + n_steps] + n0
        assert out["visited"][n0:int(w.node_off[b + 1])].sum() == n_steps
        np.testing.assert_array_equal(out["placement"][first], out["actions"][:, b])
        assert out["cur"][b] == order[n0 + n_steps]


def test_episode_loop_replays_from_a_hip_graph():
    """Sixteen steps of forward pass + transition captured once (with the reset of the state)
    and replayed three times, with eager work in between: the actions equal the eager run's."""
    import torch
    import paper_1906_08879_amd as pl
    dev = torch.device("cuda:0")
    w = make_workload("layered200", B=12)
    T = 16
    order, uniforms, placement0 = make_episode(w, T)
    eager = run_device_episode(w, T, order, uniforms, placement0)
    g = pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst)
    wt = pl.Weights(w.weights, w.D, w.H, w.n_layers, w.k_sweeps, w.group_by_device, w.weight_dtype)
    f0 = np.array(w.node_feats, dtype=np.float32)
    f0[:, 2] = 0.0
    cur0 = np.array([order[w.node_off[b]] for b in range(w.B)], dtype=np.int32)
    tf0, tp0, tc0, to, tu = (torch.from_numpy(np.ascontiguousarray(x)).to(dev)
                             for x in (f0, placement0, cur0, order, uniforms))
    tf, tp, tc = tf0.clone(), tp0.clone(), tc0.clone()
    logits = torch.empty((w.B, w.D), dtype=torch.float32, device=dev)
    act = torch.empty((T, w.B), dtype=torch.int32, device=dev)
    pl.embed_forward(g, tf, tp, tc, wt, logits)                     # first call allocates
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        graph.capture_begin()
        tf.copy_(tf0); tp.copy_(tp0); tc.copy_(tc0)
        pl.episode_run(g, wt, tf, tp, tc, to, tu, 0, T, logits, False, act, None, stream=side)
        graph.capture_end()
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        act.fill_(77)
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(act.cpu().numpy(), eager["actions"])
        np.testing.assert_array_equal(tp.cpu().numpy(), eager["placement"])
        pl.embed_forward(g, tf0, tp0, tc0, wt, logits)              # eager work between the replays
        torch.cuda.synchronize()
    del graph
    g.close()
    wt.close()


def test_ragged_batch_graphs_finish_at_different_steps():
    """Graphs of 3, 11 and 26 nodes in one batch: each episode ends after its own |V| steps and
    is left untouched afterwards, while the others go on."""
    from workloads import tiny_random_dag, weight_count
    from workloads.synthetic import Workload
    rng = np.random.default_rng(21)
    sizes, D, H = [3, 11, 26], 3, 32
    n_nodes, n_edges, srcs, dsts, feats = [], [], [], [], []
    for n in sizes:
        s, d = tiny_random_dag(rng, n, 0.3)
        n_nodes.append(n); n_edges.append(len(s)); srcs.append(s); dsts.append(d)
        feats.append(np.stack([rng.lognormal(0, 1, n), rng.lognormal(2, 1, n), np.zeros(n)], axis=1))
    w = Workload(name="ragged", B=len(sizes), D=D, H=H, n_layers=2, k_sweeps=1, group_by_device=1, weight_dtype="fp32",
                 n_nodes=np.array(n_nodes, np.int32), n_edges=np.array(n_edges, np.int32),
                 edge_src=np.concatenate(srcs).astype(np.int32), edge_dst=np.concatenate(dsts).astype(np.int32),
                 node_feats=np.concatenate(feats).astype(np.float32), placement=np.zeros(sum(sizes), np.int32),
                 cur_node=np.zeros(len(sizes), np.int32),
                 weights=rng.normal(0, 0.1, weight_count(D, H, 2, True)).astype(np.float32))
    n_steps = max(sizes) + 1
    order, uniforms, placement0 = make_episode(w, n_steps)
    out = run_device_episode(w, n_steps, order, uniforms, placement0)
    for b in range(w.B):
        check_against_replay(w, b, n_steps, order, uniforms, placement0, out, complete=True)


def ragged_workload(rng, sizes, D, H, L, wd, k=1, group=1):
    from workloads import tiny_random_dag, weight_count
    from workloads.synthetic import Workload
    n_nodes, n_edges, srcs, dsts = [], [], [], []
    for n in sizes:
        s, d = tiny_random_dag(rng, n, 0.2)
        n_nodes.append(n); n_edges.append(len(s)); srcs.append(s); dsts.append(d)
    N = sum(sizes)
    feats = np.stack([rng.lognormal(0, 1, N), rng.lognormal(2, 1, N), np.zeros(N)], axis=1)
    return Workload(name="ragged", B=len(sizes), D=D, H=H, n_layers=L, k_sweeps=k, group_by_device=group, weight_dtype=wd,
                    n_nodes=np.array(n_nodes, np.int32), n_edges=np.array(n_edges, np.int32),
                    edge_src=np.concatenate(srcs).astype(np.int32), edge_dst=np.concatenate(dsts).astype(np.int32),
                    node_feats=feats.astype(np.float32), placement=np.zeros(N, np.int32),
                    cur_node=np.zeros(len(sizes), np.int32),
                    weights=rng.normal(0, 0.02, weight_count(D, H, L, bool(group))).astype(np.float32))


# (steps per pass: 7, 4, 2, 3 of 7, 2, 1; both sides of the batch sizes where another kernel would take more copies)
@pytest.mark.parametrize("graphs,D,H,L,wd,k,group,n_steps", [
    (1, 2, 8, 2, "fp32", 1, 1, 20), (3, 4, 16, 1, "fp32", 2, 0, 9), (51, 4, 32, 2, "fp32", 1, 1, 5),
    (5, 3, 64, 1, "fp32", 1, 1, 7), (43, 2, 64, 1, "fp32", 1, 1, 4), (64, 2, 64, 2, "fp32", 2, 1, 5),
    (1, 16, 64, 2, "bf16", 1, 0, 3), (2, 8, 128, 2, "bf16", 1, 1, 8), (4, 1, 32, 2, "bf16", 1, 1, 13),
    (130, 2, 8, 2, "fp32", 1, 1, 3)])
def test_steps_taken_together_equal_single_steps_bit_for_bit(graphs, D, H, L, wd, k, group, n_steps):
    """pl_episode_run against a loop of pl_embed_forward and pl_episode_step: logits, actions, log-probabilities and
    states are the same bits, also for graphs that finish on the way, that are over or in no valid state from the
    start, and whose visiting order names a node twice; again on the same batch with fewer steps, then with more."""
    import torch
    import paper_1906_08879_amd as pl
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(1000 * graphs + H)
    sizes = [int(x) for x in rng.integers(2, 40, graphs)]
    w = ragged_workload(rng, sizes, D, H, L, wd, k, group)
    off = np.concatenate([[0], np.cumsum(sizes)])
    order = np.concatenate([rng.permutation(n) for n in sizes]).astype(np.int32)
    order[off[0] + 1] = order[off[0]]                                # the first graph visits a node twice
    cur = order[off[:-1]].copy()
    if graphs > 2:
        cur[1], cur[2] = -1, sizes[2]
    placement = rng.integers(0, D, w.n_tot).astype(np.int32)
    uniforms = rng.random((2 * n_steps, graphs), dtype=np.float32)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    wt = pl.Weights(w.weights, D, H, L, k, group, wd)
    runs = {}
    for together in (True, False):
        g = pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst)
        out = []
        f, p, c, o, u = to(w.node_feats), to(placement), to(cur), to(order), to(uniforms)
        t0 = 0
        for steps, keep in ((n_steps, True), (max(1, n_steps // 2), False), (n_steps, True)):
            t0 = 0 if t0 + steps > 2 * n_steps else t0
            logits = torch.full((steps if keep else 1, graphs, D), 7.0, device=dev)
            act = torch.full((steps, graphs), 99, dtype=torch.int32, device=dev)
            logp = torch.full((steps, graphs), 9.0, device=dev)
            if together:
                pl.episode_run(g, wt, f, p, c, o, u[t0:t0 + steps], t0, steps, logits, keep, act, logp)
            else:
                for i in range(steps):
                    l = logits[i if keep else 0]
                    pl.embed_forward(g, f, p, c, wt, l)
                    pl.episode_step(g, D, l, u[t0 + i], o, t0 + i, f, p, c, act[i], logp[i])
            t0 += steps
            torch.cuda.synchronize()
            out += [x.cpu().numpy().view(np.int32) for x in (logits, act, logp, f, p, c)]
        runs[together] = out
        g.close()
    wt.close()
    for i, (a, b) in enumerate(zip(runs[True], runs[False])):
        np.testing.assert_array_equal(a, b, err_msg=f"output {i}")


# (calls of one batch in turn: "e" runs at once, "c" is captured, "r" replays the last capture; then the number of steps, and a
# second network of another width and number of devices as "w"; a call that was captured step by step, before there were copies,
# uses the buffers of the batch's last network, as pl_embed_forward does, and is not replayed after the other one)
@pytest.mark.parametrize("graphs,D,H,wd,D2,H2", [(1, 8, 128, "bf16", 8, 64), (3, 4, 16, "fp32", 8, 128), (1, 3, 64, "fp32", 16, 64)])
@pytest.mark.parametrize("calls", [
    "e8 c4 e4 r e8 r e4 r", "e8 c8 e4 r e8 r", "e4 c4 e8 r w8 r e3 r", "w8 e1 c8 r e8 r c3 r e4 r", "e1 c8 r e8 r c8 r e4 r", "e8 w8 c3 e8 r w8 r"])
def test_captured_episodes_beside_others_on_the_same_batch(graphs, D, H, wd, D2, H2, calls):
    """Every call and every replay of a captured one equals single steps, bit for bit, whatever ran on the batch before it
    and between capture and replay."""
    import torch
    import paper_1906_08879_amd as pl
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(H + D + graphs)
    sizes = [int(x) for x in rng.integers(9, 40, graphs)]
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    w = ragged_workload(rng, sizes, D, H, 2, wd)
    off = np.concatenate([[0], np.cumsum(sizes)])
    order = np.concatenate([rng.permutation(n) for n in sizes]).astype(np.int32)
    o, cur0, u = to(order), to(order[off[:-1]]), to(rng.random((8, graphs), dtype=np.float32))
    f0 = to(w.node_feats)
    g, single = (pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst) for _ in range(2))
    side = torch.cuda.Stream()

    class Net:
        def __init__(self, D, H, wd, weights):
            self.D, self.wt = D, pl.Weights(weights, D, H, 2, 1, 1, wd)
            self.p0 = to(rng.integers(0, D, w.n_tot).astype(np.int32))

        def call(self, steps, how):
            """Reset, then the episode's first steps; returns what they write and, if captured, the graph."""
            f, p, c = torch.empty_like(f0), torch.empty_like(self.p0), torch.empty_like(cur0)
            out = (torch.full((steps, graphs, self.D), 7.0, device=dev), torch.full((steps, graphs), 9, dtype=torch.int32, device=dev),
                   torch.full((steps, graphs), 9.0, device=dev), f, p, c)
            batch = single if how == "single" else g

            def run(stream):
                f.copy_(f0); p.copy_(self.p0); c.copy_(cur0)
                if how == "single":
                    for i in range(steps):
                        pl.embed_forward(batch, f, p, c, self.wt, out[0][i])
                        pl.episode_step(batch, self.D, out[0][i], u[i], o, i, f, p, c, out[1][i], out[2][i])
                else:
                    pl.episode_run(batch, self.wt, f, p, c, o, u[:steps], 0, steps, out[0], True, out[1], out[2], stream=stream)

            torch.cuda.synchronize()
            if how != "capture":
                run(torch.cuda.current_stream())
                torch.cuda.synchronize()
                return out, None
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.stream(side):
                graph.capture_begin()
                run(side)
                graph.capture_end()
            return out, graph

    main = Net(D, H, wd, w.weights)
    other = ragged_workload(rng, sizes, D2, H2, 2, "bf16")
    wide = Net(D2, H2, "bf16", other.weights)
    want = {}

    def same(net, steps, out, what):
        if (net, steps) not in want:
            want[net, steps] = [x.cpu().numpy().view(np.int32) for x in net.call(steps, "single")[0]]
        for i, (a, b) in enumerate(zip(out, want[net, steps])):
            np.testing.assert_array_equal(a.cpu().numpy().view(np.int32), b, err_msg=f"{what}: output {i}")

    captured = None
    for at, call in enumerate(calls.split()):
        what = f"{calls}, call {at} ({call})"
        if call == "r":
            for x in captured[1]:
                x.fill_(5)
            captured[2].replay()
            torch.cuda.synchronize()
            same(main, captured[0], captured[1], what)
            continue
        steps = int(call[1:])
        net = wide if call[0] == "w" else main
        out, graph = net.call(steps, "capture" if call[0] == "c" else "eager")
        if graph is None:
            same(net, steps, out, what)
        else:
            captured = steps, out, graph
    del captured, graph
    g.close(); single.close(); main.wt.close(); wide.wt.close()


def test_only_episodes_before_a_captured_forward_pass():
    """A batch that only pl_episode_run has used, in passes of several steps, has the buffers of single passes too: a forward
    pass captured then replays with the eager one's bits."""
    import torch
    import paper_1906_08879_amd as pl
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(3)
    w = ragged_workload(rng, [17, 23], 4, 64, 2, "bf16")
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    f, p, c = to(w.node_feats), to(w.placement), to(w.cur_node)
    o = to(np.concatenate([np.arange(17), np.arange(23)]).astype(np.int32))
    u = to(rng.random((6, 2), dtype=np.float32))
    wt = pl.Weights(w.weights, 4, 64, 2, 1, 1, "bf16")
    g = pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst)
    logits, eager = (torch.empty((2, 4), device=dev) for _ in range(2))
    pl.episode_run(g, wt, f, p, c, o, u, 0, 6, logits)
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        graph.capture_begin()
        pl.embed_forward(g, f, p, c, wt, logits, stream=side)
        graph.capture_end()
    pl.embed_forward(g, f, p, c, wt, eager)
    for _ in range(3):
        logits.fill_(1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(logits, eager)
    del graph
    g.close(); wt.close()
