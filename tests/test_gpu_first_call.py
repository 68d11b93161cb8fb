"""The first call on a batch allocates its buffers and clears what has to be zero in them: on the caller's
stream.  Gradients are taken on a stream that does not wait for the null stream, while that one is busy: the first
call must not wait for its work, and a clear behind that work would land in the middle of a gradient."""
import numpy as np
import pytest

from workloads import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("forward_first", [False, True])
def test_first_calls_beside_a_busy_null_stream(forward_first):
    import torch
    import paper_1906_08879_amd as pl
    dev = torch.device("cuda:0")
    w = make_workload("nmt", B=16)
    rng = np.random.default_rng(6)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    feats, place, cur = to(w.node_feats.astype(np.float32)), to(w.placement), to(w.cur_node)
    act, co = to(rng.integers(0, w.D, w.B).astype(np.int32)), to(rng.normal(0, 1, w.B).astype(np.float32))
    wt = pl.Weights(w.weights, w.D, w.H, w.n_layers, w.k_sweeps, w.group_by_device, w.weight_dtype)
    n_par = pl.weights_count(w.D, w.H, w.n_layers, w.k_sweeps, w.group_by_device, w.weight_dtype)
    most = 300
    grads, logits = torch.empty((most, n_par), device=dev), torch.empty((most, w.B, w.D), device=dev)
    ref, ref_logits = torch.empty(n_par, device=dev), torch.empty((w.B, w.D), device=dev)
    a = torch.randn((4096, 4096), device=dev)
    b = a @ a
    g = pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst)
    pl.policy_gradient(g, feats, place, cur, wt, act, co, ref, ref_logits)
    g.close()
    side, busy = torch.cuda.Stream(), torch.cuda.Event()
    g = pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst)
    pl.graph_batch_upload(g)
    torch.cuda.synchronize()
    for _ in range(250):                                 # tens of milliseconds more than a first call takes
        torch.mm(a, a, out=b)
    busy.record()
    if forward_first:
        pl.embed_forward(g, feats, place, cur, wt, logits[0], stream=side)
    done = beside = 0
    while done < most and beside < 8:                    # gradients until a few after the null stream's work
        pl.policy_gradient(g, feats, place, cur, wt, act, co, grads[done], logits[done], stream=side)
        done += 1
        if done % 4 == 0:
            side.synchronize()
        beside += busy.query()
    torch.cuda.synchronize()
    assert done > beside                                 # the first ones were enqueued while the null stream worked
    for k in range(done):
        assert torch.equal(grads[k], ref) and torch.equal(logits[k], ref_logits), k
    g.close()
    wt.close()
