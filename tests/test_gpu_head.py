"""The policy head where its launch shape changes: a workgroup per (graph, set) or per graph (H = 128, either
side of 256 workgroups), more device groups than rows in a pass, widths whose last block of inputs is short
and widths that take the three networks one after the other.  Against the float64 oracle, with the logit
bar of tests/test_gpu_parity.py; every call must give the same bits (the workgroups of a graph hand over
through counters that have to be zero again)."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import assert_logits_close
from workloads import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,D,H,by_device", [(85, 8, 128, 1), (86, 8, 128, 1), (5, 16, 128, 1), (4, 3, 128, 0), (3, 16, 256, 1),
                                             (3, 9, 100, 1), (2, 5, 17, 1), (70, 16, 64, 1), (9, 2, 32, 0)])
def test_head_launch_shapes(B, D, H, by_device):
    import torch
    import paper_1906_08879_amd as pl
    w = make_workload("random32", B=B, D=D, H=H, group_by_device=by_device, weight_dtype="bf16" if H == 128 else "fp32")
    w.node_feats[:, :2] /= w.node_feats[:, :2].mean(axis=0)
    dev = torch.device("cuda:0")
    g = pl.GraphBatch(w.n_nodes, w.n_edges, w.edge_src, w.edge_dst)
    wt = pl.Weights(w.weights, w.D, w.H, w.n_layers, w.k_sweeps, w.group_by_device, w.weight_dtype)
    args = [torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in (w.node_feats, w.placement, w.cur_node)]
    got = []
    for _ in range(3):
        logits = torch.empty((B, D), dtype=torch.float32, device=dev)
        pl.embed_forward(g, *args, wt, logits)
        got.append(logits)
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    ref = oracle.forward_workload(w, n_threads=4, want_emb=False)["logits"]
    # (logits near zero in a row of larger ones miss a bound relative to themselves: see test_gpu_parity.py)
    assert_logits_close(got[0].cpu().numpy().astype(np.float64), ref, f"B {B} D {D} H {H}", max_fail_frac=0.01)
