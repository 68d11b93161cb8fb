"""The generic pooling kernel's two launch shapes: a graph pooled beside few others (its sets side by side) and beside
many (one workgroup per slice) gives the same bits, for graphs of one slice and of several."""
import numpy as np
import pytest

from gpu_common import custom_workload, run_library

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,group,n", [(2, 8, 1, 32), (3, 17, 0, 1), (4, 48, 1, 300), (3, 100, 1, 200), (2, 256, 1, 140)])
def test_same_bits_beside_few_and_many_graphs(D, H, group, n):
    rng = np.random.default_rng(H + n)
    one = custom_workload(rng, [n], D, H, 2, 1, group)
    few = run_library(one, want_emb=False)
    reps = 260
    many = custom_workload(rng, [1], D, H, 2, 1, group)
    for name in ("n_nodes", "n_edges", "edge_src", "edge_dst", "placement", "cur_node"):
        setattr(many, name, np.tile(getattr(one, name), reps))
    many.node_feats, many.weights, many.B = np.tile(one.node_feats, (reps, 1)), one.weights, reps
    got = run_library(many, want_emb=False)
    for b in (0, reps - 1):
        assert np.array_equal(got["pooled"][b], few["pooled"][0])
        assert np.array_equal(got["logits"][b], few["logits"][0])
