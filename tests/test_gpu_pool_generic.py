"""The generic pooling kernel's two launch shapes: a graph pooled beside few others (its sets side by side) and beside
many (one workgroup per slice) gives the same bits, for graphs of one slice and of several; narrow networks pool small
graphs beside few others in the head's workgroup, in the same order."""
import numpy as np
import pytest

from gpu_common import custom_workload, run_library

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,group,n", [(2, 8, 1, 32), (16, 16, 1, 64), (5, 8, 0, 64), (3, 16, 1, 65), (3, 17, 0, 1), (4, 48, 1, 300), (3, 100, 1, 200), (2, 256, 1, 140)])
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


@pytest.mark.parametrize("D,H,L,group,wd", [(3, 32, 2, 1, "fp32"), (1, 64, 1, 0, "fp32"), (16, 64, 2, 1, "bf16"), (5, 128, 2, 1, "bf16")])
def test_slices_of_matrix_core_pooling(D, H, L, group, wd):
    """Graphs on both sides of the sizes where a graph gets another slice, with sets of every share of it (one end of a
    chain as the current node: one set has all nodes), against the generic kernels on the same batch."""
    rng = np.random.default_rng(D + H)
    sizes = [1, 2, 16, 17, 64, 65, 128, 129, 192, 193, 512, 513, 900, 1025]
    w = custom_workload(rng, sizes, D, H, L, 1, group, wd, p_edge=0.004, w_scale=0.05)
    off = np.concatenate([[0], np.cumsum(sizes)])
    indeg = np.zeros(off[-1], int)
    e_off = np.concatenate([[0], np.cumsum(w.n_edges)])
    for b in range(len(sizes)):
        np.add.at(indeg, off[b] + w.edge_dst[e_off[b]:e_off[b + 1]], 1)
        if b % 3 == 0:
            w.cur_node[b] = int(np.argmin(indeg[off[b]:off[b + 1]]))
    got, ref = run_library(w, want_emb=False), run_library(w, want_emb=False, path=1)
    scale = np.abs(ref["pooled"]).max(axis=tuple(range(1, ref["pooled"].ndim)), keepdims=True)
    # (sums of up to a thousand fp32 terms, in other orders: a few units in 2^-24 per term)
    assert np.all(np.abs(got["pooled"] - ref["pooled"]) <= 1e-5 * scale)
