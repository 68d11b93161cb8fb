"""The weight gradients of a pass as tables of contractions: more layers than a table holds (four layers a
network, 43 contractions), slab sums that need several launches (8 and 35 thousand nodes at H = 128), two sweeps
(whose contractions must run before the earlier sweep overwrites what they read) and shapes that take the
plain kernel for every layer.  Per layer block in the 2-norm, 5e-4 (four times what a single ReLU input within
rounding of zero moves a gradient; a missing slab moves its block by about 1 / sqrt(slabs), 4e-2 or more): against
the float64 autograd oracle, which shares nothing with the tables, and against the generic fp32 kernels, which take
every contraction with another kernel but share the tables and the slab sums; equal calls give equal bits."""
import numpy as np
import pytest

from oracle import gradient as og
from tests.gpu_common import custom_workload, run_gradient

pytestmark = pytest.mark.gpu


def _assert_blocks_close(got, ref, D, H, L):
    gmax = np.abs(ref).max()
    slices, _ = og.layer_slices(D, H, L, 1)
    for name, parts in slices.items():
        for sl in parts:
            err = np.linalg.norm(got[sl] - ref[sl])
            assert err <= 5e-4 * np.linalg.norm(ref[sl]) + 1e-7 * gmax * np.sqrt(ref[sl].size), (name, err, np.linalg.norm(ref[sl]))


@pytest.mark.parametrize("sizes,D,H,L,k,wd", [
    ([32] * 1100, 4, 128, 2, 1, "bf16"), ([70, 1, 33], 3, 32, 4, 1, "fp32"), ([64, 65, 9] * 20, 8, 64, 4, 2, "bf16"),
    ([2, 40, 17], 2, 32, 1, 2, "fp32"), ([31, 12], 5, 24, 4, 1, "fp32"),
])
def test_tables_of_contractions(sizes, D, H, L, k, wd):
    rng = np.random.default_rng(H + L)
    w = custom_workload(rng, sizes, D, H, L, k, 1, wd, p_edge=0.1)
    actions = rng.integers(0, D, w.B).astype(np.int32)
    coeff = rng.normal(0, 1, w.B).astype(np.float32)
    got = run_gradient(w, actions, coeff)["grad"]
    assert np.array_equal(got, run_gradient(w, actions, coeff)["grad"])
    ref = run_gradient(w, actions, coeff, path=1)["grad"].astype(np.float64)
    _assert_blocks_close(got, ref, D, H, L)


# (every fourth graph of the large batch has a weight: one in each slab of 64 rows)
@pytest.mark.parametrize("sizes,D,H,L,k,wd,every", [
    ([16] * 500, 4, 128, 2, 1, "bf16", 4), ([70, 1, 33], 3, 32, 4, 1, "fp32", 1), ([64, 65, 9] * 8, 8, 64, 4, 2, "bf16", 1),
    ([2, 40, 17], 2, 32, 1, 2, "fp32", 1), ([31, 12], 5, 24, 4, 1, "fp32", 1),
])
def test_tables_against_the_oracle(sizes, D, H, L, k, wd, every):
    rng = np.random.default_rng(H + L)
    w = custom_workload(rng, sizes, D, H, L, k, 1, wd, p_edge=0.1)
    actions = rng.integers(0, D, w.B).astype(np.int32)
    coeff = np.where(np.arange(w.B) % every == 0, rng.normal(0, 1, w.B), 0.0).astype(np.float32)
    ref, _ = og.gradient_workload(w, actions, coeff.astype(np.float64), only=[int(b) for b in range(0, w.B, every)])
    _assert_blocks_close(run_gradient(w, actions, coeff)["grad"], ref, D, H, L)


@pytest.mark.parametrize("graphs,n,D,H,L,wd", [
    (1536, 3, 3, 32, 2, "fp32"), (1537, 3, 16, 32, 1, "fp32"), (2048, 2, 1, 64, 2, "bf16"), (2049, 2, 4, 128, 2, "bf16"),
    (1601, 70, 2, 32, 2, "fp32"), (4100, 1, 4, 32, 2, "fp32")])
def test_row_lists_of_many_graphs(graphs, n, D, H, L, wd):
    """The node sets' row lists where a graph's part of them is found in one launch and in two, at the sizes where the
    second one gets another workgroup: against the generic kernels, which have none."""
    rng = np.random.default_rng(graphs + H)
    w = custom_workload(rng, [int(x) for x in rng.integers(1, 2 * n, graphs)], D, H, L, 1, 1, wd, p_edge=0.1)
    actions, coeff = rng.integers(0, D, w.B).astype(np.int32), rng.normal(0, 1, w.B).astype(np.float32)
    got, ref = run_gradient(w, actions, coeff)["grad"], run_gradient(w, actions, coeff, path=1)["grad"].astype(np.float64)
    _assert_blocks_close(got, ref, D, H, L)


@pytest.mark.parametrize("D,H,graphs,n", [(3, 32, 9, 10417), (8, 48, 3, 21001), (16, 64, 2, 24001), (5, 256, 2, 6001),
                                              (8, 48, 5, 21001), (16, 64, 8, 24001), (5, 256, 3, 6001)])
def test_projection_gradient_of_a_large_batch(D, H, graphs, n):
    """The projection's gradient formed in one pass over d e (batches of two to twelve million elements and more) and not, against the sum of
    its graphs' gradients, each a batch of its own that takes the other kernel; device ids out of range are in no row."""
    rng = np.random.default_rng(D * H)
    w = custom_workload(rng, [1], D, H, 1, 1, 1)
    dst = np.arange(1, n, 2)                       # every second node has a parent, the first ones in a chain
    src = np.where(dst > 9, dst - 9, 0)
    N = graphs * n
    feats = np.stack([rng.lognormal(0, 1, N), rng.lognormal(1, 1, N), rng.random(N) < 0.5], axis=1).astype(np.float32)
    placement = rng.integers(-1, D + 1, N).astype(np.int32)
    cur = rng.integers(0, n, graphs).astype(np.int32)
    act, co = rng.integers(0, D, graphs).astype(np.int32), rng.normal(0, 1, graphs).astype(np.float32)

    def gradient(lo, hi):
        k = hi - lo
        w.B, w.n_nodes, w.n_edges = k, np.full(k, n, np.int32), np.full(k, len(dst), np.int32)
        w.edge_src, w.edge_dst = np.tile(src, k).astype(np.int32), np.tile(dst, k).astype(np.int32)
        w.node_feats, w.placement, w.cur_node = feats[lo * n:hi * n], placement[lo * n:hi * n], cur[lo:hi]
        return run_gradient(w, act[lo:hi], co[lo:hi])["grad"][:(D + 5) * H].reshape(D + 5, H).astype(np.float64)

    got, ref = gradient(0, graphs), sum(gradient(b, b + 1) for b in range(graphs))
    # (a row is an fp32 sum of up to N terms in two orders; its terms cancel, so the bound is against the largest row)
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref).max())
    assert np.abs(ref).max(axis=1).min() > 0
