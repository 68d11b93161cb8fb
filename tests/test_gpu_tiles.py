"""The matrix-core sweep of 32 and 64 columns (kernels_tiles.hip) where the library takes it: fp32 weights in batches just
past the sizes up to which narrow networks run in a wave's lanes (256 graphs at H = 32; 128 at H = 64 with one layer), bf16
weights and two layers at H = 64 in any batch.  Every variant of the kernel: first, middle and last of several sweeps,
kept activations, reverse pass; lists around the eight entries that are requested ahead and the sixteen of a pass, up to
130; against the oracles."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_rows_close, custom_workload, run_library
from test_gpu_batch_size import _first
from test_gpu_gradient import _compare
from test_gpu_lanes import _chain, _fan

pytestmark = pytest.mark.gpu

LISTS = [(7, 1), (8, 1), (9, 2), (14, 1), (15, 1), (16, 1), (17, 3), (24, 5), (32, 1), (33, 8), (130, 2)]


def _batch(B, D, H, L, k, wd, seed):
    graphs = ([_fan(*s) for s in LISTS] + [_chain(1 + i % 3) for i in range(B)])[:max(B, len(LISTS))]
    rng = np.random.default_rng(seed)
    w = custom_workload(rng, [g[0] for g in graphs], D, H, L, k, 1, wd, w_scale=0.07)
    w.n_edges = np.array([len(g[1]) for g in graphs], np.int32)
    w.edge_src, w.edge_dst = np.concatenate([g[1] for g in graphs]), np.concatenate([g[2] for g in graphs])
    return w


@pytest.mark.parametrize("H,L,wd,B", [(32, 1, "fp32", 257), (32, 2, "fp32", 257), (64, 1, "fp32", 129), (64, 2, "fp32", 11),
                                      (32, 1, "bf16", 11), (32, 2, "bf16", 11), (64, 1, "bf16", 11), (64, 2, "bf16", 11)])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_every_variant(H, L, wd, B, k):
    w = _batch(B, 3, H, L, k, wd, 7 * H + L + k)
    assert w.B == B
    ref = oracle.forward_workload(w, n_threads=8)
    got = run_library(w, want_class=True)
    assert_rows_close(got["emb"], ref["emb"], H, f"H {H} L {L} {wd} k {k}")
    off, e = np.concatenate([[0], np.cumsum(w.n_nodes)]), np.concatenate([[0], np.cumsum(w.n_edges)])
    for b in range(len(LISTS)):
        cls = oracle.classes(int(w.n_nodes[b]), w.edge_src[e[b]:e[b + 1]], w.edge_dst[e[b]:e[b + 1]], int(w.cur_node[b]))
        assert np.array_equal(got["classes"][off[b]:off[b + 1]], cls), b
    _compare(w, f"H {H} L {L} {wd} k {k}")


@pytest.mark.parametrize("seed", range(6))
def test_random_dags(seed):
    """Random DAGs of many densities, fp32 weights and one layer, in a batch that fills up with single nodes."""
    rng = np.random.default_rng(2000 + seed)
    H = (32, 64)[seed % 2]
    sizes = [int(x) for x in rng.integers(1, 140, size=6)] + [1] * (251 if H == 32 else 123)
    p_edge = float(rng.choice([0.01, 0.03, 0.08, 0.2, 0.5]))
    w = custom_workload(rng, sizes, int(rng.integers(1, 9)), H, 1, 1 + (seed // 2) % 3, seed % 2, "fp32", p_edge=p_edge)
    ref = oracle.forward_workload(w, n_threads=8)
    assert_rows_close(run_library(w)["emb"], ref["emb"], H, f"seed {seed} H {H} p_edge {p_edge}")


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_128_columns_beside_few_and_many_graphs(L, k):
    """Up to 128 graphs 128 columns take this file's kernel with eight waves, in more the one of kernels_mfma.hip: the
    same bits, lists of every length with near and far sources included; and every variant against the oracles."""
    many = _batch(140, 3, 128, L, k, "bf16", 900 + L + 10 * k)
    few, n = _first(many, len(LISTS))
    edge, _ = _first(many, 128)
    ref = oracle.forward_workload(few, n_threads=8)
    got, whole, limit = run_library(few, want_class=True), run_library(many, want_class=True), run_library(edge, want_class=True)
    assert_rows_close(got["emb"], ref["emb"], 128, f"L {L} k {k}")
    for other in (whole, limit):
        assert np.array_equal(got["emb"], other["emb"][:n])
        assert np.array_equal(got["classes"], other["classes"][:n])
        assert np.array_equal(got["logits"], other["logits"][:few.B])
    _compare(few, f"H 128 L {L} k {k}")
