"""The sweep kernels of narrow networks (a layer in a wave's lanes, or on matrix cores where it is wider, deeper or in
bf16): every width and depth they take, chunks of one to eight rows, rows with one source more or less than a record or a pass of a list holds, near and far; and the sizes
of a batch at which another kernel takes over.  Embeddings, gradients and node sets against the oracles."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_rows_close, custom_workload, run_library
from test_gpu_gradient import _compare

pytestmark = pytest.mark.gpu


def _fan(k_far, k_near):
    """k_far roots, a chain of nine levels of k_near nodes each, and a node whose parents are all roots and the
    chain's last level; a second such node behind it, so that the reverse direction has long lists too."""
    src, dst = [], []
    level = list(range(k_far))
    n = k_far
    for step in range(9):
        new = list(range(n, n + k_near))
        n += k_near
        for i, v in enumerate(new):
            src.append(level[i % len(level)])
            dst.append(v)
        level = new
    for v in (n, n + 1):
        for u in list(range(k_far)) + level:
            src.append(u)
            dst.append(v)
    src.append(n)
    dst.append(n + 1)
    return n + 2, np.array(src, np.int32), np.array(dst, np.int32)


def _batch(seed, D, H, L, k, wd, shapes):
    rng = np.random.default_rng(seed)
    graphs = [_fan(*s) for s in shapes]
    w = custom_workload(rng, [g[0] for g in graphs], D, H, L, k, 1, wd)
    w.n_edges = np.array([len(g[1]) for g in graphs], np.int32)
    w.edge_src, w.edge_dst = np.concatenate([g[1] for g in graphs]), np.concatenate([g[2] for g in graphs])
    return w


WIDTHS = [(8, 1), (8, 2), (16, 1), (16, 2), (32, 1), (32, 2), (64, 1), (64, 2)]
# sources of the two last nodes: lists of 2 .. 130 entries, around the 8 that are requested ahead and the H that a
# row's lanes hold; chain levels of 1 .. 8 rows and more than one chunk
SHAPES = [(2, 1), (1, 5), (1, 6), (7, 1), (8, 1), (6, 2), (9, 3), (15, 4), (16, 5), (30, 8), (33, 7), (63, 1), (64, 9), (130, 2)]


@pytest.mark.parametrize("H,L", WIDTHS)
@pytest.mark.parametrize("k,wd", [(1, "fp32"), (2, "fp32"), (1, "bf16")])
def test_every_list_length(H, L, k, wd):
    w = _batch(H + L + k, 5, H, L, k, wd, SHAPES)
    ref = oracle.forward_workload(w, n_threads=8)
    got = run_library(w, want_class=True)
    assert_rows_close(got["emb"], ref["emb"], H, f"H {H} L {L} k {k}")
    off = np.concatenate([[0], np.cumsum(w.n_nodes)])
    e = np.concatenate([[0], np.cumsum(w.n_edges)])
    for b in range(w.B):
        cls = oracle.classes(int(w.n_nodes[b]), w.edge_src[e[b]:e[b + 1]], w.edge_dst[e[b]:e[b + 1]], int(w.cur_node[b]))
        assert np.array_equal(got["classes"][off[b]:off[b + 1]], cls), (H, L, b)
    _compare(w, f"H {H} L {L} k {k} {wd}")


@pytest.mark.parametrize("H,L,B", [(32, 2, 256), (32, 2, 257), (32, 1, 257), (64, 1, 128), (64, 1, 129), (8, 2, 300)])
def test_either_side_of_the_batch_limit(H, L, B):
    w = _batch(B, 3, H, L, 1, "fp32", [(1 + i % 9, 1 + i % 3) for i in range(B)])
    ref = oracle.forward_workload(w, n_threads=8)
    assert_rows_close(run_library(w)["emb"], ref["emb"], H, f"H {H} L {L} B {B}")
    _compare(w, f"H {H} L {L} B {B}")


def _ladder(width, distance, levels):
    """`levels` levels of `width` nodes, a chunk each: a node's parents are one of the level before and, as its
    single far source, one that many chunks back that another wave stored (the mirrored row)."""
    src, dst = [], []
    for level in range(1, levels):
        for i in range(width):
            v = level * width + i
            src.append((level - 1) * width + i)
            dst.append(v)
            if level >= distance:
                src.append((level - distance) * width + width - 1 - i)
                dst.append(v)
    return levels * width, np.array(src, np.int32), np.array(dst, np.int32)


@pytest.mark.parametrize("H,L", WIDTHS)
@pytest.mark.parametrize("k", [1, 2])
def test_far_sources_of_other_waves(H, L, k):
    """Far sources at the shortest distance at which the table does not hold them any more (five chunks), one nearer and
    one further, for chunks of as many rows as two, four and eight waves take."""
    graphs = [_ladder(width, distance, 15) for width in (2, 5, 8) for distance in (4, 5, 6)]
    rng = np.random.default_rng(H + L)
    w = custom_workload(rng, [g[0] for g in graphs], 3, H, L, k, 1, "fp32", w_scale=0.05)
    w.n_edges = np.array([len(g[1]) for g in graphs], np.int32)
    w.edge_src, w.edge_dst = np.concatenate([g[1] for g in graphs]), np.concatenate([g[2] for g in graphs])
    ref = oracle.forward_workload(w, n_threads=8)
    assert_rows_close(run_library(w)["emb"], ref["emb"], H, f"H {H} L {L} k {k}")
    _compare(w, f"H {H} L {L} k {k}")


def _chain(levels):
    """One node a level: as many chunks as levels, two nodes back as a second source."""
    pairs = [(v - back, v) for v in range(levels) for back in (1, 2) if v >= back]
    src, dst = zip(*pairs) if pairs else ((), ())
    return levels, np.array(src, np.int32), np.array(dst, np.int32)


@pytest.mark.parametrize("H,L,k,wd", [(64, 2, 1, "fp32"), (64, 1, 1, "bf16"), (32, 2, 2, "bf16"), (64, 1, 3, "bf16"), (32, 2, 1, "fp32")])
def test_every_number_of_chunks(H, L, k, wd):
    """Graphs of 1 to 13 chunks: the loop's turns of four and what is left over, in the matrix-core kernel (that leaves
    in the middle of a turn, or does not where no registers are left for the test) and in the lanes."""
    graphs = [_chain(n) for n in range(1, 14)]
    rng = np.random.default_rng(H + L)
    w = custom_workload(rng, [g[0] for g in graphs], 3, H, L, k, 1, wd)
    w.n_edges = np.array([len(g[1]) for g in graphs], np.int32)
    w.edge_src, w.edge_dst = np.concatenate([g[1] for g in graphs]), np.concatenate([g[2] for g in graphs])
    ref = oracle.forward_workload(w, n_threads=8)
    assert_rows_close(run_library(w)["emb"], ref["emb"], H, f"H {H} L {L} k {k} {wd}")
    _compare(w, f"H {H} L {L} k {k} {wd}")
