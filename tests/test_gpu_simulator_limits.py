"""The simulator kernel where its layout and its lists change: child lists around the length a node's
record holds (two) and around a wave (64), transfer lists longer than a record, pending events in one
and in two DPP rows, and graphs at the LDS limit with few edges (16-bit states) and with many.
Bit for bit against the oracle, like tests/test_gpu_simulator.py."""
import numpy as np
import pytest

from tests.test_gpu_simulator import _device_both, _oracle_both
from workloads.synthetic import Workload

pytestmark = pytest.mark.gpu


def _workload(graphs, D, rng, ties):
    n_nodes = np.array([n for n, _, _ in graphs], np.int32)
    n_tot = int(n_nodes.sum())
    feats = (np.stack([rng.integers(1, 4, n_tot), rng.integers(0, 3, n_tot), np.zeros(n_tot)], axis=1) if ties else
             np.stack([rng.lognormal(0, 1, n_tot), rng.lognormal(0, 1, n_tot), np.zeros(n_tot)], axis=1))
    return Workload(name="limits", B=len(graphs), D=D, H=8, n_layers=1, k_sweeps=1, group_by_device=1,
                    weight_dtype="fp32", n_nodes=n_nodes, n_edges=np.array([len(s) for _, s, _ in graphs], np.int32),
                    edge_src=np.concatenate([s for _, s, _ in graphs]).astype(np.int32),
                    edge_dst=np.concatenate([d for _, _, d in graphs]).astype(np.int32),
                    node_feats=feats.astype(np.float32), placement=rng.integers(0, D, n_tot).astype(np.int32),
                    cur_node=np.zeros(len(graphs), np.int32), weights=np.zeros(1, np.float32))


def _fan(width):
    """A root with `width` children that all feed one node and, in pairs, a second generation."""
    src = [0] * width + list(range(1, width + 1)) + list(range(1, width + 1))
    dst = list(range(1, width + 1)) + [width + 1] * width + [width + 2 + i // 2 for i in range(width)]
    return width + 2 + (width + 1) // 2, np.array(src), np.array(dst)


def _check(w, per_child):
    rt, ev, peak, _ = _device_both(w, w.placement, 1.0, per_child)
    for b in range(w.B):
        r, e, p = _oracle_both(w, b, w.placement, 1.0, per_child)
        assert (rt[b], ev[b]) == (r, e), (b, rt[b], r, ev[b], e)
        np.testing.assert_allclose(peak[b], p, rtol=1e-6, atol=0, err_msg=f"graph {b}")


@pytest.mark.parametrize("per_child", [0, 1])
@pytest.mark.parametrize("D", [2, 8, 9, 16])
def test_child_and_transfer_lists(D, per_child):
    rng = np.random.default_rng(41 + D)
    w = _workload([_fan(k) for k in (1, 2, 3, 63, 64, 65, 130)], D, rng, ties=D % 2 == 1)
    _check(w, per_child)


@pytest.mark.parametrize("per_child", [0, 1])
@pytest.mark.parametrize("n,e", [(9090, 2), (9000, 130), (8180, 1), (4000, 7000)])
def test_graphs_at_the_size_limit(n, e, per_child):
    assert 18 * n + 13 * e <= 160 * 1024 - 32
    rng = np.random.default_rng(n)
    # (edges between different ids, lower to higher, none twice)
    pairs = set()
    while len(pairs) < e:
        a, b = sorted(int(x) for x in rng.integers(0, n, 2))
        if a != b:
            pairs.add((a, b))
    pairs = np.array(sorted(pairs))
    w = _workload([(n, pairs[:, 0], pairs[:, 1])], 8, rng, ties=False)
    _check(w, per_child)


@pytest.mark.parametrize("per_child", [0, 1])
@pytest.mark.parametrize("D", [1, 2, 16])
def test_nodes_of_thousands_of_children(D, per_child):
    """A node whose children are all on its own device, all on one other, spread, or on one other device except for the last
    few, which are the only ones on theirs; lists of one wave more or less, several of them in a graph."""
    rng = np.random.default_rng(D)

    def hubs(counts):
        src, dst, n = [], [], len(counts)
        for hub, kids in enumerate(counts):
            src += [hub] * kids
            dst += list(range(n, n + kids))
            n += kids
        return n, np.array(src), np.array(dst)

    graphs = [hubs(c) for c in ((5000,), (5000,), (5000,), (4999,), (64, 65, 63, 129, 0, 1, 2, 3, 64, 1500))]
    w = _workload(graphs, D, rng, ties=D == 2)
    off = np.concatenate([[0], np.cumsum(w.n_nodes)])
    w.placement[off[0]:off[1]] = 0
    w.placement[off[1]] = 0
    w.placement[off[1] + 1:off[2]] = D - 1
    w.placement[off[3]:off[4]] = D // 2
    w.placement[off[3]] = 0
    w.placement[off[4] - min(D, 7):off[4]] = np.arange(min(D, 7))
    _check(w, per_child)
