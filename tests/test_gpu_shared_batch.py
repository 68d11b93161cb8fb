"""One graph batch used with networks of different numbers of devices in turn: without grouping by device
they share the batch's buffers.  Logits, probabilities, pooled sums and gradients equal, bit for bit, those
of a batch of its own."""
import copy

import numpy as np
import pytest

from tests.gpu_common import custom_workload, run_gradient, run_library
from workloads import weight_count

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,wd,graphs", [(8, "fp32", 70), (32, "fp32", 64), (64, "fp32", 100), (128, "bf16", 64), (128, "bf16", 100)])
def test_networks_of_different_device_counts_on_one_batch(H, wd, graphs):
    import paper_1906_08879_amd as pl
    rng = np.random.default_rng(H + graphs)
    base = custom_workload(rng, [1 + i % 5 for i in range(graphs)], 16, H, 2, 1, 0, wd)
    nets = {}
    for D in (2, 8, 16):
        w = copy.copy(base)
        w.D, w.placement = D, base.placement % D
        w.weights = rng.normal(0, 0.1, weight_count(D, H, 2, False)).astype(np.float32)
        nets[D] = w, rng.integers(0, D, w.B).astype(np.int32), rng.normal(0, 1, w.B).astype(np.float32)
    alone = {D: (run_library(w), run_gradient(w, act, co)) for D, (w, act, co) in nets.items()}
    g = pl.GraphBatch(base.n_nodes, base.n_edges, base.edge_src, base.edge_dst)
    weights = {D: pl.Weights(w.weights, D, H, 2, 1, 0, wd) for D, (w, _, _) in nets.items()}
    for D in (2, 8, 16, 2, 16, 8):
        w, act, co = nets[D]
        got = run_library(w, handles=(g, weights[D])), run_gradient(w, act, co, handles=(g, weights[D]))
        for a, b in zip(got, alone[D]):
            for key, ref in b.items():
                if ref is not None:
                    np.testing.assert_array_equal(a[key], ref, err_msg=f"D {D}: {key}")
    g.close()
    for wt in weights.values():
        wt.close()
