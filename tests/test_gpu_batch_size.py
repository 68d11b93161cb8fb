"""What include/placeto.h says of a graph's results in batches of different sizes: the same bits, except on the two sides
of the sizes at which another kernel takes over, where they agree to rounding."""
import copy

import numpy as np
import pytest

from gpu_common import run_library
from workloads import make_workload, weight_count

pytestmark = pytest.mark.gpu


def _first(w, B):
    v = copy.copy(w)
    n, e = int(w.n_nodes[:B].sum()), int(w.n_edges[:B].sum())
    for name, m in (("n_nodes", B), ("n_edges", B), ("cur_node", B), ("edge_src", e), ("edge_dst", e), ("node_feats", n), ("placement", n)):
        setattr(v, name, getattr(w, name)[:m])
    v.B = B
    v.__post_init__()
    return v, n


@pytest.mark.parametrize("H,L,wd,B,limit", [(8, 2, "fp32", 300, None), (16, 1, "fp32", 300, None), (32, 2, "bf16", 600, None), (48, 2, "fp32", 300, None),
                                            (64, 2, "fp32", 300, None), (64, 1, "bf16", 300, None), (100, 1, "fp32", 120, None),
                                            (128, 2, "bf16", 300, None), (32, 2, "fp32", 300, 256), (64, 1, "fp32", 300, 128)])
def test_a_graph_beside_few_and_many(H, L, wd, B, limit):
    w = make_workload("layered200", B=B)
    w.H, w.n_layers, w.weight_dtype = H, L, wd
    w.weights = np.random.default_rng(H).normal(0, 0.1, weight_count(w.D, H, L, bool(w.group_by_device))).astype(np.float32)
    whole = run_library(w)
    for few in (1, 40) if limit is None else (1, limit, limit + 1):
        v, n = _first(w, few)
        part = run_library(v)
        pairs = [(whole["emb"][:n], part["emb"]), (whole["pooled"][:few], part["pooled"]), (whole["logits"][:few], part["logits"])]
        for a, b in pairs:
            if limit is None or few > limit:
                assert np.array_equal(a, b), (H, few)
            else:
                assert np.linalg.norm(a.astype(np.float64) - b) <= 2e-6 * np.linalg.norm(a.astype(np.float64)), (H, few)
