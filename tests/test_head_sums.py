"""The precision of the policy head's sums: blocks of sixteen fp32 terms added up in float64, and the terms past
the last whole block in float64 one by one, whatever the width.  The logits of a pass against the same sums
taken in numpy from the embeddings and pooled sums that the pass returned.  Both round in the same places, so
they differ by the rounding of the logit to fp32 (2^-24 of itself) and by the order of float64 sums (1e-13 of
the terms' size leaves room for a thousand of them)."""
import numpy as np
import pytest

from oracle import gradient as og
from tests.gpu_common import custom_workload, run_library

SHAPES = [(2, 8, 1, 2, "fp32"), (16, 3, 1, 2, "fp32"), (5, 17, 1, 3, "fp32"), (4, 100, 1, 2, "fp32"), (3, 255, 0, 1, "fp32"),
          (9, 24, 1, 4, "fp32"), (8, 48, 1, 2, "fp32"), (2, 256, 1, 2, "fp32"), (2, 201, 1, 2, "fp32"), (4, 64, 1, 2, "fp32"), (8, 128, 1, 2, "bf16")]


def _dense(x, W, b, relu, short_fp32):
    n = x.shape[1]
    acc = np.broadcast_to(b.astype(np.float64), (x.shape[0], W.shape[1])).copy()
    x64, W64 = x.astype(np.float64), W.astype(np.float64)
    whole = n // 16 * 16
    for k0 in range(0, n if short_fp32 else whole, 16):
        s = np.zeros(acc.shape, np.float32)
        for k in range(k0, min(k0 + 16, n)):
            s = (x64[:, k:k + 1] * W64[k] + s.astype(np.float64)).astype(np.float32)      # fused multiply-add
        acc += s
    if not short_fp32:
        acc += x64[:, whole:] @ W64[whole:]
    return np.maximum(acc, 0.0) if relu else acc


def _head(w, emb, pooled, short_fp32=False):
    """Logits [B, D] from embeddings [N, 2H] and pooled sums [B, 3, G, H], and the size of their terms.
    short_fp32 (the planted mistake): the last, short block is summed in fp32 as well."""
    import oracle
    blob = oracle.weights_as_stored(w.weights, w.D, w.H, w.n_layers, w.group_by_device, w.weight_dtype).astype(np.float32)
    slices, _ = og.layer_slices(w.D, w.H, w.n_layers, w.group_by_device)
    shapes = {name: (i, o) for name, i, o in og.layer_shapes(w.D, w.H, w.n_layers, w.group_by_device)}

    def layer(name):
        return blob[slices[name][0]].reshape(shapes[name]), blob[slices[name][1]]
    z = [emb[w.node_off[:-1] + w.cur_node]]
    for i, name in enumerate(("par", "chi", "pll")):
        x = pooled[:, i].reshape(-1, w.H)
        for l in range(w.n_layers):
            x = _dense(x, *layer(f"h_{name}.{l}"), True, short_fp32).astype(np.float32)
        z.append(x.reshape(w.B, -1))
    W1, b1 = layer("pol.0")
    # (a wide head over few graphs sums the three sets' inputs of this layer apart)
    parts = [np.concatenate(z[:2], axis=1), z[2], z[3]] if w.H >= 128 and 3 * w.B <= 256 else [np.concatenate(z, axis=1)]
    rows = np.cumsum([0] + [p.shape[1] for p in parts])
    hid = b1.astype(np.float64) + sum(_dense(p, W1[rows[i]:rows[i + 1]], np.zeros_like(b1), False, short_fp32) for i, p in enumerate(parts))
    hid = np.maximum(hid, 0.0)
    W2, b2 = (a.astype(np.float64) for a in layer("pol.1"))
    return hid @ W2 + b2, np.abs(hid) @ np.abs(W2) + np.abs(b2)


def _outside(got, ref, size):
    """Share of logits outside the bound."""
    return float(np.mean(np.abs(got.astype(np.float64) - ref) > 2.0 ** -24 * 1.01 * np.abs(ref) + 1e-13 * size))


def _workload(D, H, group, L, wd, B=24):
    rng = np.random.default_rng(1000 * H + D)
    # (output sizes of about e^2 summed over the nodes: logits are differences of larger terms)
    return custom_workload(rng, ([24, 9, 31, 17] * (B // 4 + 1))[:B], D, H, L, 1, group, wd, w_scale=0.8 / np.sqrt(H))


@pytest.mark.gpu
@pytest.mark.parametrize("D,H,group,L,wd,B", [s + (24,) for s in SHAPES] +
                         # either side of one graph per compute unit, where the launch shape changes, and of a third
                         [(3, 32, 1, 2, "fp32", 256), (3, 32, 1, 2, "fp32", 257), (9, 64, 1, 2, "fp32", 257), (2, 17, 1, 2, "fp32", 300),
                          (2, 201, 1, 2, "fp32", 85), (2, 201, 1, 2, "fp32", 86), (16, 48, 1, 2, "fp32", 257)])
def test_sums_of_the_head(D, H, group, L, wd, B):
    w = _workload(D, H, group, L, wd, B)
    got = run_library(w)
    ref, size = _head(w, got["emb"], got["pooled"])
    assert np.isfinite(ref).all() and _outside(got["logits"], ref, size) == 0.0, (D, H, np.abs(got["logits"] - ref).max())


@pytest.mark.parametrize("D,H,group,L,wd", SHAPES)
def test_bound_sees_a_short_block_in_fp32(D, H, group, L, wd):
    """The planted mistake moves logits past the bound wherever there is a short block (at H = 17 one
    product per sum is rounded, at H = 8 all of a layer of h)."""
    w = _workload(D, H, group, L, wd)
    rng = np.random.default_rng(3)
    G = D if group else 1
    emb = rng.lognormal(2, 1, (w.n_tot, 2 * H)).astype(np.float32)
    pooled = rng.lognormal(4, 1, (w.B, 3, G, H)).astype(np.float32)
    ref, size = _head(w, emb, pooled)
    wrong, _ = _head(w, emb, pooled, short_fp32=True)
    assert _outside(ref.astype(np.float32), ref, size) == 0.0
    out = _outside(wrong.astype(np.float32), ref, size)
    assert out > 0.2 if H % 16 else out == 0.0, out
