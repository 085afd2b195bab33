"""Weight gradients from the row-major tensors: expert loads at the edges of
the 64-row slabs and of the two-slab and 128-slab windows, and widths that are
not multiples of the tiles (or of 64: SwiGLU), against the oracle with the
backward's bounds (see test_gpu_backward). A few experts run on 128 x 128 tiles,
the loads with 39 experts and more on 256 x 256 tiles."""

import numpy as np
import pytest

import oracle
from gpu_util import pad_cols
from test_gpu_backward import _bf16, check_grad, run_backward
from workloads import bf16_bits_to_f32

pytestmark = pytest.mark.gpu

# Rows per expert; 8193 rows are cut into two work items.
EDGES = [0, 1, 63, 64, 65, 127, 128, 129, 0, 200, 1]
LOADS = {"edges": EDGES, "split": [8193, 0, 130], "edges132": EDGES * 12, "split39": [8193, 0, 130] + [0, 1, 65] * 12}


@pytest.mark.parametrize("d,h,swiglu,loads", [
    (320, 448, False, "edges"), (64, 64, False, "edges"), (512, 320, False, "split"), (576, 128, False, "edges"),
    (192, 33, True, "edges"), (320, 300, True, "edges"), (256, 65, True, "split"),
    (576, 448, False, "edges132"), (704, 300, True, "edges132"), (576, 448, False, "split39"),
])
def test_weight_gradient_windows(d, h, swiglu, loads):
    counts = np.array(LOADS[loads])
    E, T = len(counts), int(counts.sum())
    rng = np.random.default_rng(d + h)
    idx = rng.permutation(np.repeat(np.arange(E), counts)).astype(np.int32).reshape(T, 1)
    x, g = _bf16(rng, (T, d), 1.0), _bf16(rng, (T, d), 0.5)
    w1 = _bf16(rng, (E, (2 if swiglu else 1) * h, d), 0.1)
    w2 = _bf16(rng, (E, d, h), 0.1)
    w2p = pad_cols(w2) if swiglu else w2
    _, dw1, dw2 = run_backward(T, d, E, 1, h, idx, x, w1, w2p, g, swiglu)
    _, r1, r2 = oracle.grouped_backward(*(bf16_bits_to_f32(a) if a.dtype == np.uint16 else a
                                          for a in (x, idx, w1, w2, g)), True, act="swiglu" if swiglu else "gelu")
    check_grad(dw1, r1, "dw1")
    check_grad(dw2[..., :h], r2, "dw2")
    assert not dw2[..., h:].any()


def test_weight_gradients_keep_to_their_rows():
    # A NaN token of one expert reaches no other expert's gradients: neither
    # through padding positions nor through columns past the width.
    T, d, E, h = 700, 320, 7, 192
    rng = np.random.default_rng(3)
    idx = rng.integers(0, E, (T, 1)).astype(np.int32)
    x, g = _bf16(rng, (T, d), 1.0), _bf16(rng, (T, d), 0.5)
    w1, w2 = _bf16(rng, (E, h, d), 0.1), _bf16(rng, (E, d, h), 0.1)
    _, dw1, dw2 = run_backward(T, d, E, 1, h, idx, x, w1, w2, g)
    x[idx[:, 0] == 3] = 0x7FC0
    g[idx[:, 0] == 3] = 0x7FC0
    _, nw1, nw2 = run_backward(T, d, E, 1, h, idx, x, w1, w2, g)
    keep = np.arange(E) != 3
    assert np.isnan(nw1[3]).all() and np.isnan(nw2[3]).all()
    assert np.array_equal(dw1[keep], nw1[keep]) and np.array_equal(dw2[keep], nw2[keep])
