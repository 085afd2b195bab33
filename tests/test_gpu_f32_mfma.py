"""fp32 layers on the fp32 matrix cores against the oracle: the shortest
contraction (two slabs), slab counts that end on each of the ring's three
slots, experts with no, one and more than one tile of rows, with and without a
shared expert. Tolerance of fp32 sums in another order."""

import numpy as np
import pytest
import torch

import oracle
from gpu_util import DeviceLayer, check_close, host
from workloads import make_inputs
from workloads.configs import LayerConfig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,K,h,hs", [(1, 64, 4, 1, 64, 64), (3, 64, 3, 3, 128, 0), (65, 128, 2, 1, 64, 192),
                                          (130, 192, 5, 4, 320, 128), (257, 320, 40, 2, 448, 64)])
def test_f32_layer(T, d, E, K, h, hs):
    cfg = LayerConfig(name=f"f32_{T}_{d}", T=T, d=d, E=E, K=K, h=h, h_shared=hs, dtype="f32", bias="uniform",
                      seed=T, images=1, tokens_per_image=T)
    inp = make_inputs(cfg)
    lay = DeviceLayer(inp)
    y, idx, gate = lay.forward()
    torch.cuda.synchronize()
    o_idx, o_gate, y_ref = oracle.layer(inp.f32("x"), inp.f32("w_router"), inp.bias, inp.f32("w1"), inp.f32("w2"),
                                        inp.f32("w1s"), inp.f32("w2s"), K, cfg.lam, False)
    assert np.array_equal(host(idx), o_idx) and np.array_equal(host(gate), o_gate)
    check_close(host(y), y_ref, False, "y")
