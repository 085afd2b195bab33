"""The matrix-core router (every logit as an fp32 multiply-add chain on the
fp32 MFMAs) against the oracle, bit for bit, at the edges of its tiles: one
token, one expert, ragged last tiles of 32 and 64 tokens and experts, one slab,
row lengths that are not a multiple of 256 bytes, both wave-tile sizes (which
change at 800 000 token-expert pairs), K up to 16, ties, tiny products."""

import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2608_17402_amd import binding
from workloads import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,K,dtype,scale,dup", [
    (1, 64, 1, 1, "bf16", 0.02, 1),
    (1, 64, 16, 16, "f32", 0.02, 1),
    (31, 64, 33, 16, "bf16", 0.05, 1),
    (33, 192, 64, 8, "f32", 0.02, 2),       # 128 and 64 columns
    (65, 448, 65, 3, "bf16", 0.02, 5),
    (4097, 128, 200, 16, "bf16", 0.05, 1),  # 32 x 32 wave tiles, 64 x 64 blocks, ragged both ways
    (25601, 64, 31, 7, "bf16", 0.05, 1),    # 128-token blocks of one expert tile
    (25601, 64, 8, 2, "f32", 0.05, 1),
    (6500, 320, 129, 5, "f32", 0.02, 1),
    (70, 2112, 300, 9, "bf16", 0.005, 1),   # more than 256 experts: one wave per token in the selection
    (40, 256, 24, 4, "f32", 1e-38, 1),      # denormal products and sums
])
def test_exact_router_bitwise(T, d, E, K, dtype, scale, dup):
    rng = np.random.default_rng(T + d + E + K)
    x = rng.standard_normal((T, d)).astype(np.float32)
    wr = (rng.standard_normal(((E + dup - 1) // dup, d)) * scale).astype(np.float32)
    wr = np.repeat(wr, dup, axis=0)[:E].copy()  # identical rows tie
    bias = rng.uniform(-0.02, 0.02, E).astype(np.float32) if dup == 1 else None
    if dtype == "bf16":
        x, wr = f32_to_bf16_bits(x), f32_to_bf16_bits(wr)
        xf, wf = bf16_bits_to_f32(x), bf16_bits_to_f32(wr)
    else:
        xf, wf = x, wr
    ref_idx, ref_gate = oracle.route(xf, wf, bias if bias is not None else np.zeros(E, np.float32), K)
    desc = binding.make_desc(T, d, E, K, 64, dtype=dtype)  # every logit exactly, without the flag too
    ws = binding.alloc_workspace(desc)
    idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
    binding.moe_route(desc, dev(x), dev(wr), dev(bias), idx, gate, ws)
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ref_idx)
    assert np.array_equal(host(gate), ref_gate)
