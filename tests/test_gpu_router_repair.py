"""The bf16 pre-pass and exact repair of its candidates (more than 256 experts,
or more than 64 from 16384 tokens on) against the oracle and the all-exact
router, bit for bit: groups of identical router rows that tie exactly, up to
every expert a candidate of every token (more than the repair's slots, so every
token goes through the overflow queue), split and unsplit logits, 16 and 32
candidate slots, one-wave blocks and blocks of 64, 128 and 256 tokens, weights
in LDS for up to 256 and for up to 1024 experts, and model widths on either
side of the lines past which every logit is computed exactly."""

import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2608_17402_amd import binding
from workloads import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

CASES = [  # T, d, E, K, identical rows per group
    (300, 256, 300, 8, 1), (300, 256, 300, 8, 16), (300, 256, 300, 8, 300), (300, 1536, 1000, 12, 1),
    (300, 256, 1000, 12, 16), (301, 256, 1000, 12, 1000), (77, 2048, 512, 4, 128),
    (9001, 128, 300, 8, 1), (9001, 128, 300, 12, 64), (8200, 64, 700, 16, 700),
    (16461, 128, 300, 8, 16), (16461, 64, 1000, 12, 1), (16400, 64, 1000, 8, 1000),
    (16400, 256, 128, 8, 128), (16400, 256, 128, 12, 16), (16384, 320, 65, 8, 1), (16400, 192, 256, 16, 256),
    (33001, 128, 200, 12, 1), (33000, 64, 100, 9, 100), (65600, 128, 128, 8, 1), (65600, 64, 200, 8, 200),
    (16400, 2240, 200, 8, 1), (16390, 2624, 70, 4, 70), (16390, 2688, 70, 4, 1), (16400, 2368, 300, 8, 1),
    (16390, 2176, 520, 4, 1), (2000, 2048, 300, 8, 30), (2000, 2112, 300, 8, 30),
]


@pytest.mark.parametrize("T,d,E,K,dup", CASES)
def test_repair_bitwise(T, d, E, K, dup):
    rng = np.random.default_rng(T + d + E + K + dup)
    x = f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    base = f32_to_bf16_bits((rng.standard_normal(((E + dup - 1) // dup, d)) * 0.02).astype(np.float32))
    wr = np.repeat(base, dup, axis=0)[:E].copy()
    bias = rng.uniform(-0.02, 0.02, E).astype(np.float32) if dup == 1 else np.zeros(E, np.float32)
    ref_idx, ref_gate = oracle.route(bf16_bits_to_f32(x), bf16_bits_to_f32(wr), bias, K)
    if dup == E:
        assert np.all(ref_idx == np.arange(K)[None, :])
    xd, wd, bd = dev(x), dev(wr), dev(bias)
    for flags in (0, binding.MOE_FLAG_EXACT_ROUTER):
        desc = binding.make_desc(T, d, E, K, 64, flags=flags)
        ws = binding.alloc_workspace(desc)
        idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
        gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
        binding.moe_route(desc, xd, wd, bd, idx, gate, ws)
        torch.cuda.synchronize()
        assert np.array_equal(host(idx), ref_idx), flags
        assert np.array_equal(host(gate), ref_gate), flags
