"""Selection keys that are NaN or -inf, on every path of the router: a NaN key
(a damaged bias entry, router row or token row) counts as -inf, equal keys go
by expert index, and the chosen experts of a token are always distinct and in
range, so that what follows the routing never indexes past an expert. Indices and gates bit for
bit against the oracle, whose own rule is pinned on the CPU."""

import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2608_17402_amd import binding
from workloads import bf16_bits_to_f32, f32_to_bf16_bits


def _inputs(T, d, E, bad, dtype):
    """Router inputs with `bad` NaN bias entries and -inf ones, one NaN router
    row, and every seventh token NaN."""
    rng = np.random.default_rng(T + 3 * d + E + bad)
    x = rng.standard_normal((T, d)).astype(np.float32)
    wr = (rng.standard_normal((E, d)) * 0.02).astype(np.float32)
    bias = rng.uniform(-0.02, 0.02, E).astype(np.float32)
    order = rng.permutation(E)
    bias[order[:bad]] = np.nan
    bias[order[bad:2 * bad]] = -np.inf
    if E > 4:
        wr[order[2 * bad]] = np.nan
    if T >= 7:
        x[6::7, 3] = np.nan
    if dtype == "bf16":
        x, wr = f32_to_bf16_bits(x), f32_to_bf16_bits(wr)
        x[6::7, 3] = 0x7FC0  # the conversion rounds bit patterns: a quiet NaN, not a carry out of one
        if E > 4:
            wr[order[2 * bad]] = 0xFFC0
        return x, wr, bias, bf16_bits_to_f32(x), bf16_bits_to_f32(wr)
    return x, wr, bias, x, wr


def _select(sig, bias, K):
    """The rule, in numpy: descending keys, NaN as -inf, equal keys by index."""
    out = np.empty((sig.shape[0], K), np.int32)
    for t, s in enumerate(sig):
        key = s + bias
        out[t] = np.argsort(-np.where(np.isnan(key), -np.inf, key), kind="stable")[:K]
    return out


def test_oracle_ranks_nan_keys_last():
    rng = np.random.default_rng(1)
    for E, K in [(1, 1), (5, 5), (40, 6)]:
        sig = rng.uniform(0, 1, (30, E)).astype(np.float32)
        sig[rng.random((30, E)) < 0.3] = np.nan
        bias = np.where(rng.random(E) < 0.3, -np.inf, 0.0).astype(np.float32)
        idx, _ = oracle.topk_from_scores(sig, bias, K)
        assert np.array_equal(idx, _select(sig, bias, K))


CASES = [
    # every logit by the exact chain: 4, 8 and 16 experts per lane, more than 256 experts
    ("exact64", 40, 128, 60, 8, 5, "bf16", 0), ("exact8_all", 40, 64, 8, 8, 2, "bf16", 0),
    ("exact128", 40, 128, 100, 16, 20, "bf16", 0), ("exact256", 40, 192, 250, 3, 30, "f32", 0),
    ("exact300", 40, 128, 300, 8, 30, "f32", 0),
    ("exact300_flag", 40, 128, 300, 16, 100, "bf16", binding.MOE_FLAG_EXACT_ROUTER),
    # bf16 pre-pass and repair: small batches, 64- and 128-token blocks, 16 and 32 slots
    ("repair300", 300, 320, 300, 8, 3, "bf16", 0), ("repair1000", 300, 128, 1000, 12, 40, "bf16", 0),
    ("repair128_large", 16400, 128, 128, 8, 3, "bf16", 0), ("repair200_large", 33000, 64, 200, 12, 40, "bf16", 0),
]


@pytest.mark.gpu
@pytest.mark.parametrize("name,T,d,E,K,bad,dtype,flags", CASES, ids=[c[0] for c in CASES])
def test_nan_keys(name, T, d, E, K, bad, dtype, flags):
    x, wr, bias, xf, wf = _inputs(T, d, E, bad, dtype)
    ref_idx, ref_gate = oracle.route(xf, wf, bias, K)
    desc = binding.make_desc(T, d, E, K, 64, dtype=dtype, flags=flags)
    ws = binding.alloc_workspace(desc)
    idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
    binding.moe_route(desc, dev(x), dev(wr), dev(bias), idx, gate, ws)
    torch.cuda.synchronize()
    got = host(idx)
    assert got.min() >= 0 and got.max() < E
    assert np.all(np.diff(np.sort(got, axis=1), axis=1) > 0), "experts chosen twice"
    assert np.array_equal(got, ref_idx)
    assert np.array_equal(host(gate), ref_gate, equal_nan=True)
