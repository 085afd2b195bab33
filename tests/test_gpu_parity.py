"""Parity of the HIP path (through the C ABI) with the CPU oracle.

Routing (indices, gates) and permutation are compared bit for bit; expert
outputs and the layer output within max-abs 2e-2 / rel-L2 5e-3 (bf16) or
1e-5 / 1e-5 (fp32). Reduced-token variants of every layer shape run the
oracle over every token (several tiles per expert plus ragged tails); so do
the full-size shapes, in the launch configuration the benchmark times.
"""

import numpy as np
import pytest
import torch

import oracle
from gpu_util import DeviceLayer, check_close, dev, desc_for, host
from paper_2608_17402_amd import binding
from workloads import get_config, make_inputs

pytestmark = pytest.mark.gpu

# (config, tokens) small enough for the oracle over every token.
SMALL = [("c1", None), ("c2", 1000), ("c3", 700), ("c4", 600), ("c5", None)]


def small_id(c):
    return f"{c[0]}-T{c[1] or 'full'}"


def _layer(name, T):
    cfg = get_config(name)
    if T is not None:
        cfg = cfg.with_tokens(T)
    return cfg, make_inputs(cfg)


@pytest.fixture(scope="module", params=SMALL, ids=small_id)
def small(request):
    name, T = request.param
    cfg, inp = _layer(name, T)
    lay = DeviceLayer(inp)
    bf16 = cfg.dtype == "bf16"
    ref_idx, ref_gate = oracle.route(inp.f32("x"), inp.f32("w_router"), inp.bias, cfg.K)
    return cfg, inp, lay, bf16, ref_idx, ref_gate


def test_route_bit_exact(small):
    cfg, inp, lay, _, ref_idx, ref_gate = small
    idx, gate = lay.route()
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ref_idx)
    assert np.array_equal(host(gate), ref_gate)
    g = host(gate).astype(np.float64)
    assert np.max(np.abs(g.sum(1) - 1.0)) <= cfg.K * 2.0 ** -23


def test_route_exact_flag_agrees(small):
    # The all-exact flag is accepted and gives the same routing, bit for bit
    # (the layers here compute every logit exactly without it too; the pre-pass
    # against the exact router: test_gpu_router_repair).
    cfg, inp, lay, _, ref_idx, ref_gate = small
    d2 = desc_for(cfg, flags=binding.MOE_FLAG_EXACT_ROUTER)
    idx = torch.empty(cfg.T, cfg.K, dtype=torch.int32, device="cuda")
    gate = torch.empty(cfg.T, cfg.K, dtype=torch.float32, device="cuda")
    binding.moe_route(d2, lay.x, lay.w_router, lay.bias, idx, gate, lay.ws)
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ref_idx) and np.array_equal(host(gate), ref_gate)


@pytest.mark.parametrize("T,d,E,K", [(1, 64, 8, 2), (130, 2048, 256, 8), (77, 4096, 200, 6), (300, 4096, 64, 8),
                                     (513, 1344, 128, 1), (9001, 256, 128, 8), (16383, 192, 256, 4)])
def test_route_small_batch_widths(T, d, E, K):
    # Small batches with at most 256 experts, every logit by the matrix-core
    # chain: narrow and wide rows, 16 x 16 and 32 x 32 wave tiles, up to 16383
    # tokens, the largest batch on this path. Bit-exact against the oracle.
    from workloads import bf16_bits_to_f32, f32_to_bf16_bits

    rng = np.random.default_rng(T * 7 + d + E + K)
    x = f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    wr = f32_to_bf16_bits((rng.standard_normal((E, d)) * 0.02).astype(np.float32))
    bias = rng.uniform(-0.02, 0.02, E).astype(np.float32)
    ref_idx, ref_gate = oracle.route(bf16_bits_to_f32(x), bf16_bits_to_f32(wr), bias, K)
    desc = binding.make_desc(T, d, E, K, 64)
    ws = binding.alloc_workspace(desc)
    idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
    binding.moe_route(desc, dev(x), dev(wr), dev(bias), idx, gate, ws)
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ref_idx)
    assert np.array_equal(host(gate), ref_gate)


def _route_case(rng):
    T = int(rng.choice([1, 2, 3, 5, 17, 64, 100, 257, 513, 1025, 2047, 3000, 8200, 12000]))
    d = int(rng.choice([64, 128, 192, 320, 512, 768, 1024, 1344, 1536, 2048]))
    E = int(rng.integers(1, 257))
    K = int(rng.integers(1, min(E, 8) + 1))
    T = max(1, min(T, int(1.5e8 / (d * E))))  # the oracle's work per case
    dup = int(rng.choice([1, 1, 1, 2, 4, 16])) if E >= 16 else 1  # groups of identical rows tie exactly
    return T, d, E, K, dup


@pytest.mark.parametrize("seed", range(40))
def test_route_random_small_batches(seed):
    # Seeded random shapes of the small-batch router (every logit exactly):
    # widths 64 to 2048, E 1 to 256, K up to 8, some experts in groups of
    # identical rows, with and without a bias. Bit-exact against the oracle.
    from workloads import bf16_bits_to_f32, f32_to_bf16_bits

    rng = np.random.default_rng(5000 + seed)
    T, d, E, K, dup = _route_case(rng)
    x = f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    scale = float(rng.choice([0.01, 0.05]))
    base = f32_to_bf16_bits((rng.standard_normal(((E + dup - 1) // dup, d)) * scale).astype(np.float32))
    wr = np.repeat(base, dup, axis=0)[:E].copy()
    bias = rng.uniform(-0.03, 0.03, E).astype(np.float32) if rng.random() < 0.7 else None
    ref_idx, ref_gate = oracle.route(bf16_bits_to_f32(x), bf16_bits_to_f32(wr),
                                     bias if bias is not None else np.zeros(E, np.float32), K)
    desc = binding.make_desc(T, d, E, K, 64)
    ws = binding.alloc_workspace(desc)
    idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
    binding.moe_route(desc, dev(x), dev(wr), dev(bias) if bias is not None else None, idx, gate, ws)
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ref_idx), (T, d, E, K, dup)
    assert np.array_equal(host(gate), ref_gate), (T, d, E, K, dup)


@pytest.mark.parametrize("dup", [1, 16, 128])
def test_route_ties(dup):
    # Groups of `dup` identical router rows tie exactly for every token, up to
    # all 128 experts (the repair's overflow by ties: test_gpu_router_repair).
    T, d, E, K = 300, 256, 128, 8
    rng = np.random.default_rng(dup)
    from workloads import bf16_bits_to_f32, f32_to_bf16_bits

    x = f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    base = f32_to_bf16_bits((rng.standard_normal((E // dup, d)) * 0.05).astype(np.float32))
    wr = np.repeat(base, dup, axis=0)
    bias = np.zeros(E, np.float32)
    desc = binding.make_desc(T, d, E, K, 64)
    ws = binding.alloc_workspace(desc)
    idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
    binding.moe_route(desc, dev(x), dev(wr), dev(bias), idx, gate, ws)
    torch.cuda.synchronize()
    ref_idx, ref_gate = oracle.route(bf16_bits_to_f32(x), bf16_bits_to_f32(wr), bias, K)
    assert np.array_equal(host(idx), ref_idx) and np.array_equal(host(gate), ref_gate)
    if dup == 128:
        assert np.all(ref_idx == np.arange(K)[None, :])


@pytest.mark.parametrize("E,K", [(1, 1), (5, 3), (31, 7), (63, 8), (65, 8), (100, 16), (128, 8), (200, 4),
                                 (300, 8), (1000, 12)])
def test_route_any_expert_count(E, K):
    # The logits are padded to a multiple of 64 columns; routing must still
    # equal the oracle's, bit for bit, and (more than 256 experts: the bf16
    # pre-pass and its repair) the all-exact path's.
    from workloads import bf16_bits_to_f32, f32_to_bf16_bits

    T, d = 1500, 320
    rng = np.random.default_rng(E * 100 + K)
    x = f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    wr = f32_to_bf16_bits((rng.standard_normal((E, d)) * 0.05).astype(np.float32))
    bias = rng.uniform(-0.05, 0.05, E).astype(np.float32)
    ref_idx, ref_gate = oracle.route(bf16_bits_to_f32(x), bf16_bits_to_f32(wr), bias, K)
    for flags in (0, binding.MOE_FLAG_EXACT_ROUTER) if E > 256 else (0,):
        desc = binding.make_desc(T, d, E, K, 64, flags=flags)
        ws = binding.alloc_workspace(desc)
        idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
        gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
        binding.moe_route(desc, dev(x), dev(wr), dev(bias), idx, gate, ws)
        torch.cuda.synchronize()
        assert np.array_equal(host(idx), ref_idx), flags
        assert np.array_equal(host(gate), ref_gate), flags


def test_permute_exact(small):
    cfg, inp, lay, _, ref_idx, _ = small
    counts, offsets, slots = lay.permute(dev(ref_idx))
    torch.cuda.synchronize()
    rc, ro, rs = oracle.permute(ref_idx, cfg.E)
    assert np.array_equal(host(counts), rc)
    assert np.array_equal(host(offsets), ro)
    assert np.array_equal(host(slots), rs)


def test_grouped_mlp(small):
    cfg, inp, lay, bf16, ref_idx, _ = small
    _, ro, rs = oracle.permute(ref_idx, cfg.E)
    eo = host(lay.grouped_mlp(dev(rs), dev(ro)))
    x = inp.f32("x")
    w1, w2 = inp.f32("w1"), inp.f32("w2")
    ref = np.zeros((cfg.T * cfg.K, cfg.d))
    for e in range(cfg.E):
        seg = rs[ro[e]:ro[e + 1]]
        if seg.size:
            ref[seg] = oracle.expert_rows(x[seg // cfg.K], w1[e], w2[e], bf16)
    check_close(eo, ref, bf16, "expert_out")


def test_combine(small):
    cfg, inp, lay, bf16, ref_idx, ref_gate = small
    rng = np.random.default_rng(7)
    eo = (rng.standard_normal((cfg.T * cfg.K, cfg.d)) * 0.3).astype(np.float32)
    sh = (rng.standard_normal((cfg.T, cfg.d)) * 0.3).astype(np.float32)
    if bf16:
        from workloads import bf16_bits_to_f32, f32_to_bf16_bits

        eo_b, sh_b = f32_to_bf16_bits(eo), f32_to_bf16_bits(sh)
        eo, sh = bf16_bits_to_f32(eo_b), bf16_bits_to_f32(sh_b)
        eo_d, sh_d = dev(eo_b), dev(sh_b)
    else:
        eo_d, sh_d = dev(eo), dev(sh)
    y = lay.empty(cfg.T, cfg.d)
    binding.moe_combine(lay.desc, eo_d, dev(ref_gate), sh_d, y)
    check_close(host(y), oracle.combine(eo, ref_gate, sh, cfg.lam), bf16, "combine")
    y2 = lay.empty(cfg.T, cfg.d)
    binding.moe_combine(lay.desc, eo_d, dev(ref_gate), None, y2)
    check_close(host(y2), oracle.combine(eo, ref_gate, None, cfg.lam), bf16, "combine without shared")


def test_layer_forward(small):
    cfg, inp, lay, bf16, ref_idx, ref_gate = small
    y, idx, gate = lay.forward()
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ref_idx) and np.array_equal(host(gate), ref_gate)
    o_idx, o_gate, y_ref = oracle.layer(inp.f32("x"), inp.f32("w_router"), inp.bias, inp.f32("w1"),
                                        inp.f32("w2"), inp.f32("w1s"), inp.f32("w2s"), cfg.K, cfg.lam, bf16)
    assert np.array_equal(o_idx, ref_idx)
    check_close(host(y), y_ref, bf16, "layer y")


def test_layer_timing_events_change_nothing(small):
    """The timing hook: three events, or the outer two with the middle slot
    NULL, are recorded in order around the routed GEMMs and leave y as it is."""
    cfg, inp, lay, bf16, _, _ = small
    y0, _, _ = lay.forward()
    ev = binding.HipEvents(6)
    h = ev.handles
    for events in (h[0:3], [h[3], None, h[5]]):
        y = lay.empty(lay.desc.T, lay.desc.d)
        binding.moe_layer_forward(lay.desc, lay.x, lay.w_router, lay.bias, lay.w1, lay.w2, lay.w1s, lay.w2s, y,
                                  workspace=lay.ws, events=events)
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16) if bf16 else y, y0.view(torch.int16) if bf16 else y0)
    assert ev.elapsed_ms(0, 1) >= 0 and ev.elapsed_ms(1, 2) >= 0 and ev.elapsed_ms(3, 5) > 0
    ev.close()


def test_layer_deterministic(small):
    _, _, lay, _, _, _ = small
    y1, i1, g1 = lay.forward()
    y2, i2, g2 = lay.forward(with_routing=False)
    torch.cuda.synchronize()
    assert torch.equal(y1.view(torch.int16) if y1.dtype == torch.bfloat16 else y1,
                       y2.view(torch.int16) if y2.dtype == torch.bfloat16 else y2)


def test_layer_token_permutation_equivariance(small):
    cfg, inp, lay, _, _, _ = small
    y, _, _ = lay.forward()
    perm = np.random.default_rng(3).permutation(cfg.T)
    inp_p = make_inputs(cfg)
    inp_p.x = inp.x[perm]
    lay_p = DeviceLayer(inp_p)
    y_p, _, _ = lay_p.forward()
    torch.cuda.synchronize()
    a = host(y)[perm]
    b = host(y_p)
    assert np.array_equal(a, b)


# ------------------------------------------------------------------ edge cases


def _synthetic(T, d, E, K, h, hs, dtype, seed, bias=None, weight_std=0.02):
    from workloads.configs import LayerConfig

    cfg = LayerConfig(name=f"edge{seed}", T=T, d=d, E=E, K=K, h=h, h_shared=hs, dtype=dtype, bias="uniform",
                      seed=seed, weight_std=weight_std)
    inp = make_inputs(cfg)
    if bias is not None:
        inp.bias = np.asarray(bias, np.float32)
    return cfg, inp


EDGE = {
    "one_token": dict(T=1, d=64, E=8, K=2, h=64, hs=64, dtype="bf16"),
    "k_equals_e": dict(T=77, d=128, E=8, K=8, h=64, hs=0, dtype="bf16"),
    "single_expert": dict(T=130, d=64, E=1, K=1, h=128, hs=64, dtype="bf16"),
    "k16_e1024": dict(T=50, d=64, E=1024, K=16, h=64, hs=0, dtype="bf16"),
    "f32_ragged": dict(T=131, d=192, E=5, K=3, h=320, hs=128, dtype="f32"),
    "wide_h_odd_tiles": dict(T=257, d=320, E=6, K=2, h=448, hs=192, dtype="bf16"),
    # the descriptor's largest widths: d = h = h_s = 8192 (128 K slabs). Weights of std
    # 0.02 sqrt(1536 / 8192) keep pre-activations and outputs at the ViT-G
    # layer's magnitudes, where the bf16 bounds are stated (with std 0.02 the
    # outputs reach 8, whose bf16 spacing alone exceeds 2e-2).
    "max_widths": dict(T=40, d=8192, E=3, K=2, h=8192, hs=8192, dtype="bf16", wstd=0.02 * (1536 / 8192) ** 0.5),
    "max_width_f32": dict(T=33, d=8192, E=4, K=2, h=64, hs=128, dtype="f32", wstd=0.02 * (1536 / 8192) ** 0.5),
}


@pytest.mark.parametrize("name", sorted(EDGE))
def test_edge_layer(name):
    p = EDGE[name]
    cfg, inp = _synthetic(p["T"], p["d"], p["E"], p["K"], p["h"], p["hs"], p["dtype"], seed=len(name),
                          weight_std=p.get("wstd", 0.02))
    lay = DeviceLayer(inp)
    y, idx, gate = lay.forward()
    bf16 = cfg.dtype == "bf16"
    o_idx, o_gate, y_ref = oracle.layer(inp.f32("x"), inp.f32("w_router"), inp.bias, inp.f32("w1"),
                                        inp.f32("w2"), inp.f32("w1s"), inp.f32("w2s"), cfg.K, cfg.lam, bf16)
    assert np.array_equal(host(idx), o_idx) and np.array_equal(host(gate), o_gate)
    check_close(host(y), y_ref, bf16, name)


def test_skew_all_tokens_to_few_experts():
    # Bias +2 forces every token onto experts {1, 5}; every other expert is empty.
    E = 16
    bias = np.zeros(E, np.float32)
    bias[[1, 5]] = 2.0
    cfg, inp = _synthetic(300, 128, E, 2, 128, 0, "bf16", seed=11, bias=bias)
    lay = DeviceLayer(inp)
    y, idx, gate = lay.forward()
    counts, offsets, _ = lay.permute(idx)
    torch.cuda.synchronize()
    assert sorted(set(host(idx).reshape(-1).tolist())) == [1, 5]
    c = host(counts)
    assert c[1] == c[5] == 300 and c.sum() == 600
    o_idx, _, y_ref = oracle.layer(inp.f32("x"), inp.f32("w_router"), inp.bias, inp.f32("w1"), inp.f32("w2"),
                                   None, None, cfg.K, cfg.lam, True)
    assert np.array_equal(host(idx), o_idx)
    check_close(host(y), y_ref, True, "forced skew")


def test_shared_expert_through_grouped_mlp():
    # The shared expert as a grouped MLP with one group of every token.
    cfg, inp = _synthetic(200, 128, 4, 2, 128, 192, "bf16", seed=12)
    d1 = desc_for(cfg, E=1, K=1, h=cfg.h_shared, h_shared=0)
    ws = binding.alloc_workspace(d1)
    slots = torch.arange(cfg.T, dtype=torch.int32, device="cuda")
    offs = torch.tensor([0, cfg.T], dtype=torch.int32, device="cuda")
    out = torch.empty(cfg.T, cfg.d, dtype=torch.bfloat16, device="cuda")
    binding.moe_grouped_mlp(d1, dev(inp.x), slots, offs, dev(inp.w1s)[None], dev(inp.w2s)[None], out, ws)
    ref = oracle.expert_rows(inp.f32("x"), inp.f32("w1s"), inp.f32("w2s"), True)
    check_close(host(out), ref, True, "shared via grouped")


def test_permute_with_empty_and_full_experts():
    T, E, K = 5000, 64, 4
    rng = np.random.default_rng(5)
    # experts 0..3 take most slots, 40..63 none; distinct experts per token
    idx = np.stack([rng.choice(40, K, replace=False, p=np.r_[np.full(4, 0.2), np.full(36, 0.2 / 36)])
                    for _ in range(T)]).astype(np.int32)
    d = binding.make_desc(T, 64, E, K, 64)
    ws = binding.alloc_workspace(d)
    counts = torch.empty(E, dtype=torch.int32, device="cuda")
    offsets = torch.empty(E + 1, dtype=torch.int32, device="cuda")
    slots = torch.empty(T * K, dtype=torch.int32, device="cuda")
    binding.moe_permute(d, dev(idx), counts, offsets, slots, ws)
    rc, ro, rs = oracle.permute(idx, E)
    assert np.array_equal(host(counts), rc) and np.array_equal(host(offsets), ro)
    assert np.array_equal(host(slots), rs)


def test_errors_raise_and_enqueue_nothing():
    cfg, inp = _synthetic(10, 64, 4, 2, 64, 0, "bf16", seed=13)
    lay = DeviceLayer(inp)
    y = lay.empty(cfg.T, cfg.d)
    small_ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(binding.MoeError) as e:
        binding.moe_layer_forward(lay.desc, lay.x, lay.w_router, lay.bias, lay.w1, lay.w2, None, None, y,
                                  workspace=small_ws)
    assert e.value.status == 3


# ------------------------------------------------------------- full-size runs

FULL = ["c2", "c3", "c4", "c5"]


def _oracle_layer(inp, cfg, tokens=None):
    return oracle.layer(inp.f32("x"), inp.f32("w_router"), inp.bias, inp.f32("w1"), inp.f32("w2"),
                        inp.f32("w1s"), inp.f32("w2s"), cfg.K, cfg.lam, cfg.dtype == "bf16", tokens=tokens)


@pytest.mark.slow
@pytest.mark.parametrize("name", FULL)
def test_full_size_layer_every_token(name):
    """The benchmarked layers at full size, in the launch configuration the
    benchmark times (persistent 256-row tiles with the fused combine at ViT-L
    and ViT-G): routing, gates and the permutation bit for bit, and y of every
    token within the bf16 tolerances."""
    cfg = get_config(name)
    inp = make_inputs(cfg)
    lay = DeviceLayer(inp)
    y, idx, gate = lay.forward()
    torch.cuda.synchronize()
    print(f"[{name}] T={cfg.T}: GPU layer done, oracle over every token", flush=True)
    ref_idx, ref_gate, y_ref = _oracle_layer(inp, cfg)
    gi, gg = host(idx), host(gate)
    n_bad = int((gi != ref_idx).any(1).sum())
    assert n_bad == 0, f"{n_bad} tokens routed differently"
    assert np.array_equal(gg, ref_gate)
    counts, offsets, slots = lay.permute(idx)
    rc, ro, rs = oracle.permute(ref_idx, cfg.E)
    assert np.array_equal(host(counts), rc) and np.array_equal(host(offsets), ro)
    assert np.array_equal(host(slots), rs)
    if name == "c4":  # the skewed load reaches the tiny-group paths
        assert int((rc < 16).sum()) == 8 and int(rc.max()) == cfg.T
    yh = host(y)
    check_close(yh, y_ref, True, f"{name} y (every token)")
    # The rarest experts' tokens, on their own (tolerances over a few rows).
    rare = [e for e in np.argsort(rc)[:8] if rc[e] > 0]
    tok = np.unique(np.concatenate([rs[ro[e]:ro[e + 1]] // cfg.K for e in rare]))
    check_close(yh[tok], y_ref[tok], True, f"{name} y of the rarest experts' tokens")


@pytest.mark.slow
def test_shared_fc2_with_fused_combine_ragged_tail():
    """ViT-G shape at a token count where the shared expert runs on 256-row
    tiles, so its fc2 also performs the gate-weighted combine, with a partial
    last tile: every token matches the oracle (and the tail tile on its own),
    and a repeat is bit-identical."""
    cfg = get_config("c4").with_tokens(89 * 256 - 179)
    inp = make_inputs(cfg)
    lay = DeviceLayer(inp)
    y, idx, gate = lay.forward()
    y2, _, _ = lay.forward()
    torch.cuda.synchronize()
    assert np.array_equal(host(y).view(np.uint32), host(y2).view(np.uint32))
    o_idx, o_gate, y_ref = _oracle_layer(inp, cfg)
    assert np.array_equal(host(idx), o_idx) and np.array_equal(host(gate), o_gate)
    yh = host(y)
    check_close(yh, y_ref, True, "fused-combine y (every token)")
    tail = np.arange(88 * 256, cfg.T)
    check_close(yh[tail], y_ref[tail], True, "fused-combine y (tail tile)")


@pytest.mark.slow
@pytest.mark.parametrize("K", [1, 2, 3, 5, 7, 8])
def test_fused_combine_any_k(K):
    """The shared expert's fc2 performs the combine for every K <= 8 once it
    runs on 256-row tiles: 512 + 1 tiles with a partial last tile (77 rows).
    Every token matches the oracle (and the tail on its own); a repeat is
    bit-identical."""
    from workloads.configs import LayerConfig

    cfg = LayerConfig(name=f"fused_k{K}", T=512 * 256 + 77, d=256, E=16, K=K, h=128, h_shared=256,
                      dtype="bf16", bias="uniform", seed=40 + K)
    inp = make_inputs(cfg)
    lay = DeviceLayer(inp)
    y, idx, gate = lay.forward()
    y2, _, _ = lay.forward()
    torch.cuda.synchronize()
    assert np.array_equal(host(y).view(np.uint32), host(y2).view(np.uint32))
    o_idx, o_gate, y_ref = _oracle_layer(inp, cfg)
    assert np.array_equal(host(idx), o_idx) and np.array_equal(host(gate), o_gate)
    yh = host(y)
    check_close(yh, y_ref, True, f"fused combine K={K} (every token)")
    tail = np.arange(512 * 256, cfg.T)
    check_close(yh[tail], y_ref[tail], True, f"fused combine K={K} (tail tile)")


@pytest.mark.parametrize("d", [192, 256])
@pytest.mark.parametrize("K", [1, 3, 7, 8])
def test_fused_combine_tiled_any_k(K, d):
    """On 64-row tiles (a few hundred tokens) the shared expert's fc2 also
    performs the combine, for every K <= 8, on both tile widths (128 columns
    for d = 256, 64 for d = 192) and a ragged last tile: every token matches
    the oracle, and a repeat is bit-identical."""
    from workloads.configs import LayerConfig

    cfg = LayerConfig(name=f"fused_tiled_k{K}_d{d}", T=700, d=d, E=16, K=K, h=128, h_shared=320,
                      dtype="bf16", bias="uniform", seed=60 + K + d)
    inp = make_inputs(cfg)
    lay = DeviceLayer(inp)
    y, idx, gate = lay.forward()
    y2, _, _ = lay.forward()
    torch.cuda.synchronize()
    assert np.array_equal(host(y).view(np.uint32), host(y2).view(np.uint32))
    o_idx, o_gate, y_ref = _oracle_layer(inp, cfg)
    assert np.array_equal(host(idx), o_idx) and np.array_equal(host(gate), o_gate)
    check_close(host(y), y_ref, True, f"tiled fused combine K={K} d={d} (every token)")


@pytest.fixture(scope="module")
def persistent_layer():
    """ViT-G widths (d = 1536, h = 768, h_s = 1536) with 8 experts and K = 2
    at 22 605 tokens: about 5 650 rows per expert, so the routed GEMMs run on
    the persistent 256-row tiles with 24 (fc1) and 12 (fc2) K slabs, and the
    shared expert's fc2 (89 row tiles x 6 column tiles) carries the fused
    combine, with a partial last tile."""
    from workloads.configs import LayerConfig

    cfg = LayerConfig(name="persistent_d1536", T=89 * 256 - 179, d=1536, E=8, K=2, h=768, h_shared=1536,
                      dtype="bf16", bias="uniform", seed=77)
    inp = make_inputs(cfg)
    return cfg, inp, DeviceLayer(inp)


@pytest.mark.slow
def test_persistent_tiles_every_token(persistent_layer):
    cfg, inp, lay = persistent_layer
    y, idx, gate = lay.forward()
    torch.cuda.synchronize()
    o_idx, o_gate, y_ref = _oracle_layer(inp, cfg)
    assert np.array_equal(host(idx), o_idx) and np.array_equal(host(gate), o_gate)
    rc = np.bincount(o_idx.reshape(-1), minlength=cfg.E)
    assert rc.min() >= 512  # every expert on 256-row tiles
    check_close(host(y), y_ref, True, "persistent-tile layer y (every token)")


@pytest.mark.slow
def test_persistent_tiles_deterministic(persistent_layer):
    _, _, lay = persistent_layer
    y1, i1, g1 = lay.forward()
    y2, i2, g2 = lay.forward()
    torch.cuda.synchronize()
    assert torch.equal(i1, i2) and torch.equal(g1.view(torch.int32), g2.view(torch.int32))
    assert torch.equal(y1.view(torch.int16), y2.view(torch.int16))


@pytest.mark.slow
def test_persistent_tiles_token_permutation_equivariance(persistent_layer):
    """Permuting the tokens permutes y bit for bit: every row's arithmetic is
    the same wherever the row sits in its expert's tiles."""
    cfg, inp, lay = persistent_layer
    y, _, _ = lay.forward()
    perm = np.random.default_rng(5).permutation(cfg.T)
    inp_p = make_inputs(cfg, parts=["w_router", "bias", "w1", "w2", "w1s", "w2s"])
    inp_p.x = inp.x[perm]
    lay_p = DeviceLayer(inp_p)
    y_p, _, _ = lay_p.forward()
    torch.cuda.synchronize()
    assert np.array_equal(host(y)[perm].view(np.uint32), host(y_p).view(np.uint32))


@pytest.mark.parametrize("T", [16384 + 77, 65536 + 77])
@pytest.mark.parametrize("dup", [16, 128])
def test_route_near_ties_block_kernels(T, dup):
    """Exact ties (groups of `dup` identical router rows) at token counts that
    take the block chain kernels (64 and 256 tokens per block) with a partial
    last block: tokens whose candidates overflow go to the exact queue, and
    every token's indices and gates equal the oracle's bit for bit."""
    from workloads import bf16_bits_to_f32, f32_to_bf16_bits

    d, E, K = 256, 128, 8
    rng = np.random.default_rng(T + dup)
    x = f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    base = f32_to_bf16_bits((rng.standard_normal((E // dup, d)) * 0.05).astype(np.float32))
    wr = np.repeat(base, dup, axis=0)
    bias = np.zeros(E, np.float32)
    desc = binding.make_desc(T, d, E, K, 64)
    ws = binding.alloc_workspace(desc)
    idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
    binding.moe_route(desc, dev(x), dev(wr), dev(bias), idx, gate, ws)
    torch.cuda.synchronize()
    ref_idx, ref_gate = oracle.route(bf16_bits_to_f32(x), bf16_bits_to_f32(wr), bias, K)
    assert np.array_equal(host(idx), ref_idx) and np.array_equal(host(gate), ref_gate)


@pytest.mark.parametrize("E,dup", [(256, 1), (256, 16), (256, 128), (128, 1), (128, 16), (200, 1)])
def test_route_norms_from_logits_gemm(E, dup):
    """E experts at a token count (51 200 + 77) whose router logits run on
    256-row tiles of the persistent kernel (the logit row rounded up to 256
    columns), which also forms the token norms of the interval test; a
    partial last tile; token rows of very different norms; exact ties in
    groups of `dup` router rows (dup = 1: none), with a selection bias. Every
    token's indices and gates equal the oracle's."""
    from workloads import bf16_bits_to_f32, f32_to_bf16_bits

    T, d, K = 51200 + 77, 128, 8
    rng = np.random.default_rng(7 + dup + E)
    scale = np.exp(rng.uniform(-3.0, 1.5, (T, 1))).astype(np.float32)
    x = f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32) * scale)
    base = f32_to_bf16_bits((rng.standard_normal((E // dup, d)) * 0.05).astype(np.float32))
    wr = np.repeat(base, dup, axis=0)
    bias = rng.uniform(-0.02, 0.02, E).astype(np.float32)
    desc = binding.make_desc(T, d, E, K, 64)
    ws = binding.alloc_workspace(desc)
    idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
    binding.moe_route(desc, dev(x), dev(wr), dev(bias), idx, gate, ws)
    torch.cuda.synchronize()
    ref_idx, ref_gate = oracle.route(bf16_bits_to_f32(x), bf16_bits_to_f32(wr), bias, K)
    assert np.array_equal(host(idx), ref_idx) and np.array_equal(host(gate), ref_gate)


@pytest.mark.parametrize("E", [1, 3, 8, 64, 256, 1024])
def test_bias_update_bit_exact(E):
    """Loss-free balancing update (Eqs. (8)-(9)) through the C ABI against the
    oracle, bit for bit: random loads, a skewed load, a balanced load."""
    rng = np.random.default_rng(100 + E)
    desc = binding.make_desc(64, 64, E, 1, 64)
    for rule in (binding.MOE_BIAS_SIGN, binding.MOE_BIAS_ZSCORE):
        for case in ("random", "skewed", "balanced"):
            if case == "random":
                counts = rng.integers(0, 20000, size=E)
            elif case == "skewed":
                counts = (rng.zipf(1.2, size=E) % 65536) * 8
            else:
                counts = np.full(E, 77)
            counts = counts.astype(np.int32)
            b = rng.normal(0, 0.05, E).astype(np.float32)
            alpha = float(np.float32(rng.uniform(1e-4, 0.1)))
            db = dev(b)
            binding.moe_bias_update(desc, dev(counts), db, alpha, rule)
            torch.cuda.synchronize()
            want = oracle.bias_update(counts, b, alpha, rule)
            assert np.array_equal(host(db).view(np.uint32), want.view(np.uint32)), (rule, case)


def test_bias_update_from_permute_counts(small):
    """Route, permute and update the bias on the GPU; the counts and the new
    bias match the oracle's."""
    cfg, inp, lay, _, ref_idx, _ = small
    idx, _ = lay.route()
    counts, _, _ = lay.permute(idx)
    rc, _, _ = oracle.permute(ref_idx, cfg.E)
    assert np.array_equal(host(counts), rc)
    b0 = inp.bias if inp.bias is not None else np.zeros(cfg.E, np.float32)
    for rule in (binding.MOE_BIAS_SIGN, binding.MOE_BIAS_ZSCORE):
        db = dev(np.asarray(b0, np.float32))
        binding.moe_bias_update(lay.desc, counts, db, 1e-3, rule)
        torch.cuda.synchronize()
        want = oracle.bias_update(rc, b0, np.float32(1e-3), rule)
        assert np.array_equal(host(db).view(np.uint32), want.view(np.uint32))
