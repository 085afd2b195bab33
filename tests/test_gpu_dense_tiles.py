"""The shared expert's dense products on the tile heights below 256 rows: 128 x
128 and 128 x 64 tiles with the fused combine (K from 1 to 8) and with the
fp32 store before a separate combine (K = 9), GELU and SwiGLU, and 64-row
tiles on either side of the 128-row tiles' lines (384 tiles, 513 to 640 tiles,
widths under 384). Every row of the layer's output against torch in 64 bits
(activations and expert outputs rounded to bf16 where the library rounds
them), with the bf16 bounds of the layer tests."""

import pytest
import torch

from gpu_util import check_close
from paper_2608_17402_amd import binding

pytestmark = pytest.mark.gpu

# T, d, h_shared, K (= E), act
CASES = {
    "tiles128_k1": (6200, 1024, 1024, 1, "gelu"),
    "tiles128_k5": (6200, 1024, 1024, 5, "gelu"),
    "tiles128_k8_wide_fc1": (12500, 512, 2048, 8, "gelu"),
    "tiles128x64_k3": (7100, 960, 960, 3, "gelu"),
    "tiles128x64_k8": (16500, 448, 448, 8, "gelu"),
    "tiles128_store_k9": (6200, 1024, 1024, 9, "gelu"),
    "tiles128_sw_k7": (6200, 1024, 1000, 7, "swiglu"),
    "tiles128_sw_544": (8600, 1024, 1024, 2, "swiglu"),
    "tiles64_384minus": (6100, 1024, 1024, 2, "gelu"),
    "tiles64_544": (8600, 1024, 1024, 2, "gelu"),
    "tiles64_narrow": (26000, 320, 320, 4, "gelu"),
}


def _mlp(x, w1, w2, h, sw):
    p = x.double() @ w1.double().t()
    a = torch.nn.functional.silu(p[:, :h]) * p[:, h:] if sw else torch.nn.functional.gelu(p)
    return a.to(torch.bfloat16).double() @ w2[:, :h].double().t()


@pytest.mark.parametrize("name", CASES)
def test_shared_expert_tiles(name):
    T, d, hs, K, act = CASES[name]
    E, h, sw = K, 64, act == "swiglu"
    gen = torch.Generator(device="cuda").manual_seed(T + d + K)

    def normal(*shape, std):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(torch.bfloat16)

    rows, ld = (2 if sw else 1), (-(-hs // 64) * 64 if sw else hs)
    x, wr = normal(T, d, std=1.0), normal(E, d, std=0.02)
    w1, w2 = normal(E, rows * h, d, std=0.02), normal(E, d, h, std=0.02)
    w1s, w2s = normal(rows * hs, d, std=0.02), torch.zeros(d, ld, dtype=torch.bfloat16, device="cuda")
    w2s[:, :hs] = normal(d, hs, std=0.02)
    desc = binding.make_desc(T, d, E, K, h, hs, 0.75, "bf16", flags=binding.MOE_FLAG_SWIGLU if sw else 0)
    ws = binding.alloc_workspace(desc)
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    idx = torch.empty(T, K, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, K, dtype=torch.float32, device="cuda")
    binding.moe_layer_forward(desc, x, wr, None, w1, w2, w1s, w2s, y, idx, gate, ws)
    ref = 0.75 * _mlp(x, w1s, w2s, hs, sw)
    for e in range(E):  # K = E: every token takes every expert
        out = _mlp(x, w1[e], w2[e], h, sw).to(torch.bfloat16).double()
        ref += (gate * (idx == e)).sum(dim=1, keepdim=True).double() * out
    check_close(y.double().cpu().numpy(), ref.cpu().numpy(), True, name)
