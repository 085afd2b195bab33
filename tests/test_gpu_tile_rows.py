"""Layers of a few experts with ragged row counts (64-row tiles: the 256-row
tiles would leave most CUs idle), layers on either side of the 128-row tiles'
line (896 tiles), dense shared layers with K = 1, and launches of a few tiles
(deep rings, fewer K slabs than the ring holds). Every token against the
oracle, forward and backward, with the bounds of the random shapes (routing bit
for bit). The tile heights of larger groups: test_gpu_tile_heights."""

import pytest

import test_gpu_random_shapes as shapes
from test_gpu_random_shapes import _cid
from workloads.configs import LayerConfig

pytestmark = pytest.mark.gpu


def _layer(name, T, d, E, K, h, hs=0, act="gelu"):
    return LayerConfig(name=name, T=T, d=d, E=E, K=K, h=h, h_shared=hs, dtype="bf16", bias="uniform", seed=T + d + h,
                       act=act)


ROWS = [
    _layer("rows127", 254, 256, 2, 1, 128, 128), _layer("rows128", 256, 256, 2, 1, 128, 64),
    _layer("rows224_896tiles", 7168, 512, 128, 4, 512), _layer("rows319", 638, 128, 2, 1, 128),
    _layer("rows320", 640, 128, 2, 1, 128, 128), _layer("rows320_h320", 640, 320, 2, 1, 320, 320),
    _layer("rows130_long", 260, 768, 2, 1, 768), _layer("rows200_short", 400, 768, 2, 1, 704),
    _layer("rows210_sw", 420, 192, 4, 2, 100, 70, "swiglu"), _layer("rows130_sw_long", 260, 768, 4, 2, 710, 0, "swiglu"),
    _layer("rows200_sw_d64", 400, 64, 4, 2, 33, 65, "swiglu"), _layer("rows400_sw", 800, 128, 4, 2, 160, 0, "swiglu"),
]
WIDE = [
    _layer("rows224_d576", 7200, 576, 128, 4, 576, 64), _layer("rows224_sw", 7200, 512, 128, 4, 500, 0, "swiglu"),
    _layer("rows223_895tiles", 7167, 512, 128, 4, 512),
]
SMALL = [
    _layer("tokens1", 1, 64, 3, 2, 64, 64), _layer("tokens5", 5, 320, 70, 4, 192, 256),
    _layer("tokens65", 65, 128, 40, 8, 128, 128), _layer("tokens5_sw", 5, 192, 40, 4, 65, 100, "swiglu"),
    _layer("dense128", 6200, 1024, 2, 1, 64, 1024), _layer("dense128_sw", 6200, 1024, 2, 1, 65, 1000, "swiglu"),
]


@pytest.mark.parametrize("cfg", ROWS + WIDE + SMALL, ids=_cid)
def test_tile_rows_forward(cfg):
    shapes.test_random_shape_layer_forward(cfg)


@pytest.mark.parametrize("cfg", [c for c in ROWS + SMALL if not c.name.startswith("dense")], ids=_cid)
def test_tile_rows_backward(cfg):
    shapes.test_random_shape_backward(cfg)
