"""Kernel variants at the sizes where their dispatch changes and at the edges of their tiles, against the oracle."""
import os
import sys

import pytest

from paper_2212_05191_amd import binding as B
from paper_2212_05191_amd import workloads as wl

pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import parity  # noqa: E402
import test_gpu_backward as bwd  # noqa: E402


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    B.load()
    return torch


def _forward_and_backward(cfg, dloss=0.7):
    layer = bwd._forward_backward(cfg, chained=True, dloss=dloss)
    try:
        info = parity.check_full(cfg, layer)
        fwd, out, _ = bwd._check_steps(cfg, layer, dloss=dloss)
        errs = bwd._check_end_to_end(cfg, fwd, out, dloss=dloss)
        print(f"   forward {info}\n   backward {({k: float(f'{v:.1e}') for k, v in errs.items()})}", flush=True)
    finally:
        layer.close()


# fp32 expert GEMMs: each of the four tile shapes (picked by the number of tiles, so by experts x rows x columns), with
# row counts one off a tile edge, contraction lengths that are no multiple of the 32-deep slab (8, 40) and columns
# that end inside a tile.
F32_TILES = [
    wl.small_config("f32_tile_32x32", 130, 8, 40, 2, 1, 65, "f32", "gelu", seed=301),
    wl.small_config("f32_tile_32x64", 1100, 40, 520, 4, 2, 129, "f32", "relu", seed=302),
    wl.small_config("f32_tile_64x64", 2000, 40, 1032, 4, 4, 127, "f32", "gelu", seed=303),
    wl.small_config("f32_tile_64x128", 4000, 40, 2056, 4, 4, 257, "f32", "gelu", seed=304),
]


@pytest.mark.parametrize("cfg", F32_TILES, ids=lambda c: c.name)
def test_f32_gemm_tiles(torch_cuda, cfg):
    _forward_and_backward(cfg)
