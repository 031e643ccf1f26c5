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


# Routing: the block sizes (16, 32, 64, 256 tokens) at the batch sizes where they change, one token more and the single-block
# case; router widths on both sides of what a token's threads keep in registers; histograms summed by every block and scanned by a
# kernel of their own; the first-hop limit in each.
ROUTE_EDGES = [
    wl.small_config("route_one_block_16", 16, 64, 64, 2, 3, 2, "bf16", "relu", seed=311),
    wl.small_config("route_one_block_64_cap", 63, 72, 64, 3, 2, 9, "f32", "gelu", skew=True, seed=312, group_capacity=20),
    wl.small_config("route_two_blocks", 65, 64, 64, 1, 9, 5, "f16", "relu", seed=313),
    wl.small_config("route_256_blocks_16", 4096, 64, 64, 33, 3, 40, "bf16", "relu", seed=314, group_capacity=110),
    wl.small_config("route_16_to_32", 4097, 64, 64, 17, 4, 60, "bf16", "gelu", skew=True, seed=315),
    wl.small_config("route_32_to_64", 8193, 104, 64, 2, 8, 500, "f32", "relu", seed=316),
    wl.small_config("route_inline_to_scan", 16385, 64, 64, 4, 5, 800, "bf16", "relu", skew=True, seed=317, group_capacity=3000),
    wl.small_config("route_64_to_256", 65537, 64, 64, 3, 2, 9000, "bf16", "relu", seed=318),
    # logits left to the gate kernel: 33 to 48 columns over 64 tokens (on both sides: 32, 49), blocks of 256 tokens
    wl.small_config("route_32_columns_64", 8300, 128, 64, 24, 8, 60, "f16", "relu", seed=321),
    wl.small_config("route_33_columns_64", 8193, 136, 64, 25, 8, 60, "f32", "relu", seed=322, group_capacity=300),
    wl.small_config("route_48_columns_64", 9000, 128, 64, 40, 8, 30, "bf16", "relu", skew=True, seed=323),
    wl.small_config("route_49_columns_64", 9000, 128, 64, 41, 8, 30, "bf16", "relu", seed=324),
    wl.small_config("route_256_below_65536", 52000, 64, 64, 64, 8, 110, "bf16", "relu", seed=325),
    wl.small_config("route_256_wide_tile", 66000, 64, 64, 32, 32, 70, "bf16", "relu", skew=True, seed=326, group_capacity=2000),
    wl.small_config("route_wide_tile", 500, 64, 64, 1, 200, 4, "bf16", "relu", seed=319),
    wl.small_config("route_300_groups_cap", 300, 64, 64, 300, 2, 2, "bf16", "relu", seed=320, group_capacity=1),
]
# kernels that a case is there for (by default: logits and decision in one launch, from an LDS tile)
ROUTE_KERNELS = {
    "route_33_columns_64": ["gate_logits_kernel", "gate_logits_route_kernel", "route_first_hop_kernel<false>", "route_finish_kernel"],
    "route_48_columns_64": ["gate_logits_kernel", "gate_logits_route_kernel", "route_scan_kernel"],
    "route_64_to_256": ["gate_logits_kernel", "gate_logits_route_kernel", "route_scan_kernel"],
    "route_256_below_65536": ["gate_logits_kernel", "gate_logits_route_kernel", "route_scan_kernel"],
    "route_256_wide_tile": ["gate_logits_kernel", "gate_logits_route_kernel", "route_first_hop_kernel<true>"],
    "route_256_blocks_16": ["gate_logits_route_kernel", "route_first_hop_kernel<true>", "route_scan_kernel"],
}
# Routers too wide for a tile: per-wave histograms or one copy, block order summed inside route_finish or scanned, each with
# and without a first-hop limit.
WIDE_ROUTERS = {
    wl.small_config("wide_inline", 300, 64, 64, 1, 1024, 2, "bf16", "relu", seed=351):
        ["gate_logits_kernel", "route_decide_kernel<true>", "route_finish_kernel"],
    wl.small_config("wide_inline_hop", 500, 64, 64, 600, 2, 3, "f32", "relu", seed=352, group_capacity=1):
        ["gate_logits_kernel", "route_decide_kernel<true>", "route_first_hop_kernel<false>", "route_finish_kernel"],
    wl.small_config("wide_inline_one_copy", 700, 64, 64, 1000, 2, 2, "bf16", "relu", skew=True, seed=353, group_capacity=2):
        ["gate_logits_kernel", "route_decide_kernel<false>", "route_first_hop_kernel<false>", "route_finish_kernel"],
    wl.small_config("wide_scan", 20000, 64, 64, 2, 900, 20, "f16", "relu", seed=354):
        ["gate_logits_kernel", "route_decide_kernel<true>", "route_scan_kernel"],
    wl.small_config("wide_scan_hop", 12000, 64, 64, 48, 60, 9, "bf16", "relu", skew=True, seed=355, group_capacity=200):
        ["gate_logits_kernel", "route_decide_kernel<false>", "route_first_hop_kernel<true>"],
}


def _launched(layer, call):
    """Names of the kernels that a library call on the layer's ctx launches."""
    import ctypes
    import torch
    lib, evs = B.load(), [torch.cuda.Event(enable_timing=True) for _ in range(32)]
    for e in evs:
        e.record()
    torch.cuda.synchronize()
    arr = (ctypes.c_void_p * 32)(*[e.cuda_event for e in evs])
    assert lib.smile_kernel_timing(layer.ctx.handle, arr, 16) == 0
    call()
    torch.cuda.synchronize()
    names = [lib.smile_kernel_timing_name(layer.ctx.handle, i).decode() for i in range(lib.smile_kernel_timing_count(layer.ctx.handle))]
    assert lib.smile_kernel_timing(layer.ctx.handle, None, 0) == 0
    return names


@pytest.mark.parametrize("cfg", ROUTE_EDGES + list(WIDE_ROUTERS), ids=lambda c: c.name)
def test_routing_blocks(torch_cuda, cfg):
    """The chained forward passes (logits and routing in one launch) and the separate calls give the same bits; the
    outputs match the oracle; the kernels that the case is there for ran."""
    import numpy as np
    from test_gpu_parity import _run
    outs = {}
    for how in ("steps", "fused", "chained"):
        layer = _run(cfg, how)
        try:
            outs[how] = parity.fetch(layer)
            if how == "chained":
                parity.check_full(cfg, layer)
                names = _launched(layer, layer.forward)
                want = WIDE_ROUTERS.get(cfg) or ROUTE_KERNELS.get(cfg.name, ["gate_logits_route_kernel"])
                assert all(any(w in k for k in names) for w in want), (want, names)
                assert ("gate_logits_kernel" in want) == any("gate_logits_kernel" in k for k in names), (want, names)
        finally:
            layer.close()
    for how in ("fused", "chained"):
        for k, v in outs["steps"].items():
            if k not in ("xe", "ye"):
                np.testing.assert_array_equal(outs[how][k], v, err_msg=f"{how} {k}")


# 16-bit forward tiles of 64 rows: both sides of every line of the choice (64 x 64 tiles over the buffers: 768, 8192 for the
# up-projection, 1024, 2048 for the down-projection; 64 rows), row counts one off a tile edge, columns that end inside a
# 128- or 256-wide tile, one K slab and more slabs than a ring has stages.
FFN_TILES = [
    wl.small_config("ffn_one_row", 5, 64, 64, 2, 2, 1, "bf16", "gelu", seed=331),
    wl.small_config("ffn_up_64x64_last", 700, 64, 2048, 4, 6, 63, "bf16", "gelu", seed=332),
    wl.small_config("ffn_up_64x128_first", 700, 64, 2112, 5, 5, 64, "f16", "relu", skew=True, seed=333),
    wl.small_config("ffn_65_rows", 900, 192, 832, 3, 3, 65, "f16", "gelu", seed=334),
    wl.small_config("ffn_up_64x128_persistent", 300, 64, 4032, 13, 10, 3, "bf16", "relu", seed=335),
    wl.small_config("ffn_up_64x256", 300, 64, 4160, 16, 8, 3, "bf16", "gelu", seed=336),
    wl.small_config("ffn_down_64x64_last", 2000, 512, 576, 8, 8, 127, "bf16", "gelu", seed=337),
    wl.small_config("ffn_down_64x128", 400, 576, 640, 16, 8, 4, "bf16", "relu", seed=338),
    wl.small_config("ffn_down_64x256", 600, 576, 640, 29, 8, 4, "bf16", "gelu", skew=True, seed=339),
]


@pytest.mark.parametrize("cfg", FFN_TILES, ids=lambda c: c.name)
def test_small_ffn_tiles(torch_cuda, cfg, monkeypatch):
    """Forward (with and without expert buffers, and with both saved outputs) and backward against the oracle; the same bits
    as the 128 x 192 tile."""
    import numpy as np
    from test_gpu_parity import _run
    outs = {}
    for how, tile in (("steps", "0"), ("steps", None), ("fused", None)):
        if tile is None:
            monkeypatch.delenv("SMILE_FFN_TILE", raising=False)
        else:
            monkeypatch.setenv("SMILE_FFN_TILE", tile)
        layer = _run(cfg, how)
        try:
            outs[how, tile] = parity.fetch(layer)["y"]
        finally:
            layer.close()
    for key, y in outs.items():
        np.testing.assert_array_equal(y, outs["steps", "0"], err_msg=str(key))
    _forward_and_backward(cfg)


# ---- routing decisions must not depend on how the batch is cut into blocks.  One batch size for each block size (a single block,
# 16, 32, 64 and 256 tokens)
ROUTE_BATCHES = (40, 300, 5000, 10000, 70000)


def _route(torch, T, li, lq, bi=None, bq=None):
    """smile_route_bilevel on the first T rows of the logits; the per-token outputs as host tensors."""
    n, m = li.shape[1], lq.shape[1]
    desc = B.make_desc(T, 64, 64, n, m, 8, "f32", "relu")
    ctx, b = B.Ctx(desc), B.alloc_buffers(desc)
    li, lq = li[:T].contiguous(), lq[:T].contiguous()
    B.smile_route_bilevel(ctx, li, lq, bi, bq, b.group_idx, b.local_idx, b.pos_in_group, b.slot, b.gate, b.p_top, b.q_top,
                          b.group_count, b.local_count, b.expert_count, b.kept_count, b.p_sum, b.q_sum)
    torch.cuda.synchronize()
    ctx.close()
    return {k: getattr(b, k).cpu() for k in ("group_idx", "local_idx", "gate", "p_top", "q_top")}


@pytest.mark.parametrize("n,m", [(2, 8), (5, 3), (17, 9), (1, 129), (34, 40)])
def test_gates_do_not_depend_on_the_batch(torch_cuda, n, m):
    """A token's gate has the same bits in every block size and in the kernel for very wide routers, which adds the softmax
    denominator in column order (reached here through extra columns that a bias of -inf takes out of the sum)."""
    torch = torch_cuda
    g = torch.Generator(device="cuda:0").manual_seed(341)
    T, wide = max(ROUTE_BATCHES), max(m, min(160, 4096 // n))
    li = torch.empty(T, n, device="cuda:0").normal_(0, 1.5, generator=g)
    lq = torch.empty(T, wide, device="cuda:0").normal_(0, 1.5, generator=g)
    bq = torch.zeros(n, wide, device="cuda:0")
    bq[:, m:] = float("-inf")
    want = _route(torch, T, li, lq, None, bq)
    lq = lq[:, :m].contiguous()
    for t in ROUTE_BATCHES:
        for k, v in _route(torch, t, li, lq).items():
            assert torch.equal(v, want[k][:t]), f"T={t} {k}: {(v != want[k][:t]).sum()} of {t} differ"


@pytest.mark.parametrize("n", [4, 9, 40])
def test_rows_without_a_maximum(torch_cuda, n):
    """Logits that are not finite have unspecified results, but the same index in every block size and in the kernel for very wide
    routers: the first column above all before it, 0 where no column is above -inf."""
    torch = torch_cuda
    inf, nan = float("inf"), float("nan")
    rows = torch.zeros(6, n, device="cuda:0")
    rows[0] = -inf
    rows[1] = nan
    rows[2, 0], rows[2, 1:] = nan, -inf
    rows[3, :-1], rows[3, -1] = nan, -5.0
    rows[4] = inf
    rows[5, 1] = inf
    want = torch.tensor([0, 0, 0, n - 1, 0, 1], dtype=torch.int32)
    T = max(ROUTE_BATCHES)
    li = rows.repeat(T // 6 + 1, 1)[:T].contiguous()
    want = want.repeat(T // 6 + 1)[:T]
    for t in ROUTE_BATCHES:
        out = _route(torch, t, li, li)
        assert torch.equal(out["group_idx"], want[:t]) and torch.equal(out["local_idx"], want[:t]), t
    out = _route(torch, T, li, torch.full((T, 4000 // n), -inf, device="cuda:0"))
    assert torch.equal(out["group_idx"], want) and not out["local_idx"].any()


def test_router_logits_of_very_long_rows(torch_cuda):
    """16 rows of 286,331,200 elements: the offset of the last row does not fit 32 bits.  Every row has one element that the
    weights see, at its end."""
    torch = torch_cuda
    T, d = 16, 286331200
    assert (T - 1) * d >= 1 << 32 and d % 64 == 0
    if torch.cuda.mem_get_info()[0] < 16 << 30:
        pytest.skip("needs 16 GB of device memory")
    x = torch.zeros(T, d, dtype=torch.bfloat16, device="cuda:0")
    x[:, -1] = torch.arange(1, T + 1, device="cuda:0")
    w = torch.zeros(1, d, dtype=torch.bfloat16, device="cuda:0")
    w[0, -1] = 2.0
    li, lq = torch.empty(T, 1, device="cuda:0"), torch.empty(T, 1, device="cuda:0")
    ctx = B.Ctx(B.make_desc(T, d, 64, 1, 1, 1, "bf16", "relu"))
    B.smile_gate_logits(ctx, x, w, w, li, lq)
    torch.cuda.synchronize()
    ctx.close()
    want = 2.0 * torch.arange(1, T + 1, device="cuda:0").float()
    assert torch.equal(li[:, 0], want) and torch.equal(lq[:, 0], want)


# ---- expert biases.  Every 16-bit tile shape, plain and persistent, on columns that end inside a 128-, 192- and 256-wide tile (448, 320)
# and rows that end inside a tile; fp32 too.  6 names no shape (the library's choice); the ring tiles, 1 to 4, have one grid for both values.
def _layer_with_biases(cfg):
    import numpy as np
    from paper_2212_05191_amd.runner import GpuLayer, to_device
    layer = GpuLayer(cfg)
    rng = np.random.default_rng(9)
    b1 = wl.quantize(rng.standard_normal((cfg.N, cfg.d_ff)).astype(np.float32), cfg.dtype)
    b2 = wl.quantize(rng.standard_normal((cfg.N, cfg.d_model)).astype(np.float32), cfg.dtype)
    layer.b1, layer.b2 = to_device(b1, cfg.dtype), to_device(b2, cfg.dtype)
    for io in (layer.io, layer.io_fused):
        io.b1, io.b2 = layer.b1.data_ptr(), layer.b2.data_ptr()
    return layer, b1, b2


@pytest.mark.parametrize("persist", ["0", "1"])
@pytest.mark.parametrize("tile,dtype", [(t, "bf16") for t in range(10)] + [(t, "f16") for t in (0, 1, 2, 5, 8, 9)] + [(None, "f32"), (None, "bf16")])
def test_expert_biases_in_every_tile(torch_cuda, tile, dtype, persist, monkeypatch):
    """The separate calls against the oracle with biases; the chained, the buffer-free and the activation-saving forward passes
    (two outputs: the pre-activation has the bias too) give the same bits."""
    import numpy as np
    import oracle
    from paper_2212_05191_amd.runner import to_host
    monkeypatch.setenv("SMILE_FFN_PERSIST", persist)
    if tile is not None:
        monkeypatch.setenv("SMILE_FFN_TILE", str(tile))
    cfg = wl.small_config(f"biases_{dtype}_{tile}", 900, 320, 448, 2, 3, 170, dtype, "gelu", seed=361)
    layer, b1, b2 = _layer_with_biases(cfg)
    try:
        layer.buf.ye.zero_()
        layer.forward_steps()
        out = parity.fetch(layer)
        x, wi, wq, bi, bq = parity.host_inputs(cfg)
        r, _ = parity.check_logits_and_routing(cfg, out, x, wi, wq, bi, bq)
        xe = parity.check_dispatch_exact(cfg, out, x, r)
        w1 = np.stack([wl.gen_expert_weights(cfg, e)[0] for e in range(cfg.N)])
        w2 = np.stack([wl.gen_expert_weights(cfg, e)[1] for e in range(cfg.N)])
        ye = oracle.expert_ffn(xe, r.kept_count, w1, w2, cfg.act, dtype, b1, b2)
        mask = np.arange(cfg.capacity)[None, :] < r.kept_count[:, None]
        assert parity.normwise(out["ye"][mask], ye[mask]) <= parity.TOL[dtype]
        y = oracle.combine(ye, r.group_idx, r.local_idx, r.slot, r.gate, cfg.m_local, dtype)
        assert parity.normwise(out["y"], y) <= parity.TOL[dtype]
        for run in (layer.forward, layer.forward_fused):
            layer.buf.y.fill_(-7)
            run()
            np.testing.assert_array_equal(parity.fetch(layer)["y"], out["y"])
        layer.enable_saved_activations()
        layer.pre_save.zero_()
        layer.buf.y.fill_(-7)
        layer.forward_fused()
        np.testing.assert_array_equal(parity.fetch(layer)["y"], out["y"])
        # the pre-activation: one rounding to the storage type of a sum that is exact to fp32 rounding
        pre = np.matmul(xe.astype(np.float64), w1.astype(np.float64).transpose(0, 2, 1)) + b1[:, None, :]
        step = {"f32": 1e-5, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
        assert parity.normwise(to_host(layer.pre_save)[mask], pre[mask]) <= step
    finally:
        layer.close()


# ---- ring kernels: every tile shape against the two-stage kernels, which add the same products in the same order.  Contractions of
# three slabs, of an even and an odd number of them, and (weight gradients: a group's rows) of none, one, two and more with k-rows
# that end inside a slab; buffers of skewed experts from empty to full, so rows end anywhere in a 128- or 256-row tile; columns that end inside
# 128-, 192- and 256-wide tiles.
RING_CASES = [
    wl.small_config("ring_3_and_7_slabs", 2600, 192, 448, 3, 5, 300, "bf16", "gelu", skew=True, seed=371),
    wl.small_config("ring_4_and_5_slabs_f16", 1700, 256, 320, 4, 6, 257, "f16", "relu", skew=True, seed=372),
    wl.small_config("ring_15_slabs", 900, 960, 192, 2, 3, 170, "bf16", "relu", skew=True, seed=373, group_capacity=500),
    wl.small_config("ring_70_experts", 2000, 192, 256, 10, 7, 64, "bf16", "gelu", skew=True, seed=374),
]


@pytest.mark.parametrize("cfg", RING_CASES, ids=lambda c: c.name)
def test_ring_tiles_give_the_bits_of_the_two_stage_kernels(torch_cuda, cfg, monkeypatch):
    from paper_2212_05191_amd.runner import GpuLayer
    dy = wl.gen_output_grad(cfg)
    want = None
    for tile in range(5):   # 0: two-stage
        monkeypatch.setenv("SMILE_FFN_TILE", str(tile))
        monkeypatch.setenv("SMILE_TGEMM_TILE", str(tile))
        layer = GpuLayer(cfg)
        try:
            layer.enable_saved_activations()
            layer.forward()
            layer.prepare_backward(dy)
            for call, count in ((layer.backward, 4), (layer.forward_fused, 2)):
                names = _launched(layer, call)
                assert sum("grouped_gemm_ring" in k for k in names) == (count if tile else 0), names
            kept = layer.buf.kept_count.cpu()
            live = torch_cuda.arange(cfg.capacity)[None, :] < kept[:, None]
            got = {k: getattr(layer.buf, k).cpu() for k in ("y",)} | {k: getattr(layer.bwd, k).cpu() for k in ("dx", "dw1", "dw2")}
            got |= {"h": layer.h_save.cpu()[live], "pre": layer.pre_save.cpu()[live], "ye": layer.buf.ye.cpu()[live]}
        finally:
            layer.close()
        if want is None:
            want = got
            if cfg.name != "ring_70_experts":
                assert kept.min() < 64 and kept.max() == cfg.capacity
        for k, v in got.items():
            assert torch_cuda.equal(v, want[k]), f"tile {tile} {k}: {(v != want[k]).sum()} of {v.numel()} differ"


# Several tiles per workgroup: what a ring kernel requests of the next tile before the epilogue of this one, and the tile that it then starts
# on.  70 skewed experts (routing biases scaled so that some stay empty and most do not) give one or two row tiles and (weight gradients)
# contractions of none to three slabs side by side; narrow one way, so that every product is wide in one of the two: up, dpre and dW2 or down,
# dxe and dW1 have more tiles than the chip's 256 CUs hold workgroups.
HAND_OVER = [
    (wl.small_config("hand_over_192_to_2048", 9000, 192, 2048, 10, 7, 150, "bf16", "gelu", skew=True, seed=397), 0.45),
    (wl.small_config("hand_over_2048_to_256_f16", 9000, 2048, 256, 10, 7, 150, "f16", "relu", skew=True, seed=398), 1.4),
]


@pytest.mark.parametrize("cfg,skew", HAND_OVER, ids=lambda c: getattr(c, "name", ""))
def test_ring_tiles_one_after_the_other(torch_cuda, cfg, skew, monkeypatch):
    import numpy as np
    monkeypatch.setenv("SMILE_FFN_PERSIST", "0")   # two-stage kernels: one tile per workgroup
    layer, _, _ = _layer_with_biases(cfg)
    try:
        layer.bias_inter.mul_(skew), layer.bias_intra.mul_(skew)
        layer.enable_saved_activations()
        layer.prepare_backward(wl.gen_output_grad(cfg))
        want = None
        for tile in range(5):   # 0: two-stage
            monkeypatch.setenv("SMILE_FFN_TILE", str(tile))
            monkeypatch.setenv("SMILE_TGEMM_TILE", str(tile))
            layer.ctx.close()
            layer.ctx = B.Ctx(layer.desc)
            for t in (layer.buf.y, layer.buf.ye, layer.h_save, layer.pre_save, layer.bwd.dw1, layer.bwd.dw2, layer.bwd.dx):
                t.fill_(-7)
            got = {}
            for call, count in ((layer.forward_fused, 2), (layer.forward, 2), (layer.backward, 4)):
                names = _launched(layer, call)
                assert sum("grouped_gemm_ring" in k for k in names) == (count if tile else 0), names
                if call == layer.forward_fused:
                    got |= {"y_fused": layer.buf.y.cpu()}
                    layer.buf.y.fill_(-7)
            kept = layer.buf.kept_count.cpu().numpy()
            live = torch_cuda.arange(cfg.capacity)[None, :] < torch_cuda.from_numpy(kept)[:, None]
            got |= {"y": layer.buf.y.cpu(), "ye": layer.buf.ye.cpu()[live], "h": layer.h_save.cpu()[live], "pre": layer.pre_save.cpu()[live]}
            got |= {k: getattr(layer.bwd, k).cpu() for k in ("dx", "dw1", "dw2")}
            if want is None:
                want = got
                slabs = np.unique((kept + 63) // 64)
                assert set(slabs) == {0, 1, 2, 3}, slabs
                # live tiles of the widest shape (128 x 256; one workgroup on a CU), which has the fewest beside its slots
                assert (kept > 0).sum() * (max(cfg.d_model, cfg.d_ff) // 256) >= 512
                assert all(bool((v != 0).any()) for v in got.values())
            for k, v in got.items():
                assert torch_cuda.equal(v, want[k]), f"tile {tile} {k}: {(v != want[k]).sum()} of {v.numel()} differ"
    finally:
        layer.close()


@pytest.mark.parametrize("tile", [0, 1])
def test_gelu_of_an_overflowed_product_is_infinity(torch_cuda, tile, monkeypatch):
    """2^100 * 2^100 has no value in 32 bits; the hidden activation is then infinity, and so is a sum of positive multiples of it."""
    monkeypatch.setenv("SMILE_FFN_TILE", str(tile))
    N, C, d, F = 2, 40, 192, 256
    ctx = B.Ctx(B.make_desc(80, d, F, 1, N, C, "bf16", "gelu"))
    try:
        full = lambda *shape, value: torch_cuda.full(shape, value, dtype=torch_cuda.bfloat16, device="cuda:0")
        xe, w1, w2 = full(N, C, d, value=2.0**100), full(N, F, d, value=2.0**100), full(N, d, F, value=0.5)
        xe[1] = 2.0**-100   # a plain expert beside it: pre = d, ye = d * F / 2
        kept = torch_cuda.full((N,), C, dtype=torch_cuda.int32, device="cuda:0")
        ye = full(N, C, d, value=0.0)
        B.smile_expert_ffn(ctx, xe, kept, w1, None, w2, None, ye)
        torch_cuda.cuda.synchronize()
        assert torch_cuda.isposinf(ye[0]).all()
        assert (ye[1] == d * F / 2).all()
    finally:
        ctx.close()


@pytest.mark.parametrize("tile", [0, 1, 9])
def test_gelu_keeps_its_relative_accuracy_in_the_tail(torch_cuda, tile, monkeypatch):
    """The hidden activation of pre-activations from -5 to -12.5, where GELU falls from 1e-6 to 5e-35.  The rational erfc of the 16-bit
    kernels is off by 0.16 % at -5 and 3.4 % at -12.5 of the exact value (evaluated in 64 bits); storing it in bf16 adds 2^-9."""
    from scipy.special import ndtr
    monkeypatch.setenv("SMILE_FFN_TILE", str(tile))
    N, C, d, F = 2, 40, 192, 192
    ctx = B.Ctx(B.make_desc(80, d, F, 1, N, C, "bf16", "gelu"))
    try:
        zeros = lambda *shape: torch_cuda.zeros(shape, dtype=torch_cuda.bfloat16, device="cuda:0")
        v = -torch_cuda.linspace(5.0, 12.5, F, device="cuda:0").bfloat16()
        xe, w1, w2, ye = zeros(N, C, d), zeros(N, F, d), zeros(N, d, F), zeros(N, C, d)
        xe[:, :, 0] = 1.0
        w1[:, :, 0] = v                                     # pre-activation of column f: v[f]
        w2[:] = torch_cuda.eye(d, device="cuda:0")          # ye = h
        kept = torch_cuda.full((N,), C, dtype=torch_cuda.int32, device="cuda:0")
        B.smile_expert_ffn(ctx, xe, kept, w1, None, w2, None, ye)
        torch_cuda.cuda.synchronize()
        exact = v.double().cpu().numpy() * ndtr(v.double().cpu().numpy())
        worst = abs(ye.double().cpu().numpy() / exact - 1).max()
        assert worst <= 0.034 + 2.0 ** -8, worst
    finally:
        ctx.close()


# Wide routers whose logits the routing launch computes in one pass: 49 to 144 columns of a 16-bit type over blocks of 64 tokens, contractions of one chunk,
# of odd counts and of more chunks than waves, a block that ends early; and 145 columns beside them.
WIDE_GATE = [
    wl.small_config("gate_49_columns", 8200, 64, 64, 17, 32, 17, "bf16", "relu", seed=381),
    wl.small_config("gate_81_columns", 8200, 64, 64, 17, 64, 9, "bf16", "relu", seed=382),
    wl.small_config("gate_96_columns_f16", 8230, 192, 64, 32, 64, 5, "f16", "relu", seed=383),
    wl.small_config("gate_129_columns", 8193, 320, 64, 1, 128, 70, "bf16", "relu", seed=384),
    wl.small_config("gate_144_columns", 8255, 448, 64, 16, 128, 6, "bf16", "relu", skew=True, seed=385, group_capacity=600),
    wl.small_config("gate_145_columns", 8200, 128, 64, 1, 144, 60, "bf16", "relu", seed=386),
]


@pytest.mark.parametrize("cfg", WIDE_GATE, ids=lambda c: c.name)
def test_wide_router_in_the_routing_launch(torch_cuda, cfg):
    import numpy as np
    from test_gpu_parity import _run
    outs = {}
    for how in ("steps", "fused"):
        layer = _run(cfg, how)
        try:
            outs[how] = parity.fetch(layer)
            if how == "fused":
                assert not any("gate_logits_kernel" in k for k in _launched(layer, layer.forward_fused))
            else:
                parity.check_full(cfg, layer)
        finally:
            layer.close()
    assert "logits_intra" in outs["steps"]
    for k, v in outs["steps"].items():
        if k not in ("xe", "ye"):
            np.testing.assert_array_equal(outs["fused"][k], v, err_msg=k)


def _weight_gradients(torch_cuda, cfg, tile, monkeypatch):
    """dW1, dW2 and the names of the backward pass's expert GEMMs with SMILE_TGEMM_TILE = tile ("": the library's choice)"""
    from paper_2212_05191_amd.runner import GpuLayer
    monkeypatch.setenv("SMILE_TGEMM_TILE", tile) if tile else monkeypatch.delenv("SMILE_TGEMM_TILE", raising=False)
    layer = GpuLayer(cfg)
    try:
        layer.enable_saved_activations()
        layer.forward()
        layer.prepare_backward(wl.gen_output_grad(cfg))
        names = [k for k in _launched(layer, layer.backward) if "grouped_gemm" in k]
        return [getattr(layer.bwd, k).cpu() for k in ("dw1", "dw2")], names
    finally:
        layer.close()


def test_weight_gradients_of_one_slab(torch_cuda, monkeypatch):
    """Buffers of at most 64 rows and two 192-column tiles per CU: the two-stage kernel, with the bits of the ring."""
    cfg = wl.small_config("one_slab_130_experts", 900, 256, 384, 13, 10, 9, "bf16", "relu", skew=True, seed=391)
    got, names = _weight_gradients(torch_cuda, cfg, "", monkeypatch)
    assert sum("grouped_gemm_t_kernel" in k for k in names) >= 2, names
    ring, names = _weight_gradients(torch_cuda, cfg, "1", monkeypatch)
    assert sum("grouped_gemm_ring" in k for k in names) == 4, names
    assert all(torch_cuda.equal(a, b) for a, b in zip(got, ring))
    assert all(float(a.float().abs().sum()) > 0 for a in got)


# Weight gradients: the rows that a group is expected to contract decide, not its buffer.  192- and 128-wide tiles, both sides of their lines
# and a quarter full buffers; kernels of the two-stage form among the four products (dpre of 256 -> 1024 is one, too).
DW_ROUTES = [
    (wl.small_config("dw_192_wide_192_rows", 9 * 192, 384, 1536, 3, 3, 260, "bf16", "relu", skew=True, seed=392), 2),
    (wl.small_config("dw_192_wide_193_rows", 9 * 192 + 1, 384, 1536, 3, 3, 260, "bf16", "relu", skew=True, seed=393), 0),
    (wl.small_config("dw_192_wide_70_of_270", 9 * 70, 384, 1536, 3, 3, 270, "f16", "relu", skew=True, seed=394), 2),
    (wl.small_config("dw_128_wide_320_rows", 4 * 320, 256, 1024, 2, 2, 400, "bf16", "relu", skew=True, seed=395), 3),
    (wl.small_config("dw_128_wide_321_rows", 4 * 320 + 1, 256, 1024, 2, 2, 400, "bf16", "relu", skew=True, seed=396), 1),
]


@pytest.mark.parametrize("cfg,two_stage", DW_ROUTES, ids=lambda c: getattr(c, "name", str(c)))
def test_weight_gradients_by_expected_rows(torch_cuda, cfg, two_stage, monkeypatch):
    got, names = _weight_gradients(torch_cuda, cfg, "", monkeypatch)
    assert sum("grouped_gemm_t_kernel" in k for k in names) == two_stage and len(names) == 4, names
    for tile, want in (("0", 0), ("1", 4), ("4", 4)):
        other, names = _weight_gradients(torch_cuda, cfg, tile, monkeypatch)
        assert sum("grouped_gemm_ring" in k for k in names) == want, names
        assert all(torch_cuda.equal(a, b) for a, b in zip(got, other)), tile
    assert all(float(a.float().abs().sum()) > 0 for a in got)


# Weight gradients of short sums and many tiles (weight_gradient_kernel): experts of no row, of one slab, of several and a ragged one, tiles that end
# inside, and both sides of the lines (256 expected rows; more than four 128 x 128 tiles per CU)
SHORT_SUMS = [
    (wl.small_config("dw_short_one_slab", 900, 320, 320, 13, 10, 9, "bf16", "relu", skew=True, seed=401), 2),
    (wl.small_config("dw_short_f16_ragged", 4000, 576, 704, 8, 5, 200, "f16", "relu", skew=True, seed=402), 2),
    (wl.small_config("dw_short_256_rows", 30 * 256, 768, 704, 6, 5, 300, "bf16", "relu", skew=True, seed=403), 2),
    (wl.small_config("dw_short_257_rows", 30 * 256 + 1, 768, 704, 6, 5, 300, "bf16", "relu", skew=True, seed=404), 0),
    (wl.small_config("dw_short_four_tiles_per_cu", 2000, 256, 1024, 8, 8, 40, "bf16", "relu", skew=True, seed=405), 0),
]


@pytest.mark.parametrize("cfg,short", SHORT_SUMS, ids=lambda c: getattr(c, "name", str(c)))
def test_weight_gradients_of_short_sums(torch_cuda, cfg, short, monkeypatch):
    """The bits of the ring and of the two-stage kernel (a row's products are added in the order of k by all three)."""
    from paper_2212_05191_amd.runner import GpuLayer
    monkeypatch.delenv("SMILE_TGEMM_TILE", raising=False)
    layer = GpuLayer(cfg)
    try:
        layer.forward()
        layer.prepare_backward(wl.gen_output_grad(cfg))
        layer.bwd.dw1.fill_(-77)
        layer.bwd.dw2.fill_(-77)
        names = _launched(layer, layer.backward)
        assert sum("weight_gradient_kernel" in k for k in names) == short, names
        got = [layer.bwd.dw1.cpu(), layer.bwd.dw2.cpu()]
    finally:
        layer.close()
    for tile in ("0", "1"):
        other, _ = _weight_gradients(torch_cuda, cfg, tile, monkeypatch)
        assert all(torch_cuda.equal(a, b) for a, b in zip(got, other)), tile


# Both sides of the lines between the 64-row tiles and the others in pick_forward_tile (which tile: test_tile_choice_host.py)
PICK_TILE_EDGES = [
    wl.small_config("up_320_small_tiles", 700, 192, 640, 8, 4, 40, "bf16", "gelu", skew=True, seed=411),
    wl.small_config("up_330_small_tiles_f16", 700, 192, 704, 10, 3, 40, "f16", "relu", skew=True, seed=412),
    wl.small_config("up_one_round_of_64x128", 3000, 192, 1024, 4, 4, 256, "bf16", "gelu", skew=True, seed=413),
    wl.small_config("up_beyond_one_round_of_64x128", 3000, 192, 1024, 4, 4, 257, "bf16", "relu", skew=True, seed=414),
    wl.small_config("up_one_slab_ragged", 5000, 64, 320, 8, 5, 150, "bf16", "gelu", skew=True, seed=415),
    wl.small_config("up_two_slabs_f16", 5000, 128, 320, 8, 5, 150, "f16", "gelu", skew=True, seed=416),
    wl.small_config("down_512_of_600_live", 16 * 250, 512, 1024, 4, 4, 300, "bf16", "relu", skew=True, seed=417),
    wl.small_config("down_narrow_768", 32 * 250, 192, 768, 8, 4, 300, "bf16", "relu", skew=True, seed=418),
    wl.small_config("down_second_round", 16 * 210, 960, 1920, 4, 4, 210, "bf16", "relu", skew=True, seed=419),
    wl.small_config("down_64_rows_768", 600, 384, 768, 16, 8, 64, "bf16", "relu", skew=True, seed=420),
    wl.small_config("down_64_rows_896", 600, 448, 896, 16, 8, 64, "f16", "relu", skew=True, seed=421),
    wl.small_config("down_64_rows_64x128", 500, 1024, 1088, 8, 7, 60, "bf16", "relu", skew=True, seed=423),
    wl.small_config("down_narrow_many_experts", 72 * 120, 256, 320, 9, 8, 192, "bf16", "relu", skew=True, seed=424),
    wl.small_config("down_65_experts", 65 * 90, 448, 512, 13, 5, 90, "f16", "relu", skew=True, seed=425),
    wl.small_config("up_one_slab_192_columns", 5000, 64, 192, 8, 5, 150, "bf16", "gelu", skew=True, seed=426),
    wl.small_config("down_290_rows_of_many_experts", 104 * 290, 768, 832, 13, 8, 290, "bf16", "relu", skew=True, seed=422),
]


@pytest.mark.parametrize("cfg", PICK_TILE_EDGES, ids=lambda c: c.name)
def test_tiles_of_medium_products(torch_cuda, cfg, monkeypatch):
    """The library's tiles give the bits of 128 x 192 tiles in every form of the forward pass (every tile adds in the order of k), and are those that
    the choice by sizes names: a ring kernel or a two-stage one for each of the two products."""
    from paper_2212_05191_amd.runner import GpuLayer
    from test_tile_choice_host import forward_tile
    tiles = [forward_tile(way, cfg.N, cfg.T, cfg.capacity, cfg.d_model, cfg.d_ff) for way in ("up", "down")]
    want = ["grouped_gemm_" + ("ring" if 1 <= t <= 4 else "nt") + "_kernel" for t in tiles]
    got = {}
    for tile in ("0", ""):
        monkeypatch.setenv("SMILE_FFN_TILE", tile) if tile else monkeypatch.delenv("SMILE_FFN_TILE", raising=False)
        layer, _, _ = _layer_with_biases(cfg)
        try:
            names = [k for k in _launched(layer, layer.forward_fused) if "gemm" in k]
            assert tile or names == want, (tiles, names)
            got[tile, "y"] = layer.buf.y.cpu()
            layer.enable_saved_activations()
            layer.h_save.zero_(), layer.pre_save.zero_()
            layer.buf.y.fill_(-7)
            layer.forward()
            torch_cuda.cuda.synchronize()
            got[tile, "y_saving"], got[tile, "h"], got[tile, "pre"] = layer.buf.y.cpu(), layer.h_save.cpu(), layer.pre_save.cpu()
        finally:
            layer.close()
    assert torch_cuda.equal(got["", "y"], got["", "y_saving"]) and float(got["", "y"].float().abs().sum()) > 0
    for k in ("y", "y_saving", "h", "pre"):
        assert torch_cuda.equal(got["0", k], got["", k]), k
