"""The choice of a tile for an expert GEMM (host functions of sizes alone), on both sides of its lines.  No kernel is launched here."""
import ctypes as C

import pytest

from paper_2212_05191_amd import binding as B


class _Tuning(C.Structure):
    _fields_ = [(k, C.c_int) for k in ("ffn_tile", "tgemm_tile", "persist", "router_grad_mfma", "cus")]


class _RingArgs(C.Structure):
    _fields_ = [(k, C.c_void_p) for k in ("x", "w", "y", "y2", "aux", "bias", "rows_valid", "k_valid", "x_rows", "y_rows", "y_tok", "gate")] + \
        [(k, C.c_int) for k in ("N", "Mrows", "Nout", "K", "ldx", "ldw")] + [(k, C.c_longlong) for k in ("sx", "sw", "sy")] + \
        [("col_tiles", C.c_int), ("backwards", C.c_bool)]


T128X192, T128X256, T256X192, T128X128 = range(4)

# experts, expected rows, rows of a buffer, d_model, d_ff
CASES = [
    # many rounds: what the widths and the fill of the buffers ask for
    ("down", 128, 256, 256, 768, 3072, T256X192),      # full buffers of two row tiles
    ("down", 128, 200, 256, 768, 3072, T128X256),      # room in them
    ("down", 128, 287, 287, 768, 3072, T256X192),      # a second row tile of 31 rows, of 32 and of 80
    ("down", 128, 288, 288, 768, 3072, T128X256),
    ("down", 128, 336, 336, 768, 3072, T128X256),
    ("down", 128, 337, 337, 768, 3072, T256X192),
    ("down", 128, 384, 384, 768, 3072, T256X192),
    ("dxe", 128, 320, 320, 768, 3072, T128X256),
    ("down", 64, 300, 300, 1536, 6144, T128X256),
    ("down", 128, 320, 320, 960, 3840, T256X192),      # four tiles of 256 columns against five of 192
    ("down", 128, 320, 320, 576, 2304, T256X192),
    ("dxe", 128, 256, 256, 768, 3072, T256X192),
    ("down", 64, 256, 320, 1024, 4096, T128X128),      # 192-wide tiles pad 1024 columns by an eighth
    ("dxe", 200, 250, 256, 1024, 4096, T128X256),
    ("up", 64, 256, 320, 1024, 4096, T128X192),
    ("dpre", 16, 512, 1024, 1600, 6400, T128X192),
    ("up", 300, 200, 200, 64, 256, T128X128),          # 384 columns of tiles for 256
    ("dW", 64, 200, 256, 768, 3072, T128X192),
    # few rounds: the last one decides
    ("down", 16, 512, 512, 768, 3072, T128X192),       # one 128 x 192 tile per CU
    ("dxe", 16, 512, 1024, 1600, 6400, T128X256),      # two rounds of 128 x 256, more than one of the others
    ("down", 16, 144, 216, 1600, 6400, T128X256),      # nearly every expert has two row tiles: 224 of 256 columns, 288 of 192
    ("dxe", 64, 240, 300, 320, 1280, T128X128),        # 384 of 128 columns in one round; 256 columns would pad 320 to 512
    ("dxe", 64, 300, 600, 384, 1152, T128X192),        # three row tiles: 384 of 192 columns in one round, 576 of 128 in two
    ("dpre", 16, 128, 128, 1024, 4096, T128X128),      # 512: one round of two on a CU
    ("up", 64, 96, 120, 256, 1024, T128X128),
    ("up", 70, 96, 120, 256, 1024, T128X192),          # 560: three tiles on some CUs; 420 of 192 columns in one round
    ("down", 21, 144, 216, 1600, 6400, T128X192),      # one round against a second one of 128 x 256 for a tenth of the tiles
    ("down", 64, 208, 416, 640, 1280, T128X128),
    ("dW", 4, 128, 256, 256, 1024, T128X128),
    # the smallest and the largest sizes that the estimate meets
    ("down", 1, 1, 128, 192, 256, T128X128),
    ("up", 4096, 1, 65, 64, 4096, T128X192),
    ("up", 1, 2**31 - 1, 2**31 - 1, 64, 256, T128X128),
    ("down", 1, 2**30, 2**31 - 1, 192, 2048, T128X256),
]


@pytest.mark.parametrize("product,N,rows,cap,d,F,want", CASES, ids=lambda v: str(v))
def test_ring_tile(product, N, rows, cap, d, F, want):
    pick = B.load()._ZN5smile14pick_ring_tileERKNS_6TuningERKNS_8RingArgsEib
    pick.restype, pick.argtypes = C.c_int, [C.c_void_p, C.c_void_p, C.c_int, C.c_bool]
    mrows, nout, k = {"up": (cap, F, d), "down": (cap, d, F), "dpre": (cap, F, d), "dxe": (cap, d, F), "dW": (d, F, cap)}[product]
    a = _RingArgs(N=N, Mrows=mrows, Nout=nout, K=k, ldx=k, ldw=k, k_valid=8 if product == "dW" else None)
    tune = _Tuning(-1, -1, -1, -1, 256)
    got = pick(C.byref(tune), C.byref(a), min(rows, mrows) if product != "dW" else mrows, product in ("dpre", "dxe", "dW"))
    assert got == want


# tiles of pick_forward_tile; the ring shapes are those above, one up
T64X256, T64X64_4, T64X128, T64X64 = 5, 7, 8, 9

# direction, experts, tokens, rows of a buffer, d_model, d_ff
FORWARD_CASES = [
    # up: 64 x 64 tiles, at most one on a CU and eleven slabs or more: four stages
    ("up", 4, 96, 24, 960, 4096, T64X64_4),
    ("up", 4, 96, 24, 704, 4096, T64X64_4),
    ("up", 4, 96, 24, 640, 4096, T64X64),
    ("up", 4, 96, 24, 960, 4160, T64X64),
    ("up", 16, 240, 15, 256, 1024, T64X64),
    ("up", 12, 96, 8, 1024, 4096, T64X64),              # 768
    ("up", 13, 96, 8, 1024, 4096, T64X128),
    # up: contractions of one slab, and of two up to 4096 tiles, unless 64 x 128 tiles pad the columns
    ("up", 16, 16 * 4063, 4063, 64, 256, T64X128),
    ("up", 16, 16 * 4063, 4063, 64, 192, 0),
    ("up", 16, 8192, 512, 128, 512, T64X128),
    ("up", 32, 32 * 1024, 1024, 128, 512, T64X128),      # 4096
    ("up", 32, 32 * 1025, 1025, 128, 512, 0),
    # up: one round of two of 64 x 128 per CU, 512 of them
    ("up", 16, 3000, 256, 192, 1024, T64X128),
    ("up", 16, 3000, 257, 192, 1024, 1 + T128X128),
    # down: 512 live 64 x 64 tiles, four stages
    ("down", 16, 4000, 300, 512, 1024, T64X64_4),           # 640 in the buffers, 512 live
    ("down", 16, 4800, 300, 512, 1024, 1 + T128X128),       # 640 live
    # down: to 1024 over the buffers, the ring, of up to 64 experts
    ("down", 16, 16 * 209, 209, 960, 3840, 1 + T128X128),
    ("down", 64, 64 * 100, 100, 512, 1024, 1 + T128X128),
    ("down", 65, 65 * 90, 90, 448, 1024, T64X64_4),
    # down: narrow layers, three stages: 768 over the buffers, and of more experts 768 live
    ("down", 21, 21 * 644, 644, 192, 576, T64X64),
    ("down", 24, 24 * 644, 644, 192, 576, 1 + T128X192),
    ("down", 72, 72 * 120, 192, 256, 1024, T64X64),        # 864, 576 live
    ("down", 160, 160 * 88, 177, 128, 512, T64X64),        # 960, 640 live
    ("down", 84, 84 * 150, 190, 256, 1024, T64X64_4),      # 1008, 1008 live
    # down: buffers of at most 64 rows
    ("down", 128, 128 * 20, 26, 384, 1536, T64X64),
    ("down", 128, 256, 2, 384, 1536, T64X64_4),
    ("down", 40, 40 * 20, 26, 960, 3840, T64X64_4),
    ("down", 54, 54 * 50, 56, 1024, 4096, T64X128),
    ("down", 60, 60 * 4, 4, 1024, 4096, T64X64_4),
    ("down", 72, 72 * 20, 26, 768, 3072, T64X64_4),
    ("down", 60, 60 * 22, 22, 1088, 3264, T64X64_4),
    ("down", 65, 65 * 20, 26, 1024, 4096, T64X128),        # 1040
    ("down", 128, 128 * 20, 26, 1024, 4096, T64X128),      # 2048
    ("down", 129, 129 * 20, 26, 1024, 4096, T64X256),
]


def forward_tile(way, N, T, cap, d, F):
    pick = B.load()._ZN5smile17pick_forward_tileERKNS_6TuningEiiiiib
    pick.restype, pick.argtypes = C.c_int, [C.c_void_p] + [C.c_int] * 5 + [C.c_bool]
    tune = _Tuning(-1, -1, -1, -1, 256)
    return pick(C.byref(tune), N, cap, *((F, d) if way == "up" else (d, F)), T, way == "up")


@pytest.mark.parametrize("way,N,T,cap,d,F,want", FORWARD_CASES, ids=lambda v: str(v))
def test_forward_tile(way, N, T, cap, d, F, want):
    assert forward_tile(way, N, T, cap, d, F) == want
