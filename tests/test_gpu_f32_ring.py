"""The fp32 GEMM's tiles in a ring of loads, every row count, through the stage against the CPU oracle at the fp32 tolerance
(every element within 1e-4 of the oracle, relative to max(1, |ref|)); rows that fill no tile."""
import ctypes as C

import pytest

from paper_2505_21070_amd import binding
from test_gpu_f32_matrix import pair

_rows = binding._lib.dp_gemm_f32_rows
_rows.argtypes = [C.c_int64] * 3 + [C.c_int32]
_rows.restype = C.c_int32

# (tok_h, tok_w, frames, dim, ffn): (rows of the tile, epilogue) that this shape is here for
SHAPES = {
    (11, 31, 3, 640, 1024): {(48, "resid"), (48, "store"), (64, "gelu"), (64, "store")},
    (7, 11, 3, 128, 3072): {(48, "gelu")},
    (17, 31, 4, 384, 1536): {(64, "resid"), (80, "store"), (112, "gelu")},
    (29, 41, 3, 768, 768): {(96, "gelu"), (96, "resid"), (96, "store"), (128, "store")},
    (11, 31, 3, 128, 4096): {(128, "gelu")},
    (29, 41, 3, 1024, 256): {(112, "resid"), (112, "store")},
    (30, 52, 1, 1536, 256): {(80, "resid")},
    (16, 35, 1, 128, 4480): {(80, "gelu")},
    (31, 33, 4, 1024, 256): {(128, "resid")},
}


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_shapes_take_these_tiles(shape):
    h, w, f, D, F = shape
    M = h * w * f
    took = {(_rows(M, D, D, 3), "store"), (_rows(M, D, D, 1), "store"), (_rows(M, F, D, 1), "gelu"), (_rows(M, D, D, 1), "resid"), (_rows(M, D, F, 1), "resid")}
    assert SHAPES[shape] <= took


@pytest.mark.gpu
@pytest.mark.parametrize("tok_h,tok_w,frames,dim,ffn", SHAPES)
def test_ring_tiles(tok_h, tok_w, frames, dim, ffn):
    pair(f"ring{tok_h}x{tok_w}x{frames}/{dim}/{ffn}", frames, 0, 0, dim=dim, n_heads=dim // 128, head_dim=128, tok_h=tok_h, tok_w=tok_w, ffn_dim=ffn,
         text_dim=dim, text_len=19)
