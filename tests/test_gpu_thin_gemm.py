"""The bf16 GEMM's 32 x 64 tiles with k-tiles dealt to the wavefronts, through the stage, against the CPU oracle: fewer k-tiles
than wavefronts, exactly as many, more; rows that fill no tile; the plain store, GELU, residual and per-head epilogues."""
import pytest

from paper_2505_21070_amd import synth
from test_gemm_routes import products
from test_gpu_stage import run_pair

# (dim, heads, head_dim, ffn, tok_h, tok_w, frames): k-tiles of 64 are dim / 64 and ffn / 64
SHAPES = [
    (448, 7, 64, 576, 5, 8, 1),        # 7 and 9 k-tiles, 40 rows, separate norm and rotation kernels
    (512, 4, 128, 1088, 2, 4, 2),      # 8 and 17, 16 rows, per-head epilogue
    (768, 12, 64, 1024, 3, 8, 4),      # 12 and 16, 96 rows, heads of 64
]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_shapes_take_this_tile(shape):
    p = products(dict(dim=shape[0], ffn_dim=shape[3], tok_h=shape[4], tok_w=shape[5], block_frames=shape[6]))
    assert {k[1:] for k in p.values()} == {(32, 64, 1)}


@pytest.mark.gpu
@pytest.mark.parametrize("dim,heads,hd,ffn,tok_h,tok_w,frames", SHAPES)
def test_thin_tiles(monkeypatch, dim, heads, hd, ffn, tok_h, tok_w, frames):
    monkeypatch.setitem(synth.CONFIGS, "thin", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                    text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=frames, cache_frames=1))
    run_pair("thin", 3, True, "later")
