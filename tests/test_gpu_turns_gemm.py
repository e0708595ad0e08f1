"""The bf16 GEMM's tiles whose wavefronts take turns (128 x 256 columns, 160 x 256 with transposed sections, K cut over 128 x 128
and 128 x 256 tiles) through the stage, against the CPU oracle, at row counts that leave the last tile ragged."""
import pytest

from paper_2505_21070_amd import synth
from test_gemm_routes import config, products
from test_gpu_stage import run_pair

# (dim, heads, head_dim, ffn, tok_h, tok_w, frames): {product: (epilogue, rows, columns, stages of the tile)}
SHAPES = {
    (1408, 11, 128, 2816, 8, 41, 5): {"qkv": ("store", 128, 256, 3), "ffn1": ("gelu", 128, 256, 3)},      # 1640 rows
    (768, 6, 128, 6144, 8, 47, 5): {"qkv": ("heads", 128, 256, 3), "ffn2": ("cut", 128, 256, 3)},         # 1880 rows
    (1024, 8, 128, 2048, 8, 75, 5): {"qkv": ("heads", 160, 256, 3)},                                       # 3000 rows
    (1536, 12, 128, 1536, 8, 113, 3): {"o": ("resid", 128, 256, 3)},                                       # 2712 rows
    (640, 10, 64, 1280, 8, 53, 4): {"qkv": ("heads", 128, 128, 4)},                                        # 1696 rows
    (768, 6, 128, 6144, 8, 59, 1): {"ffn2": ("cut", 128, 128, 4)},                                         # 472 rows
}


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_shapes_take_these_tiles(shape):
    p = products(config(*shape))
    assert {k: p[k] for k in SHAPES[shape]} == SHAPES[shape]


@pytest.mark.gpu
@pytest.mark.parametrize("dim,heads,hd,ffn,tok_h,tok_w,frames", SHAPES)
def test_turns(monkeypatch, dim, heads, hd, ffn, tok_h, tok_w, frames):
    monkeypatch.setitem(synth.CONFIGS, "turns", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                     text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=frames, cache_frames=1))
    run_pair("turns", 3, True, "later")
