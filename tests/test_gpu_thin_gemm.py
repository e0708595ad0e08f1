"""The bf16 GEMM's 32 x 64 tiles with k-tiles dealt to the wavefronts, through the stage, against the CPU oracle: fewer k-tiles
than wavefronts, exactly as many, more; rows that fill no tile; the GELU, residual and per-head epilogues, and the plain store
of the text products."""
import pytest

from paper_2505_21070_amd import synth
from test_gemm_routes import config, products
from test_gpu_stage import run_pair

# (dim, heads, head_dim, ffn, tok_h, tok_w, frames): k-tiles of 64 are dim / 64 and ffn / 64
SHAPES = [
    (448, 7, 64, 576, 5, 8, 1),        # 7 and 9 k-tiles, 40 rows, heads of 64
    (512, 4, 128, 1088, 2, 4, 2),      # 8 and 17, 16 rows, heads of 128
    (768, 12, 64, 1024, 3, 8, 4),      # 12 and 16, 96 rows, heads of 64
]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_shapes_take_this_tile(shape):
    names = dict(qkv="heads", cross_q="heads", o="resid", ffn1="gelu", ffn2="resid", text_kv="store")
    assert products(config(*shape)) == {k: (e, 32, 64, 1) for k, e in names.items()}


@pytest.mark.gpu
@pytest.mark.parametrize("dim,heads,hd,ffn,tok_h,tok_w,frames", SHAPES)
def test_thin_tiles(monkeypatch, dim, heads, hd, ffn, tok_h, tok_w, frames):
    monkeypatch.setitem(synth.CONFIGS, "thin", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                    text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=frames, cache_frames=1))
    run_pair("thin", 3, True, "later")
