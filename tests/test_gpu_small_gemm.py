"""The bf16 GEMM's tiles through the stage, against the CPU oracle: fewer k-tiles than a ring has stages, exactly as many, one
more; rows and columns that fill no tile; the GELU, residual and per-head epilogues on each tile that has them, the plain
store of the projections (separate norm and rotation kernels behind it) and of the text products; the residual product with K
cut into ranges.  tests/test_gemm_routes.py asserts which kernels these shapes reach."""
import pytest

from harness import check, to_np
from paper_2505_21070_amd import synth
from test_gpu_stage import run_pair

pytestmark = pytest.mark.gpu

# (dim, heads, head_dim, ffn, tok_h, tok_w, frames): k-tiles of 64 are dim / 64 and ffn / 64
SHAPES = [
    (64, 1, 64, 64, 2, 4, 1),              # one k-tile, one tile
    (128, 1, 128, 192, 3, 8, 3),           # 2 and 3 k-tiles, 72 rows
    (256, 4, 64, 320, 5, 8, 3),            # 4 and 5, per-head epilogue with 64-column tiles, 120 rows
    (512, 4, 128, 1344, 8, 17, 9),         # 1224 rows: two and three blocks to a CU, 21 k-tiles
    (1024, 8, 128, 4096, 9, 16, 7),        # 1008 rows: 128 x 128 tiles for the FFN's first product
    (1152, 9, 128, 1152, 8, 47, 5),        # 1880 rows: three stages of 64 x 64 in every product but q|k|v, none cut
    (1152, 9, 128, 1152, 8, 49, 7),        # 2744 rows: 128 x 128 tiles there
    (1280, 10, 128, 1280, 17, 16, 4),      # 1088 rows, q|k|v on 128 x 128 tiles (270 of them fit no round: the large ones)
    (768, 6, 128, 2112, 16, 17, 5),        # 1360 rows, q|k|v on 128 x 128 tiles
    (1536, 12, 128, 1536, 8, 113, 3),      # 2712 rows: 160 x 256 tiles in every product but q|k|v, the last of them ragged
    (128, 1, 128, 2432, 14, 36, 8),        # 4032 rows: the large 192-row tile with the GELU epilogue
    (256, 2, 128, 2048, 2, 4, 1),          # 8 rows, K cut into 8 ranges of 64 x 64 tiles
    (640, 5, 128, 6144, 24, 67, 1),        # 1608 rows, 7 ranges of 160 x 256 tiles
    (640, 5, 128, 8192, 24, 67, 1),        # 8 ranges of 256 x 256 tiles
    # q | k | v as plain rows, normalised and rotated by separate kernels
    (448, 7, 64, 448, 40, 60, 1),          # 2400 rows of 128 x 128 tiles, the narrowest rows
    (1600, 25, 64, 1600, 8, 44, 2),        # 704 rows of 128 x 128 tiles, cross-q per head
    (1664, 13, 128, 1664, 24, 35, 1),      # 840 rows of large tiles, cross-q per head; the only call size of its stage
    (3136, 49, 64, 512, 8, 21, 2),         # 336 rows of 128 x 128 tiles, the widest rows
    (1088, 17, 64, 1088, 47, 64, 1),       # 3008 rows, cross-q too on 128 x 128 tiles; a stage none of whose calls store per head
]
# the same with many text tokens, whose keys and values are plain stores
TEXT_SHAPES = [
    (1152, 9, 128, 1152, 8, 47, 2, 1000),  # 288 tiles of 64 x 64: two to a CU
    (1152, 9, 128, 1152, 8, 47, 2, 1880),  # 540: three to a CU
    (1408, 11, 128, 1408, 8, 47, 2, 1880), # 165 tiles of 128 x 128
]


@pytest.mark.parametrize("dim,heads,hd,ffn,tok_h,tok_w,frames", SHAPES)
def test_small_tiles(monkeypatch, dim, heads, hd, ffn, tok_h, tok_w, frames):
    monkeypatch.setitem(synth.CONFIGS, "ring", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                    text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=frames, cache_frames=1))
    run_pair("ring", 3, True, "later")


@pytest.mark.parametrize("dim,heads,hd,ffn,tok_h,tok_w,frames", [(128, 1, 128, 192, 3, 8, 3), (512, 4, 128, 1344, 8, 17, 9), (1024, 8, 128, 4096, 9, 16, 7),
                                                                 (768, 6, 128, 2112, 16, 17, 5)])
def test_keys_are_rounded_once(monkeypatch, dim, heads, hd, ffn, tok_h, tok_w, frames):
    """Per-head stores of 64- and 128-column tiles (one shape for each) leave the keys unrounded until their row scale is
    known.  A rounding to bf16 is 1.66e-3 (relative, root mean square, for evenly spread mantissas): with the LayerNorm's output
    the first layer's keys are sqrt(2) of that from 64 bits, 2.35e-3, and would be sqrt(3), 2.87e-3, if rounded twice."""
    monkeypatch.setitem(synth.CONFIGS, "keys", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                    text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=frames, cache_frames=1))
    rep = {}
    run_pair("keys", 4, True, "later", rep)
    assert rep["keys/k"]["rel_l2"] < 2.6e-3 and rep["keys/cache_k0"]["rel_l2"] < 2.6e-3


@pytest.mark.parametrize("dim,heads,hd,ffn,tok_h,tok_w,frames,text_len", TEXT_SHAPES)
def test_text_products(monkeypatch, dim, heads, hd, ffn, tok_h, tok_w, frames, text_len):
    monkeypatch.setitem(synth.CONFIGS, "text", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                    text_len=text_len, text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=frames,
                                                    cache_frames=1))
    g, o, _, _ = run_pair("text", 3, True, "later")
    check("text/v", to_np(g.peek("text_v", 0)), o.text_v[0], "bf16")
