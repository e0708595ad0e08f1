"""The bf16 GEMM's small tiles (a ring of loads through LDS) through the stage, against the CPU oracle: fewer k-tiles than
ring stages, exactly as many, one more; rows and columns that fill no tile; the plain store, GELU, residual and per-head
epilogues on each of the three rings (64 x 64 in four and in three stages, 128 x 128 in four); the residual product with K
cut into ranges at each tile that does it.  tests/test_gemm_routes.py asserts that these shapes still reach those kernels."""
import pytest

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
]


@pytest.mark.parametrize("dim,heads,hd,ffn,tok_h,tok_w,frames", SHAPES)
def test_small_tiles(monkeypatch, dim, heads, hd, ffn, tok_h, tok_w, frames):
    monkeypatch.setitem(synth.CONFIGS, "ring", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                    text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=frames, cache_frames=1))
    run_pair("ring", 3, True, "later")
