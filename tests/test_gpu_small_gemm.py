"""The bf16 GEMM's small tiles (a ring of loads through LDS) through the stage, against the CPU oracle: fewer k-tiles than
ring stages, exactly as many, one more; rows and columns that fill no tile; every epilogue at each of the three shapes;
with and without the per-head epilogue (dim % 256);
and the residual product with K cut into ranges, at each tile."""
import pytest

from paper_2505_21070_amd import synth
from test_gpu_stage import run_pair

pytestmark = pytest.mark.gpu


# (dim, heads, head_dim, ffn, tokens): k-tiles of 64 are dim / 64 and ffn / 64
@pytest.mark.parametrize("dim,heads,hd,ffn,tok_h,tok_w,frames", [
    (64, 1, 64, 64, 2, 4, 1),              # one k-tile, one tile
    (128, 1, 128, 192, 3, 8, 3),           # 2 and 3 k-tiles, 72 rows
    (256, 4, 64, 320, 5, 8, 3),            # 4 and 5, per-head epilogue with 64-column tiles, 120 rows
    (512, 4, 128, 1344, 8, 17, 9),         # 1224 rows: two and three blocks to a CU, 21 k-tiles
    (1024, 8, 128, 4096, 9, 16, 7),        # 1008 rows: 128 x 128 tiles for the FFN's first product
    (1280, 10, 128, 1280, 17, 16, 4),      # 1088 rows, q|k|v on 128 x 128 tiles (270 of them fit no round: the large ones)
    (768, 6, 128, 2112, 16, 17, 5),        # 1360 rows, q|k|v on 128 x 128 tiles
    (128, 1, 128, 2432, 14, 36, 8),        # 4032 rows: the large 192-row tile with the GELU epilogue
    (256, 2, 128, 2048, 2, 4, 1),          # 8 rows, K cut into 8 ranges of 64 x 64 tiles
    (640, 5, 128, 6144, 24, 67, 1),        # 1608 rows, 7 ranges of 160 x 256 tiles
    (640, 5, 128, 8192, 24, 67, 1)])       # 8 ranges of 256 x 256 tiles
def test_small_tiles(monkeypatch, dim, heads, hd, ffn, tok_h, tok_w, frames):
    monkeypatch.setitem(synth.CONFIGS, "ring", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                    text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=frames, cache_frames=1))
    run_pair("ring", 3, True, "later")
