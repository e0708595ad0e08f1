"""The sum over the ranges of a cut K, one instance per number of ranges, through the stage's second FFN product against the CPU
oracle."""
import pytest

from paper_2505_21070_amd import synth
from test_gemm_routes import RESID, route
from test_gpu_stage import run_pair

# ranges: (dim, heads, head_dim, ffn, tok_h, tok_w)
SHAPES = {2: (768, 12, 64, 3072, 8, 227), 3: (512, 8, 64, 6144, 8, 65), 4: (512, 8, 64, 4096, 8, 49), 5: (768, 12, 64, 3072, 8, 25),
          6: (512, 8, 64, 4096, 8, 33), 7: (768, 12, 64, 3072, 8, 17), 8: (256, 4, 64, 2048, 8, 5)}


@pytest.mark.parametrize("parts", SHAPES)
def test_shapes_are_cut_so(parts):
    dim, _, _, ffn, tok_h, tok_w = SHAPES[parts]
    assert route(tok_h * tok_w, dim, ffn, RESID)[3] == parts


@pytest.mark.gpu
@pytest.mark.parametrize("parts", SHAPES)
def test_cut(monkeypatch, parts):
    dim, heads, hd, ffn, tok_h, tok_w = SHAPES[parts]
    monkeypatch.setitem(synth.CONFIGS, "cut", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=dim, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                   text_dim=dim, tok_h=tok_h, tok_w=tok_w, block_frames=1, cache_frames=1))
    run_pair("cut", 3, True, "later")
