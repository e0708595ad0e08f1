"""The bf16 GEMM's large tiles where only larger models reach them, through the stage, against the CPU oracle on sampled rows (each
attending over all keys): 320-row tiles with the residual epilogue, 192-row tiles with per-head and transposed stores, the last tile
ragged in both."""
import numpy as np
import pytest

from harness import check, gpu_stage, to_dev, to_np
from oracle.stage import OracleStage, token_positions
from paper_2505_21070_amd import synth
from test_gemm_routes import products

# overrides of a configuration: {product: (epilogue, rows, columns, stages of the tile)}
CASES = {
    "resid320": ("tile320_resid_bf16", {}, {"o": ("resid", 320, 256, 2), "ffn2": ("resid", 320, 256, 2)}),
    "heads192": ("tiny_bf16", dict(n_layers=1, dim=768, n_heads=6, head_dim=128, ffn_dim=256, text_dim=768, tok_h=27, tok_w=56, block_frames=3),
                 {"qkv": ("heads", 192, 256, 2)}),      # 4536 rows
}


@pytest.mark.parametrize("name", CASES)
def test_shapes_take_these_tiles(name):
    base, over, want = CASES[name]
    p = products(synth.stage_config(base, **over))
    assert {k: p[k] for k in want} == want


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_large_tiles(name):
    base, over, _ = CASES[name]
    cfg, w, text, blocks = synth.make_case(base, seed=5, strong_gate=True, **over)
    nf, S = cfg["block_frames"], cfg["block_frames"] * cfg["tok_h"] * cfg["tok_w"]
    g = gpu_stage(cfg, w, text, max_abs_frames=8)
    o = OracleStage(cfg, synth.to_numpy(w), text.numpy())
    y = g.forward(to_dev(blocks[0], cfg), nf, 0, 500.0)
    # the first and last rows of the tiles of 192 and 320, and of the block halves inside them
    edge = [r for t in (192, 320) for r in range(0, S, t // 2)]
    rows = np.unique(np.concatenate([edge, np.array(edge[1:]) - 1, [S - 1], np.random.default_rng(7).choice(S, size=40, replace=False)]))
    xin = blocks[0].numpy().astype(np.float64)
    ref, k, v = o.layer(0, xin, o.modulation(500.0), token_positions(nf, 0, cfg["tok_h"], cfg["tok_w"]), None, rows=rows)
    check(f"{name}/k", to_np(g.peek("k", 0)), k, "bf16")
    check(f"{name}/v", to_np(g.peek("v", 0)), v, "bf16")
    xres = to_np(g.peek("x_res", 0))[rows]
    check(f"{name}/x_res", xres, ref, "bf16")
    check(f"{name}/delta", xres - xin[rows], ref - xin[rows], "bf16")
    check(f"{name}/x_out", to_np(y)[rows], ref, "bf16")
