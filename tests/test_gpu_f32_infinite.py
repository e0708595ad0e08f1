"""fp32 attention where the scores that a wavefront starts with, or all of a key range, are -inf: they weigh nothing, in the kernel of
few queries or keys and in the one that shares key tiles, whole and cut."""
import numpy as np
import pytest

from harness import check
from paper_2505_21070_amd import synth
from test_gpu_f32_tiles import ranges
from test_gpu_stage import T_CUR, gpu_stage, to_dev, to_np

# heads, head_dim, token grid, text tokens, FFN (scratch), leading keys at -inf: key ranges (0: the kernel of few queries or keys)
CASES = [((2, 64, (8, 8, 1), 100, 256, 32), 0), ((2, 128, (8, 8, 2), 300, 256, 64), 0), ((2, 64, (8, 8, 2), 300, 256, 33), 0),
         ((13, 64, (8, 15, 10), 1100, 256, 32), 1), ((13, 128, (8, 15, 10), 1100, 4096, 544), 2), ((13, 64, (8, 15, 10), 1100, 4096, 352), 3)]


@pytest.mark.parametrize("case,cut", CASES)
def test_shapes_take_this_kernel(case, cut):
    heads, hd, grid, text_len, ffn, _ = case
    assert ranges(1, grid[0] * grid[1] * grid[2], text_len - grid[0] * grid[1] * grid[2], 0, heads, hd, ffn, most=grid[0] * grid[1] * grid[2]) == cut


@pytest.mark.gpu
@pytest.mark.parametrize("case,cut", CASES)
def test_leading_keys_of_infinite_scores(monkeypatch, case, cut):
    """Keys `at` are infinite in one channel, zero in the others' text rows; queries on its negative side are compared (the others'
    scores are +inf)."""
    heads, hd, grid, text_len, ffn, n = case
    c, j, at = 5, 7, slice(0, n)
    monkeypatch.setitem(synth.CONFIGS, "shape", dict(synth.CONFIGS["tiny"], n_layers=1, dim=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=ffn,
                                                     text_len=text_len, text_dim=heads * hd, tok_h=grid[0], tok_w=grid[1], block_frames=grid[2], cache_frames=1))
    cfg, w, text, blocks = synth.make_case("shape", seed=6, strong_gate=True)
    lw = w["layers"][0]
    lw["cwk"][:, c] = 0.0
    lw["cwk"][j, c], lw["cbk"][c], lw["cgk"][c], lw["cgq"][c] = 1.0, 0.0, 2.0 ** 126, 1.0
    text[:, j] = 0.0
    text[at, j] = 32.0
    g = gpu_stage(cfg, w, text, max_abs_frames=64)
    g.forward(to_dev(blocks[1], cfg), cfg["block_frames"], 0, T_CUR)
    q, k, v, got = (to_np(g.peek(what, 0)) for what in ("q", "text_k", "text_v", "cross_attn"))
    assert np.isinf(k[at, c]).all() and np.isfinite(k[n:]).all()
    rows, sl = q[:, c] < 0, slice(0, hd)                                          # channel c is the first head's
    s = q[rows, sl] @ k[:, sl].T / np.sqrt(hd)
    p = np.exp(s - s.max(1, keepdims=True))
    assert rows.any() and (p[:, at] == 0).all()
    check("f32/infinite", got[rows, sl], (p / p.sum(1, keepdims=True)) @ v[:, sl], "f32")
