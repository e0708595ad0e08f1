"""A stage whose key buffer is so long that a head's rows of V^T lie more than 2^32 bytes apart: the same block gives what it
gives with a short one, whatever the kernels' offsets can hold.  (17 GB of workspace, of which a call touches a few MB.)"""
import numpy as np
import pytest

from harness import to_dev, to_np
from paper_2505_21070_amd import synth
from test_gpu_attn_shapes import route
from test_gpu_stage import T_CUR, gpu_stage


@pytest.mark.gpu
@pytest.mark.parametrize("heads,hd,cached", [(1, 128, 1 << 24), (1, 64, 1 << 24)])
def test_attention_in_a_long_key_buffer(monkeypatch, heads, hd, cached):
    monkeypatch.setitem(synth.CONFIGS, "shape", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=128,
                                                     text_len=16, text_dim=heads * hd, tok_h=8, tok_w=8, block_frames=33, cache_frames=1))
    cfg, w, text, blocks = synth.make_case("shape", seed=9, strong_gate=True)
    S = 64 * cfg["block_frames"]
    assert route(S, S, heads, hd)[0] > 32 and hd * (2 * cached + S) > 1 << 31   # a larger block, were the buffer shorter
    out = []
    for frames in (1, cached // 64):
        g = gpu_stage(cfg, w, text, max_abs_frames=64, max_cache_frames=frames, debug_taps=1)
        g.forward(to_dev(blocks[0], cfg), cfg["block_frames"], 0, T_CUR)
        out.append(to_np(g.peek("attn", 0)))
    # two orders of the same sums over weights and results that are rounded to bf16 once each: 2^-9 at most in either
    assert np.linalg.norm(out[1] - out[0]) / np.linalg.norm(out[0]) < 4 * 2.0 ** -9
