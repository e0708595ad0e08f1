"""GPU parity of the fp32 attention that shares key tiles in LDS (at least 64 (head, 128-query) blocks and 32 key tiles): last
query tile of a block with 6 or 1 live queries or none, key ranges one and two past a tile, key ranges that start 1, 2
and 3 keys off a 16-byte boundary, cut (wide FFN: scratch for it) and whole, against the CPU oracle at the fp32
tolerance; and NaN keys in front of and behind the live range, which must not change a bit."""
import pytest
import torch

from harness import gpu_stage, to_dev, to_np
from paper_2505_21070_amd import synth
from test_gpu_f32_matrix import pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ffn", [256, 4096])
@pytest.mark.parametrize("heads,hd", [(13, 64), (13, 128)])
@pytest.mark.parametrize("tok_w,block,cache,first", [(171, 3, 3, 0), (113, 6, 4, 1), (113, 6, 4, 2), (115, 6, 4, 1)])
def test_tiles_edges(heads, hd, tok_w, block, cache, first, ffn):
    pair(f"tiles{tok_w}x{block}/{hd}/{ffn}", block, cache, first, dim=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=ffn,
         tok_h=1, tok_w=tok_w, text_len=9)


@pytest.mark.parametrize("heads,hd", [(13, 64), (13, 128)])
def test_non_finite_keys_beside_the_live_range(heads, hd):
    cfg, w, text, _ = synth.make_case("small_f32", seed=35, strong_gate=True, n_blocks=0, n_layers=1, dim=heads * hd, n_heads=heads,
                                      head_dim=hd, tok_h=1, tok_w=113)
    tok, gen = 113, torch.Generator().manual_seed(36)
    xa, xb = synth.make_block(cfg, 6, gen), synth.make_block(cfg, 5, gen)
    outs = []
    for bad in (False, True):
        if bad:
            other = torch.ones(6 * tok, dtype=torch.bool)
            other[tok:5 * tok] = False
            xa = torch.where(other[:, None], torch.full_like(xa, float("nan")), xa)
        g = gpu_stage(cfg, w, text, max_block_frames=6, max_cache_frames=4, max_abs_frames=64)
        g.forward(to_dev(xa, cfg), 6, 6, 625.0)
        g.cache_update(1, 4)
        y = g.forward(to_dev(xb, cfg), 5, 0, 500.0)
        outs.append(to_np(y))
    assert (outs[0] == outs[1]).all()
