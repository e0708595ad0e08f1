"""GPU parity of the fp32 attention that shares key tiles in LDS (at least 64 (head, 128-query) blocks and 32 key tiles): last
query tile of a block with 6 or 1 live queries or none, key ranges one and two past a tile, key ranges that start 1, 2
and 3 keys off a 16-byte boundary, cut (wide FFN: scratch for it) and whole, against the CPU oracle at the fp32
tolerance; and NaN keys in front of and behind the live range, which must not change a bit."""
import ctypes as C

import pytest
import torch

from harness import gpu_stage, to_dev, to_np
from paper_2505_21070_amd import binding, synth
from test_gpu_f32_matrix import pair

_ranges = binding._lib.dp_attn_f32_ranges
_ranges.argtypes = [C.c_int64] * 3 + [C.c_int32] * 2 + [C.c_int64]
_ranges.restype = C.c_int32


def ranges(tok, block, cache, first, heads, hd, ffn, most=None):
    """Key ranges that a block's self-attention is cut into (0: the kernel for few queries or keys)."""
    rows = ((most or block) * tok + 255) // 256 * 256
    return _ranges(block * tok, (block + cache) * tok, first * tok, heads, hd, rows * ffn)


@pytest.mark.parametrize("heads,hd,ffn,cut", [(13, 64, 256, 1), (13, 64, 4096, 4), (13, 128, 256, 1), (13, 128, 4096, 2)])
def test_shapes_take_this_kernel(heads, hd, ffn, cut):
    for tok, block, cache, first in ((171, 3, 3, 0), (113, 6, 4, 1), (113, 6, 4, 2), (115, 6, 4, 1)):
        assert ranges(tok, block, cache, first, heads, hd, ffn) == cut
    assert ranges(113, 5, 4, 1, heads, hd, 640, most=6) == 1                       # the non-finite keys' test
    # tests/test_gpu_f32_matrix.py
    assert [ranges(117, 6, 3, 1, 12, 64, f) for f in (1024, 4096)] == [1, 4]
    assert [ranges(117, 6, 3, 1, 11, 128, f) for f in (1024, 4096)] == [1, 2]
    for h, w, block, cache, first in ((1, 1, 1, 0, 0), (3, 11, 1, 1, 0), (5, 7, 3, 1, 1), (7, 9, 3, 2, 1), (6, 11, 2, 1, 1), (31, 1, 1, 0, 0)):
        assert ranges(h * w, block, cache, first, 2, hd, 640) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("ffn", [256, 4096])
@pytest.mark.parametrize("heads,hd", [(13, 64), (13, 128)])
@pytest.mark.parametrize("tok_w,block,cache,first", [(171, 3, 3, 0), (113, 6, 4, 1), (113, 6, 4, 2), (115, 6, 4, 1)])
def test_tiles_edges(heads, hd, tok_w, block, cache, first, ffn):
    pair(f"tiles{tok_w}x{block}/{hd}/{ffn}", block, cache, first, dim=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=ffn,
         tok_h=1, tok_w=tok_w, text_len=9)


@pytest.mark.gpu
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
