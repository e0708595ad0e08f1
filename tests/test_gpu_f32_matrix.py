"""GPU parity of the fp32 path's matrix kernels at the sizes where they can go wrong: edges of query, key and GEMM
tiles, rows without 16-byte alignment, key ranges that start off a 16-byte boundary, key ranges cut over blocks, all
against the CPU oracle at the fp32 tolerance (every element within 1e-4 of the oracle, relative to max(1, |ref|))."""
import pytest
import torch

from harness import check, gpu_stage, oracle_stage, to_dev, to_np
from paper_2505_21070_amd import synth

pytestmark = pytest.mark.gpu


def pair(tag, block, cache, first, **over):
    """Neighbour block, hand-over of `cache` frames from `first` on, current block; every visible result compared."""
    cfg, w, text, _ = synth.make_case("small_f32", seed=31, strong_gate=True, n_blocks=0, n_layers=1, **over)
    g = gpu_stage(cfg, w, text, max_block_frames=block, max_cache_frames=max(cache, 1), debug_taps=1, max_abs_frames=64)
    o = oracle_stage(cfg, w, text)
    gen = torch.Generator().manual_seed(32)
    xa, xb = synth.make_block(cfg, block, gen), synth.make_block(cfg, block, gen)
    g.forward(to_dev(xa, cfg), block, block, 625.0); o.forward(xa.numpy(), block, block, 625.0)
    g.cache_update(first, cache); o.cache_update(first, cache)
    taps = []
    y, r = g.forward(to_dev(xb, cfg), block, 0, 500.0), o.forward(xb.numpy(), block, 0, 500.0, taps)
    check(f"{tag}/attn", to_np(g.peek("attn")), taps[-1]["attn"], "f32")
    check(f"{tag}/cross_attn", to_np(g.peek("cross_attn")), taps[-1]["cattn"], "f32")
    check(f"{tag}/x_out", to_np(y), r, "f32")


# tokens per frame x frames: one query; one past a 32-query tile; keys starting at 1, 2, 3 mod 4 (the cache's odd frames);
# one key group of the four without a tile
@pytest.mark.parametrize("heads,hd", [(2, 64), (2, 128)])
@pytest.mark.parametrize("tok_h,tok_w,block,cache,first", [(1, 1, 1, 0, 0), (3, 11, 1, 1, 0), (5, 7, 3, 1, 1), (7, 9, 3, 2, 1),
                                                           (6, 11, 2, 1, 1), (31, 1, 1, 0, 0)])
def test_attention_tile_edges(heads, hd, tok_h, tok_w, block, cache, first):
    pair(f"edge{tok_h}x{tok_w}x{block}/{hd}", block, cache, first, dim=heads * hd, n_heads=heads, head_dim=hd, tok_h=tok_h, tok_w=tok_w,
         text_len=16 if tok_h * tok_w == 1 else 33)


# at least 64 (head, 128-query) blocks and 32 key tiles: key ranges cut over blocks, joined by the merge kernel; the FFN
# width is what bounds the scratch for it (1024: never cut, 4096: two ranges and more)
@pytest.mark.parametrize("ffn", [1024, 4096])
@pytest.mark.parametrize("heads,hd", [(12, 64), (11, 128)])
def test_attention_cut_key_ranges(heads, hd, ffn):
    pair(f"cut{hd}/{ffn}", 6, 3, 1, dim=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=ffn, tok_h=9, tok_w=13, text_len=37)


# widths that are no multiple of 4 (no 16-byte rows), shorter than a k-tile, one past a tile, on the 32 x 32 shape with K dealt
# over the wavefronts; and enough output tiles for the 128 x 128 shape, ragged in both directions, with and without
# 16-byte rows (the 64 x 64 shape runs above and below)
@pytest.mark.parametrize("tok_h,tok_w,ffn,text_dim", [(7, 9, 641, 37), (5, 13, 644, 36), (8, 8, 5, 1), (13, 5, 65, 260),
                                                      (31, 33, 16381, 64), (31, 33, 16380, 64)])
def test_gemm_edges(tok_h, tok_w, ffn, text_dim):
    pair(f"gemm{tok_h}x{tok_w}/{ffn}/{text_dim}", 1, 1, 0, dim=128, n_heads=2, head_dim=64, tok_h=tok_h, tok_w=tok_w, ffn_dim=ffn,
         text_dim=text_dim, text_len=19)


def test_gemm_middle_tiles_every_epilogue():
    pair("gemm64", 1, 1, 0, dim=1408, n_heads=11, head_dim=128, tok_h=23, tok_w=33, ffn_dim=1444, text_dim=1408, text_len=19)


@pytest.mark.parametrize("heads,hd", [(2, 64), (2, 128)])
@pytest.mark.parametrize("tok_h,tok_w,kept", [(7, 9, 0), (7, 9, 1), (3, 11, 1), (3, 11, 2)])
def test_non_finite_keys_beside_the_live_range(heads, hd, tok_h, tok_w, kept):
    """Frames of the last block that are not cached leave NaN keys and values in front of and behind the live range, inside
    its first 16-byte piece and its last key tile.  None of it may reach the result: the same bits as after a
    neighbour of finite values."""
    cfg, w, text, _ = synth.make_case("small_f32", seed=33, strong_gate=True, n_blocks=0, n_layers=1, dim=heads * hd, n_heads=heads,
                                      head_dim=hd, tok_h=tok_h, tok_w=tok_w)
    tok, gen = tok_h * tok_w, torch.Generator().manual_seed(34)
    xa, xb = synth.make_block(cfg, 3, gen), synth.make_block(cfg, 1, gen)
    outs = []
    for bad in (False, True):
        if bad:
            other = torch.ones(3 * tok, dtype=torch.bool)
            other[kept * tok:(kept + 1) * tok] = False
            xa = torch.where(other[:, None], torch.full_like(xa, float("nan")), xa)
        g = gpu_stage(cfg, w, text, max_block_frames=3, max_cache_frames=1, debug_taps=1, max_abs_frames=64)
        g.forward(to_dev(xa, cfg), 3, 3, 625.0)
        g.cache_update(kept, 1)
        y = g.forward(to_dev(xb, cfg), 1, 0, 500.0)
        assert torch.isfinite(y).all()
        outs.append((y.clone(), g.peek("attn")))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
