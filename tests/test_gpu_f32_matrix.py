"""GPU parity of the fp32 path's matrix kernels at the sizes where they can go wrong: edges of query, key and GEMM
tiles, rows without 16-byte alignment, key ranges that start off a 16-byte boundary, key ranges cut over blocks, all
against the CPU oracle at the fp32 tolerance (every element within 1e-4 of the oracle, relative to max(1, |ref|))."""
import ctypes as C

import pytest
import torch

from harness import check, gpu_stage, oracle_stage, to_dev, to_np
from paper_2505_21070_amd import binding, synth

pytestmark = pytest.mark.gpu

_tile, _run = binding._lib.dp_gemm_f32_tile, binding._lib.dp_gemm_f32_run
_tile.argtypes = [C.c_int64] * 2 + [C.c_int32]
_tile.restype = C.c_int32
_run.argtypes = [C.c_void_p, C.c_int64] * 2 + [C.c_void_p] + [C.c_int64] * 3 + [C.c_int32] + [C.c_void_p, C.c_int64] * 2 + [C.c_void_p] * 2
_run.restype = None
EPI = {"store": 0, "gelu": 1, "resid": 2}


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


# widths that are no multiple of 4 (no 16-byte rows), shorter than a k-tile, one past a tile, on the 32 x 32 tiles with K dealt
# over the wavefronts; and FFNs so wide that their first product takes 128 x 128 tiles (no 16-byte rows) or the ring's of 128 rows
@pytest.mark.parametrize("tok_h,tok_w,ffn,text_dim", [(7, 9, 641, 37), (5, 13, 644, 36), (8, 8, 5, 1), (13, 5, 65, 260),
                                                      (31, 33, 16381, 64), (31, 33, 16380, 64)])
def test_gemm_edges(tok_h, tok_w, ffn, text_dim):
    pair(f"gemm{tok_h}x{tok_w}/{ffn}/{text_dim}", 1, 1, 0, dim=128, n_heads=2, head_dim=64, tok_h=tok_h, tok_w=tok_w, ffn_dim=ffn,
         text_dim=text_dim, text_len=19)


# what the ring does not take: every tile and epilogue, K in steps of 4 with 16-byte rows and neither, one product by itself.
# 1056 tiles of 128 x 128, 256 of 64 x 64, 15 of 32 x 32, ragged in every direction
@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("epi", ["store", "gelu", "resid"])
@pytest.mark.parametrize("tile,M,N,K", [(128, 4100, 4000, 36), (64, 1000, 1020, 100), (32, 70, 132, 68)])
def test_tiles_beside_the_ring(tile, M, N, K, epi, aligned):
    if not aligned:
        N, K = N - 3, K + 1
    assert _tile(M, N, 1) == tile
    gen = torch.Generator(device="cuda").manual_seed(tile)
    A, W, b, gate = (torch.randn(s, generator=gen, device="cuda") for s in ((M, K), (K, N), (N,), (N,)))
    ld = N + 4                                         # the columns beyond N and a row beyond M stay as they are
    x = torch.randn(M + 1, ld, generator=gen, device="cuda")
    got = x.clone()
    out, resid = (None, got.data_ptr()) if epi == "resid" else (got.data_ptr(), None)
    _run(A.data_ptr(), K, W.data_ptr(), N, b.data_ptr(), M, N, K, EPI[epi], out, ld, resid, ld, gate.data_ptr(),
         torch.cuda.current_stream().cuda_stream)
    ref = A.double() @ W.double() + b.double()
    # a sum of K products and the bias, whatever its order; GELU's slope is at most 1.13 and its own arithmetic a few ulp
    bound = (K + 4) * 2.0 ** -24 * (A.abs().double() @ W.abs().double() + b.abs().double())
    if epi == "gelu":
        ref, bound = torch.nn.functional.gelu(ref, approximate="tanh"), 1.13 * bound + 1e-6 * ref.abs()
    if epi == "resid":
        ref, bound = x[:M, :N].double() + gate.double() * ref, gate.abs().double() * bound + 2.0 ** -22 * (x[:M, :N].abs().double() + ref.abs())
    assert ((got[:M, :N].double() - ref).abs() <= bound).all()
    assert torch.equal(got[M], x[M]) and torch.equal(got[:, N:], x[:, N:])


# the FFN's second product on 64 x 64 tiles, the others on the ring's
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
