"""The bf16 attention kernel's block shapes at the edges of their tiles: cross-attention against a float64 softmax over the very
q, K, V that the kernel read (peeked from the library), at the text lengths and query counts where a shape can go wrong."""
import ctypes as C

import numpy as np
import pytest

from harness import check
from paper_2505_21070_amd import binding, synth
from test_gpu_stage import T_CUR, gpu_stage, to_dev, to_np

_route = binding._lib.dp_attn_bf16_route
_route.argtypes = [C.c_int64] * 2 + [C.c_int32] * 2 + [C.POINTER(C.c_int32)]
_route.restype = None

# heads, head_dim, token grid, text tokens: (queries of a block, key groups, key ranges of the last round's blocks)
FEW, PAIRS, GROUPS = (32, 8, 1), (128, 1, 1), (128, 2, 1)
CASES = {(2, 128, (2, 4, 1), n): FEW for n in (1, 31, 32, 33, 255, 256, 257)}     # 8 queries: one to nine 32-key tiles
CASES.update({
    (2, 64, (6, 12, 3), 40): FEW, (2, 64, (6, 12, 3), 300): FEW,                  # 216 queries, 2 and 10 tiles
    (4, 128, (8, 10, 25), 1900): FEW,                                             # 252 blocks of 32 queries, 60 tiles
    (16, 64, (8, 9, 14), 70): FEW,                                                # 512 blocks of 32
    (8, 128, (8, 15, 10), 100): PAIRS, (8, 128, (8, 15, 10), 512): PAIRS,         # 1200 queries: four wavefronts, two blocks to a CU
    (16, 64, (8, 13, 10), 33): PAIRS, (16, 64, (8, 13, 10), 200): PAIRS,          # 1040 queries
    (16, 64, (8, 13, 40), 1024): (128, 1, 2),                                     # 4160: the last 16 blocks cut into key ranges
    (8, 128, (8, 15, 10), 1100): (128, 2, 2), (16, 64, (8, 13, 10), 1100): GROUPS,
})


def route(S, L, heads, hd):
    out = (C.c_int32 * 3)()
    _route(S, L, heads, hd, out)
    return tuple(out)


@pytest.mark.parametrize("heads,hd,grid,text_len", CASES)
def test_shapes_take_this_kernel(heads, hd, grid, text_len):
    assert route(grid[0] * grid[1] * grid[2], text_len, heads, hd) == CASES[heads, hd, grid, text_len]


@pytest.mark.gpu
@pytest.mark.parametrize("peaked", [False, True], ids=["plain", "peaked"])
@pytest.mark.parametrize("heads,hd,grid,text_len", CASES)
def test_cross_attention_shapes(monkeypatch, heads, hd, grid, text_len, peaked):
    """peaked: large q/k gains, so that logits of later keys exceed those of the first by more than a fixed reference can hold"""
    monkeypatch.setitem(synth.CONFIGS, "shape", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=128,
                                                     text_len=text_len, text_dim=heads * hd, tok_h=grid[0], tok_w=grid[1],
                                                     block_frames=grid[2], cache_frames=1))
    cfg, w, text, blocks = synth.make_case("shape", seed=5, strong_gate=True)
    if peaked:
        for k in ("cgq", "cgk"):
            w["layers"][0][k] = synth.round_to(w["layers"][0][k] * 12.0, "bf16")
    g = gpu_stage(cfg, w, text, max_abs_frames=64)
    g.forward(to_dev(blocks[1], cfg), cfg["block_frames"], 0, T_CUR)
    q, k, v = (to_np(g.peek(n, 0)) for n in ("q", "text_k", "text_v"))            # q: already multiplied by log2(e)/sqrt(d)
    ref = np.zeros_like(q)
    for h in range(heads):
        sl = slice(h * hd, (h + 1) * hd)
        s2 = q[:, sl] @ k[:, sl].T
        p = np.exp2(s2 - s2.max(1, keepdims=True))
        ref[:, sl] = (p / p.sum(1, keepdims=True)) @ v[:, sl]
    check("shape/cross_attn", to_np(g.peek("cross_attn", 0)), ref, "bf16")


@pytest.mark.gpu
@pytest.mark.parametrize("heads,hd,grid,text_len,at", [(2, 128, (6, 12, 3), 33, slice(32, 33)), (2, 64, (6, 12, 3), 300, slice(64, 96))])
def test_key_tiles_of_infinite_scores(monkeypatch, heads, hd, grid, text_len, at):
    """A whole 32-key tile (a ragged one of one key; a full one) whose scores are -inf weighs nothing.  Keys `at` are infinite in one
    channel, zero in the others' text rows; queries on its negative side are compared (the others' scores are +inf)."""
    c, j, D = 5, 7, heads * hd
    assert route(grid[0] * grid[1] * grid[2], text_len, heads, hd) == FEW
    monkeypatch.setitem(synth.CONFIGS, "shape", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=D, n_heads=heads, head_dim=hd, ffn_dim=128,
                                                     text_len=text_len, text_dim=D, tok_h=grid[0], tok_w=grid[1], block_frames=grid[2], cache_frames=1))
    cfg, w, text, blocks = synth.make_case("shape", seed=6, strong_gate=True)
    lw = w["layers"][0]
    lw["cwk"][:, c] = 0.0
    lw["cwk"][j, c], lw["cbk"][c], lw["cgk"][c], lw["cgq"][c] = 1.0, 0.0, 2.0 ** 125, 1.0
    text[:, j] = 0.0
    text[at, j] = 32.0
    g = gpu_stage(cfg, w, text, max_abs_frames=64)
    g.forward(to_dev(blocks[1], cfg), cfg["block_frames"], 0, T_CUR)
    q, k, v, got = (to_np(g.peek(n, 0)) for n in ("q", "text_k", "text_v", "cross_attn"))
    assert np.isinf(k[at, c]).all() and np.isfinite(np.delete(k, np.r_[at], 0)).all()
    rows, sl = q[:, c] < 0, slice(0, hd)                                          # channel c is the first head's
    s2 = q[rows, sl] @ k[:, sl].T
    p = np.exp2(s2 - s2.max(1, keepdims=True))
    assert rows.any() and (p[:, at] == 0).all()
    check("shape/infinite", got[rows, sl], (p / p.sum(1, keepdims=True)) @ v[:, sl], "bf16")
