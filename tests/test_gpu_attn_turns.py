"""The bf16 attention kernel whose wavefronts take turns (many keys, heads of 128) and the one with a pinned order, in blocks of eight
wavefronts at the edges of their tiles: cross-attention against a float64 softmax over the
very q, K, V that the kernel read, with one and with two key groups, whole and with key ranges that are merged; last tiles of one
key, one short of a tile and a whole one; queries that fill no block; overflow of the fixed reference; tiles of -inf scores."""
import ctypes as C

import numpy as np
import pytest

from harness import check
from paper_2505_21070_amd import binding, synth
from test_gpu_attn_shapes import route
from test_gpu_stage import T_CUR, gpu_stage, to_dev, to_np

# heads, head_dim, token grid, text tokens: (queries of a block, key groups, key ranges of the last round's blocks)
CASES = {(16, 128, (8, 15, 17), n): (256, 1, 1) for n in (513, 575, 576)}          # 2040 queries: 128 blocks, 9 tiles
CASES.update({(16, 128, (8, 15, 17), n): (256, 1, 2) for n in (1025, 1088)})       # 17 tiles: 8 and 9
CASES.update({(32, 64, (8, 15, 17), n): (256, 1, 1) for n in (1025, 1087, 1088)})  # 256 blocks
CASES.update({(8, 128, (8, 15, 10), n): (128, 2, 1) for n in (513, 576, 639, 640)})         # 1200 queries: 5 + 4 and 5 + 5 tiles
CASES.update({(16, 64, (8, 13, 10), n): (128, 2, 1) for n in (1025, 1151, 1152)})  # 1040 queries: 9 + 8, 9 + 9
# with enough keys for turns
TURNS = {(32, 128, (8, 15, 17), n): (256, 1, 1) for n in (2241, 2304)}             # 2040 queries: 256 blocks, 36 tiles
TURNS.update({(16, 128, (8, 15, 17), n): (256, 1, 2) for n in (5057, 5119, 5184)}) # 128 blocks: 80 and 81 tiles, 40 and 41 in a range
TURNS.update({(13, 128, (8, 15, 10), n): (128, 2, 1) for n in (2369, 2432, 2495, 2496)})    # 1200 queries: 19 + 19 and 20 + 19 tiles
TURNS.update({(10, 128, (8, 163, 1), n): (128, 2, 2) for n in (4033, 4160)})       # 1304 queries: 64 and 65 tiles, 16 + 16 and 17 + 16 in a range
CASES.update(TURNS)

_turns = binding._lib.dp_attn_bf16_turns
_turns.argtypes, _turns.restype = [C.c_int64] * 2 + [C.c_int32] * 2, C.c_int


def layer(monkeypatch, heads, hd, grid, text_len, seed):
    monkeypatch.setitem(synth.CONFIGS, "shape", dict(synth.CONFIGS["tiny_bf16"], n_layers=1, dim=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=128,
                                                     text_len=text_len, text_dim=heads * hd, tok_h=grid[0], tok_w=grid[1],
                                                     block_frames=grid[2], cache_frames=1))
    return synth.make_case("shape", seed=seed, strong_gate=True)


def operands(cfg, w, text, blocks):
    g = gpu_stage(cfg, w, text, max_abs_frames=64)
    g.forward(to_dev(blocks[1], cfg), cfg["block_frames"], 0, T_CUR)
    return (to_np(g.peek(n, 0)) for n in ("q", "text_k", "text_v", "cross_attn"))   # q: already multiplied by log2(e)/sqrt(d)


def softmax2(s2):
    p = np.exp2(s2 - s2.max(1, keepdims=True))
    return p / p.sum(1, keepdims=True)


@pytest.mark.parametrize("heads,hd,grid,text_len", CASES)
def test_shapes_take_this_kernel(heads, hd, grid, text_len):
    S = grid[0] * grid[1] * grid[2]
    assert route(S, text_len, heads, hd) == CASES[heads, hd, grid, text_len]
    assert bool(_turns(S, text_len, heads, hd)) == ((heads, hd, grid, text_len) in TURNS)


@pytest.mark.gpu
@pytest.mark.parametrize("peaked", [False, True], ids=["plain", "peaked"])
@pytest.mark.parametrize("heads,hd,grid,text_len", CASES)
def test_turns(monkeypatch, heads, hd, grid, text_len, peaked):
    """peaked: large q/k gains, so that logits of later keys exceed those of the first by more than a fixed reference can hold"""
    cfg, w, text, blocks = layer(monkeypatch, heads, hd, grid, text_len, 5)
    if peaked:
        for k in ("cgq", "cgk"):
            w["layers"][0][k] = synth.round_to(w["layers"][0][k] * 12.0, "bf16")
    q, k, v, got = operands(cfg, w, text, blocks)
    ref = np.concatenate([softmax2(q[:, i:i + hd] @ k[:, i:i + hd].T) @ v[:, i:i + hd] for i in range(0, heads * hd, hd)], axis=1)
    check("turns/cross_attn", got, ref, "bf16")


@pytest.mark.gpu
@pytest.mark.parametrize("heads,hd,grid,text_len,at", [(16, 128, (8, 15, 17), 575, slice(512, 575)), (16, 128, (8, 15, 17), 576, slice(64, 128)),
                                                       (8, 128, (8, 15, 10), 640, slice(256, 320)), (32, 64, (8, 15, 17), 1025, slice(1024, 1025))])
def test_tiles_of_infinite_scores(monkeypatch, heads, hd, grid, text_len, at):
    """A whole key tile (the ragged one that the walk starts with; one inside it; the one a key group starts with) whose scores are
    -inf weighs nothing.  Keys `at` are infinite in one channel, zero in the others' text rows; queries on its negative side are
    compared (the others' scores are +inf)."""
    c, j = 5, 7
    cfg, w, text, blocks = layer(monkeypatch, heads, hd, grid, text_len, 6)
    lw = w["layers"][0]
    lw["cwk"][:, c] = 0.0
    lw["cwk"][j, c], lw["cbk"][c], lw["cgk"][c], lw["cgq"][c] = 1.0, 0.0, 2.0 ** 125, 1.0
    text[:, j] = 0.0
    text[at, j] = 32.0
    q, k, v, got = operands(cfg, w, text, blocks)
    assert np.isinf(k[at, c]).all() and np.isfinite(np.delete(k, np.r_[at], 0)).all()
    rows, sl = q[:, c] < 0, slice(0, hd)                                          # channel c is the first head's
    p = softmax2(q[rows, sl] @ k[:, sl].T)
    assert rows.any() and (p[:, at] == 0).all()
    check("turns/infinite", got[rows, sl], p @ v[:, sl], "bf16")


# heads, head_dim, token grid, text tokens, keys at -inf, head that has them: (queries of a block, key groups, key ranges of the last
# round's blocks)
RANGES = [((8, 128, (8, 15, 10), 1100, np.r_[0:576], 0), (128, 2, 2)),         # all keys of a range, in both key groups
          ((16, 64, (8, 13, 40), 1024, np.r_[0:512], 15), (128, 1, 2)),        # the same in blocks of four wavefronts; a head of the last round
          ((8, 128, (8, 15, 10), 512, np.r_[0:32, 448:480], 0), (128, 1, 1)),  # the keys that the one and the other pass start with
          ((16, 64, (8, 15, 17), 600, np.r_[0:32, 576:600], 0), (256, 1, 1)),
          ((8, 128, (8, 15, 10), 640, np.r_[0:32, 288:352, 608:640], 0), (128, 2, 1)),
          ((16, 128, (8, 15, 17), 5184, np.r_[0:2560], 0), (256, 1, 2)),       # in turns: a whole range,
          ((10, 128, (8, 163, 1), 4096, np.r_[0:2048], 0), (128, 2, 2)),       # both groups of one,
          ((13, 128, (8, 15, 10), 2496, np.r_[0:32, 1248:1312, 2432:2464], 0), (128, 2, 1))]     # where each group and pass starts


@pytest.mark.gpu
@pytest.mark.parametrize("case,taken", RANGES)
def test_ranges_of_infinite_scores(monkeypatch, case, taken):
    """A whole key range of a cut work id whose scores are -inf weighs nothing, nor do such scores where both passes start (the fixed
    reference fails there, and the online softmax has none yet).  Keys and queries as in the test above."""
    heads, hd, grid, text_len, at, head = case
    assert route(grid[0] * grid[1] * grid[2], text_len, heads, hd) == taken
    c, j = head * hd + 5, 7
    cfg, w, text, blocks = layer(monkeypatch, heads, hd, grid, text_len, 6)
    lw = w["layers"][0]
    lw["cwk"][:, c] = 0.0
    lw["cwk"][j, c], lw["cbk"][c], lw["cgk"][c], lw["cgq"][c] = 1.0, 0.0, 2.0 ** 125, 1.0
    text[:, j] = 0.0
    text[at, j] = 32.0
    q, k, v, got = operands(cfg, w, text, blocks)
    assert np.isinf(k[at, c]).all() and np.isfinite(np.delete(k, at, 0)).all()
    rows, sl = q[:, c] < 0, slice(head * hd, (head + 1) * hd)
    p = softmax2(q[rows, sl] @ k[:, sl].T)
    assert rows.any() and (p[:, at] == 0).all()
    check("turns/infinite", got[rows, sl], p @ v[:, sl], "bf16")
