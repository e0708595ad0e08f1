"""Which kernel of the bf16 GEMM each product of the GPU parity tests takes (host only): the shapes of those tests are chosen
to reach every tile with every epilogue it has, and a change of the dispatch rules must not quietly take them elsewhere.
Whether a projection stores per head is the library's own answer for that call."""
import ctypes as C

import pytest

import test_gpu_small_gemm
from paper_2505_21070_amd import binding, synth

STORE, GELU, RESID, HEADS = range(4)
SCRATCH_FLOATS = 1 << 24                   # of a stage: 64 MiB, or less where 8 partial results are smaller than that

_route = binding._lib.dp_gemm_bf16_route
_route.argtypes = [C.c_int64] * 3 + [C.c_int32] * 2 + [C.c_int64, C.POINTER(C.c_int32)]
_route.restype = None
_heads = binding._lib.dp_gemm_bf16_heads
_heads.argtypes = [C.c_int64] * 2 + [C.c_int32] * 2
_heads.restype = C.c_int32


def route(M, N, K, epi):
    """(rows, columns, LDS stages of the tile, K ranges)"""
    out = (C.c_int32 * 4)()
    _route(M, N, K, epi, 0, SCRATCH_FLOATS, out)
    return tuple(out)


def products(c):
    """{product: (epilogue name, rows, columns, stages)} of one bf16 stage configuration: a forward of its block, and the text
    side at init"""
    S, D, F, Lt, Td = c["block_frames"] * c["tok_h"] * c["tok_w"], c["dim"], c["ffn_dim"], c["text_len"], c["text_dim"]
    names = {STORE: "store", GELU: "gelu", RESID: "resid", HEADS: "heads"}
    out = {}

    def add(name, M, N, K, epi):
        r = route(M, N, K, epi)
        out[name] = (names[epi] if r[3] == 1 else "cut",) + r[:3]
    for name, N in (("qkv", 3 * D), ("cross_q", D)):
        add(name, S, N, D, HEADS if _heads(S, N, D, c["head_dim"]) else STORE)
    add("o", S, D, D, RESID)                                                       # the cross-attention's too
    add("ffn1", S, F, D, GELU)
    add("ffn2", S, D, F, RESID)
    add("text_kv", Lt, D, D, STORE)
    if Td != D:
        add("text1", Lt, D, Td, GELU)
        add("text2", Lt, D, D, STORE)
    return out


def tokens(p):
    """those of a forward"""
    return {k: v for k, v in p.items() if not k.startswith("text")}


def config(dim, heads, hd, ffn, tok_h, tok_w, frames, text_len=16):
    return dict(dim=dim, head_dim=hd, ffn_dim=ffn, tok_h=tok_h, tok_w=tok_w, block_frames=frames, text_len=text_len, text_dim=dim)


def parity_configs():
    """the bf16 configurations that a GPU test compares with the oracle"""
    import test_gpu_thin_gemm
    import test_gpu_turns_gemm
    cfgs = {n: c for n, c in synth.CONFIGS.items() if c["dtype"] == "bf16"}
    for m in (test_gpu_small_gemm, test_gpu_thin_gemm, test_gpu_turns_gemm):
        cfgs.update((str(s), config(*s)) for s in m.SHAPES)
    cfgs.update((str(s), config(*s)) for s in test_gpu_small_gemm.TEXT_SHAPES)
    return cfgs


SMALL = [(32, 64, 1), (64, 64, 4), (64, 64, 3), (128, 128, 4)]
LARGE = [(128, 256, 3), (160, 256, 3), (192, 256, 2), (256, 256, 2), (320, 256, 2)]
NEEDED = ([(e,) + t for t in SMALL + LARGE for e in ("store", "gelu", "resid")] +
          [("heads",) + t for t in SMALL + [(128, 256, 3), (160, 256, 3), (256, 256, 2)]] +
          [("cut",) + t for t in ((64, 64, 4), (128, 128, 4), (128, 256, 3), (160, 256, 3), (256, 256, 2))])


@pytest.mark.parametrize("kernel", NEEDED, ids=lambda k: "-".join(map(str, k)))
def test_every_tile_and_epilogue_is_compared_with_the_oracle(kernel):
    where = [f"{n}/{p}" for n, c in parity_configs().items() for p, k in products(c).items() if k == kernel]
    assert where, f"no parity test reaches {kernel}"


def test_nothing_else_is_reached():
    assert {k for c in parity_configs().values() for k in products(c).values()} == set(NEEDED)


@pytest.mark.parametrize("name,tile,but", [
    ("tile192_bf16", (192, 256, 2), {"qkv": (256, 256, 2)}), ("tile256_bf16", (256, 256, 2), {}),
    ("tile320_bf16", (160, 256, 3), {"qkv": (320, 256, 2), "ffn1": (320, 256, 2)}),
    (str((1152, 9, 128, 1152, 8, 47, 5)), (64, 64, 3), {"qkv": (160, 256, 3)}),
    (str((1152, 9, 128, 1152, 8, 49, 7)), (128, 128, 4), {"qkv": (256, 256, 2)})])
def test_whole_layers_on_one_tile(name, tile, but):
    for p, k in tokens(products(parity_configs()[name])).items():
        assert k[0] != "cut" and k[1:] == but.get(p, tile), (p, k)


# the separate norm, rotation and transposition kernels behind plain stores, at each width of the row kernels' registers:
# (q | k | v, cross-q) of one shape
@pytest.mark.parametrize("name,qkv,cross", [
    ("tile192_bf16", "store", "store"), ("tile256_bf16", "store", "store"), ("tile320_bf16", "store", "store"),
    (str((448, 7, 64, 448, 40, 60, 1)), "store", "heads"), (str((1600, 25, 64, 1600, 8, 44, 2)), "store", "heads"),
    (str((1664, 13, 128, 1664, 24, 35, 1)), "store", "heads"), (str((3136, 49, 64, 512, 8, 21, 2)), "store", "heads"), (str((1088, 17, 64, 1088, 47, 64, 1)), "store", "store"),
    ("dim2176_bf16", "heads", "heads"), ("dim2752_bf16", "heads", "heads"), ("dim6144_bf16", "heads", "heads")])
def test_projections_store(name, qkv, cross):
    p = products(parity_configs()[name])
    assert (p["qkv"][0], p["cross_q"][0]) == (qkv, cross)
