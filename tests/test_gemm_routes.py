"""Which kernel of the bf16 GEMM each product of the GPU parity tests takes (host only): the shapes of those tests are chosen
to reach every tile with every epilogue it has, and a change of the dispatch rules must not quietly take them elsewhere."""
import ctypes as C

import pytest

from paper_2505_21070_amd import binding, synth
from test_gpu_small_gemm import SHAPES

STORE, GELU, RESID, HEADS = range(4)
SCRATCH_FLOATS = 1 << 24                   # of a stage: 64 MiB, or less where 8 partial results are smaller than that

_route = binding._lib.dp_gemm_bf16_route
_route.argtypes = [C.c_int64] * 3 + [C.c_int32] * 2 + [C.c_int64, C.POINTER(C.c_int32)]
_route.restype = None


def route(M, N, K, epi, transposed=0):
    """(rows, columns, LDS stages of the tile, K ranges)"""
    out = (C.c_int32 * 4)()
    _route(M, N, K, epi, transposed, SCRATCH_FLOATS, out)
    return tuple(out)


def products(c):
    """{product: (epilogue name, rows, columns, stages)} of one bf16 stage configuration"""
    S, D, F = c["block_frames"] * c["tok_h"] * c["tok_w"], c["dim"], c["ffn_dim"]
    proj = HEADS if D % 256 == 0 else STORE
    names = {STORE: "store", GELU: "gelu", RESID: "resid", HEADS: "heads"}
    out = {}
    for name, N, K, epi, t in (("qkv", 3 * D, D, proj, 1), ("cross_q", D, D, proj, 0), ("o", D, D, RESID, 0), ("cross_o", D, D, RESID, 0),
                               ("ffn1", F, D, GELU, 0), ("ffn2", D, F, RESID, 0)):
        r = route(S, N, K, epi, t)
        out[name] = (names[epi] if r[3] == 1 else "cut",) + r[:3]
    return out


def parity_configs():
    """the bf16 configurations that a GPU test compares with the oracle"""
    cfgs = {n: c for n, c in synth.CONFIGS.items() if c["dtype"] == "bf16"}
    for s in SHAPES:
        cfgs[str(s)] = dict(dim=s[0], ffn_dim=s[3], tok_h=s[4], tok_w=s[5], block_frames=s[6])
    return cfgs


RINGS, LARGE = [(64, 64, 4), (64, 64, 3), (128, 128, 4)], [(160, 256, 3), (192, 256, 2), (256, 256, 2), (320, 256, 2)]
NEEDED = ([(e,) + t for t in RINGS + LARGE for e in ("store", "gelu", "resid")] +
          [("heads",) + t for t in RINGS + [(160, 256, 3), (256, 256, 2)]] +
          [("cut",) + t for t in ((64, 64, 4), (160, 256, 3), (256, 256, 2))])


@pytest.mark.parametrize("kernel", NEEDED, ids=lambda k: "-".join(map(str, k)))
def test_every_tile_and_epilogue_is_compared_with_the_oracle(kernel):
    where = [f"{n}/{p}" for n, c in parity_configs().items() for p, k in products(c).items() if k == kernel]
    assert where, f"no parity test reaches {kernel}"


@pytest.mark.parametrize("name,tile,but", [
    ("tile192_bf16", (192, 256, 2), {"qkv": (256, 256, 2)}), ("tile256_bf16", (256, 256, 2), {}),
    ("tile320_bf16", (160, 256, 3), {"qkv": (320, 256, 2), "ffn1": (320, 256, 2)}),
    (str((1152, 9, 128, 1152, 8, 47, 5)), (64, 64, 3), {"qkv": (160, 256, 3)}),
    (str((1152, 9, 128, 1152, 8, 49, 7)), (128, 128, 4), {"qkv": (256, 256, 2)})])
def test_whole_layers_on_one_tile(name, tile, but):
    for p, k in products(parity_configs()[name]).items():
        assert k[0] != "cut" and k[1:] == but.get(p, tile), (p, k)
