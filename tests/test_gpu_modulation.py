"""The modulation vectors against the CPU oracle at the fp32 tolerance on both storage types: one slice of the channels, slices of
unequal width, the widest that the first two products share a launch for and the first beyond it, features other than 256 (their own
launch), timesteps at both ends."""
import numpy as np
import pytest

from harness import check, gpu_stage, oracle_stage, to_dev, to_np
from paper_2505_21070_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dim,freq", [(64, 256), (192, 256), (448, 256), (576, 256), (1984, 256), (2048, 256), (2112, 256), (576, 64), (128, 320)])
def test_modulation(dim, freq, dtype):
    cfg, w, text, blocks = synth.make_case("tiny_bf16", seed=9, strong_gate=False, n_layers=2, dim=dim, n_heads=dim // 64, head_dim=64, ffn_dim=64,
                                           text_dim=dim, tok_h=2, tok_w=4, block_frames=1, cache_frames=0, freq_dim=freq, dtype=dtype)
    g, o = gpu_stage(cfg, w, text, max_abs_frames=8), oracle_stage(cfg, w, text)
    for t in (0.0, 437.5, 999.0):
        g.forward(to_dev(blocks[0], cfg), 1, 0, t)
        e0 = o.modulation(t)
        for l in range(2):
            check(f"mod/{dim}/{freq}/{t}", to_np(g.peek("mod", l)), o.layers[l]["mod"] + e0, "f32")
            assert np.linalg.norm(to_np(g.peek("mod", l)) - (o.layers[l]["mod"] + e0)) < 1e-6 * np.linalg.norm(o.layers[l]["mod"] + e0)
