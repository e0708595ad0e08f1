"""The one-kernel patch embedding and output head at the edges of their ranges, against the CPU oracle: token counts that
are no multiple of a block's 16 or 32 tokens, channel groups that do not divide by the eight wavefronts, one to four
fragments of values per token and the first width beyond them (which takes the GEMMs, as does a head wider than 5120),
embeddings of a wide token on both sides of the line between the kernel and the GEMM,
buffers that start off a 16-byte boundary, and outputs that overlap their input."""
import numpy as np
import pytest
import torch

from harness import check, to_dev, to_np
from paper_2505_21070_amd import synth
from test_gpu_ends import make_ends

pytestmark = pytest.mark.gpu


def setup(dim, channels, tok_h, tok_w, frames):
    cfg = synth.stage_config("tiny_bf16", dim=dim, tok_h=tok_h, tok_w=tok_w)
    w = {"stage": synth.make_weights(dict(cfg, n_layers=0), seed=41)["stage"]}
    g, o = make_ends(cfg, w, channels, frames, seed=41)
    gen = torch.Generator().manual_seed(42)
    return cfg, w, g, o, synth.make_latent(cfg, frames, channels, gen), synth.make_block(cfg, frames, gen)


@pytest.mark.parametrize("dim,channels,tok_h,tok_w,frames", [
    (64, 16, 1, 1, 1), (320, 16, 3, 5, 3), (576, 32, 7, 9, 2), (128, 48, 5, 7, 1), (1024, 64, 4, 5, 1), (128, 80, 3, 11, 1),
    (2560, 64, 20, 80, 1), (2560, 64, 20, 82, 1), (768, 64, 20, 51, 6),
    (2176, 16, 3, 5, 1), (3136, 16, 3, 6, 1), (5120, 16, 3, 7, 1), (5184, 16, 2, 3, 1), (128, 16, 64, 65, 1), (128, 16, 63, 65, 1)])
def test_embed_and_head_edges(dim, channels, tok_h, tok_w, frames):
    cfg, _, g, o, lat, tokens = setup(dim, channels, tok_h, tok_w, frames)
    tag = f"{dim}/{channels}/{tok_h}x{tok_w}x{frames}"
    check(f"{tag}/embed", to_np(g.embed(lat.cuda())), o.embed(lat.numpy().astype(np.float64)), "bf16")
    v = g.head(to_dev(tokens, cfg), 437.0, frames)
    check(f"{tag}/head", to_np(v).reshape(-1, channels), o.head(tokens.numpy().astype(np.float64), 437.0, frames).reshape(-1, channels), "bf16")


def test_buffers_off_a_16_byte_boundary():
    from paper_2505_21070_amd import binding as B
    cfg, w, g, _, lat, tokens = setup(320, 16, 3, 5, 3)

    def shifted(t):                                   # the same values one element further on
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)
    x = to_dev(tokens, cfg)
    assert torch.equal(g.embed(shifted(lat.cuda())), g.embed(lat.cuda()))
    ref = g.head(x, 437.0, 3)
    assert torch.equal(g.head(shifted(x), 437.0, 3), ref)
    out = shifted(torch.full_like(ref, float("nan")))
    B.head_forward_static(cfg, g._keep, 16, x, 437.0, 3, out)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_output_may_overlap_the_input(dtype):
    """An output that shares memory with the input: same values as with buffers of their own.  65536 tokens are several
    times what is resident at once, so a kernel that stores while others still have input to load gives other values."""
    from paper_2505_21070_amd import binding as B
    dim, side, frames, channels = 64, 64, 16, 16
    cfg = synth.stage_config("tiny_bf16", dim=dim, tok_h=side, tok_w=side, dtype=dtype)
    w = {"stage": synth.make_weights(dict(cfg, n_layers=0), seed=43)["stage"]}
    g, _ = make_ends(cfg, w, channels, frames, seed=43)
    gen = torch.Generator().manual_seed(44)
    lat, x = synth.make_latent(cfg, frames, channels, gen).cuda(), to_dev(synth.make_block(cfg, frames, gen), cfg)
    stream = torch.cuda.current_stream().cuda_stream
    want_x, want_v = g.embed(lat), g.head(x, 437.0, frames)
    room = max(lat.numel() * 4, x.numel() * x.element_size())

    def place(t, offset):                            # t's values inside a buffer of three times the room
        buf = torch.zeros(3 * room, dtype=torch.uint8, device="cuda")
        at = buf[offset:offset + t.numel() * t.element_size()].view(t.dtype)
        at.copy_(t.reshape(-1))
        return buf, at.view(t.shape)

    for off in (-room // 2, -256, 0, 256, room // 2):       # of the output against the input
        buf, src = place(lat, room)
        out = buf[room + off:room + off + want_x.numel() * want_x.element_size()].view(want_x.dtype).view(want_x.shape)
        B._check(B._lib.dp_embed_forward(g._h, src.data_ptr(), out.data_ptr(), frames, stream), "overlap")
        assert torch.equal(out, want_x), f"embed, output {off} bytes from the latent"
        for static in (False, True):
            buf, src = place(x, room)
            out = buf[room + off:room + off + want_v.numel() * 4].view(torch.float32).view(want_v.shape)
            if static:
                B.head_forward_static(cfg, g._keep, channels, src, 437.0, frames, out)
            else:
                B._check(B._lib.dp_head_forward(g._h, src.data_ptr(), 437.0, out.data_ptr(), frames, stream), "overlap")
            assert torch.equal(out, want_v), f"head (static {static}), output {off} bytes from the tokens"
