"""The output head that streams its tokens (bf16, more than 2048 channels) at 16, 32 and 64 tokens per block, against the CPU oracle:
channel counts that leave the shares uneven, last blocks of one and of all but one token, two groups of 64 output values, rows
whose mean is far from zero (what cancels is the mean, in the statistics and in the product)."""
import numpy as np
import pytest
import torch

from harness import check, to_dev, to_np
from paper_2505_21070_amd import binding as B
from test_gpu_ends_fused import setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("far", [False, True], ids=["plain", "far"])
@pytest.mark.parametrize("dim,channels,tok_h,tok_w,frames", [
    (2112, 16, 1, 1, 1), (2112, 32, 3, 16, 1), (2240, 16, 1, 4096, 1),     # 16 tokens a block: 1, 48 and 4096 of them
    (2112, 16, 1, 4097, 1), (2304, 32, 1, 4095, 1), (2112, 16, 1, 8191, 1),   # 32: one token in the last block, one missing
    (2112, 16, 1, 8193, 1), (2176, 32, 1, 8192, 2)])                       # 64
def test_streamed_head(dim, channels, tok_h, tok_w, frames, far):
    cfg, _, g, o, _, tokens = setup(dim, channels, tok_h, tok_w, frames)
    if far:                                                                # rows at -60 .. 60, still of spread one
        tokens = (tokens.float() + torch.linspace(-60, 60, tokens.shape[0])[:, None]).to(torch.bfloat16).float()
    v = to_np(g.head(to_dev(tokens, cfg), 437.0, frames)).reshape(-1, channels)
    ref = o.head(tokens.numpy().astype(np.float64), 437.0, frames).reshape(-1, channels)
    check(f"{dim}/{channels}/{tok_w}/head", v, ref, "bf16")
    # one rounding to bf16 (of the modulated weights; 2^-9 at most, 1.66e-3 in the mean square) per product, no other
    assert np.linalg.norm(v - ref) / np.linalg.norm(ref) < 2.0 ** -9


@pytest.mark.parametrize("channels,frames", [(16, 1), (32, 3)])
def test_tokens_off_a_16_byte_boundary(channels, frames):
    """One arithmetic serves every pointer: the same bits wherever the tokens start, from the handle and from the static call."""
    cfg, _, g, _, _, tokens = setup(2112, channels, 5, 16, frames)
    x = to_dev(tokens, cfg)
    buf = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
    buf[1:] = x.reshape(-1)
    ref = g.head(x, 437.0, frames)
    assert torch.equal(g.head(buf[1:].view(x.shape), 437.0, frames), ref)
    out = torch.full_like(ref, float("nan"))
    B.head_forward_static(cfg, g._keep, channels, buf[1:].view(x.shape), 437.0, frames, out)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("dim,channels,n", [(2112, 16, 8193), (2112, 32, 8193), (5120, 16, 8200)])
def test_a_token_does_not_depend_on_the_others(dim, channels, n):
    """A whole call and the same tokens fed in parts, at 64, 32 and 16 tokens a block: the same bits."""
    cfg, _, g, _, _, tokens = setup(dim, channels, 1, 1, n)
    x = to_dev(tokens, cfg)
    whole = g.head(x, 437.0, n)
    for first, count in ((0, 4097 if channels == 16 else 2049), (5, 1000), (n - 1, 1)):
        assert torch.equal(g.head(x[first:first + count], 437.0, count), whole[first:first + count])


@pytest.mark.parametrize("channels", [16, 32])
def test_static_call_gives_the_handle_s_bits(channels):
    """The static array holds the modulated weights behind the packed ones and their sums in the first product's place: a large call,
    a smaller one and the large one again, each as the handle has it."""
    cfg, _, g, _, _, tokens = setup(2112, channels, 1, 1, 4100)
    x = to_dev(tokens, cfg)
    for n, t in ((4100, 437.0), (33, 812.0), (4100, 437.0)):
        ref = g.head(x[:n], t, n)
        out = torch.full_like(ref, float("nan"))
        B.head_forward_static(cfg, g._keep, channels, x[:n], t, n, out)
        assert torch.equal(out, ref)


@pytest.mark.parametrize("channels", [16, 32])
def test_streamed_output_may_overlap_the_tokens(channels):
    """An output that shares memory with the tokens, at more blocks than are resident at once: the values of one that does not."""
    n, dim = 16384, 2112
    cfg, _, g, _, _, tokens = setup(dim, channels, 1, 1, n)
    x = to_dev(tokens, cfg)
    want = g.head(x, 437.0, n)
    size, out_size = x.numel() * 2, want.numel() * 4
    for off in (-(out_size // 2), 0, size // 2):             # bytes of the output against the tokens
        buf = torch.zeros(size + 2 * out_size, dtype=torch.uint8, device="cuda")
        src = buf[out_size:out_size + size].view(torch.bfloat16).view(x.shape)
        src.copy_(x)
        out = buf[out_size + off:2 * out_size + off].view(torch.float32).view(want.shape)
        B._check(B._lib.dp_head_forward(g._h, src.data_ptr(), 437.0, out.data_ptr(), n, torch.cuda.current_stream().cuda_stream), "overlap")
        assert torch.equal(out, want), off


@pytest.mark.parametrize("dim,channels,n", [(3136, 64, 5), (3136, 64, 4099), (5120, 48, 17), (5120, 48, 4097)])
def test_wide_heads_of_more_channels(dim, channels, n):
    """More than 32 latent channels stay with the kernel that holds a token in registers: eight and ten groups of channels a
    wavefront, 16 and 32 tokens a block."""
    cfg, _, g, o, _, tokens = setup(dim, channels, 1, 1, n)
    check(f"{dim}/{channels}/{n}/head", to_np(g.head(to_dev(tokens, cfg), 437.0, n)).reshape(-1, channels),
          o.head(tokens.numpy().astype(np.float64), 437.0, n).reshape(-1, channels), "bf16")
