"""GPU parity: skiparse_permute / skiparse_unpermute through the C ABI against the oracle, byte for byte."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu

CASES = [  # B, heads, D, T, H, W, s, torch dtype
    (1, 2, 64, 2, 8, 8, 2, torch.float32),      # the tiny workload's grid, fp32 rows of 512 B
    (2, 3, 128, 3, 8, 12, 2, torch.bfloat16),
    (1, 5, 128, 2, 9, 18, 3, torch.bfloat16),   # s = 3
    (3, 1, 64, 1, 16, 32, 4, torch.bfloat16),   # s = 4, short rows (128 B)
    (2, 40, 128, 1, 4, 8, 2, torch.bfloat16),   # 10 KiB rows as at the 768P shape
    (2, 2, 64, 2, 3, 5, 1, torch.bfloat16),     # s = 1: plain copy
    (1, 7, 128, 2, 8, 8, 2, torch.uint8),       # one-byte elements, 896-byte rows (ragged tail of 16-byte chunks)
]


def _random_bits(shape, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    nbytes = int(np.prod(shape)) * torch.empty((), dtype=dtype).element_size()
    raw = torch.randint(0, 256, (nbytes,), generator=g, dtype=torch.uint8)
    return raw.view(dtype).reshape(shape)


@pytest.mark.parametrize("B,heads,D,T,H,W,s,dtype", CASES)
@pytest.mark.parametrize("pattern", ["token", "group"])
def test_permute_roundtrip_bit_exact(B, heads, D, T, H, W, s, dtype, pattern):
    import paper_2605_28691_amd as sk

    if pattern == "group" and (H % (s * s) or W % (s * s)):
        pytest.skip("group-wise needs multiples of s^2")
    x = _random_bits((B, T * H * W, heads, D), dtype, seed=B * 100 + s)
    xb = x.view(torch.uint8).reshape(B, T * H * W, -1).numpy()
    want = oracle.permute(xb, T, H, W, s, pattern)
    xd = x.cuda()
    yd = sk.skiparse_permute(xd, T, H, W, s, pattern)
    got = yd.cpu().view(torch.uint8).reshape(want.shape).numpy()
    assert np.array_equal(got, want)
    back = sk.skiparse_unpermute(yd, T, H, W, s, pattern)
    assert torch.equal(back.cpu().view(torch.uint8), x.view(torch.uint8))
    # unpermute on its own, from the oracle's permuted bytes
    yo = torch.from_numpy(want).view(dtype).reshape(yd.shape).cuda()
    assert torch.equal(sk.skiparse_unpermute(yo, T, H, W, s, pattern).cpu().view(torch.uint8), x.view(torch.uint8))


@pytest.mark.parametrize("name", ["480p", "768p"])
def test_permute_full_size(name):
    """The benchmark shapes in full, every byte compared (bf16 rows of 3 KiB / 10 KiB)."""
    import paper_2605_28691_amd as sk

    w = si.WORKLOADS[name]
    g = torch.Generator().manual_seed(w.seed)
    x = torch.randint(-32768, 32767, (w.B, w.N, w.heads, w.D), generator=g, dtype=torch.int16).view(torch.bfloat16)
    xd = x.cuda()
    for pattern in w.patterns:
        want = oracle.permute(x.view(torch.int16).numpy(), w.T, w.H, w.W, w.s, pattern)
        yd = sk.skiparse_permute(xd, w.T, w.H, w.W, w.s, pattern)
        assert torch.equal(yd.cpu().view(torch.int16), torch.from_numpy(want))
        back = sk.skiparse_unpermute(yd, w.T, w.H, w.W, w.s, pattern)
        assert torch.equal(back.view(torch.int16), xd.view(torch.int16))
        del yd, back, want


def test_permute_does_not_touch_neighbouring_memory():
    """Canary bytes around the destination stay intact."""
    import paper_2605_28691_amd as sk

    B, heads, D, T, H, W, s = 1, 3, 64, 2, 8, 8, 2
    n = B * T * H * W * heads * D
    x = torch.randn((B, T * H * W, heads, D)).to(torch.bfloat16).cuda()
    buf = torch.full((n + 4096,), 7.0, dtype=torch.bfloat16, device="cuda")
    out = buf[2048 : 2048 + n].view(s * s * B, T * H * W // (s * s), heads, D)
    sk.skiparse_permute(x, T, H, W, s, "group", out=out)
    torch.cuda.synchronize()
    assert (buf[:2048] == 7.0).all() and (buf[2048 + n :] == 7.0).all()


@pytest.mark.parametrize("B,heads,D,T,H,W,s,dtype", [
    (1, 2, 64, 2, 8, 8, 2, torch.float32),
    (2, 3, 128, 3, 8, 12, 2, torch.bfloat16),
    (1, 5, 128, 2, 9, 18, 3, torch.bfloat16),
    (3, 1, 64, 1, 16, 32, 4, torch.bfloat16),
    (1, 7, 128, 2, 8, 8, 2, torch.uint8),
    (2, 2, 64, 2, 3, 5, 1, torch.bfloat16),
])
@pytest.mark.parametrize("from_pattern", ["token", "group"])
def test_switch_pattern_bit_exact(B, heads, D, T, H, W, s, dtype, from_pattern):
    """skiparse_switch_pattern against the oracle's composition unpermute(from) -> permute(other), byte for byte."""
    import paper_2605_28691_amd as sk

    y = _random_bits((s * s * B, T * H * W // (s * s), heads, D), dtype, seed=7 * B + s)
    yb = y.view(torch.uint8).reshape(y.shape[0], y.shape[1], -1).numpy()
    want = oracle.switch_pattern(yb, T, H, W, s, from_pattern)
    got = sk.skiparse_switch_pattern(y.cuda(), T, H, W, s, from_pattern)
    assert np.array_equal(got.cpu().view(torch.uint8).reshape(want.shape).numpy(), want)


def test_switch_pattern_768p_equals_two_step():
    """At the 768P shape: the one-step switch equals unpermute + permute done by the library itself (both already checked
    against the oracle), in both directions."""
    import paper_2605_28691_amd as sk

    w = si.WORKLOADS["768p"]
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randint(-32768, 32767, (w.B, w.N, w.heads, w.D), generator=g, dtype=torch.int16, device="cuda").view(torch.bfloat16)
    tsa = sk.skiparse_permute(x, w.T, w.H, w.W, w.s, "token")
    gsa = sk.skiparse_permute(x, w.T, w.H, w.W, w.s, "group")
    assert torch.equal(sk.skiparse_switch_pattern(tsa, w.T, w.H, w.W, w.s, "token").view(torch.int16), gsa.view(torch.int16))
    assert torch.equal(sk.skiparse_switch_pattern(gsa, w.T, w.H, w.W, w.s, "group").view(torch.int16), tsa.view(torch.int16))


# Rows up to 768 B are moved in batches by one wavefront: rows of 1 to 63 chunks of 16 bytes, batches that do not divide the number of
# rows, s = 1 (a copy), all three directions, canaries behind the destination.
@pytest.mark.parametrize("row_bytes", [16, 48, 128, 336, 496, 1008])
@pytest.mark.parametrize("B,T,H,W,s", [(1, 5, 36, 36, 2), (1, 7, 36, 36, 3), (3, 5, 32, 16, 4), (1, 41, 11, 13, 1), (1, 260, 16, 16, 2)])
def test_short_rows_bit_exact(row_bytes, B, T, H, W, s):
    import paper_2605_28691_amd as sk

    x = _random_bits((B, T * H * W, 1, row_bytes), torch.uint8, seed=row_bytes + s)
    xd = x.cuda()
    pad = 4096
    for pattern, other in (("token", "group"), ("group", "token")):
        want = oracle.permute(x.numpy().reshape(B, T * H * W, row_bytes), T, H, W, s, pattern)
        want_other = oracle.permute(x.numpy().reshape(B, T * H * W, row_bytes), T, H, W, s, other)
        shape = (s * s * B, T * H * W // (s * s), 1, row_bytes)
        bufs = [torch.full((x.numel() + pad,), 7, dtype=torch.uint8, device="cuda") for _ in range(3)]
        y, z = (b[: x.numel()].view(shape) for b in bufs[:2])
        back = bufs[2][: x.numel()].view(x.shape)
        sk.skiparse_permute(xd, T, H, W, s, pattern, out=y)
        sk.skiparse_switch_pattern(y, T, H, W, s, pattern, out=z)
        sk.skiparse_unpermute(z, T, H, W, s, other, out=back)
        assert np.array_equal(y.cpu().numpy().reshape(want.shape), want)
        assert np.array_equal(z.cpu().numpy().reshape(want_other.shape), want_other)
        assert torch.equal(back.cpu(), x)
        assert all(bool((b[x.numel() :] == 7).all()) for b in bufs)


@pytest.mark.parametrize("row_bytes", [16, 48])
def test_short_rows_in_full_batches(row_bytes):
    """134,640 rows: batches of 64 rows, one a lane (fewer rows get smaller batches), the last of 48."""
    test_short_rows_bit_exact(row_bytes, 1, 33, 68, 60, 2)


# Longer rows are moved in parts: rows just above a batch, of one part, of one part and a chunk, of parts that are not full, of many.
@pytest.mark.parametrize("row_bytes", [784, 1024, 1040, 1280, 1792, 2304, 10240, 10256])
@pytest.mark.parametrize("B,T,H,W,s", [(1, 2, 16, 16, 2), (2, 1, 18, 9, 3), (1, 3, 5, 7, 1)])
def test_long_rows_bit_exact(row_bytes, B, T, H, W, s):
    test_short_rows_bit_exact(row_bytes, B, T, H, W, s)
