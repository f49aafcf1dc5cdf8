"""Activations at sizes around every change of launch shape (small workgroups, tiles shrunk to the number of compute
units): an element's values do not depend on its neighbours, so every shape gives the bits of the plain one (pieces
and lanes fixed by the knobs), with guard words behind every output."""
import pytest
import torch

from paper_2210_10246_amd import binding as B

pytestmark = pytest.mark.gpu

KI, MI = 1 << 10, 1 << 20
SIZES = [8, 2041, 640 * KI, 640 * KI + 1, 3 * MI, 3 * MI + 517, 4 * MI, 4 * MI + 1, 8 * MI, 8 * MI + 8, 9 * MI + 3, 5003 * 3072,
         16 * MI, 16 * MI + 1, 17 * MI + 511, 24 * MI - 1, 24 * MI] + [2267024 + left for left in range(8)]
GUARD = 64


def guarded(n, dtype):
    buf = torch.full((n + GUARD,), 7, dtype=dtype, device="cuda")
    return buf[:n], buf[n:]


F32_SIZES = [1, 1021, 1024, 1025, 2047, 256 * KI - 1, 256 * KI, 256 * KI + 1, 300 * KI + 3]


@pytest.mark.parametrize("kind", ["erf", "silu"])
@pytest.mark.parametrize("n", SIZES)
def test_every_shape_gives_the_same_bits(n, kind):
    check(n, kind, torch.bfloat16, {0: 1, 1: 1})


@pytest.mark.parametrize("kind", ["erf", "silu"])
@pytest.mark.parametrize("n", F32_SIZES)
def test_every_float32_shape_gives_the_same_bits(n, kind):
    check(n, kind, torch.float32, {0: 4, 1: 4, 15: 64})


def check(n, kind, dtype, plain):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x, dy = ((3 * torch.randn(n, generator=g, device="cuda")).to(dtype) for _ in range(2))

    def both():
        (y, y_end), (mask, mask_end) = guarded(n, dtype), guarded(B.mask_words(n), torch.int32)
        dx, dx_end = guarded(n, dtype)
        if kind == "silu":
            B.tempo_silu_fwd(x, y, mask)
            B.tempo_silu_bwd(dy, y, mask, dx)
        else:
            B.tempo_gelu_fwd(x, y, mask, kind)
            B.tempo_gelu_bwd(dy, y, mask, dx, kind)
        assert all((end == 7).all() for end in (y_end, mask_end, dx_end))
        return y, mask, dx

    got = both()
    old = {key: B.tempo_get_launch_param(key) for key in plain}
    try:
        for key, value in plain.items():
            B.tempo_set_launch_param(key, value)
        want = both()
    finally:
        for key, value in old.items():
            B.tempo_set_launch_param(key, value)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
