"""bfloat16 activations at sizes around every change of launch shape (small workgroups, tiles shrunk to the number of
compute units): the values are looked up per bit pattern, so every shape gives the bits of the plain one (pieces
per lane fixed by the knobs), with guard words behind every output."""
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


@pytest.mark.parametrize("kind", ["erf", "silu"])
@pytest.mark.parametrize("n", SIZES)
def test_every_shape_gives_the_same_bits(n, kind):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x, dy = ((3 * torch.randn(n, generator=g, device="cuda")).to(torch.bfloat16) for _ in range(2))

    def both():
        (y, y_end), (mask, mask_end) = guarded(n, torch.bfloat16), guarded(B.mask_words(n), torch.int32)
        dx, dx_end = guarded(n, torch.bfloat16)
        if kind == "silu":
            B.tempo_silu_fwd(x, y, mask)
            B.tempo_silu_bwd(dy, y, mask, dx)
        else:
            B.tempo_gelu_fwd(x, y, mask, kind)
            B.tempo_gelu_bwd(dy, y, mask, dx, kind)
        assert all((end == 7).all() for end in (y_end, mask_end, dx_end))
        return y, mask, dx

    got = both()
    old = B.tempo_get_launch_param(0), B.tempo_get_launch_param(1)
    try:
        B.tempo_set_launch_param(0, 1)
        B.tempo_set_launch_param(1, 1)
        want = both()
    finally:
        B.tempo_set_launch_param(0, old[0])
        B.tempo_set_launch_param(1, old[1])
    assert all(torch.equal(a, b) for a, b in zip(got, want))
