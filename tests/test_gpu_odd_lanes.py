"""Attention rows on 12, 24, 48, 96, 160, 224, 320 and 384 lanes, several of which lie across the waves of a
workgroup: both ends of every range of pieces per row, ragged and aligned, with row counts that leave
lane groups of the last workgroup without a row, under every mask: a causal forward has shapes of its own.
The checks are those of the ragged rows: the oracle, every source of the keep bits, in place, guard words behind
every output."""
import pytest

from test_gpu_ragged_rows import B, check_attention  # noqa: F401

pytestmark = pytest.mark.gpu

# pieces per row (8 bfloat16 or 4 float32 elements): the first and last of each range, and their neighbours
PIECES = [8, 9, 12, 13, 16, 17, 24, 25, 33, 48, 49, 65, 88, 89, 96, 97, 129, 160, 161, 192, 193, 208, 209, 224, 225,
          257, 320, 321, 352, 353]


@pytest.mark.parametrize("mask", ["none", "padding", "causal"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("cut", [0, 3])     # elements short of whole pieces
@pytest.mark.parametrize("pieces", PIECES)
def test_attention(B, pieces, cut, dt, mask):
    rows = 13 if pieces <= 48 else (5 if pieces <= 224 else 2)
    check_attention(B, pieces * (8 if dt == "bf16" else 4) - cut, rows, dt, mask)
