"""Which layer sizes the encoder's own products take, and that a layer without a GPU is made of its parts."""
import ctypes

import pytest
import torch

from paper_2210_10246_amd import binding, modules


class Encoder(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_int64) for n in ("batch", "seq", "hidden", "heads", "ffn")]
                + [(n, ctypes.c_float) for n in ("eps1", "eps2", "p")]
                + [(n, ctypes.c_uint64) for n in ("seed", "offset")] + [("kind", ctypes.c_int)]
                + [("pointer%d" % i, ctypes.c_void_p) for i in range(24)])


@pytest.mark.parametrize("sizes,takes", [
    ((2, 128, 768, 12, 3072), 1), ((1, 1, 4, 1, 4), 1), ((8, 256, 1024, 16, 4096), 1), ((1, 4096, 512, 8, 2048), 1),
    # where the library's products are faster: many rows, long sequences, wide layers, wide heads
    ((16, 256, 1024, 16, 4096), 0), ((1, 7168, 256, 4, 1024), 1), ((1, 8192, 256, 4, 1024), 0), ((1, 16384, 64, 1, 256), 0),
    ((1, 256, 2048, 16, 8192), 1), ((1, 257, 2048, 16, 8192), 0), ((1, 16, 4096, 32, 16384), 1), ((1, 80, 4096, 32, 16384), 0),
    ((1, 1, 5120, 40, 20480), 0), ((1, 1, 8192, 64, 32768), 0), ((1, 1900, 512, 1, 2048), 1), ((1, 4096, 512, 1, 2048), 0),
    ((1, 1024, 1024, 1, 4096), 0), ((1, 1024, 1024, 4, 4096), 1), ((1, 900, 1536, 12, 6144), 1),
    ((2, 128, 66, 3, 256), 0), ((2, 128, 64, 4, 254), 0), ((2, 8, 64, 3, 256), 0),   # no whole pieces, no whole heads
    ((0, 8, 64, 4, 256), 0), ((2, 0, 64, 4, 256), 0),
    ((2, 8, 64, 0, 256), 0), ((2, 8, 64, -4, 256), 0), ((2, 8, 64, 4 - (1 << 32), 256), 0), ((2, 8, 64, 4 + (1 << 32), 256), 0),
    ((-2, -8, 64, 4, 256), 0), ((1 << 62, 4, 64, 4, 256), 0), ((2, 8, 1 << 62, 4, 256), 0),
    ((1, 1, 4, 1, 1 << 23), 1), ((1, 1, 4, 1, 1 << 26), 0), ((1, 1, 80000, 1250, 4), 0),   # few rows, more tiles than are counted
    ((1 << 21, 1, 4, 1, 4), 0), ((1 << 19, 64, 8, 2, 8), 0), ((1, 40000, 64, 1, 64), 0),   # more tiles than are counted
])
def test_sizes_the_one_call_takes(sizes, takes):
    assert binding.load().tempo_encoder_takes(ctypes.byref(Encoder(*sizes))) == takes


def test_a_layer_without_a_gpu_is_made_of_its_parts():
    layer = modules.TempoEncoderLayer(8, 2, 16)
    assert layer._as_one(torch.zeros(1, 2, 8), None) is None
    with pytest.raises(ValueError):
        layer(torch.zeros(1, 2, 8))              # its kernels want CUDA tensors
