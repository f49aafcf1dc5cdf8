"""The native and the ctypes half of the binding make the same call: same outputs, on the current
stream, and the same refusals (the native half hands over whatever it does not take).  Which half made a
call is seen from what the native function returned: a status, or None for a call handed over."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2210_10246_amd import binding
    binding.load()
    return binding


class Spy:
    """Stands in for the native module and keeps what each of its functions returned."""

    def __init__(self, native):
        self._native, self.returned = native, []

    def __getattr__(self, name):
        fn = getattr(self._native, name)

        def call(*args):
            r = fn(*args)
            self.returned.append((name, r))
            return r
        return call


@pytest.fixture
def spy(B, monkeypatch):
    s = Spy(B._native)
    monkeypatch.setattr(B, "_native", s)
    return s


def calls(B, dt):
    """{entry point: (function of stream -> outputs)}, each on buffers of its own."""
    g = torch.Generator(device="cuda")
    g.manual_seed(3)

    def rand(*shape, dtype=dt):
        return torch.randn(*shape, generator=g, device="cuda").to(dtype)

    x, dy, gamma, beta = rand(6, 40), rand(6, 40), 1 + 0.1 * rand(40, dtype=torch.float32), rand(40, dtype=torch.float32)
    s, dout = rand(2, 3, 5, 24), rand(2, 3, 5, 24)
    key_len = torch.tensor([24, 11], dtype=torch.int32, device="cuda")
    mask, keep = (torch.zeros(B.mask_words(t.numel()), dtype=torch.int32, device="cuda") for t in (x, s))
    B.tempo_gelu_fwd(x, torch.empty_like(x), mask)
    probs = torch.empty_like(s)
    B.tempo_attn_softmax_dropout_fwd(s, key_len, False, probs, torch.empty_like(s), keep, 0.1, 7, 2**40)
    keep_bytes = torch.empty(s.numel(), dtype=torch.uint8, device="cuda")
    B.tempo_mask_bits_to_bytes(keep, keep_bytes, s.numel())
    y, rstd = torch.empty_like(x), torch.empty(6, device="cuda")
    B.tempo_layernorm_fwd(x, gamma, beta, y, rstd)
    ws = torch.empty(B.tempo_layernorm_bwd_workspace_bytes(6, 40), dtype=torch.uint8, device="cuda")

    def out(fn, outputs, *args, **kw):
        def run(stream):
            o = [torch.full_like(t, 3) for t in outputs]
            fn(*[o[a[0]] if isinstance(a, tuple) else a for a in args], stream=stream, **kw)
            return o
        return run

    return {
        "gelu_fwd": out(B.tempo_gelu_fwd, [x, mask], x, (0,), (1,), "tanh"),
        "gelu_bwd": out(B.tempo_gelu_bwd, [x], dy, x, mask, (0,)),
        "silu_fwd": out(B.tempo_silu_fwd, [x, mask], x, (0,), (1,)),
        "silu_bwd": out(B.tempo_silu_bwd, [x], dy, x, mask, (0,)),
        "layernorm_fwd": out(B.tempo_layernorm_fwd, [y, rstd, rstd], x, gamma, beta, (0,), (1,), (2,), 1e-3),
        "layernorm_fwd_eps0": out(B.tempo_layernorm_fwd, [y, rstd], x, gamma, beta, (0,), (1,), None, 0),
        "layernorm_bwd": out(B.tempo_layernorm_bwd, [y, gamma, beta], dy, y, gamma, beta, rstd, (0,), (1,), (2,), ws),
        "layernorm_bwd_static": out(B.tempo_layernorm_bwd_static, [y, gamma, beta], dy, y, gamma, beta, rstd, (0,),
                                    (1,), (2,)),
        "attn_fwd": out(B.tempo_attn_softmax_dropout_fwd, [s, s, keep], s, key_len, True, (0,), (1,), (2,), 0.1, 7, 2**40),
        "attn_fwd_p0": out(B.tempo_attn_softmax_dropout_fwd, [s, keep], s, None, 0, (0,), None, (1,), 0, 7, 1),
        "attn_bwd": out(B.tempo_attn_softmax_dropout_bwd, [s, s], dout, probs, keep, (0,), (1,), 0.1),
        "attn_bwd_regen": out(B.tempo_attn_softmax_dropout_bwd_regen, [s, s], dout, probs, (0,), (1,), 0.1, 7, 2**40),
        "attn_bwd_bytemask": out(B.tempo_attn_softmax_dropout_bwd_bytemask, [s], dout, probs, keep_bytes, (0,), None, 0.1),
    }


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_native_and_ctypes_calls_agree(B, dt, spy):
    side = torch.cuda.Stream()
    for name, run in calls(B, dt).items():
        spy.returned.clear()
        want = run(torch.cuda.current_stream())          # an explicit stream: the ctypes half
        assert spy.returned == []
        got = run(None)
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            on_side = run(None)                          # the native half follows the current stream
        side.synchronize()
        assert [r for _, r in spy.returned] == [0, 0], name
        assert all(name.removesuffix("_p0").removesuffix("_eps0").replace("attn_", "attn_softmax_dropout_") in called
                   for called, _ in spy.returned), name
        for w, a, b in zip(want, got, on_side):
            assert torch.equal(w, a) and torch.equal(w, b), name


def test_native_half_refuses_what_the_ctypes_half_refuses(B, spy):
    x = torch.zeros(64, device="cuda")
    m = torch.zeros(2, dtype=torch.int32, device="cuda")
    with pytest.raises(ValueError, match="mask must have at least 2"):
        B.tempo_gelu_fwd(x, torch.empty_like(x), m[:1])
    with pytest.raises(ValueError, match="y must be"):
        B.tempo_gelu_fwd(x, x.bfloat16(), m)
    with pytest.raises(ValueError, match="contiguous CUDA"):
        B.tempo_gelu_fwd(x, torch.empty(128, device="cuda")[::2], m)
    with pytest.raises(ValueError, match="contiguous CUDA"):
        B.tempo_gelu_fwd(x, x.cpu(), m)
    with pytest.raises(KeyError):
        B.tempo_gelu_fwd(x, torch.empty_like(x), m, "sigmoid")
    # a number of another type: taken by ctypes or not, but never by the native half
    B.tempo_layernorm_fwd(x.view(4, 16), *torch.ones(2, 16, device="cuda"), x.view(4, 16).clone(),
                          torch.empty(4, device="cuda"), None, np.float32(0.5))
    assert [r for _, r in spy.returned] == [None] * 6    # all handed over
    spy.returned.clear()
    with pytest.raises(B.TempoError, match="16-byte") as e:
        B.tempo_gelu_fwd(x, torch.empty(65, device="cuda")[1:], m)
    assert e.value.status == 2
    with pytest.raises(B.TempoError):
        B.tempo_attn_softmax_dropout_bwd_regen(x.view(1, 1, 8, 8), x.view(1, 1, 8, 8), x.view(1, 1, 8, 8), None, 1.5, 1, 1)
    y, r, g = torch.empty(4, 16, device="cuda"), torch.empty(4, device="cuda"), torch.ones(16, device="cuda")
    with pytest.raises(B.TempoError, match="workspace"):
        B.tempo_layernorm_bwd(y, y.clone(), g, g, r, y.clone(), g.clone(), g.clone(), torch.empty(16, device="cuda"))
    assert [r for _, r in spy.returned] == [2, 1, 3]     # refused by the library itself
