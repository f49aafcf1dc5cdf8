"""A forward over a large tensor gives the bits of forwards over its parts, whatever launch shapes the two sizes
take, at aligned and ragged rows."""
import pytest
import torch

from paper_2210_10246_amd import binding as B

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _x(shape, dtype, seed=3):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dtype)


@pytest.mark.parametrize("dtype,mib", [(torch.bfloat16, 61), (torch.bfloat16, 71), (torch.float32, 61), (torch.float32, 90)])
@pytest.mark.parametrize("cols", [1024, 1003])
def test_layernorm_fwd(dtype, mib, cols):
    esize = 2 if dtype == torch.bfloat16 else 4
    rows = mib * MIB // (cols * esize) + 1
    x = _x((rows, cols), dtype)
    gamma, beta = 1.0 + _x((cols,), torch.float32, 4) / 10, _x((cols,), torch.float32, 5)

    def fwd(x):
        y, rstd = torch.empty_like(x), torch.empty(x.shape[0], dtype=torch.float32, device="cuda")
        B.tempo_layernorm_fwd(x, gamma, beta, y, rstd, None, 1e-5)
        return y, rstd

    y, rstd = fwd(x)
    step = rows // 4 // 8 * 8            # quarters, 16-byte aligned
    for r in range(0, rows, step):
        ys, rs = fwd(x[r:r + step])
        assert torch.equal(y[r:r + step], ys) and torch.equal(rstd[r:r + step], rs)


@pytest.mark.parametrize("mib", [59, 60, 64, 65, 130])
def test_gelu_fwd_bf16(mib):
    n = mib * MIB // 2 + 5
    x = _x((n,), torch.bfloat16)

    def fwd(x):
        y, mask = torch.empty_like(x), torch.empty(B.mask_words(x.numel()), dtype=torch.int32, device="cuda")
        B.tempo_gelu_fwd(x, y, mask, "erf")
        return y, mask

    y, mask = fwd(x)
    step = 1 << 23
    for e in range(0, n, step):
        ys, ms = fwd(x[e:e + step])
        assert torch.equal(y[e:e + step], ys) and torch.equal(mask[e // 32:e // 32 + ms.numel()], ms)


@pytest.mark.parametrize("dtype,heads,seq", [(torch.bfloat16, 150, 840), (torch.bfloat16, 100, 333), (torch.float32, 30, 1024),
                                             (torch.float32, 120, 333), (torch.bfloat16, 20, 2600)])
@pytest.mark.parametrize("causal", [False, True])
def test_attention_fwd(dtype, heads, seq, causal):
    scores = _x((1, heads, seq, seq), dtype)
    p, seed, offset = 0.25, 11, 5

    def fwd(s, p):
        probs, out = torch.empty_like(s), torch.empty_like(s)
        keep = torch.empty(B.mask_words(s.numel()), dtype=torch.int32, device="cuda")
        B.tempo_attn_softmax_dropout_fwd(s, None, causal, probs, out, keep, p, seed, offset)
        return probs, out, keep

    probs, out, keep = fwd(scores, p)
    step = 8                             # heads: whole groups of 8 elements
    for h in range(0, heads, step):
        part = scores[:, h:h + step].contiguous()
        assert torch.equal(probs[:, h:h + step], fwd(part, 0.0)[0])
    bits = (keep.view(-1, 1) >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1
    bits = bits.view(-1)[:scores.numel()].view(scores.shape).bool()
    scale = torch.tensor(1.0) / (torch.tensor(1.0) - torch.tensor(p))
    assert torch.equal(out, torch.where(bits, (probs.float() * scale.cuda()).to(dtype), torch.zeros_like(out)))
