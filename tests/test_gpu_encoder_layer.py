"""TempoEncoderLayer as one native call each way against the same layer made of its parts: outputs, gradients, and which of
the two routes a call takes."""
import math
import threading

import numpy as np
import pytest
import torch
import torch.nn.functional as F

from oracle import tempo_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2210_10246_amd import binding, modules
    binding.load()
    return modules


@pytest.fixture
def taken(M, monkeypatch):
    """Whether each call of the layer so far was made as one."""
    made, fwd = [], M.B.encoder_fwd

    def spy(*args):
        r = fwd(*args)
        made.append(r is not None)
        return r
    monkeypatch.setattr(M.B, "encoder_fwd", spy)
    return made


def layer_of(M, hidden, heads, ffn, **kw):
    torch.manual_seed(11)
    layer = M.TempoEncoderLayer(hidden, heads, ffn, eps=1e-5, **kw).cuda().train()
    with torch.no_grad():
        for ln in (layer.ln1, layer.ln2):
            ln.weight.add_(0.1 * torch.randn_like(ln.weight))
            ln.bias.add_(0.1 * torch.randn_like(ln.bias))
    return layer


def inputs(batch, seq, hidden):
    g = torch.Generator(device="cuda")
    g.manual_seed(seq)
    x, dy = (torch.randn(batch, seq, hidden, generator=g, device="cuda") for _ in range(2))
    return x.requires_grad_(), dy


def step(layer, x, dy, key_len=None, wanted=None):
    layer.core.offset = 4
    out = layer(x, key_len)
    wanted = [x, *layer.parameters()] if wanted is None else wanted
    return [out.detach(), *torch.autograd.grad(out, wanted, dy)]


def parts(M, monkeypatch, *args):
    with monkeypatch.context() as m:
        m.setattr(M.TempoEncoderLayer, "_as_one", lambda *a: None)
        return step(*args)


# Tiles of 32 and 64 rows, columns and steps of k of 16, 32 and 64: one short of them, whole, one more; head sizes and
# sequences that are no multiple of a piece's 4, and the smallest ones.  On 256 compute units the last ten come to every tile
# that launch_matmul() and launch_matmul_group() choose, with and without GELU; with test_options_reach_the_kernels and
# test_gelu_at_the_end_of_a_product every one of the 37 kernels of matmul.hip runs.
@pytest.mark.parametrize("batch,seq,hidden,heads,ffn", [
    (1, 1, 32, 2, 64), (2, 31, 64, 4, 100), (3, 33, 96, 3, 36), (2, 33, 64, 2, 72), (1, 65, 128, 2, 512), (2, 130, 40, 5, 44), (5, 7, 192, 12, 768),
    (1, 64, 64, 1, 4), (3, 63, 12, 3, 260), (2, 256, 256, 4, 1024), (4, 97, 512, 8, 2048), (1, 3, 1024, 16, 4096),
    (1, 128, 512, 8, 3072), (4, 256, 256, 4, 1024), (4, 515, 192, 12, 772), (1, 1, 128, 2, 3080), (1, 515, 64, 1, 64),
    (1, 130, 512, 8, 2052), (8, 333, 320, 5, 264), (1, 16, 2560, 20, 512)])
@pytest.mark.parametrize("padded", [False, True])
def test_one_call_matches_the_parts(M, monkeypatch, taken, batch, seq, hidden, heads, ffn, padded):
    layer = layer_of(M, hidden, heads, ffn, p_attn=0.1)
    x, dy = inputs(batch, seq, hidden)
    key_len = torch.arange(seq, seq - batch, -1, device="cuda", dtype=torch.int32).clamp(min=1) if padded else None
    got = step(layer, x, dy, key_len)
    assert taken == [True] and layer.core.offset == 5
    want = parts(M, monkeypatch, layer, x, dy, key_len)
    # float32 sums of up to 4096 products in another order: about sqrt(4096) 2^-24 = 4e-6 of the result's norm, and what
    # five products in a row make of it; an absolute 1e-6 for the key bias, whose gradient is 0 but for rounding
    for i, (a, b) in enumerate(zip(got, want)):
        assert (a - b).norm() <= 2e-5 * b.norm() + 1e-6 * a.numel() ** 0.5, i


def in_64_bits(layer, x, dy, keep):
    """Output and gradients of the layer in plain float64."""
    p = [t.detach().double().requires_grad_() for t in (x, *layer.parameters())]
    wqkv, bqkv, wproj, bproj, w1, b1, w2, b2, g1, be1, g2, be2 = p[1:]
    (Bn, S, H), A = x.shape, layer.heads
    q, k, v = F.linear(p[0], wqkv, bqkv).view(Bn, S, 3, A, H // A).permute(2, 0, 3, 1, 4)
    probs = torch.softmax(torch.matmul(q, k.transpose(-1, -2)) / math.sqrt(H // A), dim=-1) * keep
    ctxt = torch.matmul(probs, v).permute(0, 2, 1, 3).reshape(Bn, S, H)
    y = F.layer_norm(p[0] + F.linear(ctxt, wproj, bproj), (H,), g1, be1, 1e-5)
    out = F.layer_norm(y + F.linear(F.gelu(F.linear(y, w1, b1)), w2, b2), (H,), g2, be2, 1e-5)
    return [out.detach(), *torch.autograd.grad(out, p, dy.double())]


@pytest.mark.parametrize("batch,seq,hidden,heads,ffn", [(2, 128, 768, 12, 3072), (4, 97, 512, 8, 2048), (1, 515, 64, 1, 64),
                                                        (8, 256, 256, 4, 1024)])
def test_as_exact_as_the_parts(M, monkeypatch, taken, batch, seq, hidden, heads, ffn):
    layer = layer_of(M, hidden, heads, ffn, p_attn=0.1)
    x, dy = inputs(batch, seq, hidden)
    K = O.dropout_keep(batch * heads * seq * seq, 0.1, layer.core.seed, 5).reshape(batch, heads, seq, seq)
    scale = float(np.float32(1.0) / (np.float32(1.0) - np.float32(0.1)))
    exact = in_64_bits(layer, x, dy, torch.from_numpy(K).cuda().double() * scale)
    got, want = step(layer, x, dy), parts(M, monkeypatch, layer, x, dy)
    assert taken == [True]
    order = [n for n, _ in layer.named_parameters()]
    for name, a, b, e in zip(["out", "x", *order], got, want, exact, strict=True):
        if name == "qkv.bias":                    # without the keys', whose gradient is rounding alone
            a, b, e = (torch.cat([t[:hidden], t[2 * hidden:]]) for t in (a, b, e))
        one, made = ((t.double() - e).norm() / e.norm() for t in (a, b))
        print(name, f"{one:.2e} {made:.2e}")
        # rounding of the same number of sums in another order; inputs or sums of a bit less would double it
        assert one <= 1.5 * made, name


# tanh at sizes that come to every tile of the backward's product with GELU
@pytest.mark.parametrize("kind,store,training,batch,seq,hidden,heads,ffn", [
    ("tanh", True, True, 2, 50, 128, 2, 256), ("tanh", True, True, 2, 256, 256, 4, 1024), ("tanh", True, True, 4, 97, 512, 8, 2048),
    ("tanh", True, True, 1, 3, 1024, 16, 4096), ("tanh", True, True, 4, 256, 256, 4, 1024), ("erf", False, True, 2, 50, 128, 2, 256),
    ("erf", True, False, 2, 50, 128, 2, 256)])
def test_options_reach_the_kernels(M, monkeypatch, taken, kind, store, training, batch, seq, hidden, heads, ffn):
    layer = layer_of(M, hidden, heads, ffn)
    layer.act.kind, layer.core.store_mask = kind, store
    layer.train(training)
    x, dy = inputs(batch, seq, hidden)
    got = step(layer, x, dy)
    assert taken == [True]
    for a, b in zip(got, parts(M, monkeypatch, layer, x, dy)):
        assert (a - b).norm() <= 2e-5 * b.norm() + 1e-6 * a.numel() ** 0.5


# Sizes whose products take other tiles alone than beside others: with values of k split over 1, 2, 4 and 8 waves.
@pytest.mark.parametrize("batch,seq,hidden,heads,ffn", [(3, 20, 64, 4, 128), (2, 128, 768, 12, 3072), (1, 77, 512, 8, 2048),
                                                        (4, 130, 256, 4, 1028), (3, 63, 12, 3, 260),
                                                        (2, 31, 1024, 16, 4096)])
def test_gradients_of_a_part_of_the_inputs(M, taken, batch, seq, hidden, heads, ffn):
    """Whatever is asked for has the bits it has when everything is."""
    layer = layer_of(M, hidden, heads, ffn)
    x, dy = inputs(batch, seq, hidden)
    every = [x, *layer.parameters()]
    full = step(layer, x, dy)[1:]
    for names in ([0], [2], [3, 4], [5], [7, 8], [9], [11, 12], [0, 6], [1, 10]):
        for t in every:
            t.requires_grad_(any(t is every[i] for i in names))
        got = step(layer, x, dy, None, [every[i] for i in names])[1:]
        for i, g in zip(names, got):
            assert torch.equal(g, full[i]), names
    assert all(taken)
    for t in every:
        t.requires_grad_(True)


def test_without_gradients(M, taken):
    layer = layer_of(M, 64, 4, 128)
    x, dy = inputs(2, 9, 64)
    want = step(layer, x, dy)[0]
    for mode in (torch.no_grad, torch.inference_mode):
        with mode():
            layer.core.offset = 4
            assert torch.equal(layer(x), want)
    assert taken == [True] * 3


def test_calls_that_are_made_of_the_parts(M, monkeypatch, taken):
    """Whatever could see or change the layer's parts, or that the kernels do not take."""
    layer = layer_of(M, 64, 4, 128)
    x, dy = inputs(2, 8, 64)
    want = step(layer, x, dy)
    assert taken == [True]
    taken.clear()
    seen = []
    hook = layer.fc1.register_forward_hook(lambda m, i, o: seen.append(o.shape))
    got = step(layer, x, dy)
    hook.remove()
    assert seen == [(2, 8, 128)] and torch.allclose(got[0], want[0], atol=1e-5)
    with torch.autocast("cuda", dtype=torch.bfloat16):
        layer(x)
    proj, layer.proj = layer.proj, torch.nn.Sequential(layer.proj)
    step(layer, x, dy, None, [x])
    layer.proj = proj
    step(layer, x.transpose(0, 1).contiguous().transpose(0, 1).detach().requires_grad_(), dy, None, list(layer.parameters()))
    with torch.device("cuda"):                   # a function mode
        step(layer, x, dy)
    with monkeypatch.context() as m:
        plain = torch.nn.Linear.forward
        m.setattr(torch.nn.Linear, "forward", lambda self, t: 2 * plain(self, t))
        assert not torch.allclose(step(layer, x, dy)[0], want[0], atol=1e-2)
    assert not any(taken)
    # gradients that are differentiated again: connected as the parts' are
    out = layer(x)
    (g,) = torch.autograd.grad(out, [layer.fc2.weight], dy, create_graph=True)
    with monkeypatch.context() as m:
        m.setattr(M.TempoEncoderLayer, "_as_one", lambda *a: None)
        layer.core.offset -= 1
        (h,) = torch.autograd.grad(layer(x), [layer.fc2.weight], dy, create_graph=True)
    # of the forward that was made, whose products differ from the library's as in test_one_call_matches_the_parts
    assert g.requires_grad == h.requires_grad and (g - h).norm() <= 2e-5 * h.norm() + 1e-6 * h.numel() ** 0.5


def test_odd_heads_are_made_of_the_parts(M, taken):
    layer = layer_of(M, 66, 3, 128)              # 22 columns a head
    x, dy = inputs(2, 8, 66)
    step(layer, x, dy)
    assert taken == [False]


def test_hooks_on_what_is_kept(M, taken):
    layer = layer_of(M, 64, 4, 128)
    x, dy = inputs(2, 40, 64)
    want = step(layer, x, dy)
    with torch.autograd.graph.save_on_cpu():
        got = step(layer, x, dy)
    assert taken == [True, True]
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_replays_of_a_captured_step(M, taken):
    layer = layer_of(M, 64, 4, 128)
    x, dy = inputs(2, 40, 64)
    want = step(layer, x, dy)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        step(layer, x, dy)
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            got = step(layer, x, dy)
        for _ in range(3):
            for t in got:
                t.zero_()
            graph.replay()
            st.synchronize()
            for a, b in zip(got, want):
                assert torch.equal(a, b)
            step(layer, x, dy)
    assert all(taken)


def test_create_graph(M, monkeypatch):
    """Weights that a layer's own input depends on, a bias, key_len: gradients and what is differentiated again."""
    layer = layer_of(M, 64, 4, 128)
    x, dy = inputs(2, 40, 64)

    def both():
        layer.core.offset = 4
        key_len = torch.tensor([40, 23], device="cuda", dtype=torch.int32)
        out = layer(layer(x, key_len), key_len)
        key_len.fill_(1)
        grads = torch.autograd.grad(out, [x, *layer.parameters()], dy, create_graph=True)
        penalty = sum(g.square().mean() for g in grads if g.requires_grad)
        return [*grads, *torch.autograd.grad(penalty, [x, *layer.parameters()], materialize_grads=True)]
    got = both()
    with monkeypatch.context() as m:
        m.setattr(M.TempoEncoderLayer, "_as_one", lambda *a: None)
        want = both()
    # two layers and their backwards of products summed in another order (see test_one_call_matches_the_parts), and one more of each
    for i, (a, b) in enumerate(zip(got, want)):
        assert a.requires_grad == b.requires_grad and (a - b).norm() <= 6e-5 * b.norm() + 1e-6 * a.numel() ** 0.5, i


@pytest.mark.parametrize("frozen", [("qkv.weight", "proj.weight", "fc1.weight", "fc2.weight"), ("qkv.", "proj."), ("qkv.", "proj.", "ln1."), ("proj.",), ("qkv.", "proj.", "ln1.", "fc1."),
                                    ("fc1.", "fc2."), ("qkv.", "proj.", "ln1.", "fc1.", "fc2.")])
@pytest.mark.parametrize("x_needs", [True, False])
def test_frozen_halves(M, monkeypatch, taken, frozen, x_needs):
    """The native backward from what a partly frozen layer keeps."""
    layer = layer_of(M, 128, 4, 260)
    x, dy = inputs(3, 70, 128)
    x.requires_grad_(x_needs)
    for name, p in layer.named_parameters():
        p.requires_grad_(not name.startswith(frozen))
    wanted = [x] * x_needs + [p for p in layer.parameters() if p.requires_grad]

    def kept():
        seen = {}

        def pack(t):
            seen[t.untyped_storage().data_ptr()] = t.untyped_storage().nbytes()
            return t
        with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t):
            got = step(layer, x, dy, None, wanted)
        return got, sum(seen.values())
    got, few = kept()
    assert taken == [True]
    with monkeypatch.context() as m:
        m.setattr(M.TempoEncoderLayer, "_as_one", lambda *a: None)
        want, most = kept()
    assert few <= most
    for a, b in zip(got, want, strict=True):      # the bound of test_one_call_matches_the_parts
        assert (a - b).norm() <= 2e-5 * b.norm() + 1e-6 * a.numel() ** 0.5


def test_what_hooks_give_back_in_another_layout(M, taken):
    layer = layer_of(M, 64, 4, 128)
    x, dy = inputs(2, 40, 64)
    want = step(layer, x, dy)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.t().contiguous().t() if t.shape == (128, 64) else t, lambda t: t):
        got = step(layer, x, dy)
    assert taken == [True, True]
    for a, b in zip(got, want, strict=True):
        assert (a - b).norm() <= 2e-5 * b.norm() + 1e-6 * a.numel() ** 0.5


def test_threads_that_share_a_layer_draw_other_bits(M, monkeypatch):
    layer, drawn = layer_of(M, 64, 4, 128), []
    x, _ = inputs(2, 8, 64)
    fwd = M.B.encoder_fwd

    def spy(*args):
        r = fwd(*args)
        drawn.append(r[0])
        return r
    monkeypatch.setattr(M.B, "encoder_fwd", spy)

    def calls():
        with torch.no_grad():
            for _ in range(200):
                layer(x)
    threads = [threading.Thread(target=calls) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert sorted(drawn) == list(range(1, 801)) and layer.core.offset == 800


def specials(M, kind, n):
    """n values around GELU's minimum, of every size and sign, infinities and NaN."""
    star = {"erf": O.GELU_XSTAR_F32["erf"], "tanh": O.GELU_XSTAR_F32["tanh"]}[kind]
    star = torch.tensor(float(star))
    at = [star, star.nextafter(torch.tensor(0.0)), star.nextafter(torch.tensor(-9.0))]
    odd = [0.0, -0.0, 1e-42, -1e-42, 1e-8, -1e-8, 40.0, -40.0, 3e38, -3e38, math.inf, -math.inf, math.nan]
    v = torch.cat([torch.stack(at), torch.tensor(odd)])
    fill = torch.linspace(-8, 8, n)
    fill[torch.arange(0, n, 7)] = v[torch.arange(0, n, 7) // 7 % len(v)]
    return fill.cuda()


def same_values(a, b):
    """NaN for NaN, all else equal (a product's sum starts at +0, so that -0 does not come out of it)."""
    return torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(0, math.inf, -math.inf), b.nan_to_num(0, math.inf, -math.inf))


# Sizes at which the first feed-forward product takes each of its four tiles.
@pytest.mark.parametrize("batch,seq,hidden,heads,ffn", [(2, 33, 64, 2, 1024), (8, 64, 64, 4, 1024), (4, 97, 512, 8, 2048),
                                                        (1, 16, 2560, 20, 512)])
@pytest.mark.parametrize("kind", ["erf", "tanh"])
def test_gelu_at_the_end_of_a_product(M, batch, seq, hidden, heads, ffn, kind):
    """Values and mask bits are those of tempo_gelu_fwd."""
    layer = layer_of(M, hidden, heads, ffn)
    layer.act.kind = kind
    pre = specials(M, kind, ffn)
    with torch.no_grad():
        layer.fc1.weight.zero_()                  # so that what GELU gets is the bias
        layer.fc1.bias.copy_(pre)
    x, _ = inputs(batch, seq, hidden)
    h, side = forward(M, layer, x)[6:8]
    rows = pre.expand(batch * seq, ffn).contiguous()
    y, mask = torch.empty_like(rows), torch.empty_like(side)
    M.B.tempo_gelu_fwd(rows, y, mask, kind)
    assert same_values(h, y), [(v, a, b) for v, a, b in zip(pre.tolist(), h[0].tolist(), y[0].tolist()) if a != b]
    assert torch.equal(side, mask)


def forward(M, layer, x):
    made = M.B.encoder_fwd(x, None, layer.core.__dict__, layer.heads, 1e-5, 1e-5, 0.1, 7, layer.act.kind, *params_of(layer))
    assert made is not None
    return made[1:]


def params_of(layer):
    return [t for m in (layer.qkv, layer.proj, layer.fc1, layer.fc2, layer.ln1, layer.ln2) for t in (m.weight, m.bias)]


@pytest.mark.parametrize("hidden,heads,ffn", [(64, 2, 1024), (128, 2, 3080), (512, 8, 8192)])
@pytest.mark.parametrize("kind", ["erf", "tanh"])
def test_gelu_backward_at_the_end_of_a_product(M, hidden, heads, ffn, kind):
    """The gradient that reaches the first feed-forward layer is that of tempo_gelu_bwd: for one token it is its bias gradient."""
    layer = layer_of(M, hidden, heads, ffn)
    layer.act.kind = kind
    with torch.no_grad():                         # so that each column of h gets one gradient of the layer's output
        layer.fc2.weight.zero_()
        layer.fc2.weight[torch.arange(ffn) % hidden, torch.arange(ffn)] = 1.0
    x, dy = inputs(1, 1, hidden)
    qkv, probs, keep, ctxt, y1, rstd1, h, side, y2, rstd2 = forward(M, layer, x)
    pre = specials(M, kind, ffn)
    M.B.tempo_gelu_fwd(pre, h.view(-1), side, kind)
    wqkv, _, wproj, _, w1, _, w2, _, g1, be1, g2, be2 = params_of(layer)
    grads = M.B.encoder_bwd(dy, (1 << 13) - 1, heads, ffn, 0.1, 7, 1, kind, x, wqkv, wproj, w1, w2, g1, be1, g2, be2, qkv, probs,
                            keep, ctxt, y1, rstd1, h, side, y2, rstd2)
    db1, db2 = grads[6], grads[8]
    dh, want = db2[torch.arange(ffn) % hidden], torch.empty(ffn, device="cuda")
    M.B.tempo_gelu_bwd(dh.contiguous(), h.view(-1), side, want, kind)
    assert same_values(db1, want)
