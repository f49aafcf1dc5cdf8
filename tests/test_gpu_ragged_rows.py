"""Rows whose length is no multiple of a 16-byte piece, against the oracle: both sides of every
shape of the ragged kernels (shorter than a piece, one element more than a piece, the last lane of a
group, one or several pieces per lane, one or several waves per row), every mask source, in place,
and with guard words behind every output."""
import numpy as np
import pytest
import torch

from helpers import TOL, rel_err
from oracle import tempo_oracle as O

pytestmark = pytest.mark.gpu

TDT = {"f32": torch.float32, "bf16": torch.bfloat16}
GUARD = 64


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2210_10246_amd import binding
    binding.load()
    return binding


def dev(a, dt):
    return torch.from_numpy(np.ascontiguousarray(a)).to(TDT[dt]).cuda()


def host(t):
    return t.detach().cpu().to(torch.float64).numpy()


def stored(rng, shape, dt, scale=1.0):
    return O.round_to_dtype(rng.standard_normal(shape) * scale, dt)


def guarded(shape, dtype, init=None):
    """A tensor of that shape with GUARD elements of 7 behind it."""
    n = int(np.prod(shape))
    buf = torch.full((n + GUARD,), 7, dtype=dtype, device="cuda")
    if init is not None:
        buf[:n] = init.reshape(-1)
    return buf[:n].view(shape), buf[n:]


# row length, rows: the last row ends inside a mask word, on one, or one element before one
ATTN_ROWS = [(1, 33), (3, 21), (5, 13), (7, 9), (9, 7), (15, 3), (31, 5), (33, 9), (63, 3), (65, 2), (127, 3),
             (129, 5), (253, 3), (255, 2), (257, 3), (333, 5), (505, 2), (511, 3), (513, 3), (769, 2),
             (1023, 3), (1025, 2), (1535, 2), (2047, 2), (2049, 2), (3071, 1), (4093, 2), (4095, 1),
             (8191, 1)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("Sk,Sq", ATTN_ROWS)
def test_attention_ragged_rows(B, Sk, Sq, dt):
    check_attention(B, Sk, Sq, dt, {1: "causal", 3: "padding"}.get(Sk % 4, "none"))


def check_attention(B, Sk, Sq, dt, mask):
    rng = np.random.default_rng(Sk)
    shape = (2, 1, Sq, Sk)
    p, seed, offset = np.float32(0.2), 0x123456789ABC, 5
    causal = mask == "causal"
    key_len = np.array([Sk, max(1, Sk * 2 // 3)], dtype=np.int32) if mask == "padding" else None
    s = stored(rng, shape, dt, 0.5)
    P_ref, out_ref, K_ref = O.attn_softmax_dropout_fwd(s, key_len, causal, p, seed, offset, dt)
    sd = dev(s, dt)
    kd = None if key_len is None else torch.from_numpy(key_len).cuda()
    n = s.size
    for in_place in (False, True):
        Pd, g0 = guarded(shape, TDT[dt], sd if in_place else None)
        od, g1 = guarded(shape, TDT[dt])
        md, g2 = guarded((B.mask_words(n),), torch.int32)
        B.tempo_attn_softmax_dropout_fwd(Pd if in_place else sd, kd, causal, Pd, od, md, float(p), seed, offset)
        assert np.array_equal(md.cpu().numpy().view(np.uint32), O.pack_bits(K_ref))
        assert rel_err(host(Pd), P_ref) <= TOL[dt]
        assert rel_err(host(od), out_ref) <= TOL[dt]
        for g in (g0, g1, g2):
            assert (g == 7).all()
    dout = stored(rng, shape, dt)
    dS_ref, out_re_ref = O.attn_softmax_dropout_bwd(dout, P_ref, K_ref, p, dt)
    dod, Pd2 = dev(dout, dt), dev(P_ref, dt)
    keep = torch.from_numpy(np.ascontiguousarray(K_ref).reshape(-1).astype(np.uint8)).cuda()
    results = []
    for source in ("bits", "regen", "bytes"):
        dsd, g0 = guarded(shape, TDT[dt], dod)
        rd, g1 = guarded(shape, TDT[dt])
        if source == "bits":       # in place: dscores is dout
            B.tempo_attn_softmax_dropout_bwd(dsd, Pd2, md, dsd, rd, float(p))
        elif source == "regen":
            B.tempo_attn_softmax_dropout_bwd_regen(dod, Pd2, dsd, rd, float(p), seed, offset)
        else:
            B.tempo_attn_softmax_dropout_bwd_bytemask(dod, Pd2, keep, dsd, rd, float(p))
        assert rel_err(host(dsd), dS_ref) <= TOL[dt], source
        assert rel_err(host(rd), out_re_ref) <= TOL[dt], source
        assert (g0 == 7).all() and (g1 == 7).all(), source
        results.append((dsd, rd))
    for dsd, rd in results[1:]:
        assert torch.equal(dsd, results[0][0]) and torch.equal(rd, results[0][1])


# columns, rows: rows enough for one batch, for several, or for workgroups that loop
LN_ROWS = [(4, 5), (5, 40), (7, 9), (9, 3), (63, 70), (65, 130), (127, 9), (129, 4100), (255, 17), (258, 1030),
           (385, 33), (511, 2100), (513, 41), (770, 700), (1001, 1300), (1023, 19), (1025, 600), (1535, 300),
           (1537, 20), (2047, 300), (2049, 9), (3070, 7), (3073, 300), (4095, 5), (4097, 260), (4100, 270),
           (6145, 3), (8191, 270),
           # fewer and more than 64 rows per compute unit (the row shapes of the backward differ), eight waves per row
           (259, 64), (515, 700), (515, 16400), (5003, 300)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("M,N", LN_ROWS)
def test_layernorm_ragged_rows(B, M, N, dt):
    rng = np.random.default_rng(M)
    x = O.round_to_dtype(2.0 * rng.standard_normal((N, M)) + 0.5, dt)
    gamma = O.round_to_dtype(1 + 0.1 * rng.standard_normal(M), "f32")
    beta = O.round_to_dtype(0.1 * rng.standard_normal(M), "f32")
    dy = stored(rng, (N, M), dt)
    y, rstd, mean = O.layernorm_fwd(x, gamma, beta, 1e-5, dt)
    gd, bd = dev(gamma, "f32"), dev(beta, "f32")
    yd, g0 = guarded((N, M), TDT[dt], dev(x, dt))            # in place
    rd, g1 = guarded((N,), torch.float32)
    md, g2 = guarded((N,), torch.float32)
    B.tempo_layernorm_fwd(yd, gd, bd, yd, rd, md, 1e-5)
    assert rel_err(host(yd), y) <= TOL[dt]
    assert rel_err(host(rd), rstd) <= TOL["f32"]
    assert rel_err(host(md), mean) <= TOL["f32"]
    assert all((g == 7).all() for g in (g0, g1, g2))

    dx_ref, dg_ref, db_ref = O.layernorm_bwd(dy, y, gamma, beta, rstd, dt)
    size = B.tempo_layernorm_bwd_workspace_bytes(N, M)
    runs = []
    for _ in range(2):
        dxd, g0 = guarded((N, M), TDT[dt], dev(dy, dt))      # in place
        dgd, g1 = guarded((M,), torch.float32)
        dbd, g2 = guarded((M,), torch.float32)
        ws, g3 = guarded(((size + 15) // 16 * 16,), torch.uint8)
        B.tempo_layernorm_bwd(dxd, dev(y, dt), gd, bd, dev(rstd, "f32"), dxd, dgd, dbd, ws)
        assert rel_err(host(dxd), dx_ref) <= TOL[dt]
        assert rel_err(host(dgd), dg_ref) <= TOL["f32"]
        assert rel_err(host(dbd), db_ref) <= TOL["f32"]
        assert all((g == 7).all() for g in (g0, g1, g2, g3))
        runs.append((dxd, dgd, dbd))
    assert all(torch.equal(a, b) for a, b in zip(*runs))     # fixed summation order


@pytest.mark.parametrize("extremes", [False, True])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("M,N", [(5, 40), (63, 70), (255, 17), (511, 2100), (1001, 300), (2047, 300), (4097, 20), (8191, 9),
                                 # more rows than the backward takes in one launch
                                 (9, 700), (63, 1000), (257, 650), (1001, 700), (2047, 645), (4097, 650), (8191, 641)])
def test_layernorm_backward_where_beta_is_much_larger_than_gamma(B, M, N, dt, extremes):
    """xhat = (y - beta) / gamma: the subtraction cancels, so it has to come first.  It is exact or
    rounded once and the quotient within two units in the last place, whatever beta / gamma is;
    subtracting beta / gamma from y / gamma instead is off by 2^-24 |beta / gamma|, here 6e-4."""
    rng = np.random.default_rng(M)
    gamma = O.round_to_dtype(0.01 * (1 + 0.1 * rng.standard_normal(M)), "f32")
    beta = O.round_to_dtype(100 * (1 + 0.1 * rng.standard_normal(M)), "f32")
    if extremes:  # columns whose gamma has no float32 reciprocal, or one close to the end of the range
        gamma[M // 2], beta[M // 2] = 2.0 ** -130, 0.0
        gamma[M // 3], beta[M // 3] = 2.0 ** 100, 0.0
    x = O.round_to_dtype(rng.standard_normal((N, M)), dt)
    y, rstd, _ = O.layernorm_fwd(x, gamma, beta, 1e-5, dt)
    dy = stored(rng, (N, M), dt)
    refs = O.layernorm_bwd(dy, y, gamma, beta, rstd, dt)
    dxd = dev(dy, dt)
    dgd, dbd = torch.empty(M, device="cuda"), torch.empty(M, device="cuda")
    ws = torch.empty(B.tempo_layernorm_bwd_workspace_bytes(N, M), dtype=torch.uint8, device="cuda")
    B.tempo_layernorm_bwd(dxd, dev(y, dt), dev(gamma, "f32"), dev(beta, "f32"), dev(rstd, "f32"), dxd, dgd, dbd, ws)
    for name, got, ref, d in zip(("dx", "dgamma", "dbeta"), (dxd, dgd, dbd), refs, (dt, "f32", "f32")):
        assert rel_err(host(got), ref) <= TOL[d], name


@pytest.mark.parametrize("Sk", [31, 255, 333, 1001])
def test_attention_probabilities_of_equal_scores_are_correctly_rounded(B, Sk):
    """Equal scores: every exponential is 1 and the sum of a causal row's i + 1 of them exact, so P is
    1 / (i + 1) to the last bit if the reciprocal is correctly rounded."""
    s = torch.zeros(1, 1, Sk, Sk, device="cuda")
    P = torch.empty_like(s)
    md = torch.empty(B.mask_words(s.numel()), dtype=torch.int32, device="cuda")
    B.tempo_attn_softmax_dropout_fwd(s, None, True, P, None, md, 0.1, 1, 2)
    want = torch.tril((1.0 / torch.arange(1, Sk + 1, dtype=torch.float64)).float()[:, None].expand(Sk, Sk))
    assert torch.equal(P[0, 0].cpu(), want)
