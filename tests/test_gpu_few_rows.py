"""LayerNorm backward of few rows: one launch where dx is apart from dy, two where it is dy, and the row kernel with
its partial sums where dgamma is an input too.  All against float64, at the edges of the column walk's steps
(128 rows), of the row shapes and of the rule (640 rows, 320 of the longest float32 ones)."""
import pytest
import torch

from paper_2210_10246_amd import binding as B

pytestmark = pytest.mark.gpu

DT = {"f32": torch.float32, "bf16": torch.bfloat16}
# float32 sums of at most 641 rows or 8192 columns, added as trees of short runs: well below 1e-5 of the result's
# root mean square; bfloat16 outputs (dx): half an ulp, 2^-9, of each value
TOL = {"f32": 1e-5, "bf16": 2.0 ** -8}
GUARD = 64


def guarded(n, dtype):
    buf = torch.full((n + GUARD,), 7, dtype=dtype, device="cuda")
    return buf[:n], buf[n:]


def inputs(M, N, dt):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    gamma, beta = 1.0 + 0.1 * normal(M), 0.1 * normal(M)
    xhat = torch.nn.functional.layer_norm(normal(N, M), (M,))
    y, dy = (gamma * xhat + beta).to(DT[dt]), normal(N, M).to(DT[dt])
    return gamma, beta, y, dy, 0.5 + torch.rand(N, generator=g, device="cuda")


def close(got, want, tol):
    want = want.double().reshape(-1)
    floor = torch.maximum(want.abs(), want.square().mean().sqrt())
    return bool(((got.double().reshape(-1) - want).abs() <= tol * floor).all())


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 9, 128, 129, 640, 641])
@pytest.mark.parametrize("M", [8, 9, 31, 32, 33, 255, 256, 260, 512, 515, 768, 1024, 1027, 2048, 2052, 2056, 4100, 6148, 8191, 8192])
def test_layernorm_bwd(M, N, dt):
    gamma, beta, y, dy, rstd = inputs(M, N, dt)
    h = (y.double() - beta.double()) / gamma.double()
    q = dy.double() * gamma.double()
    dx = rstd.double()[:, None] * (q - h * (q * h).mean(-1, keepdim=True) - q.mean(-1, keepdim=True))
    want = dx, (dy.double() * h).sum(0), dy.double().sum(0)

    ws = torch.empty(B.tempo_layernorm_bwd_workspace_bytes(N, M), dtype=torch.uint8, device="cuda")
    for case in ("apart", "dx is dy", "dgamma is gamma"):
        dg, dg_end = guarded(M, torch.float32)
        db, db_end = guarded(M, torch.float32)
        out, out_end = guarded(N * M, DT[dt])
        out = out.view(N, M)
        src = dy
        if case == "dx is dy":
            out.copy_(dy)
            src = out
        if case == "dgamma is gamma":
            dg.copy_(gamma)
        B.tempo_layernorm_bwd(src, y, dg if case == "dgamma is gamma" else gamma, beta, rstd, out, dg, db, ws)
        for got, ref, tol in ((out, want[0], TOL[dt]), (dg, want[1], 1e-5), (db, want[2], 1e-5)):
            assert close(got, ref, tol), (case, float((got.double() - ref).abs().max()))
        assert (dg_end == 7).all() and (db_end == 7).all() and (out_end == 7).all()


# Where one launch is slower, the row kernel has to run: it adds dgamma and dbeta in an order of its own, so that their
# bits tell.  Its bits come from a call that is always its own, the one with dgamma in gamma's place.
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("N,M", [(321, 6148), (640, 8192), (321, 4097), (640, 8191)])
def test_long_float32_rows_take_the_row_kernel(N, M, in_place, dt="f32"):
    gamma, beta, y, dy, rstd = inputs(M, N, dt)
    ws = torch.empty(B.tempo_layernorm_bwd_workspace_bytes(N, M), dtype=torch.uint8, device="cuda")

    def bwd(in_place, aliased):
        src = dy.clone()
        dx = src if in_place else torch.empty_like(dy)
        dgamma, dbeta = gamma.clone(), torch.empty_like(beta)
        B.tempo_layernorm_bwd(src, y, dgamma if aliased else gamma, beta, rstd, dx, dgamma, dbeta, ws)
        return dx, dgamma, dbeta

    assert all(torch.equal(a, b) for a, b in zip(bwd(in_place, False), bwd(False, True)))
