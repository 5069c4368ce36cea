"""The tiled products at sizes around their tile edges: ragged row, column and
k tiles, operands smaller than one tile, in every tile shape.  The inputs lie
between NaNs, so an element read past an operand's end shows in the result."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

F64 = torch.float64
SHAPES = ["128x128", "128x64", "64x64", None]  # None: the default table, smaller tiles for few
# (naux, nbf, nocc): k of 3 to 130, rows of 4 to 17161 with every remainder class
SIZES = [(3, 2, 1), (7, 5, 2), (16, 16, 3), (17, 31, 8), (33, 65, 1), (130, 63, 9), (31, 131, 2)]


def _guarded(x):
    """x on the device with 64 NaNs before and after it."""
    buf = torch.full((x.numel() + 128,), float("nan"), dtype=x.dtype, device="cuda:0")
    view = buf[64:64 + x.numel()].view(x.shape)
    view.copy_(x)
    return view


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2210_17093_amd.qsgw as q
    with q.Context() as c:
        yield c


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("naux,nbf,nocc", SIZES)
def test_products_at_tile_edges(ctx, naux, nbf, nocc, shape, precision):
    import paper_2210_17093_amd.qsgw as q
    prec, u = {"fp64": (q.PREC_FP64, 2.0 ** -53), "fp32": (q.PREC_FP32, 2.0 ** -24)}[precision]
    mo2 = shape if shape != "128x64" else "64x64"
    ctx.set_tiles(shape and f"mo1={shape},mo2={mo2},casida={mo2},rho={shape},sigma={shape},"
                  "rho_target=64")
    try:
        g = torch.Generator().manual_seed(naux * 1000 + nbf)
        B = torch.randn(naux, nbf, nbf, generator=g, dtype=F64)
        B = B + B.transpose(1, 2)
        C = torch.randn(nbf, nbf, generator=g, dtype=F64)
        ntr = nocc * (nbf - nocc)
        s0, ns = min(2, ntr - 1), max(1, ntr - 3)
        eps = torch.cat([-2.0 - torch.rand(nocc, generator=g, dtype=F64),
                         1.0 + torch.rand(nbf - nocc, generator=g, dtype=F64)])
        Z = torch.randn(ntr, ntr, generator=g, dtype=F64)
        Om = 1.0 + torch.rand(ntr, generator=g, dtype=F64)
        Bd = _guarded(B)
        Bmo = q.qsgw_mo_transform(ctx, Bd, _guarded(C), precision=prec)
        M, sd = q.qsgw_rpa_build(ctx, Bd, _guarded(eps), nocc, precision=prec)
        w = q.qsgw_residues(ctx, Bd, _guarded(sd), _guarded(Z), _guarded(Om), nocc, s0, ns,
                            precision=prec)
        V = q.qsgw_sigma_qs(ctx, _guarded(w), _guarded(eps), _guarded(Om[s0:s0 + ns]), nocc, 0.5)
        torch.cuda.synchronize()
        Bmo, M, sd, w, V = (t.cpu() for t in (Bmo, M, sd, w, V))
    finally:
        ctx.set_tiles(None)

    # each sum of K products of rounded factors is off by at most (K + 6) u of
    # the sum of its terms' sizes; 10 covers the scalings before and after it
    def close(got, ref, size, K):
        assert torch.all((got - ref).abs() <= (K + 10) * u * size + 64 * 2.0 ** -53 * size)

    close(Bmo, C.T @ B @ C, C.abs().T @ B.abs() @ C.abs(), 2 * nbf)
    D = (eps[None, nocc:] - eps[:nocc, None]).reshape(-1)
    X = B[:, :nocc, nocc:].reshape(naux, -1) * D.sqrt()
    close(M, 4.0 * (X.T @ X) + torch.diag(D * D), 4.0 * (X.abs().T @ X.abs()) + torch.diag(D * D),
          naux)
    Zs, Os = Z[s0:s0 + ns], Om[s0:s0 + ns]
    rho = (X @ Zs.T) * torch.sqrt(2.0 / Os)
    rho_size = (X.abs() @ Zs.abs().T) * torch.sqrt(2.0 / Os)
    flat = B.reshape(naux, -1)
    close(w, (flat.T @ rho).reshape(nbf, nbf, ns),
          (flat.abs().T @ rho_size).reshape(nbf, nbf, ns), naux + ntr)
    sign = torch.where(torch.arange(nbf) < nocc, 1.0, -1.0).to(F64)
    x = eps[:, None, None] - eps[None, :, None] + sign[None, :, None] * Os[None, None, :]
    a = w * x / (x * x + 0.25)  # [m][k][s]
    G = a.reshape(nbf, -1) @ w.reshape(nbf, -1).T
    S = a.abs().reshape(nbf, -1) @ w.abs().reshape(nbf, -1).T
    # FP64 throughout; the pole's own rounding (terms below 16) moves a weight
    # by at most 4 u 16 / eta^2
    W = w.abs().reshape(nbf, -1) @ w.abs().reshape(nbf, -1).T
    off = (nbf * ns + 64) * 2.0 ** -53 * 0.5 * (S + S.T) + 4 * 2.0 ** -53 * 16 * 4.0 * W
    assert torch.all((V - 0.5 * (G + G.T)).abs() <= off)
