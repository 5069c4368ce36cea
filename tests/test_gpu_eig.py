"""The two-stage Casida eigensolver (QSGW_EIG_TWO_STAGE: dense -> band ->
tridiagonal -> divide and conquer -> both back-transformations) against the
oracle's dense eigensolve of the same Casida matrix (Eq. (12) in Hermitian
form, scipy eigh), through the C-ABI.

Sizes start at the smallest the two-stage path takes (256 transitions, four
panels of 64) and include ragged last panels, an auxiliary basis smaller
than the band (rank-deficient panels), a rank-one coupling, a matrix that is
already diagonal (every reflector trivial) and repeated transition energies
(degenerate eigenvalues).  Eigenvectors are compared through what is unique:
the eigenvalues, the eigen-residual and orthonormality, and the first qsGW
iteration that consumes them.
"""
import numpy as np
import pytest

import oracle as O
from qsgw_inputs import make_problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

QP_TOL = 1e-8  # Ha

SHAPES = [  # nbf, naux, nocc -> transitions
    (40, 160, 8),    # 256: four full panels
    (57, 120, 7),    # 350: ragged last panel
    (70, 280, 12),   # 696
    (90, 60, 13),    # 1001: N_aux = 60 < 64, every panel rank-deficient
    (130, 260, 17),  # 1921
]


@pytest.fixture(scope="module")
def q():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2210_17093_amd.qsgw as q
    return q


@pytest.fixture(scope="module")
def ctx(q):
    c = q.Context()
    c.set_eigensolver(q.EIG_TWO_STAGE)
    yield c
    c.close()


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def check_eigenpairs(M, Z, Om, Om_ref):
    """Z: rows are eigenvectors (row-major view of the column-major output)."""
    n = M.shape[0]
    np.testing.assert_allclose(Om, Om_ref, rtol=1e-11)
    assert np.max(np.abs(Z @ Z.T - np.eye(n))) <= 1e-11
    res = M @ Z.T - Z.T * (Om ** 2)[None, :]
    assert np.max(np.abs(res)) <= 1e-11 * np.abs(M).max()


@pytest.mark.parametrize("shape", SHAPES)
def test_two_stage_matches_oracle(q, ctx, shape):
    nbf, naux, nocc = shape
    print("two-stage eigensolve", shape, flush=True)
    p = make_problem(nbf, naux, nocc, max(1, naux // 2), 0.99, 3)
    B_mo = O.mo_transform(p.B_ao, p.C0)
    M_ref, sq_ref = O.rpa_hermitian(B_mo, p.eps0, nocc)
    Om_ref, _ = O.rpa_solve(M_ref, sq_ref)
    Z, Om = q.qsgw_rpa_solve(ctx, dev(M_ref))
    check_eigenpairs(M_ref, host(Z), host(Om), Om_ref)


def test_two_stage_rank_one_coupling(q, ctx):
    """N_aux = 1: M = Delta^2 + u u^T, every panel below the band has rank <= 1."""
    print("two-stage eigensolve, rank-one coupling", flush=True)
    p = make_problem(60, 1, 9, 1, 0.99, 5, coupling=1.0)
    B_mo = O.mo_transform(p.B_ao, p.C0)
    M_ref, sq_ref = O.rpa_hermitian(B_mo, p.eps0, 9)
    Om_ref, _ = O.rpa_solve(M_ref, sq_ref)
    Z, Om = q.qsgw_rpa_solve(ctx, dev(M_ref))
    check_eigenpairs(M_ref, host(Z), host(Om), Om_ref)


def test_two_stage_diagonal_matrix(q, ctx):
    """No coupling (B_mo = 0): M = diag(Delta^2), every reflector is the identity;
    the eigenvectors are signed unit vectors."""
    print("two-stage eigensolve, diagonal matrix", flush=True)
    nbf, nocc = 50, 8
    eps = np.concatenate([np.sort(np.random.default_rng(1).uniform(-30, -0.3, nocc)),
                          np.sort(np.random.default_rng(2).uniform(0.05, 20, nbf - nocc))])
    M_ref, sq_ref = O.rpa_hermitian(np.zeros((3, nbf, nbf)), eps, nocc)
    Om_ref, _ = O.rpa_solve(M_ref, sq_ref)
    Z, Om = q.qsgw_rpa_solve(ctx, dev(M_ref))
    Zh = host(Z)
    check_eigenpairs(M_ref, Zh, host(Om), Om_ref)
    np.testing.assert_allclose(np.abs(Zh).max(axis=1), 1.0, atol=1e-13)


def test_two_stage_degenerate_eigenvalues(q, ctx):
    """Evenly spaced orbital energies repeat every transition energy many
    times; a rank-two coupling lifts only part of each degeneracy."""
    print("two-stage eigensolve, degenerate eigenvalues", flush=True)
    nbf, nocc = 48, 8
    eps = np.concatenate([-1.0 - 0.5 * np.arange(nocc)[::-1], 0.5 + 0.5 * np.arange(nbf - nocc)])
    rng = np.random.default_rng(4)
    B = 0.05 * rng.standard_normal((2, nbf, nbf))
    B = 0.5 * (B + B.transpose(0, 2, 1))
    M_ref, sq_ref = O.rpa_hermitian(B, eps, nocc)
    Om_ref, _ = O.rpa_solve(M_ref, sq_ref)
    assert np.sum(np.diff(Om_ref) < 1e-12) > 100  # many exact multiplets
    Z, Om = q.qsgw_rpa_solve(ctx, dev(M_ref))
    check_eigenpairs(M_ref, host(Z), host(Om), Om_ref)


def test_two_stage_inside_iteration(q, ctx):
    """One qsGW iteration with the two-stage Casida eigensolve against the
    oracle step (quasiparticle energies to 1e-8 Ha)."""
    print("two-stage eigensolve inside qsgw_iterate", flush=True)
    nbf, naux, nocc = 70, 280, 12
    p = make_problem(nbf, naux, nocc, naux // 2, 0.99, 0)
    h_ref = O.hf_core(p.B_ao, p.C0, p.eps0, nocc)
    st = O.qsgw_step(p.B_ao, h_ref, p.C0, p.eps0, nocc, 1e-3)
    B = dev(p.B_ao)
    C = dev(p.C0.copy())
    e = dev(p.eps0.copy())
    h = q.qsgw_hf_core(ctx, B, C, e, nocc)
    q.qsgw_iterate(ctx, B, h, nocc, e, C, 1e-3, tol=0.0, max_iter=1)
    assert np.max(np.abs(host(e) - st["eps"])) <= QP_TOL


def test_eigensolver_choice_errors(q, ctx):
    with pytest.raises(q.QsgwError):
        ctx.set_eigensolver(7)
    ctx.set_eigensolver(q.EIG_TWO_STAGE)


def test_two_stage_full_size_properties(q):
    """The 10,400-transition Casida matrix of the N_b = 300 workload: the
    eigen-residual and orthonormality of the two-stage result (FP64 products
    on the device), its eigenvalues against rocSOLVER's one-stage dsyevd, and
    the trace identity sum Omega^2 = tr M."""
    from qsgw_inputs import make_config
    print("two-stage eigensolve at 10,400 transitions", flush=True)
    p = make_config("cfg2")
    d = torch.device("cuda:0")
    with q.Context() as c:
        B_mo = q.qsgw_mo_transform(c, torch.from_numpy(p.B_ao).to(d), torch.from_numpy(p.C0).to(d))
        M, _ = q.qsgw_rpa_build(c, B_mo, torch.from_numpy(p.eps0).to(d), p.nocc)
        del B_mo
        c.set_eigensolver(q.EIG_ROCSOLVER)
        _, Om1 = q.qsgw_rpa_solve(c, M.clone())
        c.set_eigensolver(q.EIG_TWO_STAGE)
        Z, Om2 = q.qsgw_rpa_solve(c, (Mc := M.clone()))
        n = p.ntr
        lam = Om2 * Om2
        R = torch.mm(M, Z.T) - Z.T * lam[None, :]
        resid = float(R.abs().max() / M.abs().max())
        del R
        G = torch.mm(Z, Z.T)
        G.diagonal().sub_(1.0)
        orth = float(G.abs().max())
        del G, Mc
        rel = float(((Om2 - Om1).abs() / Om1).max())
        tr = float(M.diagonal().sum())
        torch.cuda.synchronize()
    print(f"  residual {resid:.2e}, orthonormality {orth:.2e}, eigenvalues vs dsyevd {rel:.2e}",
          flush=True)
    assert resid <= 1e-11 and orth <= 1e-11 and rel <= 1e-11
    assert abs(float(lam.sum()) - tr) <= 1e-12 * tr


@pytest.mark.parametrize("prec,s_block", [("fp64", 0), ("fp64", 200), ("fp32", 0), ("fp32", 250),
                                          ("bf16x3", 0), ("bf16x3", 300)])
def test_projected_iteration_matches_oracle(q, ctx, prec, s_block):
    """qsgw_iterate with the two-stage solver hands the residue step rho' of
    every excitation straight from the eigensolver (projection of Bt on the
    eigenvectors, Z never formed): one iteration against the oracle step,
    FP64 to 1e-8 Ha and the reduced-precision products to 1 meV, in one
    excitation block or in streamed blocks with a ragged last one; the
    diagonal outputs against the oracle's definition; a replayed iteration
    reproduces the full one bitwise."""
    print("projected iteration", prec, s_block, flush=True)
    nbf, naux, nocc = 70, 200, 11
    eta = 1e-3
    p = make_problem(nbf, naux, nocc, naux // 2, 0.99, 0)
    h_ref = O.hf_core(p.B_ao, p.C0, p.eps0, nocc)
    st = O.qsgw_step(p.B_ao, h_ref, p.C0, p.eps0, nocc, eta)
    pr = {"fp64": q.PREC_FP64, "fp32": q.PREC_FP32, "bf16x3": q.PREC_SPLIT_BF16}[prec]
    B = dev(p.B_ao)
    C = dev(p.C0.copy())
    e = dev(p.eps0.copy())
    h = q.qsgw_hf_core(ctx, B, C, e, nocc)
    diag = torch.zeros((nbf, 4), dtype=torch.float64, device="cuda")
    q.qsgw_iterate(ctx, B, h, nocc, e, C, eta, tol=0.0, max_iter=1, precision=pr, s_block=s_block,
                   diag=diag)
    err = np.max(np.abs(host(e) - st["eps"]))
    assert err <= (QP_TOL if prec == "fp64" else 1.0 / 27211.386), err
    if prec == "fp64":
        d = host(diag)
        for m in (0, nocc - 1, nocc, nbf - 1):
            ref = O.sigma_element(st["w"], p.eps0, st["Omega"], nocc, eta, m, m, [p.eps0[m]])[0]
            assert abs(d[m, 0] - ref.real) <= 1e-8 * max(1.0, abs(ref.real))
            assert abs(d[m, 1] - ref.imag) <= 1e-8 * max(1.0, abs(ref.imag))
    e_full = host(e)
    e2, C2 = dev(p.eps0.copy()), dev(p.C0.copy())
    q.qsgw_iterate(ctx, B, h, nocc, e2, C2, eta, tol=0.0, max_iter=1, precision=pr,
                   s_block=s_block, replay_eig=True)
    np.testing.assert_array_equal(host(e2), e_full)


@pytest.mark.parametrize("case", ["degenerate", "rank_one", "uncoupled"])
def test_projected_iteration_deflation(q, ctx, case):
    """The projection's tridiagonal merge deflates most of its poles when the
    Casida spectrum is degenerate (evenly spaced orbital energies: every
    transition energy repeats), when the coupling has rank one (N_aux = 1) and
    when there is almost none (the torn tridiagonal is nearly diagonal): one
    qsgw_iterate step against the oracle step to 1e-8 Ha."""
    print("projected iteration with deflation:", case, flush=True)
    if case == "degenerate":
        # a rank-two coupling lifts only part of each multiplet: 185 of the 320
        # eigenvalues repeat
        nbf, naux, nocc = 48, 2, 8
        p = make_problem(nbf, naux, nocc, 2, 0.99, 6, coupling=0.05)
        eps0 = np.concatenate([-1.0 - 0.5 * np.arange(nocc)[::-1],
                               0.5 + 0.5 * np.arange(nbf - nocc)])
    elif case == "rank_one":
        nbf, naux, nocc = 60, 1, 9
        p = make_problem(nbf, naux, nocc, 1, 0.99, 5, coupling=1.0)
        eps0 = p.eps0
    else:
        nbf, naux, nocc = 50, 30, 8
        p = make_problem(nbf, naux, nocc, 15, 0.99, 7, coupling=1e-7)
        eps0 = p.eps0
    eta = 1e-3
    h_ref = O.hf_core(p.B_ao, p.C0, eps0, nocc)
    st = O.qsgw_step(p.B_ao, h_ref, p.C0, eps0, nocc, eta)
    B = dev(p.B_ao)
    C = dev(p.C0.copy())
    e = dev(eps0.copy())
    h = q.qsgw_hf_core(ctx, B, C, e, nocc)
    q.qsgw_iterate(ctx, B, h, nocc, e, C, eta, tol=0.0, max_iter=1)
    assert np.max(np.abs(host(e) - st["eps"])) <= QP_TOL


@pytest.mark.parametrize("leaf,case", [(64, "random"), (16, "degenerate"), (40, "rank_one")])
def test_projected_divide_and_conquer_levels(q, ctx, leaf, case):
    """The projection's divide and conquer with small leaves (tile table key
    dc_leaf), so that merges of merged halves run (four to five levels, each
    half carrying the unit column whose projection is its boundary row): one
    qsgw_iterate step against the oracle step to 1e-8 Ha."""
    print("projected divide and conquer, leaf", leaf, case, flush=True)
    if case == "random":
        nbf, naux, nocc = 70, 280, 12
        p = make_problem(nbf, naux, nocc, naux // 2, 0.99, 0)
        eps0 = p.eps0
    elif case == "degenerate":
        nbf, naux, nocc = 48, 2, 8
        p = make_problem(nbf, naux, nocc, 2, 0.99, 6, coupling=0.05)
        eps0 = np.concatenate([-1.0 - 0.5 * np.arange(nocc)[::-1],
                               0.5 + 0.5 * np.arange(nbf - nocc)])
    else:
        nbf, naux, nocc = 60, 1, 9
        p = make_problem(nbf, naux, nocc, 1, 0.99, 5, coupling=1.0)
        eps0 = p.eps0
    eta = 1e-3
    h_ref = O.hf_core(p.B_ao, p.C0, eps0, nocc)
    st = O.qsgw_step(p.B_ao, h_ref, p.C0, eps0, nocc, eta)
    B = dev(p.B_ao)
    C = dev(p.C0.copy())
    e = dev(eps0.copy())
    h = q.qsgw_hf_core(ctx, B, C, e, nocc)
    ctx.set_tiles(f"dc_leaf={leaf}")
    try:
        assert f"dc_leaf={leaf}" in ctx.get_tiles()
        q.qsgw_iterate(ctx, B, h, nocc, e, C, eta, tol=0.0, max_iter=1)
    finally:
        ctx.set_tiles(None)
    assert np.max(np.abs(host(e) - st["eps"])) <= QP_TOL


def test_projected_iteration_per_column_panels(q, ctx):
    """The dense -> band stage with the per-column panel launches (tile table
    panel_coop=0) instead of the cooperative one, and both divide-and-conquer
    depths: one qsgw_iterate step against the oracle step to 1e-8 Ha."""
    print("projected iteration, per-column panel QR", flush=True)
    nbf, naux, nocc = 70, 280, 12
    p = make_problem(nbf, naux, nocc, naux // 2, 0.99, 0)
    h_ref = O.hf_core(p.B_ao, p.C0, p.eps0, nocc)
    st = O.qsgw_step(p.B_ao, h_ref, p.C0, p.eps0, nocc, 1e-3)
    B = dev(p.B_ao)
    C = dev(p.C0.copy())
    e = dev(p.eps0.copy())
    h = q.qsgw_hf_core(ctx, B, C, e, nocc)
    ctx.set_tiles("panel_coop=0,dc_leaf=100")
    try:
        assert "panel_coop=0" in ctx.get_tiles()
        q.qsgw_iterate(ctx, B, h, nocc, e, C, 1e-3, tol=0.0, max_iter=1)
    finally:
        ctx.set_tiles(None)
    assert np.max(np.abs(host(e) - st["eps"])) <= QP_TOL


@pytest.mark.parametrize("n", [256, 257, 258, 319, 320, 321, 322, 705])
def test_two_stage_window_edges(q, ctx, n):
    """Orders around the 64-row windows of the bulge chasing: a last window of
    one, two, 63 and 64 rows at the first sweep, and of every length later."""
    print("two-stage eigensolve, order", n, flush=True)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n))
    M_ref = A @ A.T / n + np.diag(np.linspace(1.0, 50.0, n))
    M_ref = 0.5 * (M_ref + M_ref.T)
    Z, Om = q.qsgw_rpa_solve(ctx, dev(M_ref))
    check_eigenpairs(M_ref, host(Z), host(Om), np.sqrt(np.linalg.eigvalsh(M_ref)))


def test_two_stage_tall_panels(q, ctx):
    """An order whose first panels are spread over more than 64 workgroups (a
    second round of partial sums a column): residual, norm and order of some of
    the eigenpairs, and the trace."""
    n = 16_577
    print("two-stage eigensolve, order", n, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randn(n, n, generator=g, dtype=torch.float64, device="cuda") / n ** 0.5
    A = 0.5 * (A + A.T)
    A.diagonal().add_(torch.linspace(10.0, 60.0, n, dtype=torch.float64, device="cuda"))
    Z, Om = q.qsgw_rpa_solve(ctx, A.clone())
    ev = Om * Om
    assert bool((ev[1:] >= ev[:-1]).all())
    assert abs(float(ev.sum() - A.diagonal().sum())) <= 1e-11 * n * 62
    some = torch.linspace(0, n - 1, 24, device="cuda").long()
    Zs = Z[some]  # rows are eigenvectors
    assert float((Zs @ Z.T - torch.eye(n, dtype=torch.float64, device="cuda")[some]).abs().max()) <= 1e-11
    assert float((Zs @ A - ev[some, None] * Zs).abs().max()) <= 1e-11 * 62


@pytest.mark.parametrize("n", [3073, 6143])
def test_two_stage_large_tridiagonals(q, ctx, n):
    """Orders of the two-stage solver whose whole tridiagonal problem is solved by
    the merges with formed eigenvectors, up to the largest: residual, norm and
    order of some of the eigenpairs, and the trace."""
    print("two-stage eigensolve, order", n, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn(n, n, generator=g, dtype=torch.float64, device="cuda") / n ** 0.5
    A = 0.5 * (A + A.T)
    A.diagonal().add_(torch.linspace(10.0, 60.0, n, dtype=torch.float64, device="cuda"))
    Z, Om = q.qsgw_rpa_solve(ctx, A.clone())
    ev = Om * Om
    assert bool((ev[1:] >= ev[:-1]).all())
    assert abs(float(ev.sum() - A.diagonal().sum())) <= 1e-11 * n * 62
    some = torch.linspace(0, n - 1, 24, device="cuda").long()
    Zs = Z[some]  # rows are eigenvectors
    eye = torch.eye(n, dtype=torch.float64, device="cuda")[some]
    assert float((Zs @ Z.T - eye).abs().max()) <= 1e-11
    assert float((Zs @ A - ev[some, None] * Zs).abs().max()) <= 1e-11 * 62


@pytest.mark.parametrize("n", [3073, 5001])
def test_automatic_solver_above_one_stage_orders(q, n):
    """The default choice just above the one-stage solver's orders and between:
    the two-stage solver, and still the lower triangle alone counts."""
    print("automatic eigensolver, order", n, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn(n, n, generator=g, dtype=torch.float64, device="cuda") / n ** 0.5
    A = 0.5 * (A + A.T)
    A.diagonal().add_(torch.linspace(10.0, 60.0, n, dtype=torch.float64, device="cuda"))
    given = torch.tril(A) + torch.triu(torch.ones_like(A), 1)
    with q.Context() as c:
        Z, Om = q.qsgw_rpa_solve(c, given)
        torch.cuda.synchronize()
    ev = Om * Om
    assert bool((ev[1:] >= ev[:-1]).all())
    some = torch.linspace(0, n - 1, 24, device="cuda").long()
    Zs = Z[some]
    eye = torch.eye(n, dtype=torch.float64, device="cuda")[some]
    assert float((Zs @ Z.T - eye).abs().max()) <= 1e-11
    assert float((Zs @ A - ev[some, None] * Zs).abs().max()) <= 1e-11 * 62
