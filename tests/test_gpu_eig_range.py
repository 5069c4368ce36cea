"""Values that leave the range of FP64 inside a call: the eigensolvers return an
error code or, where the eigenvalues themselves can be represented, the right
eigenpairs, and the context goes on working."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2210_17093_amd.qsgw as q
    return q


@pytest.fixture()
def ctx(q):
    c = q.Context()
    yield c
    c.close()


def spd(n, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, max(2, n // 4))) * 0.3
    return np.diag(rng.uniform(0.1, 2500.0, n)) + X @ X.T


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def check_solve(q, ctx, M, scale=1.0):
    """Eigenpairs of scale * M (scale a power of two) against LAPACK's of M, with
    the bounds of the other eigensolver tests."""
    n = M.shape[0]
    ref = np.linalg.eigvalsh(M)
    Z, Om = q.qsgw_rpa_solve(ctx, dev(M * scale))
    torch.cuda.synchronize()
    norm = np.abs(ref).max()
    bound = 1e-13 * max(4.0, np.sqrt(n))
    lam = (Om.cpu().numpy() / np.sqrt(scale)) ** 2
    assert np.max(np.abs(lam - ref)) <= bound * norm
    assert float((Z @ Z.T - torch.eye(n, dtype=torch.float64, device="cuda")).abs().max()) <= bound
    assert float((Z @ dev(M) - dev(lam)[:, None] * Z).abs().max()) <= bound * norm


@pytest.mark.parametrize("nbf", [40, 80, 300])
def test_overflow_before_the_eigensolve_is_an_error(q, ctx, nbf):
    """C^T h C overflows, so the Fock matrix is not finite."""
    print("fock overflow", nbf, flush=True)
    eye = np.eye(nbf)
    h = spd(nbf, nbf) * 1e200
    args = [dev(np.zeros((3, nbf, nbf))), dev(np.zeros((3, nbf, nbf))), dev(h), dev(0.0 * eye),
            dev(0.0 * eye), 4, 3, dev(np.zeros(nbf)), dev(np.zeros(nbf)), dev(eye * 1e60),
            dev(eye * 1e60)]
    with pytest.raises(q.QsgwError) as ei:
        q.qsgw_fock_unrestricted(ctx, *args)
    assert ei.value.code == q.ERR_NONFINITE and "not finite" in str(ei.value)
    check_solve(q, ctx, spd(nbf, 1))


def test_batch_with_a_zero_gap_names_the_molecule(q):
    """A molecule of 80 functions whose HOMO and LUMO are equal: its Casida matrix
    has a zero eigenvalue.  The call says which molecule it is, and the others of
    the batch take their iteration as they do alone."""
    from qsgw_inputs import make_problem
    stream = torch.cuda.Stream()
    c = q.Context(stream)
    try:
        mols, alone = [], []
        with torch.cuda.stream(stream):
            for nbf, seed in ((33, 1), (80, 2), (20, 3), (95, 4)):
                p = make_problem(nbf, 4 * nbf, nbf // 6, 2 * nbf, 0.99, 900 + seed)
                B, C, e = dev(p.B_ao), dev(p.C0), p.eps0.copy()
                h = q.qsgw_hf_core(c, B, C, dev(e), p.nocc)
                if nbf == 80:
                    e[p.nocc] = e[p.nocc - 1]
                else:
                    e1, C1 = dev(e), C.clone()
                    q.qsgw_iterate(c, B, h, p.nocc, e1, C1, 1e-3, tol=0.0, max_iter=1)
                    alone.append(e1)
                mols.append(dict(B_ao=B, h=h, nocc=p.nocc, eps=dev(e), C=C.clone()))
            print("batch with a zero gap", flush=True)
            with pytest.raises(q.QsgwError) as ei:
                q.qsgw_iterate_batched(c, mols, 1e-3, tol=0.0, max_iter=1)
        assert ei.value.code == q.ERR_INVALID_ARG and "molecule 1:" in str(ei.value)
        good = [m["eps"] for m in mols if m["eps"].shape[0] != 80]
        for a, b in zip(alone, good):
            assert float((a - b).abs().max()) <= 1e-8
        stream.synchronize()
    finally:
        c.close()


@pytest.mark.parametrize("n", [1, 5, 24, 95, 300, 1100, 3200])
@pytest.mark.parametrize("power", [-1000, -600, 600, 1000])
def test_entries_whose_squares_leave_the_range(q, ctx, n, power):
    """A matrix of entries near 2^power (orders on both sides of the solvers' limit)."""
    print("eigensolve of 2^%d, order %d" % (power, n), flush=True)
    check_solve(q, ctx, spd(n, n), 2.0 ** power)


@pytest.mark.parametrize("n", [24, 95, 300, 3200])
@pytest.mark.parametrize("t", [1e-150, 1e-156, 1e-159, 1e-162, 1e-200])
def test_couplings_whose_squares_underflow(q, ctx, n, t):
    """Columns whose sums of squares are zero or have lost their bits."""
    print("eigensolve with couplings of %g, order %d" % (t, n), flush=True)
    M = spd(n, n)
    M[n // 3:, :n // 3] *= t
    M[:n // 3, n // 3:] *= t
    M[n // 3:, n // 3:] = np.diag(np.diag(M)[n // 3:]) + t * (M[n // 3:, n // 3:])
    check_solve(q, ctx, M)


@pytest.mark.parametrize("nbf", [24, 120, 300])
def test_blocks_of_very_different_scale(q, ctx, nbf):
    """A symmetric matrix (the core Hamiltonian of a call without interaction) of
    four blocks down to the smallest normal numbers: its eigenvectors are
    orthonormal and its residuals small beside its largest eigenvalue."""
    print("blocks of different scale", nbf, flush=True)
    h = np.zeros((nbf, nbf))
    k = nbf // 4
    for b, s in enumerate((1.0, 1e-152, 1e-163, 1e-304)):
        o = b * k
        A = spd(k, b + 1)
        h[o:o + k, o:o + k] = s * (A - 0.5 * np.diag(np.diag(A)))
    eye = np.eye(nbf)
    Ca, Cb, ea, eb = dev(eye), dev(eye), dev(np.zeros(nbf)), dev(np.zeros(nbf))
    zero = dev(np.zeros((3, nbf, nbf)))
    q.qsgw_fock_unrestricted(ctx, zero, zero, dev(h), dev(0.0 * eye), dev(0.0 * eye), 4, 3, ea, eb,
                             Ca, Cb)
    ref = np.linalg.eigvalsh(h)
    norm = np.abs(ref).max()
    bound = 1e-13 * max(4.0, np.sqrt(nbf))
    for C, e in ((Ca, ea), (Cb, eb)):
        assert float((C.T @ C - dev(eye)).abs().max()) <= bound
        assert float((dev(h) @ C - C * e[None, :]).abs().max()) <= bound * norm
        assert np.max(np.abs(e.cpu().numpy() - ref)) <= bound * norm


@pytest.mark.parametrize("iters", [1, 3])
def test_batch_reports_the_eigensolve_that_failed(q, iters):
    """A Fock matrix of a batch overflows: the call says so and names the molecule,
    whatever the numbers that the eigensolve leaves look like afterwards."""
    from qsgw_inputs import make_problem
    stream = torch.cuda.Stream()
    c = q.Context(stream)
    try:
        mols = []
        with torch.cuda.stream(stream):
            for nbf, seed in ((33, 1), (80, 2), (20, 3)):
                p = make_problem(nbf, 4 * nbf, nbf // 6, 2 * nbf, 0.99, 900 + seed)
                B, C, e = dev(p.B_ao), dev(p.C0), dev(p.eps0)
                h = q.qsgw_hf_core(c, B, C, e, p.nocc)
                if nbf == 80:
                    h, C = torch.full_like(h, 1e308), C * 1e3
                mols.append(dict(B_ao=B, h=h, nocc=p.nocc, eps=e, C=C))
            print("batch with a Fock matrix that overflows", iters, flush=True)
            with pytest.raises(q.QsgwError) as ei:
                q.qsgw_iterate_batched(c, mols, 1e-3, tol=0.0, max_iter=iters)
        assert ei.value.code == q.ERR_NONFINITE
        assert "molecule 1: batched Fock eigensolve" in str(ei.value)
    finally:
        c.close()
