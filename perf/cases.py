"""Timed workloads of libqsgw, called through its public entry points.

Every case is something a program built on the library does: whole qsGW
iterations of one molecule (closed or open shell, each precision variant), a
batch of uneven molecules, the stages called one by one, a streamed residue
block of the 600-basis workload, the qsMP2 potential, the four-index transform
and one training step plus inference of the warm-start network.  Inputs follow
the recipe of ``qsgw_inputs.generator`` (drawn on the GPU here): a symmetric RI
tensor, Haar-orthogonal orbitals, orbital energies in [-30, 20] Ha, and the
one-body matrix that makes them a Hartree-Fock fixed point.

``exact`` restates each case in plain FP64 torch without the library.
"""
import math

import torch

from paper_2210_17093_amd import qsgw as q

DEV = "cuda:0"
F64 = torch.float64
F32 = torch.float32
PREC = {"fp64": q.PREC_FP64, "fp32": q.PREC_FP32, "split_bf16": q.PREC_SPLIT_BF16}
COUPLING = 0.1  # the generator's coupling scale
PAD = 32  # packed per-molecule arrays start on multiples of this many values

_kept = {}


def _session():
    """The one stream and library context a program keeps for its life."""
    if not _kept:
        _kept["stream"] = torch.cuda.Stream()
        _kept["ctx"] = q.Context(_kept["stream"])
    return _kept["stream"], _kept["ctx"]


# ------------------------------------------------------------------ cases --
def listed():
    return [
        # the 24-basis workload stage by stage with the HOMO/LUMO spectral
        # functions on its 201-point grid: the smallest calls, all latency
        dict(name="stages_24", kind="stages", nbf=24, nocc=5, nomega=201),
        # one small molecule, FP32 matrix-core variant, two iterations
        dict(name="iterate_61_fp32", kind="iterate", nbf=61, nocc=10, precision="fp32", iters=2),
        # one ordinary molecule of odd size at the upper end of the batched distribution
        dict(name="iterate_117_fp64", kind="iterate", nbf=117, nocc=20, precision="fp64", iters=1),
        # a larger molecule, split-BF16 variant
        dict(name="iterate_213_split_bf16", kind="iterate", nbf=213, nocc=29,
             precision="split_bf16", iters=1),
        # the 300-basis workload, plain FP64 iteration with its Casida eigensolve
        dict(name="iterate_300_fp64", kind="iterate", nbf=300, nocc=40, precision="fp64", iters=1),
        # open-shell iteration of a doublet
        dict(name="open_shell_83", kind="open_shell", nbf=83, nocc=14, iters=1),
        # a batch of uneven molecules (20 to 120 basis functions) with hipGraph
        # segments, as the batched and learned workloads run them
        dict(name="batch_48_split_bf16", kind="batch", nmol=48, lo=20, hi=120, shapes=4,
             precision="split_bf16", iters=2, graph=True),
        # what precedes the eigensolve of a mid-size molecule: the MO transform
        # and the Casida matrix of 18,232 transitions
        dict(name="build_397_fp64", kind="build", nbf=397, nocc=53, precision="fp64"),
        # one streamed excitation block of the 600-basis workload (41,600
        # transitions): residues with their pole-weighted copy, qsGW product
        dict(name="block_600_fp64", kind="block", nbf=600, nocc=80, s_begin=20000, s_count=640,
             precision="fp64"),
        # the qsMP2 potential of one molecule
        dict(name="mp2_131", kind="mp2", nbf=131, nocc=22),
        # a slab of the four-index transform without the RI factorisation
        dict(name="ao2mo_150_slab_24", kind="ao2mo", nbf=150, slab=24),
        # the warm-start network: one Adam step on the training protocol's
        # minibatch of 4096 states and BF16 inference over a held-out batch
        dict(name="learn_4096", kind="learn", rows=4096, infer=17920),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("stages", "iterate", "iterate", "iterate", "open_shell", "batch", "build",
                       "block", "mp2", "ao2mo", "learn"))
    if kind == "stages":
        nbf = rng.randint(12, 60)
        return dict(kind=kind, nbf=nbf, nocc=_occ(rng, nbf), nomega=rng.randint(1, 301))
    if kind == "iterate":
        nbf = _log_int(rng, 20, 230)
        return dict(kind=kind, nbf=nbf, nocc=_occ(rng, nbf), iters=rng.randint(1, 2),
                    precision=rng.choice(sorted(PREC)))
    if kind == "open_shell":
        nbf = _log_int(rng, 20, 110)
        return dict(kind=kind, nbf=nbf, nocc=max(2, _occ(rng, nbf)), iters=1)
    if kind == "batch":
        lo = rng.randint(12, 60)
        return dict(kind=kind, nmol=_log_int(rng, 2, 48), lo=lo, hi=rng.randint(lo + 10, 120),
                    shapes=rng.randint(0, 10 ** 6), precision=rng.choice(sorted(PREC)),
                    iters=rng.randint(1, 2), graph=rng.random() < 0.5)
    if kind == "build":
        nbf = _log_int(rng, 60, 400)
        return dict(kind=kind, nbf=nbf, nocc=round(nbf / 7.5), precision=rng.choice(sorted(PREC)))
    if kind == "block":
        nbf = _log_int(rng, 60, 600)
        nocc = round(nbf / 7.5)
        count = rng.randint(64, 640)
        return dict(kind=kind, nbf=nbf, nocc=nocc, s_count=count, precision="fp64",
                    s_begin=rng.randint(0, nocc * (nbf - nocc) - count))
    if kind == "mp2":
        nbf = _log_int(rng, 20, 150)
        return dict(kind=kind, nbf=nbf, nocc=_occ(rng, nbf))
    if kind == "ao2mo":
        nbf = _log_int(rng, 20, 150)
        return dict(kind=kind, nbf=nbf, slab=rng.randint(1, min(nbf, 40)))
    return dict(kind=kind, rows=_log_int(rng, 64, 4096), infer=_log_int(rng, 20, 20000))


def _occ(rng, nbf):
    return max(1, round(nbf / rng.uniform(5.5, 8.0)))


def _batch_shapes(case):
    """(nbf, nocc) of each molecule: nbf uniform in [lo, hi], nocc = round(nbf / 6)."""
    g = torch.Generator().manual_seed(case["shapes"])
    nbf = torch.randint(case["lo"], case["hi"] + 1, (case["nmol"],), generator=g).tolist()
    return [(n, int(n / 6.0 + 0.5)) for n in nbf]


# ----------------------------------------------------------------- inputs --
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, dtype=F64, device=DEV)


def _energies(g, nbf, nocc):
    occ = -30.0 + 29.7 * torch.rand(nocc, generator=g, dtype=F64, device=DEV)
    virt = 0.05 + 19.95 * torch.rand(nbf - nocc, generator=g, dtype=F64, device=DEV)
    return torch.cat([occ.sort().values, virt.sort().values])


def _haar(g, n):
    Q, R = torch.linalg.qr(_normal(g, n, n))
    return (Q * torch.sign(torch.diagonal(R))).contiguous()


def _ri_tensor(g, nbf, decay=0.99):
    """B^P_mn = sum_r L_Pr U_rm U_rn with N_aux = 4 nbf, rank 2 nbf."""
    naux, rank = 4 * nbf, 2 * nbf
    U = _normal(g, rank, nbf)
    Q, _ = torch.linalg.qr(_normal(g, naux, rank))
    s = decay ** torch.arange(rank, dtype=F64, device=DEV)
    s = s * math.sqrt(COUPLING * 0.5 / (3.0 * float((s * s).sum())))
    B = ((Q * s) @ (U[:, :, None] * U[:, None, :]).reshape(rank, nbf * nbf)).reshape(naux, nbf, nbf)
    return (0.5 * (B + B.transpose(1, 2))).contiguous()


def _mean_field(B, C_s, nocc_s):
    """J of both spins' density and K of each spin's, AO basis."""
    D_s = [C[:, :no] @ C[:, :no].T for C, no in zip(C_s, nocc_s)]
    flat = B.reshape(B.shape[0], -1)
    J = ((flat @ sum(D_s).reshape(-1)) @ flat).reshape(B.shape[1:])
    K = []
    for C, no in zip(C_s, nocc_s):
        X = (B.reshape(-1, B.shape[1]) @ C[:, :no]).reshape(B.shape[0], B.shape[1], no)
        X = X.transpose(0, 1).reshape(B.shape[1], -1)
        K.append(X @ X.T)
    return J, K


def _molecule(g, nbf, nocc):
    """(B_ao, h, eps0, C0): a Hartree-Fock fixed point of the drawn integrals."""
    B = _ri_tensor(g, nbf)
    eps = _energies(g, nbf, nocc)
    C = _haar(g, nbf)
    J, K = _mean_field(B, [C, C], [nocc, nocc])
    h = (C * eps) @ C.T - J + K[0]
    return B, (0.5 * (h + h.T)).contiguous(), eps, C


def _inputs(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind in ("stages", "iterate", "open_shell"):
        return dict(zip(("B", "h", "eps", "C"), _molecule(g, case["nbf"], case["nocc"])))
    if kind == "batch":
        return dict(mols=[_molecule(g, n, no) for n, no in _batch_shapes(case)])
    if kind == "build":
        nbf, nocc = case["nbf"], case["nocc"]
        return dict(B=_ri_tensor(g, nbf), eps=_energies(g, nbf, nocc), C=_haar(g, nbf))
    if kind == "block":
        nbf, nocc = case["nbf"], case["nocc"]
        ntr = nocc * (nbf - nocc)
        eps = _energies(g, nbf, nocc)
        delta = (eps[None, nocc:] - eps[:nocc, None]).reshape(-1)
        v = _normal(g, ntr)
        v /= v.norm()
        Z = torch.outer(-2.0 * v, v)  # a reflection: orthogonal, dense
        Z.diagonal().add_(1.0)
        return dict(B=_ri_tensor(g, nbf), eps=eps, Z=Z, sqrt_delta=delta.sqrt(),
                    Omega=(delta.sort().values * 1.01 + 0.01).contiguous())
    if kind == "mp2":
        nbf, nocc = case["nbf"], case["nocc"]
        G = _normal(g, 4 * nbf, nbf, nbf)
        B = math.sqrt(COUPLING * 0.5 / (4 * nbf)) * 0.5 * (G + G.transpose(1, 2))
        return dict(B=B.contiguous(), eps=_energies(g, nbf, nocc))
    if kind == "ao2mo":
        nbf = case["nbf"]
        flat = _ri_tensor(g, nbf).reshape(-1, nbf * nbf)
        return dict(eri=(flat.T @ flat).reshape(nbf, nbf, nbf, nbf), C=_haar(g, nbf))

    def uniform(n, fan):
        return (2.0 * torch.rand(n, generator=g, dtype=F32, device=DEV) - 1.0) / math.sqrt(fan)
    z = torch.zeros(128, dtype=F32, device=DEV)
    P = torch.cat([uniform(128 * 16, 16), z, uniform(128 * 128, 128), z, uniform(128, 128), z[:1]])
    X = torch.randn(case["rows"], 16, generator=g, dtype=F32, device=DEV)
    T = torch.randn(case["rows"], generator=g, dtype=F32, device=DEV)
    Xi = torch.randn(case["infer"], 16, generator=g, dtype=F32, device=DEV)
    return dict(P=P, X=X, T=T, Xi=Xi)


def _padded(n):
    return (n + PAD - 1) // PAD * PAD


def prepare(case, seed):
    stream, ctx = _session()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        s = dict(_inputs(case, seed), case=case)
        kind = case["kind"]
        if kind == "stages":
            s["omega"] = torch.linspace(-2.0, 2.0, case["nomega"], dtype=F64, device=DEV)
            s["states"] = torch.tensor([case["nocc"] - 1, case["nocc"]], device=DEV)
        elif kind == "iterate":
            s.update(e=s["eps"].clone(), Cw=s["C"].clone(), Vc=torch.zeros_like(s["C"]))
        elif kind == "open_shell":
            s.update(e=[s["eps"].clone() for _ in "ab"], Cw=[s["C"].clone() for _ in "ab"])
        elif kind == "batch":
            # every molecule's energies and orbitals as slices of one buffer
            sizes = [(_padded(e.numel()), _padded(C.numel())) for _, _, e, C in s["mols"]]
            start = torch.zeros(sum(a + b for a, b in sizes), dtype=F64, device=DEV)
            work = start.clone()
            runs, at = [], 0
            for (B, h, e, C), (a, b) in zip(s["mols"], sizes):
                n = e.numel()
                start[at:at + n] = e
                start[at + a:at + a + n * n] = C.reshape(-1)
                runs.append(dict(B_ao=B, h=h, eps=work[at:at + n],
                                 C=work[at + a:at + a + n * n].view(n, n)))
                at += a + b
            for r, (_, no) in zip(runs, _batch_shapes(case)):
                r["nocc"] = no
            s.update(start=start, work=work, runs=runs)
        elif kind == "build":
            n, ntr = case["nbf"], case["nocc"] * (case["nbf"] - case["nocc"])
            s.update(B_mo=torch.empty_like(s["B"]),
                     M=torch.empty(ntr, ntr, dtype=F64, device=DEV),
                     sd=torch.empty(ntr, dtype=F64, device=DEV))
        elif kind == "block":
            s["w"] = torch.empty(case["nbf"], case["nbf"], case["s_count"], dtype=F64, device=DEV)
            s["V"] = torch.zeros(case["nbf"], case["nbf"], dtype=F64, device=DEV)
        elif kind == "ao2mo":
            s["out"] = torch.empty((case["slab"],) + (case["nbf"],) * 3, dtype=F64, device=DEV)
        elif kind == "learn":
            s.update(Pw=s["P"].clone(), m=torch.zeros_like(s["P"]), v=torch.zeros_like(s["P"]),
                     grad=torch.empty_like(s["P"]), loss=torch.empty(1, dtype=F64, device=DEV))
    torch.cuda.current_stream().wait_stream(stream)
    return s


# -------------------------------------------------------------------- run --
ETA = 0.05  # the paper's qsGW broadening (Ha), at which the iteration converges
ETA_BLOCK = 1e-3  # the stated broadening of the 600-basis workload
LR = 2e-3


def run(s):
    stream, ctx = _session()
    with torch.cuda.stream(stream):
        return _RUN[s["case"]["kind"]](ctx, s, s["case"])


def _run_stages(ctx, s, c):
    nocc = c["nocc"]
    B_mo = q.qsgw_mo_transform(ctx, s["B"], s["C"])
    M, sd = q.qsgw_rpa_build(ctx, B_mo, s["eps"], nocc)
    Z, Om = q.qsgw_rpa_solve(ctx, M)
    w, wh = q.qsgw_residues(ctx, B_mo, sd, Z, Om, nocc, weighted=True, eps=s["eps"], eta=ETA)
    V = q.qsgw_sigma_qs(ctx, w, s["eps"], Om, nocc, ETA, wh=wh)
    spec = q.qsgw_sigma_diag(ctx, w, s["eps"], Om, nocc, ETA, s["omega"], s["states"])
    self_ = q.qsgw_sigma_diag_self(ctx, w, s["eps"], Om, nocc, ETA, s["states"])
    return dict(Omega=Om, V=V, spec=spec, self=self_, B_mo=B_mo)


def _run_iterate(ctx, s, c):
    s["e"].copy_(s["eps"])
    s["Cw"].copy_(s["C"])
    q.qsgw_iterate(ctx, s["B"], s["h"], c["nocc"], s["e"], s["Cw"], ETA, tol=1e-6,
                   max_iter=c["iters"], Vc=s["Vc"], precision=PREC[c["precision"]])
    return dict(eps=s["e"], C=s["Cw"], Vc=s["Vc"])


def _run_open_shell(ctx, s, c):
    for e, C in zip(s["e"], s["Cw"]):
        e.copy_(s["eps"])
        C.copy_(s["C"])
    q.qsgw_iterate_unrestricted(ctx, s["B"], s["h"], c["nocc"], c["nocc"] - 1, s["e"][0],
                                s["Cw"][0], s["e"][1], s["Cw"][1], ETA, tol=1e-6,
                                max_iter=c["iters"])
    return dict(eps=s["e"], C=s["Cw"])


def _run_batch(ctx, s, c):
    s["work"].copy_(s["start"])
    q.qsgw_iterate_batched(ctx, s["runs"], ETA, tol=1e-6, max_iter=c["iters"], graph=c["graph"],
                           precision=PREC[c["precision"]])
    return s["work"]


def _run_build(ctx, s, c):
    p = PREC[c["precision"]]
    q.qsgw_mo_transform(ctx, s["B"], s["C"], B_mo=s["B_mo"], precision=p)
    q.qsgw_rpa_build(ctx, s["B_mo"], s["eps"], c["nocc"], M=s["M"], sqrt_delta=s["sd"], precision=p)
    return dict(B_mo=s["B_mo"], M=s["M"], sqrt_delta=s["sd"])


def _run_block(ctx, s, c):
    b, n = c["s_begin"], c["s_count"]
    w, wh = q.qsgw_residues(ctx, s["B"], s["sqrt_delta"], s["Z"], s["Omega"], c["nocc"], s_begin=b,
                            s_count=n, w=s["w"], weighted=True, eps=s["eps"], eta=ETA_BLOCK)
    V = q.qsgw_sigma_qs(ctx, w, s["eps"], s["Omega"][b:b + n], c["nocc"], ETA_BLOCK, out=s["V"],
                        wh=wh)
    return dict(w=w, wh=wh, V=V)


def _run_mp2(ctx, s, c):
    return q.qsgw_mp2_sigma(ctx, s["B"], s["eps"], c["nocc"], ETA)


def _run_ao2mo(ctx, s, c):
    return q.qsgw_ao2mo_4center(ctx, s["eri"], s["C"], m_count=c["slab"], out=s["out"])


def _run_learn(ctx, s, c):
    s["Pw"].copy_(s["P"])
    s["m"].zero_()
    s["v"].zero_()
    q.qsgw_mlp_train_step(ctx, s["Pw"], s["m"], s["v"], 1, LR, s["X"], s["T"], grad=s["grad"],
                          loss=s["loss"])
    y = q.qsgw_mlp_forward_bf16(ctx, s["P"], s["Xi"])
    return dict(params=s["Pw"], m=s["m"], v=s["v"], grad=s["grad"], loss=s["loss"], y=y)


_RUN = {"stages": _run_stages, "iterate": _run_iterate, "open_shell": _run_open_shell,
        "batch": _run_batch, "build": _run_build, "block": _run_block, "mp2": _run_mp2,
        "ao2mo": _run_ao2mo, "learn": _run_learn}


# ------------------------------------------------------------------- work --
def _iteration_work(nbf, nocc):
    """One closed-shell iteration: MO transform, Casida product, eigensolve
    (reduction 4/3 n^3 and the projection of N_aux columns), residues on pairs,
    qsGW product, Fock build and its eigensolve.  Bytes: B_ao and h read once."""
    b, a, t = float(nbf), 4.0 * nbf, float(nocc * (nbf - nocc))
    flops = (3 * b + 1) * b * b * a + t * (t + 1) * a + 4 / 3 * t ** 3 + 4 * t * t * a
    flops += b * (b + 1) * t * a + 2 * b ** 3 * t
    flops += b * (b + 1) * a * nocc + 2 * a * b * b + 12 * b ** 3
    return flops, 8 * (a * b * b + 6 * b * b)


def work(case):
    k = case["kind"]
    if k == "learn":
        n, m = case["rows"], case["infer"]
        w = 16 * 128 + 128 * 128 + 128
        return dict(flops=6.0 * n * w + 2.0 * m * w,
                    bytes=4.0 * (17 * (n + m) + 7 * q.MLP_NPARAMS))
    if k == "ao2mo":
        n, s = float(case["nbf"]), case["slab"]
        return dict(flops=8 * s * n ** 4, bytes=8 * (n ** 4 + s * n ** 3))
    if k == "batch":
        w = [_iteration_work(n, no) for n, no in _batch_shapes(case)]
        return dict(flops=case["iters"] * sum(f for f, _ in w),
                    bytes=case["iters"] * sum(x for _, x in w))
    nbf, nocc = case["nbf"], case["nocc"]
    b, a, t = float(nbf), 4.0 * nbf, float(nocc * (nbf - nocc))
    if k == "iterate":
        f, x = _iteration_work(nbf, nocc)
        return dict(flops=case["iters"] * f, bytes=case["iters"] * x)
    if k == "stages":
        f, x = _iteration_work(nbf, nocc)
        return dict(flops=f + 20.0 * b * t * case["nomega"], bytes=x + 8 * (2 * a * b * b))
    if k == "open_shell":
        t2 = t + (nocc - 1) * (nbf - nocc + 1)
        f = 2 * (3 * b + 1) * b * b * a + t2 * (t2 + 1) * a + 4 / 3 * t2 ** 3 + 4 * t2 * t2 * a
        f += 2 * (b * (b + 1) * t2 * a + 2 * b ** 3 * t2)
        return dict(flops=case["iters"] * f, bytes=case["iters"] * 8 * (a * b * b + 12 * b * b))
    if k == "build":
        return dict(flops=(3 * b + 1) * b * b * a + t * (t + 1) * a,
                    bytes=8 * (2 * a * b * b + t * t))
    if k == "block":
        s = case["s_count"]
        return dict(flops=2 * a * t * s + b * (b + 1) * a * s + 2 * b ** 3 * s,
                    bytes=8 * (a * b * b + t * s + 2 * b * b * s))
    return dict(flops=b * (b + 1) * t * a + 2 * b ** 3 * t, bytes=8 * (a * b * b + b * b))  # mp2


# ------------------------------------------------------------------ exact --
def _transform(B, C):
    return (C.T @ (B @ C)).contiguous()


def _weights(eps, Omega, nocc, eta):
    """Re 1/(eps_m - eps_k +- (Omega_s - i eta)) as a function of m: [k][s]."""
    sign = torch.where(torch.arange(eps.numel(), device=DEV) < nocc, 1.0, -1.0).to(F64)

    def at(m):
        x = eps[m] - eps[:, None] + sign[:, None] * Omega[None, :]
        return x / (x * x + eta * eta)
    return at


def _sigma_qs(w, eps, Omega, nocc, eta):
    n = eps.numel()
    at, flat, G = _weights(eps, Omega, nocc, eta), w.reshape(n, -1), []
    for m in range(n):
        G.append(flat @ (flat[m] * at(m).reshape(-1)))
    G = torch.stack(G)
    return 0.5 * (G + G.T)


def _casida(B_s, eps_s, nocc_s, factor):
    """Omega and rho[P][s] = sum_t B_t sqrt(Delta_t) Z_ts sqrt(factor / (2 Omega_s))
    of M = Delta^2 + factor sqrt(Delta) K sqrt(Delta)."""
    Bt = torch.cat([B[:, :no, no:].reshape(B.shape[0], -1) for B, no in zip(B_s, nocc_s)], 1)
    D = torch.cat([(e[None, no:] - e[:no, None]).reshape(-1) for e, no in zip(eps_s, nocc_s)])
    X = Bt * D.sqrt()
    M = factor * (X.T @ X)
    M.diagonal().add_(D * D)
    lam, Z = torch.linalg.eigh(M)
    Om = lam.sqrt()
    return Om, (X @ Z) * torch.sqrt(factor / (2.0 * Om))


def _diagonalize(F):
    e, C = torch.linalg.eigh(0.5 * (F + F.T))
    top = C.gather(0, C.abs().argmax(0, keepdim=True))
    return e, (C * torch.where(top < 0, -1.0, 1.0)).contiguous()


def _residue(B, rho):
    n = B.shape[1]
    return (B.reshape(-1, n * n).T @ rho).reshape(n, n, -1)


def _step(B, h, eps_s, C_s, nocc_s, factor):
    """One iteration of every spin (one entry per spin; a closed shell has one)."""
    B_s = [_transform(B, C) for C in C_s]
    Om, rho = _casida(B_s, eps_s, nocc_s, factor)
    both = (C_s * 2, nocc_s * 2) if len(C_s) == 1 else (C_s, nocc_s)
    J, K = _mean_field(B, *both)
    out = []
    for i, C in enumerate(C_s):
        V = C @ _sigma_qs(_residue(B_s[i], rho), eps_s[i], Om, nocc_s[i], ETA) @ C.T
        out.append(_diagonalize(h + J - K[i] + V) + (V,))
    return out


def exact(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    if kind == "iterate":
        e, C, nocc = x["eps"], x["C"], case["nocc"]
        for _ in range(case["iters"]):
            ((e, C, V),) = _step(x["B"], x["h"], [e], [C], [nocc], 4.0)
        return dict(eps=e, C=C, Vc=V)
    if kind == "open_shell":
        e, C = [x["eps"]] * 2, [x["C"]] * 2
        for _ in range(case["iters"]):
            out = _step(x["B"], x["h"], e, C, [case["nocc"], case["nocc"] - 1], 2.0)
            e, C = [o[0] for o in out], [o[1] for o in out]
        return dict(eps=e, C=C)
    if kind == "batch":
        parts = []
        for (B, h, e, C), (_, nocc) in zip(x["mols"], _batch_shapes(case)):
            for _ in range(case["iters"]):
                ((e, C, _),) = _step(B, h, [e], [C], [nocc], 4.0)
            for v in (e, C.reshape(-1)):
                parts.append(torch.nn.functional.pad(v, (0, _padded(v.numel()) - v.numel())))
        return torch.cat(parts)
    if kind == "stages":
        nocc, eps = case["nocc"], x["eps"]
        B = _transform(x["B"], x["C"])
        Om, rho = _casida([B], [eps], [nocc], 4.0)
        w = _residue(B, rho)
        om = torch.linspace(-2.0, 2.0, case["nomega"], dtype=F64, device=DEV)
        sign = torch.where(torch.arange(case["nbf"], device=DEV) < nocc, 1.0, -1.0).to(F64)
        spec, own = [], []
        for m in (nocc - 1, nocc):
            pole = sign[:, None] * Om[None, :] - eps[:, None]
            d = torch.complex(om[:, None, None] + pole, (-ETA * sign)[None, :, None] + 0 * pole)
            spec.append((w[m] ** 2 / d).sum((1, 2)))
            d = torch.complex(eps[m] + pole, (-ETA * sign)[:, None] + 0 * pole)
            v, dv = (w[m] ** 2 / d).sum(), -(w[m] ** 2 / d ** 2).sum()
            own.append(torch.stack([v.real, v.imag, dv.real]))
        return dict(Omega=Om, V=_sigma_qs(w, eps, Om, nocc, ETA), spec=torch.stack(spec),
                    self=torch.stack(own), B_mo=B)
    if kind == "build":
        nocc, eps = case["nocc"], x["eps"]
        B = _transform(x["B"], x["C"])
        D = (eps[None, nocc:] - eps[:nocc, None]).reshape(-1)
        X = B[:, :nocc, nocc:].reshape(B.shape[0], -1) * D.sqrt()
        M = 4.0 * (X.T @ X)
        M.diagonal().add_(D * D)
        return dict(B_mo=B, M=M, sqrt_delta=D.sqrt())
    if kind == "block":
        nocc, eps, b, n = case["nocc"], x["eps"], case["s_begin"], case["s_count"]
        X = x["B"][:, :nocc, nocc:].reshape(x["B"].shape[0], -1) * x["sqrt_delta"]
        Om = x["Omega"][b:b + n]
        w = _residue(x["B"], (X @ x["Z"][b:b + n].T) * torch.sqrt(2.0 / Om))
        at = _weights(eps, Om, nocc, ETA_BLOCK)
        wh = torch.stack([w[m] * at(m) for m in range(case["nbf"])])
        G = wh.reshape(case["nbf"], -1) @ w.reshape(case["nbf"], -1).T
        return dict(w=w, wh=wh, V=0.5 * (G + G.T))
    if kind == "mp2":
        return _exact_mp2(x["B"], x["eps"], case["nocc"])
    if kind == "ao2mo":
        n, s, C = case["nbf"], case["slab"], x["C"]
        T = (C[:, :s].T @ x["eri"].reshape(n, -1)).reshape(s, n, n * n)
        T = (C.T @ T).reshape(s * n, n, n)
        return ((C.T @ T) @ C).reshape(s, n, n, n)
    return _exact_learn(case, x)


def _exact_mp2(B, eps, nocc):
    nbf, naux = eps.numel(), B.shape[0]
    nv = nbf - nocc
    flat = B.reshape(naux, -1)
    Bia = B[:, :nocc, nocc:].reshape(naux, -1)
    L = (flat.T @ Bia).reshape(nbf, nbf, nocc, nv)  # (mp|ia)
    Bia_p = L  # (np|ia): the direct term of the right operand
    pi_an = L[:, nocc:].permute(0, 3, 2, 1)  # [n][p virt][i][a] = (na|ip), with (ip) as (i, p)
    pa_in = L[:, :nocc].permute(0, 2, 1, 3)  # [n][p occ][i][a] = (ni|pa)
    X = torch.cat([pa_in, pi_an], 1)
    R = 2.0 * Bia_p - X
    ei, ea = eps[:nocc, None], eps[None, nocc:]
    G = []
    for n in range(nbf):
        occ = eps[n] + (ea - ei)[None] - eps[:nocc, None, None]
        virt = eps[n] - (ea - ei)[None] - eps[nocc:, None, None]
        d = torch.cat([occ, virt])
        G.append(L.reshape(nbf, -1) @ (R[n] * d / (d * d + ETA * ETA)).reshape(-1))
    G = torch.stack(G, 1)
    return 0.5 * (G + G.T)


def _exact_learn(case, x):
    def bf16(t):
        return t.to(F32).to(torch.bfloat16).to(F64)

    def unpack(p):
        parts, at = [], 0
        for shape in ((128, 16), (128,), (128, 128), (128,), (128,), (1,)):
            n = math.prod(shape)
            parts.append(p[at:at + n].reshape(shape))
            at += n
        return parts
    gelu = torch.nn.functional.gelu
    P = x["P"].to(F64).requires_grad_(True)
    W1, b1, W2, b2, w3, b3 = unpack(P)
    y = gelu(gelu(x["X"].to(F64) @ W1.T + b1) @ W2.T + b2) @ w3 + b3
    loss = ((y - x["T"].to(F64)) ** 2).mean()
    (g,) = torch.autograd.grad(loss, P)
    W1, b1, W2, b2, w3, b3 = (t.detach() for t in (W1, b1, W2, b2, w3, b3))
    A = bf16(gelu(bf16(x["Xi"].to(F64)) @ bf16(W1).T + b1))
    A = bf16(gelu(A @ bf16(W2).T + b2))
    m, v = 0.1 * g, 0.001 * g * g
    p = P.detach() - LR * g / (g.abs() + 1e-8)
    return dict(params=p, m=m, v=v, grad=g, loss=loss.detach().reshape(1), y=A @ bf16(w3) + b3)
