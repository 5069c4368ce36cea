"""Calls whose HIP runtime refuses something: cooperative launches, large
allocations.  A child process loads a small library that stands before the
runtime's own entry and refuses it; the answers are those of a process where
nothing is refused."""
import os
import shutil
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COOP = """
static int calls;
int hipLaunchCooperativeKernel(void) { ++calls; return 720; } /* too large */
int refused(void) { return calls; }
"""


def run_child(tmp_path, source, code):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("no host compiler")
    src, so = tmp_path / "refuse.c", tmp_path / "refuse.so"
    src.write_text(source)
    subprocess.run([cc, "-O1", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    head = f"""
import ctypes, sys
shim = ctypes.CDLL({str(so)!r}, mode=ctypes.RTLD_GLOBAL)
sys.path[:0] = [{ROOT!r}, {os.path.join(ROOT, "tests")!r}]
import numpy as np
import torch
import paper_2210_17093_amd.qsgw as q
"""
    r = subprocess.run([sys.executable, "-u", "-c", head + code], cwd=ROOT, timeout=100,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    print(r.stdout, flush=True)


def test_refused_cooperative_launches(tmp_path):
    """Dense eigensolves of one and of many problems, and a two-stage one."""
    run_child(tmp_path, COOP, """
from test_gpu_eig_range import check_solve, spd, dev
from qsgw_inputs import make_problem
c = q.Context()
for n in (60, 129, 300, 1100, 3200):
    print("refused cooperative launch, order", n, flush=True)
    before = shim.refused()
    check_solve(q, c, spd(n, n))
    assert (shim.refused() > before) == (n > 128), n
mols, alone = [], []
for nbf, seed in ((20, 3), (60, 1), (75, 2)):
    p = make_problem(nbf, 4 * nbf, nbf // 6, 2 * nbf, 0.99, 900 + seed)
    B, C, e = dev(p.B_ao), dev(p.C0), dev(p.eps0)
    h = q.qsgw_hf_core(c, B, C, e, p.nocc)
    e1, C1 = e.clone(), C.clone()
    c.set_eigensolver(q.EIG_ROCSOLVER)
    q.qsgw_iterate(c, B, h, p.nocc, e1, C1, 1e-3, tol=0.0, max_iter=1)
    c.set_eigensolver(q.EIG_AUTO)
    alone.append(e1)
    mols.append(dict(B_ao=B, h=h, nocc=p.nocc, eps=e, C=C))
print("refused cooperative launch, batch", flush=True)
q.qsgw_iterate_batched(c, mols, 1e-3, tol=0.0, max_iter=1)
for a, m in zip(alone, mols):
    assert float((a - m["eps"]).abs().max()) <= 1e-8
c.close()
""")


def test_rocsolver_choice_reaches_every_eigensolve(tmp_path):
    """A context set to EIG_ROCSOLVER asks for no cooperative launch: Casida and
    Fock eigensolves, single and batched.  (Without that choice all of them do.)"""
    run_child(tmp_path, COOP, """
from test_gpu_eig_range import dev
from qsgw_inputs import make_problem
c = q.Context()
p = make_problem(140, 200, 9, 100, 0.99, 77)
B, C, e = dev(p.B_ao), dev(p.C0), dev(p.eps0)
h = q.qsgw_hf_core(c, B, C, e, p.nocc)
def calls(solver, step):
    c.set_eigensolver(solver)
    before = shim.refused()
    step()
    return shim.refused() - before
def single():
    q.qsgw_iterate(c, B, h, p.nocc, e.clone(), C.clone(), 1e-3, tol=0.0, max_iter=1)
def batch():
    q.qsgw_iterate_batched(c, [dict(B_ao=B, h=h, nocc=p.nocc, eps=e.clone(), C=C.clone())], 1e-3,
                           tol=0.0, max_iter=1)
for step in (single, batch):
    print("eigensolver choice", step.__name__, flush=True)
    assert calls(q.EIG_AUTO, step) == 2
    assert calls(q.EIG_ROCSOLVER, step) == 0
c.close()
""")
