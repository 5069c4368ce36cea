"""The tile shape of an FP64 product: which one the table and the rule for small
products choose (csrc/tiles.hpp compiled for the host), and, on the device, that
a table which names no shape, or the default one written out and set again,
launches the kernels of the default."""
import ctypes as ct
import json
import os
import shutil
import subprocess
import sys

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2210_17093_amd", "csrc")
S64, S128x64, S128, S32 = 0, 1, 2, 4
MO1, MO2, CASIDA, RHO, SIGMA, EXCHANGE = range(6)
SRC = """
#include "tiles.hpp"
using namespace qsgw;
extern "C" int table(int k, int set, int tri, long M, long N, long batch, long nz) {
  Tiles t;
  if (set >= 0) t.shape[k] = set;
  t.dc_leaf = 512;
  t.persistent = 1;
  return table_shape(t, (Tunable)k, tri != 0, M, N, batch, nz);
}
extern "C" int fitting(int shape, int tri, long M, long N, long batch, long nz) {
  return fitting_shape(shape, tri != 0, M, N, batch, nz);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    tmp = tmp_path_factory.mktemp("tiles")
    src, out = tmp / "tiles.cpp", tmp / "libtiles.so"
    src.write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o",
                    str(out)], check=True)
    lib = ct.CDLL(str(out))
    lib.table.argtypes = [ct.c_int] * 3 + [ct.c_long] * 4
    lib.fitting.argtypes = [ct.c_int] * 2 + [ct.c_long] * 4
    return lib


# (order, shape): symmetric product of 128 x 128 tiles; 22 tiles a side are 253, 23 are 276
@pytest.mark.parametrize("n,want", [(95, S32), (1000, S32), (1408, S32), (1409, S64), (2816, S64),
                                    (2817, S128), (18232, S128)])
def test_the_rule(lib, n, want):
    assert lib.fitting(S128, 1, n, n, 1, 1) == want


@pytest.mark.parametrize("k,default", [(MO1, S128x64), (MO2, S64), (CASIDA, S128), (RHO, S128),
                                       (SIGMA, S64), (EXCHANGE, S64)])
@pytest.mark.parametrize("M,N,batch,nz", [(95, 95, 1, 1), (24, 24, 96, 1), (2304, 2304, 1, 1),
                                          (60, 60, 1, 200), (9000, 9000, 1, 1)])
def test_a_table_without_the_product_s_shape_chooses_as_the_default(lib, k, default, M, N, batch, nz):
    tri = int(k in (MO2, CASIDA, EXCHANGE))
    want = lib.fitting(default, tri, M, N, batch, nz)
    assert lib.table(k, -1, tri, M, N, batch, nz) == want
    assert lib.table(k, default, tri, M, N, batch, nz) == want
    for other in (S64, S128x64, S128):
        if other != default:
            assert lib.table(k, other, tri, M, N, batch, nz) == other


CHILD = """
import json, sys
sys.path[:0] = [sys.argv[1]]
import torch
import paper_2210_17093_amd.qsgw as q
from qsgw_inputs import make_problem
p = make_problem(60, 240, 10, 120, 0.99, 5)
ctx = q.Context()
B, e = torch.from_numpy(p.B_ao).cuda(), torch.from_numpy(p.eps0).cuda()
ctx.set_tiles(None)
default = ctx.get_tiles()
out = {}
for spec in ("", "dc_leaf=512", "persistent=1", "panel_coop=0", "mo1=64x64", default, "casida=64x64"):
    ctx.set_tiles(spec)
    q.qsgw_rpa_build(ctx, B, e, p.nocc)
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        q.qsgw_rpa_build(ctx, B, e, p.nocc)
        torch.cuda.synchronize()
    out["default table" if spec == default else spec] = sorted(
        ev.name for ev in prof.events() if "gemm" in ev.name)
print("KERNELS " + json.dumps(out), flush=True)
"""


@pytest.mark.gpu
def test_launched_kernels_follow_the_table():
    """(In a process of its own: the profiler stays loaded in the one that uses it.)"""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, root], cwd=root, timeout=100,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    lines = [x for x in r.stdout.splitlines() if x.startswith("KERNELS ")]
    assert lines, r.stdout[-2000:]
    out = json.loads(lines[0][len("KERNELS "):])
    other = out.pop("casida=64x64")
    want = out.pop("")
    assert want and other != want
    for spec, got in out.items():
        assert got == want, spec
