"""Host code of the library without a GPU: the library runs on a stand-in for
the HIP runtime (hip_stub.c), in a process of its own, and the calls it makes
are looked at. Kernels do nothing there, so results are not.
"""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2112_01852_amd", "libqdwf.so")

PRELUDE = """
import ctypes, os, sys, unittest.mock
stub = ctypes.CDLL({stub!r}, ctypes.RTLD_GLOBAL)
stub.stub_log.restype = ctypes.c_char_p
C = ctypes.CDLL({lib!r})
sys.modules["torch"] = unittest.mock.MagicMock()   # torch brings its own HIP runtime
sys.path.insert(0, {root!r})
from paper_2112_01852_amd import qdwf as q
lib = q.lib()

def buf(n):
    raw = (ctypes.c_char * (n + 4096))()
    at = ctypes.addressof(raw)
    keep.append(raw)
    return (at + 255) // 256 * 256
keep = []

def log(word=""):
    lines = [l for l in stub.stub_log().decode().splitlines() if l.startswith(word)]
    stub.stub_clear()
    return lines

def action(L, Ls, b=1.5, c=0.5):
    a = q.qdwf_action()
    a.L[:], a.Ls, a.bc[:], a.M5, a.mf, a.b, a.c = L, Ls, (1, 1, 1, -1), 1.8, 0.1, b, c
    return a

def context(L, Ls):
    ctx = ctypes.c_void_p()
    a = action(L, Ls)
    assert lib.qdwf_create(ctypes.byref(a), 0, ctypes.byref(ctx)) == 0
    V = L[0] * L[1] * L[2] * L[3]
    assert lib.qdwf_set_gauge(ctx, buf(V * 72 * 8), 0, None) == 0
    stub.stub_clear()
    return ctx, V * Ls * 24

def hops():
    # grid, block and LDS bytes of each hop launched
    return [tuple(int(v) for v in l.split()[2:]) for l in log("kernel") if "hop" in l]
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not os.path.exists(LIB):
        pytest.skip("libqdwf.so not built (run __graft_entry__.build())")
    stub = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", "-o", stub, os.path.join(HERE, "hip_stub.c")],
                   check=True)

    def child(code, **env):
        p = subprocess.run([sys.executable, "-c", PRELUDE.format(stub=stub, lib=LIB, root=ROOT) + code],
                           capture_output=True, text=True, timeout=120,
                           env={k: v for k, v in dict(os.environ, **env).items() if v is not None})
        assert p.returncode == 0, p.stdout + p.stderr
        return p.stdout

    return child


PAD = """
for L, Ls, prec in (((4, 4, 4, 4), 8, 0), ((4, 4, 4, 4), 16, 0), ((8, 8, 8, 8), 8, 1), ((8, 8, 4, 4), 16, 2)):
    ctx, n = context(L, Ls)
    f, g = buf(n * 8), buf(n * 8)
    ws = buf(lib.qdwf_workspace_bytes(ctx, q.QDWF_OP_MDAGM, prec, 1))
    for pad in (0, 8192, 22528, 24576, 45056, 49152):
        os.environ["QDWF_HOP_LDS_PAD"] = str(pad)
        for d in (0, 1):
            assert lib.qdwf_apply_D(ctx, g, f, d, prec, q.QDWF_RIRI, 1, None) == 0, (L, Ls, prec, pad)
        assert lib.qdwf_apply_MdagM(ctx, g, f, prec, q.QDWF_RIRI, 1, ws, None) == 0, (L, Ls, prec, pad)
        for grid, block, lds in hops():
            assert pad <= lds <= 65536
"""


def test_a_padded_small_launch_takes_a_form_that_fits(run):
    run(PAD)
