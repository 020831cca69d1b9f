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

TUNER = """
for L, Ls, prec in (((4, 4, 4, 4), 8, 0), ((8, 8, 8, 8), 8, 1), ((8, 8, 8, 8), 16, 2)):
    ctx, n = context(L, Ls)
    f, g, ws = buf(n * 8), buf(n * 8), buf(lib.qdwf_workspace_bytes(ctx, q.QDWF_OP_TUNE, prec, 1))
    mws = buf(lib.qdwf_workspace_bytes(ctx, q.QDWF_OP_MDAGM, prec, 1))

    def launches():
        stub.stub_clear()
        for d in (0, 1):
            assert lib.qdwf_apply_D(ctx, g, f, d, prec, q.QDWF_RIRI, 1, None) == 0
        assert lib.qdwf_apply_MdagM(ctx, g, f, prec, q.QDWF_RIRI, 1, mws, None) == 0
        return hops()

    plain = launches()
    ms = (ctypes.c_double * 2)()
    assert lib.qdwf_tune(ctx, prec, q.QDWF_RIRI, 1, ws, None, ms) == 0
    # every launch takes the same time on the stand-in: nothing beats the untuned one
    tuned = launches()
    assert tuned == plain, (L, Ls, prec, plain, tuned)
    lib.qdwf_destroy(ctx)
    # a context that reads the result from the cache launches the same
    ctx, n = context(L, Ls)
    assert launches() == plain
    lib.qdwf_destroy(ctx)
"""


def test_tuning_keeps_the_untuned_launch_where_nothing_beats_it(run, tmp_path):
    run(TUNER, QDWF_TUNE_CACHE=str(tmp_path / "tune.jsonl"))


OLD_CACHE = """
L, Ls, prec = (4, 4, 4, 4), 8, 0
path = os.environ.pop("QDWF_TUNE_CACHE")
ctx, n = context(L, Ls)
f, g = buf(n * 8), buf(n * 8)

def launched(ctx):
    stub.stub_clear()
    assert lib.qdwf_apply_D(ctx, g, f, 0, prec, q.QDWF_RIRI, 1, None) == 0
    return hops()

plain = launched(ctx)
ws = buf(lib.qdwf_workspace_bytes(ctx, q.QDWF_OP_TUNE, prec, 1))
os.environ["QDWF_TUNE_CACHE"] = path
assert lib.qdwf_tune(ctx, prec, q.QDWF_RIRI, 1, ws, None, None) == 0
lib.qdwf_destroy(ctx)
import json
line = json.loads(open(path).readline())
assert line["split"] == 1
del line["split"]
line.update(threads=128, nrb=1, xcd=0, lds_pad=0, sweep=0)
for split, same in ((None, True), (0, False), (1, True)):
    entry = dict(line) if split is None else dict(line, split=split)
    entry["ms"] = entry.pop("ms")
    open(path, "w").write(json.dumps(entry) + "\\n")
    ctx, n = context(L, Ls)
    shape = (ctypes.c_int32 * 4)()
    assert lib.qdwf_tuned_shape(ctx, prec, q.QDWF_RIRI, 0, 1, shape) == 0
    assert list(shape) == [128, 1, 0, 0]
    assert (launched(ctx) == plain) == same, (split, plain)
    lib.qdwf_destroy(ctx)
"""


def test_cache_lines_with_and_without_the_form(run, tmp_path):
    run(OLD_CACHE, QDWF_TUNE_CACHE=str(tmp_path / "tune.jsonl"))

POOL = """
name = {name!r}
prm = q.qdwf_solve_params(system=0, inner_prec=q.QDWF_F16, layout=q.QDWF_RIRI, max_iter=100, tol=1e-10,
                          delta=0.1, x0_is_guess=0, check_every=8, use_graph=0)
L = (4, 4, 4, 4)

def submit(pool, Ls):
    a, n = action(L, Ls), 256 * Ls * 24
    r = q.qdwf_request(act=a, U=buf(256 * 72 * 8), b=buf(n * 8), x_out=buf(n * 8), params=prm)
    i = ctypes.c_uint64()
    assert lib.qdwf_pool_submit(pool, ctypes.byref(r), ctypes.byref(i)) == 0

class Device:
    # what the host knows to be over, from the calls in order
    def __init__(self):
        self.of, self.seen, self.left, self.n = {{}}, {{}}, set(), 0

    def feed(self, lines):
        for l in lines:
            w = l.split()
            if len(w) > 1 and w[1] == "FAILS":
                continue
            if w[0] == "hipGraphLaunch":
                self.n += 1
                self.of.setdefault(w[2], set()).add(self.n)
                self.left.add(self.n)
            elif w[0] == "hipEventRecord":
                self.seen[w[1]] = set(self.of.get(w[2], ()))
            elif w[0] == "hipStreamWaitEvent":
                self.of.setdefault(w[1], set()).update(self.seen.get(w[2], ()))
            elif w[0] == "hipEventSynchronize":
                self.left -= self.seen.get(w[1], set())
            elif w[0] == "hipStreamSynchronize":
                self.left -= self.of.get(w[1], set())
            elif w[0] == "hipGraphExecDestroy" or w[0] == "hipMemcpyAsync" and int(w[1]) > 100000:
                # the graph, or the table and its staging, of a round that may be running
                assert not self.left, l

n = 1
while True:
    need = lib.qdwf_pool_overhead_bytes(4)
    for Ls in (8, 16, 28):
        need += lib.qdwf_request_bytes(ctypes.byref(action(L, Ls)), ctypes.byref(prm)) + 4096
    pool = ctypes.c_void_p()
    assert lib.qdwf_pool_create(0, buf(need), need, 4, ctypes.byref(prm), ctypes.byref(pool)) == 0
    for Ls in (16, 28):
        submit(pool, Ls)
    D = Device()
    D.feed(log())
    stub.stub_fail(name.encode(), n)
    lib.qdwf_pool_step(pool, None, None)
    lines = log()
    D.feed(lines)
    stub.stub_fail(b"", 0)
    submit(pool, 8)
    assert lib.qdwf_pool_step(pool, None, None) == 0
    D.feed(log())
    assert D.n >= 2
    lib.qdwf_pool_destroy(pool)
    D.feed(log())
    if not any(" FAILS " in l for l in lines):
        break
    n += 1
print(n, "calls of", name)
assert n > 1
"""


@pytest.mark.parametrize("name", ["hipEventRecord", "hipStreamWaitEvent", "hipGraphLaunch", "hipMemcpyAsync"])
def test_a_round_that_fails_half_way_is_waited_for(run, name):
    run(POOL.format(name=name))
