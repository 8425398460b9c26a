"""Which kernels a step launches, and that the tile-shape tuner times the
launches that the step makes (no GPU: the library runs against
routes_mock.cpp in a process of its own)."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r'''
import ctypes, os, sys
lib = ctypes.CDLL(%r)
V, D, I = ctypes.c_void_p, ctypes.c_double, ctypes.c_int
class Desc(ctypes.Structure):
    _fields_ = [("dim", I), ("nx", I), ("ny", I), ("lx", D), ("ly", D), ("p", I), ("eq", I), ("velocity", D * 2),
                ("gamma", D), ("limiter", I), ("gmin", D), ("gmax", D), ("vel_rows", V), ("vel_cols", V), ("bc", I * 2)]
dim, nx, ny, p, eq = map(int, sys.argv[1:6])
d = Desc(dim=dim, nx=nx, ny=ny, lx=1, ly=1, p=p, eq=eq, gamma=1.4)
d.velocity[0] = d.velocity[1] = 1.0
h = V()
assert lib.idp_dg_create(ctypes.byref(d), None, ctypes.byref(h)) == 0
lib.idp_dg_num_nodes.restype = ctypes.c_long
u = (D * (4 * lib.idp_dg_num_nodes(h)))()
out = I(-1)
def say(s):
    ctypes.CDLL(None).puts(s.encode())
for v in (0, 1):
    assert lib.idp_dg_set_tile_shape(h, v) == 0
    tx, ty = I(), I()
    lib.idp_dg_tile_dims(h, ctypes.byref(tx), ctypes.byref(ty))
    say("shape %%d tiles %%d" %% (v, -(-nx // tx.value) * -(-ny // ty.value)))
    assert lib.idp_dg_step_cfl(h, u, D(0.5)) == 0
say("step")
assert lib.idp_dg_step(h, u, D(1e-3)) == 0
lib.idp_dg_set_tile_shape(h, 0)
say("tune")
assert lib.idp_dg_tune(h, u, D(0.5), 1, ctypes.byref(out)) == 0
say("kept %%d" %% out.value)
b, hs, us = V(), (V * 1)(h), (V * 1)(ctypes.cast(u, V))
assert lib.idp_dg_batch_create(hs, 1, None, ctypes.byref(b)) == 0
say("batch tune")
assert lib.idp_dg_batch_tune(b, us, D(0.5), 1) == 0
''' % os.path.join(ROOT, "paper_2004_08503_amd", "libidp_dg.so")


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("routes"))
    so = os.path.join(d, "routes_mock.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "routes_mock.cpp")], check=True)

    def run(*args):
        r = subprocess.run([sys.executable, "-c", DRIVER] + [str(a) for a in args], capture_output=True, text=True,
                           env=dict(os.environ, LD_PRELOAD=so), timeout=120)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
        out, key = {}, None
        for line in r.stdout.splitlines():
            if re.match(r"shape|step$|tune$|kept|batch tune$", line):
                key = " ".join(line.split()[:2]) if line.startswith("shape") else line
                out[key] = []
                if line.startswith("shape"):
                    out[key + " tiles"] = int(line.split()[-1])
                continue
            if key:
                out[key].append(line)
        return out
    return run


def kinds(launches):
    return [re.match(r"_ZN3idp\d+([a-z0-9_]+?)(I|E)", k).group(1) for k in launches]


FOLD = ["maxdt_kernel", "stage_fold_kernel", "stage_kernel", "stage_kernel"]
PLAIN = ["maxdt_kernel", "min_reduce_kernel", "stage_kernel", "stage_kernel", "stage_kernel"]
LARGE = ["maxdt_kernel", "chunk_min_kernel", "min_reduce_kernel", "stage_kernel", "stage_kernel", "stage_kernel"]
ONE_TILE = ["maxdt_kernel", "stage_kernel", "stage_kernel", "stage_kernel"]


def expected(tiles):
    return ONE_TILE if tiles == 1 else FOLD if tiles <= 1024 else PLAIN if tiles <= 32768 else LARGE


@pytest.mark.parametrize("args", [(2, 3, 3, 4, 2), (2, 96, 96, 4, 2), (2, 97, 96, 4, 2), (2, 128, 128, 3, 1),
                                  (2, 96, 32, 8, 2), (2, 97, 32, 8, 2), (2, 900, 900, 4, 2), (1, 1000, 1, 3, 2),
                                  (1, 31 * 1024, 1, 3, 1)])
def test_launches_and_tuner(routes, args):
    r = routes(*args)
    for v in (0, 1):
        assert kinds(r["shape %d" % v]) == expected(r["shape %d tiles" % v])
    # one warm-up and two rounds of one step per shape, each the step's own launches
    t = r["tune"]
    a, b = r["shape 0"], r["shape 1"]
    assert t == a + b + 2 * (["event"] + a + ["event"] + ["event"] + b + ["event"])
    assert "kept 0" in r
    # a batch has neither of the short routes
    assert not {"stage_fold_kernel", "step1_kernel"} & set(kinds([k for k in r["batch tune"] if k != "event"]))
    assert len(r["batch tune"]) > 8


@pytest.mark.parametrize("args", [(1, 1, 1, 8, 0), (1, 60, 1, 3, 1), (1, 60, 1, 3, 2)])
def test_one_workgroup(routes, args):
    r = routes(*args)
    assert kinds(r["shape 0"]) == kinds(r["shape 1"]) == kinds(r["step"]) == ["step1_kernel"]
    assert r["shape 0"] == r["shape 1"]
    assert r["tune"] == [] and "kept 0" in r      # one kernel whatever the shape: nothing to choose
    assert "stage_kernel" in kinds([k for k in r["batch tune"] if k != "event"])


@pytest.mark.parametrize("eq,nodes", [(0, 766), (1, 766), (2, 510)])
@pytest.mark.parametrize("p", [1, 3, 8])
def test_one_workgroup_limit(routes, eq, nodes, p):
    """The last mesh of one launch and the one after it (Euler gains nothing
    from one launch past eight waves)."""
    nx = nodes // (p + 1)
    assert kinds(routes(1, nx, 1, p, eq)["step"]) == ["step1_kernel"]
    r = routes(1, nx + 1, 1, p, eq)
    assert kinds(r["step"]) == ["stage_kernel"] * 3 and kinds(r["shape 0"]) == FOLD
