"""What the library asks of the HIP runtime, and what it does where the
runtime refuses: a child process loads hip_calls.c in front of the runtime,
which notes a few calls and passes them on or refuses them."""

import json
import os
import shutil
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, json, os, sys
calls = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
calls.calls_end.restype = ctypes.c_char_p
import torch
from paper_1905_11722_amd import rcdp as rc, workloads as W
torch.cuda.set_device(0)
"""


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    """Runs a program behind hip_calls.c; returns what it passed to answer()."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if shutil.which("gcc") is None:
        pytest.skip("no C compiler")
    lib = str(tmp_path_factory.mktemp("hip_calls") / "hip_calls.so")
    subprocess.check_call(["gcc", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                           os.path.join(ROOT, "tests", "hip_calls.c"), "-o", lib, "-ldl"])

    def run(program):
        source = PRELUDE + program + "\nprint('ANSWER', json.dumps(answer()), flush=True)\n"
        r = subprocess.run([sys.executable, "-c", source, lib], cwd=ROOT, capture_output=True,
                           text=True, timeout=100)
        assert r.returncode == 0, r.stdout + r.stderr
        return json.loads(r.stdout.split("ANSWER", 1)[1])
    return run


def test_fill_window(child):
    """fill_ms covers every kernel of a solve but the selection's: the first
    event comes before the first launch, the last one before the last launch,
    for every fill, one table and a batch of them (one selection each)."""
    logs = child("""
def answer():
    out = {}
    g = W.chain(120, seed=3, tmax=9, mmax=9)
    B = (3 * sum(g.M)) // 2
    for path in ("level", "block", "wide", "wavefront"):
        os.environ["RCDP_FILL"] = path
        fam = rc.Graph.create(g).build_family("pruned")
        fam.solve(B, "tc").free()                    # the family's lazy parts
        for name, call in (("solve", lambda: [fam.solve(B, "tc")]),
                           ("dominance", lambda: [fam.solve_dominance(B)]),
                           ("sweep", lambda: [s for _, s in fam.sweep([B, B + 1], "tc")])):
            calls.calls_start()
            sols = call()
            out[path + " " + name] = calls.calls_end().decode()
            for s in sols:
                s.free()
    return out
""")
    assert len(logs) == 12
    for name, log in logs.items():
        assert log.count("E") in (2, 4), (name, log)     # 4: around the wavefront kernel too
        assert log.startswith("EL") and log.endswith("EL"), (name, log)


def test_no_pinned_memory(child):
    """rc_graph_create and rc_min_budget where pinned host memory cannot be
    had and the pool holds none (a call whose wait reports an error gives its
    buffer up): the same graph and budget as with it."""
    got = child("""
def answer():
    g = W.random_dag(90, 0.06, 5, tmax=40, mmax=30)
    calls.calls_refuse_pinned(1)
    h = rc.Graph.create(g)
    calls.calls_refuse_pinned(0)
    fam, ref = h.build_family("pruned"), rc.Graph.create(g).build_family("pruned")
    same = bool((fam.sets() == ref.sets()).all()) and fam.info == ref.info
    want = ref.min_budget()
    failed = 0
    calls.calls_refuse_pinned(1)
    for _ in range(16):
        calls.calls_fail_sync(0)
        try:
            fam.min_budget()
        except rc.RcError as e:
            failed += e.status == rc.E_DEVICE
        calls.calls_fail_sync(-1)
    got = fam.min_budget()
    try:
        h.build_family("pruned")
        pinned = True
    except rc.RcError as e:
        pinned = e.status != rc.E_NOMEM
    calls.calls_refuse_pinned(0)
    return dict(same=same, want=want, got=got, failed=failed, pinned=pinned)
""")
    assert got["same"] and got["got"] == got["want"]
    assert got["failed"] == 16 and not got["pinned"]
