"""librel's host side on a HIP runtime that computes nothing (hip_stub.cpp), in a
process of its own: which kernels a call launches, what memory it takes, and what
it does when there is none."""
from __future__ import annotations

import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

_PRELUDE = """
import ctypes, sys
sys.path.insert(0, {root!r})
from paper_2608_13696_amd import rel
stub = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)  # before librel: its runtime
stub.stub_limit.argtypes = [ctypes.c_size_t]
stub.stub_used.restype = ctypes.c_size_t
stub.stub_kill.argtypes = stub.stub_revive.argtypes = [ctypes.c_void_p]
stub.stub_log.restype = ctypes.c_char_p
L = rel.lib()
P, BIG = ctypes.byref, 1 << 62  # (no kernel runs: a column is an address)
def new_ctx(stream=0x1000):
    h = ctypes.c_void_p()
    assert L.rel_ctx_create(0, ctypes.c_void_p(stream), P(h)) == 0
    return h
def column():
    column.at += 1 << 20
    return column.at
column.at = 1 << 40
def kernels():
    out = [line.rsplit(" ", 1) for line in stub.stub_log().decode().splitlines()]
    stub.stub_clear_log()
    return [(name, int(grid)) for name, grid in out]
def launched(names, part):
    return any(part in name for name, _ in names)
def table(ctx, m, opts=None):
    t = ctypes.c_void_p()
    st = L.rel_join_build(ctx, column(), None, m, opts, P(t))
    return st, t
def groups(cap):
    return rel.GroupsOut(column(), column(), column(), column(), cap, column())
def fact(n):
    return rel.Fact(column(), column(), column(), column(), column(), n)
def dim(m):
    return rel.Dim(column(), column(), column(), m)
def query(ctx, n, m, by, plan=None):
    out = groups(max(n, 1))
    return L.rel_filter_join_agg(ctx, P(fact(n)), P(dim(m)), P(rel.Query(1000, rel.GROUP_BY[by])), plan and P(plan), P(out), None)
def groupby(ctx, n, hint=0, placement="auto"):
    return L.rel_groupby_agg(ctx, column(), column(), column(), None, n, P(rel.TableOpts(hint, rel.PLACE[placement], 0.0)), P(groups(n)))
"""


def run(tmp_path_factory, body: str):
    """Runs `body` behind the prelude; a failing assertion there fails the test."""
    so = os.path.join(str(tmp_path_factory.getbasetemp()), "libhip_stub.so")
    if not os.path.exists(so):
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I/opt/rocm/include", "-Wno-unused-result",
                               "-o", so, os.path.join(HERE, "hip_stub.cpp")])
    code = _PRELUDE.format(root=ROOT, so=so) + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
