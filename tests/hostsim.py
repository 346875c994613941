"""Runs the library's host code without a GPU: a child process loads tests/fake_hip.cpp (kernel
launches are only logged) ahead of libstotree.so and drives the C entry points through the binding."""
import functools
import os
import subprocess
import sys
import tempfile
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PROLOGUE = """
import ctypes as C, re, sys
import numpy as np
sys.path[:0] = [{root!r}, {here!r}]
fake = C.CDLL({lib!r}, mode=C.RTLD_GLOBAL)
fake.fake_calls.restype = C.c_char_p
import treegen
from paper_2107_01745_amd import stotree as st
L = st.lib()


def calls():
    out = fake.fake_calls().decode().splitlines()
    fake.fake_clear()
    return out


def launches(log=None):
    "names of the kernels launched since the last look, without namespaces and argument lists"
    out = []
    for ln in calls() if log is None else log:
        if ln.startswith("launch "):
            mangled = ln.split()[1]
            m = re.search(r"[0-9]+([a-z][a-z0-9_]*_kernel)(I\\S*?E)?E[vNPil]", mangled)
            out.append(m.group(1) + (m.group(2) or "") if m else mangled)
    return out


_keep = []


def buf(n):
    a = np.zeros(int(n))
    _keep.append(a)
    return a.ctypes.data


def problem(branching, nx, nu, seed=0):
    return treegen.draw_problem(treegen.uniform_tree(branching), nx, nu, np.random.default_rng(seed))


def factor(*probs):
    tf = st.tree_factor(probs[0], stream=0) if len(probs) == 1 else st.tree_factor_batch(list(probs), stream=0)
    calls()
    return tf


def sweep(tf, nrhs=1, y=None, x=None, u=None):
    rc = L.dual_grad(tf.handle, buf(nrhs * tf.x0_len), y or buf(nrhs * tf.m), 0, nrhs, x or buf(nrhs * tf.x_len),
                     u or buf(nrhs * tf.u_len), None)
    return rc, launches()
"""


@functools.lru_cache(maxsize=None)
def _fake_lib():
    out = os.path.join(tempfile.mkdtemp(prefix="stotree_fake_hip_"), "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "fake_hip.cpp")], check=True)
    return out


def run(body):
    """The child's standard output; raises with its errors if an assertion in body fails."""
    code = PROLOGUE.format(root=ROOT, here=HERE, lib=_fake_lib()) + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout
