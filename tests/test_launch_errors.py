"""Launch errors reach the caller: every kernel launch, transform and copy of a step in turn fails, and
the step says so.  Runs without a device, on a stand-in for the HIP runtime (tests/fake_hip.cpp), in a
process of its own."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = r"""
import ctypes as C, math, sys
F = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # before the library: its symbols come first
F.fake_fail_at.argtypes = [C.c_long]
F.fake_calls.restype = C.c_long
F.fake_refuse_new.argtypes = [C.c_size_t]
import numpy as np
from paper_2411_17294_amd import tfs
L = tfs.lib()


def plan(dim, points, scheme, stride):
    w, lam = np.array([1.0, 0.5]), np.array([0.0, 3.0])
    dp = lambda a: a.ctypes.data_as(C.POINTER(C.c_double))
    d = tfs.PlanDesc(dim, 2, points, stride, 0, 0.5, 1.0, 0.1, 1e-3, 8, dp(w), dp(lam), 0, 0, None, scheme, 0, 1)
    h = C.c_void_p()
    tfs.check(L.tfs_plan_create(C.byref(d), C.byref(h)))
    return h


def transport(shape, stride, iters):
    d = len(shape)
    h = C.c_void_p()
    tfs.check(L.tfs_transport_create(d, (C.c_int64 * d)(*shape), (C.c_double * d)(*[6.0] * d), 0.1, stride, iters, C.byref(h)))
    return h


def buf(n):
    return np.zeros(n)


def steps(shape, whole, method, tol, scheme):
    d, P = len(shape), math.prod(shape)
    c = d * (d + 1) // 2
    p, tr = plan(d, P, scheme, P), transport(shape, P, 3)
    if not whole:
        tfs.check(L.tfs_transport_set_batched(tr, 0))
    tfs.check(L.tfs_transport_set_method(tr, method))
    tfs.check(L.tfs_transport_set_tolerance(tr, tol, 1))
    ka, u, X, Y, tau, diag = buf(d * d * P), buf(d * P), buf(2 * c * P), buf(4 * c * P), buf(c * P), buf(6)
    q = lambda a: a.ctypes.data
    for n in (0, 1):
        step = lambda: L.tfs_transport_step(tr, p, n, q(ka), None, q(u), None, q(X), q(Y), q(tau), q(diag))
        F.fake_fail_at(-1)
        assert step() == 0
        total = F.fake_calls()
        assert total > 5
        lost = []
        for k in range(total):
            F.fake_fail_at(k)
            if step() == 0:
                lost.append(k)
        F.fake_fail_at(-1)
        assert not lost, f"{shape} method {method} scheme {scheme} n={n}: calls {lost} of {total} failed unseen"
        print(shape, method, scheme, n, total, flush=True)
    L.tfs_transport_destroy(tr)
    L.tfs_plan_destroy(p)


exec(sys.argv[2])
print("ok")
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
    return so


def child(fake, code):
    r = subprocess.run([sys.executable, "-c", CHILD, fake, code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr


@pytest.mark.parametrize("shape", [(400, 405), (12, 16), (8, 6, 10)])
@pytest.mark.parametrize("method", [0, 1])
def test_transport_step_reports_every_failed_call(fake, shape, method):
    """Line kernels (400 x 405), batched transforms and single planes; both solvers, with and without
    the early exit; the start and the step after it."""
    code = "\n".join(f"steps({shape}, {whole}, {method}, {tol}, {scheme})"
                     for whole in (True, False) for tol in (0.0, 1e-9) for scheme in (0, 1))
    child(fake, code)


def test_line_kernels_keep_no_batched_plans(fake):
    """A transport object holds the two single-plane plans, and the four batched ones only where it uses
    them."""
    child(fake, """
for shape, n in (((400, 405), 2), ((12, 16), 6), ((8, 6, 10), 6)):
    tr = transport(shape, math.prod(shape), 3)
    assert F.fake_plans() == n and L.tfs_transport_batched(tr) == 1, (shape, F.fake_plans())
    tfs.check(L.tfs_transport_set_batched(tr, 0))
    assert F.fake_plans() == 2 and L.tfs_transport_batched(tr) == 0, (shape, F.fake_plans())
    tfs.check(L.tfs_transport_set_batched(tr, 1))
    assert F.fake_plans() == n and L.tfs_transport_batched(tr) == 1, (shape, F.fake_plans())
    tfs.check(L.tfs_transport_destroy(tr))
    assert F.fake_plans() == 0
""")


def test_no_host_memory_for_the_line_kernels(fake):
    """No exception leaves the C entry: without memory for the tables the object uses the library's
    transforms."""
    child(fake, """
F.fake_refuse_new(4096)
tr = transport((400, 405), 162000, 3)
F.fake_refuse_new(0)
assert F.fake_plans() == 6 and L.tfs_transport_batched(tr) == 1
tfs.check(L.tfs_transport_destroy(tr))
""")
