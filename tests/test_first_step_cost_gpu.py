"""The first step of a run and its adjoint cost what they move: ratios of two calls on one device,
far from either side's spread."""
import pytest
import torch

from oracle import soe as osoe
from paper_2411_17294_amd import tfs

pytestmark = pytest.mark.gpu


def best_us(f, reps=10):
    f()
    torch.cuda.synchronize()
    out = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            f()
        b.record()
        torch.cuda.synchronize()
        out.append(a.elapsed_time(b) / reps * 1e3)
    return min(out)


def test_first_exponential_step_reads_no_modes():
    """At n = 0 the modes are -q_k X^0: the step writes m c values a point and reads none, a later one
    reads as many as it writes."""
    P, m = 1 << 20, 32
    w, lam, _ = osoe.soe_fit(0.5, m, 1e-3, 1.0)
    p = tfs.Plan(2, P, w, lam, 0.5, 1.0, 0.1, 1e-3, 8, scheme="exp")
    X, Y, tau, _ = p.alloc()
    k = p.kappa_tensor()
    t = [best_us(lambda: p.step(n, k, k, X, Y, tau)) for n in (0, 3)]
    print(f"exponential step: n=0 {t[0]:.1f} us, n=3 {t[1]:.1f} us", flush=True)
    assert t[0] < 0.75 * t[1]


def test_start_adjoint_is_not_slower_with_fp64_gradients():
    """FP64 velocity gradients add 36 bytes a point to 1500 of modes."""
    P, m = 500000, 32
    w, lam, _ = osoe.soe_fit(0.5, m, 1e-3, 1.0)
    t = []
    for kappa in ("fp32", "fp64"):
        p = tfs.Plan(3, P, w, lam, 0.5, 1.0, 0.1, 1e-3, 8, precision="fp32_modes", kappa=kappa)
        X, Y, tau, _ = p.alloc()
        ka, Xb, Hb = p.kappa_tensor(), torch.zeros_like(X), torch.zeros_like(Y)
        kb = torch.zeros((9, p.stride), dtype=torch.float64, device="cuda")
        pb = torch.zeros(p.pbar_size, dtype=torch.float64, device="cuda")
        t.append(best_us(lambda: p.step_adjoint(0, ka, None, X[0], None, X[1], Y, Y, Xb, Hb, pb, taubar=tau, kappabar_a=kb)))
    print(f"start adjoint: FP32 gradients {t[0]:.1f} us, FP64 {t[1]:.1f} us", flush=True)
    assert t[1] < 1.3 * t[0]
