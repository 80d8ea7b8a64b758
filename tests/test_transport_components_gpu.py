"""The transport solve on 2-D grids of line kernels with tensor components of different size: the
ordinary state of a sheared fluid has X_xx far above X_yy, and each component's rounding stays its
own."""
import math

import pytest
import torch

from oracle import soe as osoe
from paper_2411_17294_amd import tfs
from paper_2411_17294_amd.transport import Transport

pytestmark = pytest.mark.gpu


def sheared(shape, seed, cross):
    """u = (U(y), cross V), its gradient (scale `cross` outside the shear), smooth base field."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    y = 2 * math.pi * torch.arange(shape[0], dtype=torch.float64, device="cuda")[:, None] / shape[0]
    x = 2 * math.pi * torch.arange(shape[1], dtype=torch.float64, device="cuda")[None, :] / shape[1]

    def smooth():
        a = torch.randn(6, dtype=torch.float64, device="cuda", generator=g)
        return (1.0 + a[0] ** 2 + 0.3 * torch.sin(y + a[1]) * torch.cos(2 * x + a[2]) + 0.3 * torch.cos(3 * y - x + a[3])).reshape(-1)
    u = torch.stack([cross * smooth(), smooth()])
    # kappa_ij = d u_i / d x_j; axis 1 carries the flow, axis 0 the shear direction
    kappa = torch.stack([cross * smooth(), cross ** 2 * smooth(), smooth(), -cross * smooth()])
    return 0.2 * u, 0.3 * kappa, torch.stack([smooth() for _ in range(3)])


@pytest.mark.parametrize("shape", [(405, 960), (400, 405), (1000, 486)])
@pytest.mark.parametrize("scheme", ["bdf2", "exp"])
@pytest.mark.parametrize("small", [1e-4, 1e-6])
def test_each_component_keeps_its_own_precision(shape, scheme, small):
    """Every component against the same steps with the library's transforms one plane at a time,
    relative to its own largest value: two transforms of n points at rounding unit 1.1e-16 differ by
    a few units times log2 n each way, 1e-14 over a solve; the bar is 1e-13."""
    P, m, dt, N = shape[0] * shape[1], 6, 1e-3, 3
    w, lam, _ = osoe.soe_fit(0.5, m, dt, 1.0)
    u, kap, base = sheared(shape, sum(shape), small)
    # (0, 0), (1, 1), (0, 1): the flow direction is axis 1
    X0 = 1e-2 * base * torch.tensor([small, 1.0, math.sqrt(small)], dtype=torch.float64, device="cuda")[:, None]
    out = []
    for whole in (True, False):
        p = tfs.Plan(2, P, w, lam, 0.5, 1.0, 0.1, dt, N, precision="fp64", scheme=scheme)
        st = p.stride
        pad = lambda f: torch.nn.functional.pad(f, (0, st - P)).contiguous()
        tr = Transport(p, shape, (2 * math.pi, 3.0), 0.05, 8)
        if not whole:
            tr.set_batched(False)
        print(f"shape={shape} {scheme} small={small} whole fields {whole}", flush=True)
        X, Y, tau, _ = p.alloc()
        X[0, :, :P] = X0
        ka, ua = pad(kap), pad(u)
        for n in range(N):
            tr.step(n, ka, ka, ua, ua, X, Y, tau)
        torch.cuda.synchronize()
        out.append(X[N % 2, :, :P].clone())
    for s in range(3):
        top = float(out[1][s].abs().max())
        e = float((out[0][s] - out[1][s]).abs().max()) / top
        print(f"  component {s}: size {top:.1e}, difference {e:.1e}", flush=True)
        assert e < 1e-13, s


@pytest.mark.parametrize("shape", [(405, 960), (729, 225), (972, 400), (640, 600), (500, 1024), (1024, 375)])
@pytest.mark.parametrize("method,scheme", [("splitting", "bdf2"), ("gmres", "bdf2"), ("splitting", "exp")])
def test_line_kernels_over_the_sizes_that_take_them(shape, method, scheme):
    """Odd numbers of rows, and row and column lengths of every radix, in a ragged layout, normwise as
    for the other transforms."""
    P, m, dt, N = shape[0] * shape[1], 6, 1e-3, 3
    w, lam, _ = osoe.soe_fit(0.5, m, dt, 1.0)
    u, kap, base = sheared(shape, sum(shape), 1.0)
    out = []
    for whole in (True, False):
        p = tfs.Plan(2, P, w, lam, 0.5, 1.0, 0.1, dt, N, precision="fp64", scheme=scheme, stride=P + 37, tile=0)
        pad = lambda f: torch.nn.functional.pad(f, (0, p.stride - P)).contiguous()
        tr = Transport(p, shape, (2 * math.pi, 3.0), 0.05, 6)
        if not whole:
            tr.set_batched(False)
        tr.set_method(method)
        print(f"shape={shape} {method} {scheme} whole fields {whole}", flush=True)
        X, Y, tau, diag = p.alloc()
        X[0, :, :P] = 1e-2 * base
        levels = [(pad(kap * (1 + 0.1 * n)), pad(u * (1 - 0.1 * n))) for n in range(N)]
        for n in range(N):
            (ka, ua), (kb, ub) = levels[n], levels[max(n - 1, 0)]
            tr.step(n, ka, kb, ua, ub, X, Y, tau, diag)
        torch.cuda.synchronize()
        out.append((X[N % 2, :, :P].clone(), tau[:, :P].clone(), Y.clone(), diag.clone()))
    for a, b, name in zip(out[0], out[1], ("X", "tau", "modes", "diag")):
        e = float((a - b).abs().max() / b.abs().max())
        print(f"  {name}: {e:.1e}", flush=True)
        assert e < 1e-12, name
