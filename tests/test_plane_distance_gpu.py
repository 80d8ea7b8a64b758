"""Grid planes an odd number of values apart: the transport and the coupled step give what they give
with planes an even distance apart (real transforms of even length go in pairs of values)."""
import math

import pytest
import torch

from oracle import soe as osoe
from paper_2411_17294_amd import tfs
from paper_2411_17294_amd.ns import Solver
from paper_2411_17294_amd.transport import Transport

pytestmark = pytest.mark.gpu

SHAPES = [(24, 32), (24, 33), (8, 12, 10), (6, 10, 9)]


def fields(shape, count, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((count, math.prod(shape)), dtype=torch.float64, device="cuda", generator=g)


def close(a, b, name):
    """Rounding of two orders of the same transforms over a few steps: 1e-12 normwise."""
    e = float((a - b).abs().max() / b.abs().max())
    print(f"  {name}: {e:.1e}", flush=True)
    assert e < 1e-12, name


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("extra", [1, 2])
def test_transport_planes(shape, extra):
    d, P, m, dt = len(shape), math.prod(shape), 4, 1e-3
    w, lam, _ = osoe.soe_fit(0.5, m, dt, 1.0)
    u, kap, X0 = fields(shape, d, 1), fields(shape, d * d, 2), fields(shape, d * (d + 1) // 2, 3)
    out = []
    for stride in (P + P % 2, P + P % 2 + extra):
        p = tfs.Plan(d, P, w, lam, 0.5, 1.0, 0.1, dt, 4, stride=stride, tile=0)
        pad = lambda f: torch.nn.functional.pad(f, (0, p.stride - P)).contiguous()
        tr = Transport(p, shape, (2 * math.pi,) * d, 0.1, 4)
        print(f"transport {shape} stride {p.stride} whole fields {tr.batched}", flush=True)
        X, Y, tau, _ = p.alloc()
        X[0, :, :P] = 1e-2 * X0
        for n in range(3):
            tr.step(n, pad(0.1 * kap), pad(0.1 * kap), pad(0.1 * u), pad(0.1 * u), X, Y, tau)
        torch.cuda.synchronize()
        out.append((X[1, :, :P].clone(), tau[:, :P].clone()))
    close(out[1][0], out[0][0], "X")
    close(out[1][1], out[0][1], "tau")


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("extra", [1, 2])
def test_coupled_planes(shape, extra):
    d, P, m, dt = len(shape), math.prod(shape), 4, 1e-3
    w, lam, _ = osoe.soe_fit(0.5, m, dt, 1.0)
    u0, X0 = fields(shape, d, 1), fields(shape, d * (d + 1) // 2, 3)
    out = []
    for stride in (P + P % 2, P + P % 2 + extra):
        p = tfs.Plan(d, P, w, lam, 0.5, 1.0, 0.1, dt, 4, stride=stride, tile=0)
        sol = Solver(p, shape, (2 * math.pi,) * d, 0.9, dt)
        print(f"coupled {shape} stride {p.stride} whole fields {sol.batched}", flush=True)
        X, Y, tau, _ = p.alloc()
        u, kappa, uh, fh = sol.alloc()
        X[0, :, :P] = 1e-2 * X0
        u[:, :P] = 0.1 * u0
        sol.init(u, uh, kappa)
        for n in range(3):
            sol.step(n, u, uh, fh, kappa, X, Y, tau)
        torch.cuda.synchronize()
        out.append((u[:, :P].clone(), kappa[:, :P].clone(), X[1, :, :P].clone(), tau[:, :P].clone()))
    for a, b, name in zip(out[1], out[0], ("u", "kappa", "X", "tau")):
        close(a, b, name)
