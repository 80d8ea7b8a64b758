"""The 2-D FP64 kernel of whole grids (two points and all components a lane) at a ragged end: an even
number of points that fills neither its last wave nor its last block, against the component-split
kernel.  Same bits: a point's arithmetic does not depend on the launch."""
import math

import pytest
import torch

from oracle import soe as osoe
from paper_2411_17294_amd import tfs
from paper_2411_17294_amd.transport import Transport

pytestmark = pytest.mark.gpu


def run(P, vec, step, spatial=False, N=3, m=5):
    w, lam, _ = osoe.soe_fit(0.4, m, 1e-3, 0.1)
    p = tfs.Plan(2, P, w, lam, 0.4, 1.0, 0.1, 1e-3, N, precision="fp64", mode_form="y")
    p.tune("vec", vec)
    g = torch.Generator(device="cuda").manual_seed(7)

    def field(n, rms):
        f = torch.zeros((n, p.stride), dtype=torch.float64, device="cuda")
        f[:, :P] = rms * torch.randn((n, P), dtype=torch.float64, device="cuda", generator=g)
        return f
    X, Y, tau, diag = p.alloc()
    X[0] = field(3, 1e-2)
    ka, kb, u = field(4, 0.3), field(4, 0.3), field(2, 0.1)
    rate = field(1, 1.0).abs_()
    if spatial:
        p.set_spatial(rate, 5)
    step(p, N, ka, kb, u, X, Y, tau, diag)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(X).all()) and float(tau.abs().max()) > 0
    return X, Y, tau, diag


@pytest.mark.parametrize("spatial", [False, True])
def test_ragged_end_gives_the_same_bits(spatial):
    P = 2 * 512 * 256 * 4 - 2 * 37          # 8 full rounds of 256 blocks less 74 points

    def step(p, N, ka, kb, u, X, Y, tau, diag):
        for n in range(N):
            p.step(n, ka, kb, X, Y, tau, diag if n == N - 1 else None)
    a, b = run(P, 2, step, spatial), run(P, 1, step, spatial)
    for x, y in zip(a[:3], b[:3]):
        assert torch.equal(x, y)
    assert torch.equal(a[3][:4], b[3][:4]) and float(a[3][5]) == float(b[3][5]) == 0.0
    # a sum of P positive terms in two orders: P eps in the worst case, far less in either
    assert abs(float(a[3][4] - b[3][4])) < 1e-12 * abs(float(b[3][4]))


def test_ragged_split_step_gives_the_same_bits():
    """The transport step's form, without the local solve (1022 x 1026 points)."""
    shape = (1022, 1026)

    def step(p, N, ka, kb, u, X, Y, tau, diag):
        tr = Transport(p, shape, (2 * math.pi, 3.0), 0.1, 2)
        for n in range(N):
            tr.step(n, ka, kb, u, u, X, Y, tau, diag)
    a, b = run(shape[0] * shape[1], 2, step), run(shape[0] * shape[1], 1, step)
    for x, y in zip(a[:3], b[:3]):
        assert torch.equal(x, y)
