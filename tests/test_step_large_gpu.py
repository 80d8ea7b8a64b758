"""A 3-D FP64 exponential step large enough that each block takes consecutive blocks of points: the same
bits as the field cut into two smaller plans (points are independent)."""
import pytest
import torch

from oracle import soe as osoe
from paper_2411_17294_amd import tfs

pytestmark = pytest.mark.gpu


def test_consecutive_blocks_give_the_same_bits():
    P, m, N = (1 << 21) + 77, 3, 3
    cut = P // 2
    w, lam, _ = osoe.soe_fit(0.4, m, 1e-3, 0.1)
    g = torch.Generator(device="cuda").manual_seed(3)
    X0 = 1e-2 * torch.randn((6, P), dtype=torch.float64, device="cuda", generator=g)
    kap = torch.randn((9, P), dtype=torch.float64, device="cuda", generator=g)

    def run(lo, hi):
        n = hi - lo
        p = tfs.Plan(3, n, w, lam, 0.4, 1.0, 0.1, 1e-3, N, scheme="exp")
        X, Y, tau, diag = p.alloc()
        X[0, :, :n] = X0[:, lo:hi]
        k = p.kappa_tensor()
        k[:, :n] = kap[:, lo:hi]
        plain = torch.zeros((m, 6, p.stride), dtype=torch.float64, device="cuda")
        for i in range(N):
            p.step(i, k, k, X, Y, tau, diag)
        p.modes_to_plain(N, X, Y, plain)
        torch.cuda.synchronize()
        assert float(diag[5]) == 0.0
        return X[N % 2, :, :n].clone(), tau[:, :n].clone(), plain[:, :, :n].clone()
    whole, parts = run(0, P), (run(0, cut), run(cut, P))
    for a, b, c in zip(whole, *parts):
        assert torch.equal(a, torch.cat((b, c), dim=-1))
