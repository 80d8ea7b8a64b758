"""Forward steps whose layout allows no wide access (an odd plane stride, a pointer between two wide
elements), with enough points for whole blocks: the same bits as one point a lane."""
import pytest
import torch

from oracle import soe as osoe
from paper_2411_17294_amd import tfs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,prec,kappa", [(2, "fp64", "fp64"), (3, "fp64", "fp64"), (2, "fp32_modes", "fp64"), (3, "fp32_modes", "fp32")])
@pytest.mark.parametrize("scheme,spatial", [("bdf2", False), ("exp", False), ("bdf2", True), ("exp", True)])
@pytest.mark.parametrize("tile,offset", [(0, 0), (20, 1)])
def test_same_bits_as_one_point_a_lane(d, prec, kappa, scheme, spatial, tile, offset):
    """tile 0: an odd stride; tile 20: a wave crosses several tiles, and every field starts one element
    past a wide boundary.  196608 points are whole rounds of blocks for every width, 105 more a ragged
    end."""
    if spatial and kappa == "fp32":
        pytest.skip("the spatial form takes FP64 gradients")
    P, m, N = 196608 + 105, 5, 4
    w, lam, _ = osoe.soe_fit(0.4, m, 1e-3, 0.1)
    out = []
    for vec in (0, 1):
        p = tfs.Plan(d, P, w, lam, 0.4, 1.0, 0.1, 1e-3, N, precision=prec, kappa=kappa, scheme=scheme, tile=tile)
        p.tune("vec", vec)
        g = torch.Generator(device="cuda").manual_seed(7)

        def field(n, dtype=torch.float64, rms=0.0):
            """n planes, `offset` elements past an aligned start."""
            f = torch.zeros(n * p.stride + offset, dtype=dtype, device="cuda")[offset:]
            if rms:
                f.view(n, p.stride)[:, :P] = rms * torch.randn((n, P), dtype=torch.float64, device="cuda", generator=g)
            return f
        X = field(p.x_levels * p.c)
        X[:p.c * p.stride] = field(p.c, rms=1e-2)
        Y, tau = field(p.mode_levels * m * p.c, p.mode_dtype), field(p.c)
        ka, kb = field(d * d, p.kappa_dtype, 1.0), field(d * d, p.kappa_dtype, 1.0)
        rate = field(1, rms=1.0).abs_() if spatial else None
        if spatial:
            p.set_spatial(rate, 3)
        diag = torch.zeros(6, dtype=torch.float64, device="cuda")
        print(f"d={d} {prec} {scheme} spatial={spatial} tile={tile} vec={vec} stride={p.stride}", flush=True)
        for n in range(N):
            p.step(n, ka, kb, X, Y, tau, diag if n % 2 else None)
        torch.cuda.synchronize()
        out.append((X, Y, tau))
    assert bool(torch.isfinite(out[0][0]).all()) and float(out[0][2].abs().max()) > 0
    for a, b in zip(*out):
        assert torch.equal(a, b)


def test_an_odd_stride_costs_its_cache_lines():
    """The same step with an odd and an even stride: a wave's kilobyte of a plane spans nine cache lines
    instead of eight, and the loads are narrower.  Two calls on one device, far from either's spread
    (1.25; with one point a lane 1.9)."""
    P, m = 1 << 18, 32
    w, lam, _ = osoe.soe_fit(0.5, m, 1e-3, 1.0)
    t = []
    for stride in (P, P + 1):
        p = tfs.Plan(3, P, w, lam, 0.5, 1.0, 0.1, 1e-3, 8, precision="fp32_modes", scheme="exp", stride=stride, tile=0)
        X, Y, tau, _ = p.alloc()
        k = p.kappa_tensor()
        best = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                p.step(3, k, k, X, Y, tau)
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b) / 20 * 1e3)
        t.append(min(best))
    print(f"even stride {t[0]:.1f} us, odd {t[1]:.1f} us", flush=True)
    assert t[1] < 1.6 * t[0]
