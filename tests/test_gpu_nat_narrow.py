"""General attention on grids of a few lons: workgroups of one to four lon groups.

Reference: the float64 oracle on the same rounded operands.  Tolerances
(relative L2): float32 2e-6 (scores of size 20 rounded at 2^-24 give
probabilities good to 1.2e-6); bf16 5e-3 (probabilities and outputs rounded to
8 bits: 1.7e-3 rms each at the most).
"""
import numpy as np
import pytest

import wm_synth as S
from oracle import wm_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2503_22235_amd as wm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    wm.lib()
    ctx = wm.wm_ctx_create(0)
    yield wm, torch, ctx
    torch.cuda.synchronize()
    ctx.close()


# Z, Y, X, Kz, Ky, Kx, periodic mask: lon groups per workgroup 1, 1, 2, 2, 3, 3, 4, 3, 3
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims", [(9, 11, 1, 3, 5, 1, 0), (33, 9, 2, 7, 9, 1, 2), (5, 21, 3, 3, 5, 3, 4), (5, 9, 4, 3, 9, 3, 0),
                                  (3, 18, 5, 3, 13, 5, 4), (6, 7, 6, 5, 7, 5, 1), (4, 8, 8, 3, 5, 7, 5), (4, 9, 9, 3, 5, 9, 0),
                                  (3, 9, 17, 3, 3, 7, 4)])
def test_narrow_grids(env, dims, bf16):
    wm, torch, ctx = env
    z, y, x, kz, ky, kx, mask = dims
    print("narrow", dims, "bf16" if bf16 else "f32", flush=True)
    r = np.random.default_rng(sum(dims))
    dt = torch.bfloat16 if bf16 else torch.float32
    g = S.Grid(Z=z, Y=y, X=x, C=96, heads=3, Kz=kz, Ky=ky, Kx=kx, periodic_mask=mask)
    q, k, v = (torch.from_numpy(r.standard_normal((2, z * y * x, 3, 32)).astype(np.float32)).to(dt).cuda() for _ in range(3))
    rpb = torch.from_numpy(r.standard_normal((3, 2 * kz - 1, 2 * ky - 1, 2 * kx - 1)).astype(np.float32)).cuda()
    out = torch.full_like(q, float("nan"))
    wm.wm_nat_forward(ctx, g, 2, int(bf16), q, k, v, rpb, out)
    f = lambda t: t.double().cpu().numpy()
    ref = np.stack([O.nat_c(f(q[b]), f(k[b]), f(v[b]), f(rpb), g) for b in range(2)])
    assert O.rel_l2(f(out), ref) <= (5e-3 if bf16 else 2e-6)


def test_few_lons_cost_no_idle_waves(env):
    """Two lons or eight, the same tokens, groups and halo: about the same time
    (four times as long when three of four waves walk a halo for nothing)."""
    wm, torch, ctx = env
    times = {}
    for X in (2, 8):
        Y = 65536 // X
        print("few lons", X, flush=True)
        g = S.Grid(Z=4, Y=Y, X=X, C=256, heads=8, Kz=3, Ky=5, Kx=1, periodic_mask=0)
        gen = torch.Generator(device="cuda").manual_seed(1)
        q, k, v = (torch.randn((1, 4 * Y * X, 8, 32), generator=gen, device="cuda") for _ in range(3))
        rpb = torch.randn((8, 5, 9, 1), generator=gen, device="cuda")
        out = torch.empty_like(q)
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(3):
                wm.wm_nat_forward(ctx, g, 1, 0, q, k, v, rpb, out)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        times[X] = best
    print("  ms", times, flush=True)
    assert times[2] < 2 * times[8]
