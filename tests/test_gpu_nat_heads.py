"""The ring attention kernels walk several heads per workgroup on large grids,
the next head's first levels in flight while the last of one are computed.
Every head has to come out as it does alone (one head per workgroup), bit for
bit, also where scores far above a query's own make a workgroup walk a head a
second time.
"""
import pytest

import wm_synth as S

pytestmark = pytest.mark.gpu

# heads: 4, 2 and 1 of them per workgroup at this grid
HEADS = [16, 14, 13]


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


@pytest.mark.parametrize("sharp", [False, True])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("H", HEADS)
def test_heads_alone_and_together(env, H, fp8, sharp):
    wm, torch, ctx = env
    Z, Y, X = 8, 90, 180
    print("heads", H, "fp8" if fp8 else "bf16", "sharp" if sharp else "", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, Z * Y * X, H, 32), generator=gen, device="cuda") for _ in range(3))
    if sharp:                     # every third head
        q[:, :, 1::3] *= 12.0
        k[:, :, 1::3] *= 8.0
    for t in (q, k, v):           # one largest magnitude, and so one e4m3 scale, for all heads
        m = t.abs().max()
        t[0, 0, :, 0] = m
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    rpb = torch.randn((H, 9, 13, 13), generator=gen, device="cuda")
    prec = 2 if fp8 else 1
    grid = lambda h: S.Grid(Z=Z, Y=Y, X=X, C=32 * h, heads=h, Kz=5, Ky=7, Kx=7, periodic_mask=4)
    out = torch.empty_like(q)
    wm.wm_nat_forward(ctx, grid(H), 1, prec, q, k, v, rpb, out)
    assert torch.isfinite(out.float()).all()
    for h in range(H):
        one = [t[:, :, h:h + 1].contiguous() for t in (q, k, v)]
        alone = torch.empty_like(one[0])
        wm.wm_nat_forward(ctx, grid(1), 1, prec, *one, rpb[h:h + 1].contiguous(), alone)
        assert torch.equal(out[:, :, h:h + 1], alone), h
