"""Attention with any window and any periodic axes (float32, and bf16 outside
the tiled kernels' windows) where its workgroups can go wrong: halos of more
units than one pass lists, lon counts that are no multiple of a workgroup's,
windows as long as their axis, every kind of border, bias tables too long for
LDS, and rows beyond 32-bit byte offsets.

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

# Z, Y, X, Kz, Ky, Kx, periodic mask
GRIDS = [
    (1, 1, 1, 1, 1, 1, 4),
    (2, 3, 7, 1, 1, 1, 0),
    (5, 9, 7, 5, 7, 7, 4),
    (6, 7, 19, 3, 5, 9, 4),
    (3, 5, 11, 3, 5, 5, 0),
    (7, 9, 13, 5, 7, 7, 7),
    (9, 17, 18, 9, 17, 17, 4),
    (9, 17, 23, 9, 17, 17, 0),
    (1, 2, 1030, 1, 1, 1027, 4),
    (1, 1, 1030, 1, 1, 1029, 0),
]


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


def _grid(z, y, x, kz, ky, kx, mask, C):
    return S.Grid(Z=z, Y=y, X=x, C=C, heads=C // 32, Kz=kz, Ky=ky, Kx=kx, periodic_mask=mask)


def _inputs(torch, shape, tbl, dt, seed):
    r = np.random.default_rng(seed)
    qkv = [torch.from_numpy(r.standard_normal(shape).astype(np.float32)).to(dt).cuda() for _ in range(3)]
    return qkv, torch.from_numpy(r.standard_normal(tbl).astype(np.float32)).cuda()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims", GRIDS)
def test_general_windows(env, dims, bf16):
    wm, torch, ctx = env
    z, y, x, kz, ky, kx, mask = dims
    print("general window", dims, "bf16" if bf16 else "f32", flush=True)
    dt = torch.bfloat16 if bf16 else torch.float32
    g = _grid(*dims, C=128)
    (q, k, v), rpb = _inputs(torch, (2, z * y * x, 4, 32), (4, 2 * kz - 1, 2 * ky - 1, 2 * kx - 1), dt, sum(dims))
    out = torch.full_like(q, float("nan"))
    wm.wm_nat_forward(ctx, g, 2, int(bf16), q, k, v, rpb, out)
    f = lambda t: t.double().cpu().numpy()
    ref = np.stack([O.nat_c(f(q[b]), f(k[b]), f(v[b]), f(rpb), g) for b in range(2)])
    err = O.rel_l2(f(out), ref)
    print("  rel_l2", err, flush=True)
    assert err <= (5e-3 if bf16 else 2e-6)


def test_not_finite_stays_local(env):
    """A NaN value reaches the queries whose window holds it, and no query
    more than a window and a query group away."""
    wm, torch, ctx = env
    dims = (5, 23, 14, 3, 5, 5, 4)
    print("not finite", dims, flush=True)
    g = _grid(*dims, C=128)
    (q, k, v), rpb = _inputs(torch, (1, 5 * 23 * 14, 4, 32), (4, 5, 9, 9), torch.float32, 5)
    clean, out = torch.empty_like(q), torch.empty_like(q)
    wm.wm_nat_forward(ctx, g, 1, 0, q, k, v, rpb, clean)
    v.view(5, 23, 14, 4, 32)[2, 11, 13] = float("nan")
    wm.wm_nat_forward(ctx, g, 1, 0, q, k, v, rpb, out)
    out, clean = out.view(5, 23, 14, 4, 32), clean.view(5, 23, 14, 4, 32)
    assert torch.isnan(out[1:4, 9:14, [11, 12, 13, 0, 1]]).all()
    assert torch.equal(out[:, :7], clean[:, :7]) and torch.equal(out[:, 16:], clean[:, 16:])
    assert torch.equal(out[:, :, 3:10], clean[:, :, 3:10])


def test_far_rows(env):
    """Rows past 4 GiB: each head gives what it gives as a tensor of its own."""
    wm, torch, ctx = env
    z, y, x, C = 1, 97, 1361, 8160
    print("far rows", z, y, x, C, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((1, y * x, C), generator=gen, device="cuda") for _ in range(3))
    assert q.numel() * 4 > 1 << 32
    rpb = torch.randn((C // 32, 1, 5, 5), generator=gen, device="cuda")
    out = torch.empty_like(q)
    wm.wm_nat_forward(ctx, _grid(z, y, x, 1, 3, 3, 4, C), 1, 0, q, k, v, rpb, out)
    heads = [0, 100, 200, 254]
    cut = lambda t: torch.stack([t.view(1, y * x, C // 32, 32)[:, :, h] for h in heads], 2).contiguous()
    got, near = cut(out), torch.empty((1, y * x, 4, 32), device="cuda")
    wm.wm_nat_forward(ctx, _grid(z, y, x, 1, 3, 3, 4, 128), 1, 0, cut(q), cut(k), cut(v), rpb[heads].contiguous(), near)
    assert (got - near).norm() <= 1e-6 * near.norm()
