"""float32 linear maps on split operands: what a row holds reaches that row only."""
import numpy as np
import pytest

import wm_synth as S

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


@pytest.mark.parametrize("M,N,K", [(70, 64, 96), (5200, 1024, 512)])
def test_rows_beside_one_that_is_not_finite(env, M, N, K):
    """A row with an infinity, a NaN or an overflowing sum leaves the bits of the
    rows beside it (64- and 128-wide tiles); so does such a feature of w."""
    wm, torch, ctx = env
    print("rows beside", M, N, K, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(7)
    a = torch.randn((M, K), generator=gen, device="cuda")
    w = torch.randn((N, K), generator=gen, device="cuda")
    b = torch.randn(N, generator=gen, device="cuda")
    run = lambda a, w: wm.wm_linear(M, N, K, wm.WM_F32, a, w, b, 0, out := torch.empty((M, N), device="cuda")) or out
    clean = run(a, w)
    rows, cols = [3, 37, M - 1], [5, N - 2]
    a2, w2 = a.clone(), w.clone()
    a2[3, 9], a2[37, 1], a2[M - 1] = float("inf"), float("nan"), 3e38
    w2[5, 7], w2[N - 2, 3] = float("nan"), float("-inf")
    out = run(a2, w2)
    keep = torch.ones((M, N), dtype=torch.bool, device="cuda")
    keep[rows], keep[:, cols] = False, False
    assert torch.equal(out[keep], clean[keep])
    assert torch.isnan(out[37]).all() and torch.isnan(out[:, 5]).all()
    assert not torch.isfinite(out[3]).any() and not torch.isfinite(out[:, N - 2]).any()


def test_state_beside_one_that_has_diverged(env):
    """Two float32 states of 405 tokens, so that a wave's rows lie in both: the
    healthy one comes out as it does alone."""
    wm, torch, ctx = env
    print("state beside", flush=True)
    g = S.Grid(Z=3, Y=9, X=15, C=128, heads=4, Kz=3, Ky=5, Kx=5)
    p = wm.wm_processor_create(ctx, g, 2, 4, wm.WM_F32, S.processor_params(g, 2, 1))
    x = torch.from_numpy(S.latent_state(g, 2, 6)).cuda()
    alone = x[1:].clone()
    x[0, 1, 4, 7] = float("nan")
    x[0, 2, 8, 14] = float("inf")
    wm.wm_processor_step(ctx, p, 2, x)
    wm.wm_processor_step(ctx, p, 1, alone)
    assert torch.equal(x[1:], alone)
    assert not torch.isfinite(x[0]).all()
    p.close()
