"""float32 linear maps on split operands: what a row holds reaches that row only,
and operands of any size keep all their bits."""
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


@pytest.mark.parametrize("ea,ew", [(-126, 0), (-126, 60), (60, -126), (-112, 0), (0, -118), (-60, -60), (110, 0), (0, 120), (-126, 126), (60, 60)])
@pytest.mark.parametrize("M,N,K", [(70, 64, 96), (5200, 1024, 160)])
def test_powers_of_two_commute(env, M, N, K, ea, ew):
    """Operands in +-[1, 2) times powers of two, so that no float32 operation
    rounds differently: the result is that of the operands themselves times both
    powers, bit for bit, down to the smallest normal operands."""
    wm, torch, ctx = env
    print("powers of two", M, N, K, ea, ew, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M)

    def draw(r, c):
        t = torch.rand((r, c), generator=gen, device="cuda") + 1.0
        return torch.where(torch.rand((r, c), generator=gen, device="cuda") < 0.5, -t, t)

    a, w, b = draw(M, K), draw(N, K), torch.zeros(N, device="cuda")
    run = lambda a, w: wm.wm_linear(M, N, K, wm.WM_F32, a, w, b, 0, out := torch.empty((M, N), device="cuda")) or out
    ref = run(a, w)
    exact = a.double() @ w.double().T
    assert (ref.double() - exact).norm() < 2e-6 * exact.norm()
    pow2 = lambda e: torch.tensor(2.0, dtype=torch.float64).pow(e).item()
    out = run(a * pow2(ea), w * pow2(ew))
    # (in float64: the powers of a product may lie beyond float32's range)
    got = out.double() / pow2(ea) / pow2(ew)
    rel = (got - exact).norm() / exact.norm()
    print("  rel_l2", rel.item(), flush=True)
    assert rel < 2e-6
    big = max(ea, ew) >= 104 or ea + ew >= 70        # (past the split's range: float32 MFMAs, another order of the sums)
    small = ea + ew < -110                           # (sums may fall below the smallest normal number)
    if not big and not small:
        assert torch.equal(got, ref.double())


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


def test_nan_rows_and_features(env):
    """Every row of a state or every feature of w NaN, and NaN rows beside an
    infinity and an overflow: what float32 arithmetic gives."""
    wm, torch, ctx = env
    M, N, K = 200, 192, 160
    print("nan rows", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(2)
    b = torch.zeros(N, device="cuda")
    run = lambda a, w: wm.wm_linear(M, N, K, wm.WM_F32, a, w, b, 0, out := torch.empty((M, N), device="cuda")) or out
    a, w = torch.rand((M, K), generator=gen, device="cuda") + 0.5, torch.rand((N, K), generator=gen, device="cuda") + 0.5
    clean = run(a, w)
    assert torch.isnan(run(torch.full_like(a, float("nan")), w)).all()
    assert torch.isnan(run(a, torch.full_like(w, float("nan")))).all()
    a2, w2 = a.clone(), w.clone()
    a2[::2, 3] = float("nan")               # every other row
    a2[1, 7], a2[65, 9] = float("inf"), -float("inf")
    a2[3] = 3e38
    w2[5, 150], w2[130, 0] = float("nan"), float("nan")
    out = run(a2, w2)
    assert torch.isnan(out[::2]).all() and torch.isnan(out[:, [5, 130]]).all()
    rest = torch.ones(N, dtype=torch.bool, device="cuda")
    rest[[5, 130]] = False
    assert (out[1, rest] == float("inf")).all() and (out[65, rest] == -float("inf")).all() and (out[3, rest] == float("inf")).all()
    rows = [r for r in range(1, M, 2) if r not in (1, 3, 65)]
    assert torch.equal(out[rows][:, rest], clean[rows][:, rest])


def test_diverged_state_costs_little_more(env):
    """A float32 map of NaN rows takes less than 1.5 times a finite one's time
    (three times where every sum was done again)."""
    wm, torch, ctx = env
    M, N, K = 64800, 512, 512
    print("diverged, time", flush=True)
    w, b, out = torch.randn((N, K), device="cuda"), torch.zeros(N, device="cuda"), torch.empty((M, N), device="cuda")
    times = []
    for a in (torch.randn((M, K), device="cuda"), torch.full((M, K), float("nan"), device="cuda")):
        best = float("inf")
        for _ in range(5):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            for _ in range(3):
                wm.wm_linear(M, N, K, wm.WM_F32, a, w, b, 0, out)
            t[1].record()
            torch.cuda.synchronize()
            best = min(best, t[0].elapsed_time(t[1]))
        times.append(best)
    print("  ms", times, flush=True)
    assert times[1] < 1.5 * times[0]
