"""The wide GEMM tiles (N a multiple of 256) at the edges of their ranges: one
K stage per tile (K = 64 bf16, 128 e4m3), odd stage counts, one row, rows just
off a tile, several feature tiles or row blocks per workgroup; and residual
rows that straddle states.

Reference: float64 on the same rounded operands.  Tolerances (relative L2):
bf16 outputs 5e-3 (a bf16 rounding is 1.1e-3 rms, 3.9e-3 at most); the float32
residual update 1e-5 in bf16 (float32 sums of exact products) and 1e-4 in e4m3
(the 128-deep MFMA sums its products at less than float32 precision).
"""
import numpy as np
import pytest

import wm_synth as S
from oracle import wm_oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [(1, 256, 1), (255, 512, 1), (257, 256, 2), (513, 1536, 3), (700, 2048, 1), (770, 512, 5), (300, 3072, 2)]


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


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("M,N,stages", SHAPES)
def test_wide_tiles(env, M, N, stages, epi, fp8):
    wm, torch, ctx = env
    K = stages * (128 if fp8 else 64)
    print("wide tiles", M, N, K, "epilogue", epi, "fp8" if fp8 else "bf16", flush=True)
    r = np.random.default_rng(M + N + K)
    dt = torch.float8_e4m3fn if fp8 else torch.bfloat16
    a = torch.from_numpy(r.standard_normal((M, K)).astype(np.float32)).cuda().to(dt)
    w = torch.from_numpy((r.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)).cuda().to(dt)
    b = torch.from_numpy((0.1 * r.standard_normal(N)).astype(np.float32)).cuda()
    x0 = torch.from_numpy(r.standard_normal((M, N)).astype(np.float32)).cuda()

    def run(rows):
        out = x0[:rows].clone() if epi == 2 else torch.empty((rows, N), dtype=torch.bfloat16, device="cuda")
        if fp8:
            wm.wm_linear_fp8(rows, N, K, a, 1.0, w, 1.0, b, epi, out)
        else:
            wm.wm_linear(rows, N, K, wm.WM_BF16, a, w, b, epi, out)
        return out

    out = run(M)
    ref = a.float().double().cpu().numpy() @ w.float().double().cpu().numpy().T + b.double().cpu().numpy()
    if epi == 2:
        ref = x0.double().cpu().numpy() + ref
    elif epi == 1:
        ref = O.gelu(ref)
    assert O.rel_l2(out.double().cpu().numpy(), ref) < ((1e-4 if fp8 else 1e-5) if epi == 2 else 5e-3)
    # a row's result does not depend on how many rows follow it
    for rows in {1, M // 2 + 1}:
        assert torch.equal(run(rows), out[:rows])


@pytest.mark.parametrize("prec", [1, 2])
def test_states_straddling_waves(env, prec):
    """C = 512 states of 405 tokens in separate buffers: the rows of a wave of
    the residual epilogues (64) lie in two states; bit-identical to the step
    on the stacked states."""
    wm, torch, ctx = env
    g = S.Grid(Z=3, Y=9, X=15, C=512, heads=16, Kz=3, Ky=5, Kx=5)
    B = 3
    print("straddling states prec", prec, flush=True)
    p = wm.wm_processor_create(ctx, g, 2, 4, prec, S.processor_params(g, 2, 1))
    x = S.latent_state(g, B, 6)
    xb = torch.from_numpy(x).cuda()
    wm.wm_processor_step(ctx, p, B, xb)
    bufs = [torch.from_numpy(x[b:b + 1].copy()).cuda() for b in range(B)]
    wm.wm_processor_step_states(ctx, p, B, torch.tensor([t.data_ptr() for t in bufs], dtype=torch.int64, device="cuda"))
    for b in range(B):
        assert torch.equal(bufs[b], xb[b:b + 1])
    p.close()


@pytest.mark.parametrize("prec", [1, 2])
@pytest.mark.parametrize("C,shape", [(128, (5, 45, 90)), (256, (5, 20, 22)), (512, (8, 60, 36))])
def test_tile_choice_does_not_show(env, C, shape, prec):
    """The GEMM tiles depend on the number of rows (64, 128 or 256 rows; 64 or
    128 with the fused LayerNorm): a state alone and in a batch of 4 runs on
    different ones and gets the same bits."""
    wm, torch, ctx = env
    g = S.Grid(Z=shape[0], Y=shape[1], X=shape[2], C=C, heads=C // 32, Kz=3, Ky=5, Kx=5)
    print("tile choice", C, shape, "prec", prec, flush=True)
    p = wm.wm_processor_create(ctx, g, 1, 4, prec, S.processor_params(g, 1, 1))
    x = torch.from_numpy(S.latent_state(g, 1, 6)).cuda()
    xb = x.repeat(4, 1, 1, 1, 1).contiguous()
    xb[1:3].neg_()
    xs = x.clone()
    wm.wm_processor_step(ctx, p, 4, xb)
    wm.wm_processor_step(ctx, p, 1, xs)
    assert torch.equal(xb[:1], xs) and torch.equal(xb[3:], xs)
    p.close()


@pytest.mark.parametrize("M,N,K", [(1, 64, 32), (63, 192, 96), (65, 128, 64), (129, 384, 32), (700, 512, 2048), (5200, 1024, 160)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_f32_split(env, M, N, K, epi):
    """float32 maps run as six bf16 products of three-way split operands, on
    64- or 128-wide tiles: as exact as float32 arithmetic.  Bound: a sum of K
    products rounded K / 32 * 6 times, each by at most 2^-24 of a partial sum
    of at most sqrt(K) |a||w| here: 2^-24 sqrt(6 K / 32), plus 3e-7 for the
    GELU's erf and 2^-24 for the store; held with a factor of 2."""
    wm, torch, ctx = env
    print("f32", M, N, K, epi, flush=True)
    r = np.random.default_rng(M + N + K + epi)
    a = torch.from_numpy(r.standard_normal((M, K)).astype(np.float32)).cuda()
    w = torch.from_numpy((r.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)).cuda()
    b = torch.from_numpy((0.1 * r.standard_normal(N)).astype(np.float32)).cuda()
    x0 = torch.from_numpy(r.standard_normal((M, N)).astype(np.float32)).cuda()
    out = x0.clone()
    wm.wm_linear(M, N, K, wm.WM_F32, a, w, b, epi, out)
    ref = a.double().cpu().numpy() @ w.double().cpu().numpy().T + b.double().cpu().numpy()
    if epi == 2:
        ref = x0.double().cpu().numpy() + ref
    elif epi == 1:
        ref = O.gelu(ref)
    tol = 2 * (2.0 ** -24 * (np.sqrt(6 * K / 32) + 1) + (6e-7 if epi == 1 else 0))
    assert O.rel_l2(out.double().cpu().numpy(), ref) < tol
    out1 = x0[:1].clone()
    wm.wm_linear(1, N, K, wm.WM_F32, a, w, b, epi, out1)
    assert torch.equal(out1, out[:1])


@pytest.mark.parametrize("M,N", [(70, 64), (5200, 1024)])
def test_f32_not_finite(env, M, N):
    """Infinities, NaN and values next to the largest float32 in the operands
    give what float32 arithmetic gives: the split's parts alone would give NaN
    for inf * 1 and for a value that rounds up to infinity in bf16."""
    wm, torch, ctx = env
    K = 64
    print("f32 not finite", M, N, flush=True)
    r = np.random.default_rng(5)
    a = r.integers(-4, 5, (M, K)).astype(np.float32)
    w = r.integers(1, 5, (N, K)).astype(np.float32)
    big = np.finfo(np.float32).max
    a[3, 5], a[4, 6], a[5, 7] = np.inf, -np.inf, np.nan
    a[6] = 0.0
    a[6, 9] = big
    w[:, 9] = 1.0                    # row 6: the largest float32 times 1
    a[7] = big                       # row 7: overflows
    w[2, 11] = np.inf
    a[:, 11] = np.abs(a[:, 11]) + 1  # inf times a positive value (NaN and inf rows keep theirs)
    a[6, 11] = 1.0
    b = np.zeros(N, np.float32)
    dev = [torch.from_numpy(t).cuda() for t in (a, w, b)]
    out = torch.empty((M, N), device="cuda")
    wm.wm_linear(M, N, K, wm.WM_F32, dev[0], dev[1], dev[2], 0, out)
    with np.errstate(all="ignore"):
        ref = a.astype(np.float64) @ w.astype(np.float64).T
        ref[6] = np.where(np.arange(N) == 2, np.inf, big)      # (+ w[n, 11], far below big's last bit)
        ref = ref.astype(np.float32)
    got = out.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    ok = ~np.isnan(ref)
    assert np.array_equal(got[ok], ref[ok])
