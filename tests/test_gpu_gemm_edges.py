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
