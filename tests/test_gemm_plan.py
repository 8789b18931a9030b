"""Tile choice of the linear maps, and the 256-wide tiles that it sends large
ones to: one K stage and odd numbers of them, several feature tiles or row
blocks per workgroup (with a short last group), rows just off a tile, and
residual rows that straddle states.

The choice is read from the host header by a small program built here, so that
the sizes below stay on the tiles that they are meant for.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import wm_synth as S
from oracle import wm_oracle as O

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_22235_amd", "csrc")

# M, N, K stages of 128 bytes, epilogue, feature tiles (N = 512: row blocks) per workgroup
WIDE = [(59907, 2048, 1, 0, 4), (80131, 1536, 1, 1, 2), (32259, 2048, 2, 1, 4), (64259, 1536, 2, 0, 3),
        (120067, 1024, 3, 0, 1), (31235, 1536, 5, 2, 3), (20227, 3072, 5, 1, 4), (126211, 512, 5, 2, 2),
        (58371, 512, 8, 0, 2), (20739, 2048, 8, 2, 3), (41475, 768, 8, 1, 1)]
SLICE = 2999                                # rows: too few for a 256-wide tile at these sizes
STATES = S.Grid(Z=5, Y=37, X=31, C=512, heads=16, Kz=3, Ky=5, Kx=5)     # 5735 tokens: 39 (mod 64)
NSTATES = 3


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text('#include "gemm_plan.hpp"\nextern "C" void plan(int M, int N, int nk, int n256, int wmax, int resid, int *o)'
                   '{ auto t = wm::plan_tiles(M, N, nk, n256, wmax, resid); o[0] = t.bm; o[1] = t.tpw; o[2] = t.rw; }\n'
                   'extern "C" int wide(int N) { return wm::wide_max(N); }\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    L = ctypes.CDLL(str(lib))

    def run(M, N, nk, resid, wmax=None):
        o = (ctypes.c_int * 3)()
        L.plan(M, N, nk, N % 256 == 0, L.wide(N) if wmax is None else wmax, resid, o)
        return tuple(o)
    return run


@pytest.mark.parametrize("M,N,nk,resid,times", [
    # us: 64 x 64, 128 x 128, and 256 x 256 by tiles per workgroup
    (130000, 2048, 1, 0, (232, 195, 185, 162, 176, 151)), (130000, 1536, 1, 0, (182, 149, 144, 129, 126)),
    (520000, 1024, 1, 0, (485, 393, 365)), (520000, 384, 1, 0, (196, 160)),
    (130000, 3072, 1, 0, (340, 295, 292, 263, 254, 251)), (130000, 1536, 2, 0, (222, 194, 169, 149, 150)),
    (520000, 512, 2, 0, (322, 272, 224, 212)), (130000, 4096, 1, 1, (918, 824, 862, 843, 889, 856)),
    (520000, 1536, 1, 1, (1396, 1306, 1413, 1396, 1418)), (520000, 512, 2, 1, (499, 456, 466, 471)),
    (130000, 3072, 3, 1, (774, 719, 768, 743, 765, 793)), (4000, 1536, 1, 0, (8.4, 9, 14.2, 23.4, 31.9)),
    (40000, 256, 1, 1, (17.6, 20.5, 22.7))])
def test_short_contractions_get_a_fast_tile(plan, M, N, nk, resid, times):
    """K of one to four stages: the tile is within a tenth of the fastest one measured."""
    bm, tpw, _ = plan(M, N, nk, resid)
    assert times[{64: 0, 128: 1, 256: 1 + tpw}[bm]] <= 1.1 * min(times)


def test_plans_are_legal(plan):
    """Over rows, columns, stages and limits: a 256-wide tile only where N allows
    one, no more of them per workgroup than the limit, row walks for N = 512."""
    r = np.random.default_rng(1)
    for _ in range(3000):
        M, N, nk = int(np.exp(r.uniform(0, 16))), 128 * int(r.integers(1, 33)), int(r.integers(1, 130))
        wmax, resid = int(r.integers(1, 5)), int(r.integers(0, 2))
        bm, tpw, rw = plan(M, N, nk, resid, wmax)
        assert bm in (64, 128, 256) and 1 <= tpw <= wmax and (bm == 256 or tpw == 1)
        assert bm != 256 or N % 256 == 0
        assert not rw or N == 512


def test_sizes_of_the_gpu_tests_are_wide(plan):
    for M, N, nk, epi, w in WIDE:
        assert plan(M, N, nk, epi == 2)[:2] == (256, w), (M, N, nk)
        assert plan(SLICE, N, nk, epi == 2)[0] < 256
    T, g = STATES.Z * STATES.Y * STATES.X, STATES
    for stage in (128, 64):                   # e4m3, bf16: MLP2 of the stacked states
        assert plan(NSTATES * T, g.C, 4 * g.C // stage, 1)[0] == 256
        assert plan(T, g.C, 4 * g.C // stage, 1)[0] < 256
    assert T % 64 and NSTATES * T > 64 * 256 >= T     # the fused LayerNorm's 128-row tiles, and its 64-row ones


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


@pytest.mark.gpu
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("M,N,stages,epi,walk", WIDE)
def test_wide_and_narrow_tiles_agree(env, M, N, stages, epi, walk, fp8):
    """All rows at once (256-wide tiles) against slices of them (narrow tiles), bit
    for bit, and some rows against float64 on the same rounded operands (relative
    L2: bf16 outputs 5e-3, whose rounding is 1.1e-3 rms; the float32 residual
    update 1e-5, in e4m3 1e-4, as the 128-deep MFMA sums at less than float32)."""
    wm, torch, ctx = env
    K = stages * (128 if fp8 else 64)
    print("wide", M, N, K, "epilogue", epi, "fp8" if fp8 else "bf16", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    dt = torch.float8_e4m3fn if fp8 else torch.bfloat16
    a = torch.randn((M, K), generator=gen, device="cuda").to(dt)
    w = (torch.randn((N, K), generator=gen, device="cuda") / K ** 0.5).to(dt)
    b = 0.1 * torch.randn(N, generator=gen, device="cuda")
    x0 = torch.randn((M, N), generator=gen, device="cuda") if epi == 2 else None

    def run(lo, hi):
        out = x0[lo:hi].clone() if epi == 2 else torch.empty((hi - lo, N), dtype=torch.bfloat16, device="cuda")
        if fp8:
            wm.wm_linear_fp8(hi - lo, N, K, a[lo:hi], 1.0, w, 1.0, b, epi, out)
        else:
            wm.wm_linear(hi - lo, N, K, wm.WM_BF16, a[lo:hi], w, b, epi, out)
        return out

    out = run(0, M)
    for lo in range(0, M, SLICE):
        hi = min(lo + SLICE, M)
        assert torch.equal(run(lo, hi), out[lo:hi]), lo
    rows = torch.cat([torch.arange(3), torch.randint(0, M, (90,)), torch.arange(M - 3, M)]).cuda()
    ref = a[rows].double().cpu().numpy() @ w.double().cpu().numpy().T + b.double().cpu().numpy()
    if epi == 2:
        ref = x0[rows].double().cpu().numpy() + ref
    elif epi == 1:
        ref = O.gelu(ref)
    assert O.rel_l2(out[rows].double().cpu().numpy(), ref) < ((1e-4 if fp8 else 1e-5) if epi == 2 else 5e-3)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [1, 2])
def test_states_straddling_wide_tiles(env, prec):
    """C = 512 states of 5735 tokens, three in separate buffers (128-row tiles of the
    fused LayerNorm, 256-wide ones of MLP2; a wave's rows lie in two states):
    bit-identical to the stacked states and to each state alone (narrow tiles)."""
    wm, torch, ctx = env
    g, B = STATES, NSTATES
    print("straddling wide tiles prec", prec, flush=True)
    p = wm.wm_processor_create(ctx, g, 1, 4, prec, S.processor_params(g, 1, 1))
    x = torch.from_numpy(S.latent_state(g, B, 6)).cuda()
    bufs, alone = ([x[b:b + 1].clone() for b in range(B)] for _ in range(2))
    wm.wm_processor_step(ctx, p, B, x)
    wm.wm_processor_step_states(ctx, p, B, torch.tensor([t.data_ptr() for t in bufs], dtype=torch.int64, device="cuda"))
    for b in range(B):
        wm.wm_processor_step(ctx, p, 1, alone[b])
        assert torch.equal(bufs[b], x[b:b + 1]) and torch.equal(alone[b], x[b:b + 1]), b
    p.close()


# a model of width 128: MLP1 has one (e4m3) or two (bf16) K stages, and two states
# send it to 256-wide tiles that walk row blocks
NARROW = S.Grid(Z=8, Y=90, X=180, C=128, heads=4, Kz=3, Ky=3, Kx=3)


def test_narrow_model_changes_tiles(plan):
    T, C = NARROW.Z * NARROW.Y * NARROW.X, NARROW.C
    for stage in (128, 64):
        assert plan(T, 4 * C, C // stage, 0)[0] == 128 and plan(2 * T, 4 * C, C // stage, 0) == (256, 2, 1)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [1, 2])
def test_narrow_model_alone_and_in_a_batch(env, prec):
    """The same bits for a state alone (128-wide tiles) and beside another."""
    wm, torch, ctx = env
    print("narrow model prec", prec, flush=True)
    p = wm.wm_processor_create(ctx, NARROW, 1, 4, prec, S.processor_params(NARROW, 1, 1))
    gen = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn((2, NARROW.Z, NARROW.Y, NARROW.X, NARROW.C), generator=gen, device="cuda")
    alone = [x[b:b + 1].clone() for b in range(2)]
    wm.wm_processor_step(ctx, p, 2, x)
    for b in range(2):
        wm.wm_processor_step(ctx, p, 1, alone[b])
        assert torch.equal(alone[b], x[b:b + 1]), b
    p.close()
