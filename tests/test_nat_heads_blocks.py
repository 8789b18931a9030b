"""Several heads per workgroup in the blocks' attention (head-major rows): the
next head's levels are in flight while the last of one are computed, also where
scores far above a query's own send a workgroup on a second walk.

A state that repeats itself in lon gives, on a grid three times as long, three
times the output of the short grid, bit for bit: lon tiles of 8 fall on the same
tokens.  The short grid is small enough for one head per workgroup.  The number
of heads is read from the host header by a small program built here.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import wm_synth as S

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_22235_amd", "csrc")
HEAD_MAJOR, TOKEN_MAJOR, E4M3 = 0, 1, 2
REPEAT = 3

# precision, states, short grid, heads per workgroup on the long grid
CASES = [("fp8", 1, (8, 104, 56, 5, 7, 7), 2), ("fp8", 4, (8, 104, 56, 5, 7, 7), 4), ("fp8", 1, (5, 96, 56, 3, 5, 5), 2),
         ("fp8", 2, (5, 96, 56, 3, 3, 3), 2), ("bf16", 1, (5, 96, 56, 3, 5, 5), 2), ("bf16", 2, (5, 96, 56, 3, 3, 3), 2),
         ("bf16", 1, (8, 104, 56, 5, 7, 7), 1)]


def _grid(dims, lon=1):
    z, y, x, kz, ky, kx = dims
    return S.Grid(Z=z, Y=y, X=lon * x, C=512, heads=16, Kz=kz, Ky=ky, Kx=kx)


@pytest.fixture(scope="module")
def heads(tmp_path_factory):
    d = tmp_path_factory.mktemp("heads")
    src, lib = d / "heads.cpp", d / "heads.so"
    src.write_text('#include "nat_plan.hpp"\nextern "C" int heads(long tiles, int H, int Kz, int rows)'
                   '{ return wm::nat_heads(tiles, H, Kz, (wm::NatRows)rows); }\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    f = ctypes.CDLL(str(lib)).heads
    f.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return f


def _tiles(g, B):
    return B * -(-g.Z // 4) * -(-g.Y // 4) * -(-g.X // 8)


# us with 1, 2 and 4 heads
@pytest.mark.parametrize("tiles,H,Kz,rows,times", [
    (1058, 16, 5, HEAD_MAJOR, (282.3, 282.0, 283.6)), (552, 16, 5, HEAD_MAJOR, (139.8, 144.4, 150.3)),
    (782, 16, 5, HEAD_MAJOR, (208.9, 212.8, 217.6)), (288, 4, 5, HEAD_MAJOR, (23.6, 25.7, 35.4)),
    (1058, 16, 3, HEAD_MAJOR, (204.4, 194.5, 196.9)), (288, 32, 3, HEAD_MAJOR, (110.6, 105.9, 106.6)),
    (288, 4, 3, HEAD_MAJOR, (21.3, 21.8, 34.2)), (1058, 4, 3, HEAD_MAJOR, (55.7, 56.0, 61.5)),
    (1058, 16, 5, TOKEN_MAJOR, (398.4, 371.2, 363.9)), (1058, 4, 5, TOKEN_MAJOR, (78.0, 82.6, 92.7)),
    (1058, 16, 5, E4M3, (256.2, 246.4, 245.5)), (768, 16, 5, E4M3, (185.0, 177.3, 179.0)),
    (288, 4, 5, E4M3, (24.7, 27.4, 39.5)), (1152, 32, 3, E4M3, (384.6, 361.4, 353.6)),
    (552, 4, 5, E4M3, (39.5, 43.6, 52.2))])
def test_heads_per_workgroup_follow_the_times(heads, tiles, H, Kz, rows, times):
    """Within 2.5% of the fastest, and no slower than one head by more than 1%."""
    t = times[{1: 0, 2: 1, 4: 2}[heads(tiles, H, Kz, rows)]]
    assert t <= 1.025 * min(times) and t <= 1.01 * times[0]


def test_more_heads_than_one_are_worth_their_traffic(heads):
    """bf16 blocks with window 5x7x7 walk one head: two take the same time and fetch a quarter more."""
    for tiles in (1, 500, 1058, 4232, 100000):
        assert heads(tiles, 16, 5, HEAD_MAJOR) == 1


def test_cases_walk_the_heads_they_are_meant_to(heads):
    for prec, B, dims, n in CASES:
        rows = E4M3 if prec == "fp8" else HEAD_MAJOR
        assert heads(_tiles(_grid(dims, REPEAT), B), 16, dims[3], rows) == n, (prec, B, dims)
        assert heads(_tiles(_grid(dims), 1), 16, dims[3], rows) == 1


@pytest.mark.gpu
@pytest.mark.parametrize("sharp", [False, True])
@pytest.mark.parametrize("prec,B,dims,n", CASES)
def test_repeated_states(prec, B, dims, n, sharp):
    """sharp: in every third head a bias of -100 at the query's own key puts all
    other scores some 144 (log2) above it, past what either precision's weights
    hold, so that each workgroup walks these heads twice."""
    import torch
    import paper_2503_22235_amd as wm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("repeated states", prec, B, dims, n, "sharp" if sharp else "", flush=True)
    ctx = wm.wm_ctx_create(0)
    g1, g3 = _grid(dims), _grid(dims, REPEAT)
    params = S.processor_params(g1, 1, 1)
    if sharp:
        at = 0
        for name, shape in S.block_param_layout(g1):
            size = int(np.prod(shape))
            if name == "rpb":
                params[at:at + size].reshape(shape)[1::3, g1.Kz - 1, g1.Ky - 1, g1.Kx - 1] = -100.0
            at += size
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((B, g1.Z, g1.Y, g1.X, g1.C), generator=gen, device="cuda")
    x3 = x.repeat(1, 1, 1, REPEAT, 1)
    p1, p3 = (wm.wm_processor_create(ctx, g, 1, 4, {"bf16": wm.WM_BF16, "fp8": wm.WM_FP8_E4M3}[prec], params) for g in (g1, g3))
    wm.wm_processor_step(ctx, p3, B, x3)
    for b in range(B):
        alone = x[b:b + 1].clone()
        wm.wm_processor_step(ctx, p1, 1, alone)
        assert torch.isfinite(alone).all()
        assert torch.equal(x3[b:b + 1], alone.repeat(1, 1, 1, REPEAT, 1)), b
    for h in (p1, p3, ctx):
        h.close()
