"""Tile choice of the linear maps.  It is read from the host header by a small
program built here.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_22235_amd", "csrc")


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
