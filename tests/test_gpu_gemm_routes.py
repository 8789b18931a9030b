"""Linear maps on the less usual routes of the dispatch."""
import numpy as np
import pytest

from oracle import wm_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2503_22235_amd as wm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    wm.lib()
    yield wm, torch


@pytest.mark.parametrize("M,N,K", [(3, 64, 64), (70, 192, 128), (2000, 1088, 64)])
def test_gelu_of_64_wide_maps(env, M, N, K):
    """N = 64 (mod 128), bf16: GELU with erf good to 3e-7.  The pre-activation is
    the bias alone (a = 0), so the output is the GELU of a known float32, rounded
    once to bf16.  Rounding is monotonic: the output lies between the rounded ends
    of GELU +- d, d being erf's error times |z| / 2 and 24 float32 roundings (the
    16th power's among them) of the part |z| / 2 (1 - erf)."""
    wm, torch = env
    print("gelu", M, N, K, flush=True)
    a = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda")
    w = torch.randn((N, K), device="cuda").bfloat16()
    z = np.linspace(-4.5, 3.0, N).astype(np.float32)
    out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    wm.wm_linear(M, N, K, wm.WM_BF16, a, w, torch.from_numpy(z).cuda(), 1, out)
    z = z.astype(np.float64)
    ref = O.gelu(z)
    d = 1.5e-7 * np.abs(z) + 24 * 2.0 ** -23 * np.minimum(np.abs(ref), np.abs(z) / 2)
    ends = [torch.from_numpy(ref + s * d).bfloat16().double().numpy() for s in (-1, 1)]
    got = out.double().cpu().numpy()
    assert ((ends[0] <= got) & (got <= ends[1])).all()
