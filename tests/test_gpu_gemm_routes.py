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


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("extra", [0, 64])
def test_weights_of_2_gib(env, extra, bf16):
    """Weights past 32-bit offsets, with 128- and 64-wide tiles: sampled features of
    every row against float64 (relative L2: bf16 outputs 5e-3, whose rounding is
    1.1e-3 rms; float32 2 (sqrt(K / 4) + 1) 2^-24, a rounding per four products)."""
    wm, torch = env
    K, M = 1024, 131
    N = (1 << (20 if bf16 else 19)) + extra
    print("2 GiB of weights", N, "bf16" if bf16 else "f32", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N)
    dt = torch.bfloat16 if bf16 else torch.float32
    w = torch.randn((N, K), generator=gen, device="cuda", dtype=dt)
    a = torch.randn((M, K), generator=gen, device="cuda", dtype=dt)
    b = torch.randn(N, generator=gen, device="cuda")
    out = torch.empty((M, N), dtype=dt, device="cuda")
    wm.wm_linear(M, N, K, wm.WM_BF16 if bf16 else wm.WM_F32, a, w, b, 0, out)
    cols = torch.cat([torch.arange(70), torch.randint(0, N, (300,)), torch.arange(N - 70, N)]).cuda()
    ref = (a.double() @ w[cols].double().T + b[cols].double()).cpu().numpy()
    err = O.rel_l2(out[:, cols].double().cpu().numpy(), ref)
    print("  rel_l2", err, flush=True)
    assert err < (5e-3 if bf16 else 2 * (np.sqrt(K / 4) + 1) * 2.0 ** -24)


def test_weights_of_2_gib_keep_the_wide_tile(env):
    """N a multiple of 128 runs on 128-wide tiles, in half the time of 64-wide ones."""
    wm, torch = env
    K, M, times = 1024, 700, []
    for N in (1 << 20, (1 << 20) + 64):
        print("2 GiB of weights, time", N, flush=True)
        w = torch.randn((N, K), device="cuda", dtype=torch.bfloat16)
        a = torch.randn((M, K), device="cuda", dtype=torch.bfloat16)
        b, out = torch.zeros(N, device="cuda"), torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        best = float("inf")
        for _ in range(4):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            wm.wm_linear(M, N, K, wm.WM_BF16, a, w, b, 0, out)
            t[1].record()
            torch.cuda.synchronize()
            best = min(best, t[0].elapsed_time(t[1]))
        times.append(best)
    print("  ms", times, flush=True)
    assert times[0] < 0.75 * times[1]


@pytest.mark.parametrize("bf16,N", [(False, 192), (False, 128), (True, 192)])
@pytest.mark.parametrize("which", ["a", "w", "bias and out"])
def test_operands_at_odd_elements(env, which, bf16, N):
    """Tensors that start one element into a buffer: the direct loads to LDS are
    for 16-byte aligned operands (other kernel, other order of the sums: relative
    L2 as in test_weights_of_2_gib)."""
    wm, torch = env
    M, K = 77, 128
    print("odd elements", which, N, "bf16" if bf16 else "f32", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N)
    dt = torch.bfloat16 if bf16 else torch.float32

    def place(t, odd):
        if not odd:
            return t.contiguous()
        buf = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
        v = buf[1:1 + t.numel()].view(t.shape)
        v.copy_(t)
        return v

    a = place(torch.randn((M, K), generator=gen, device="cuda").to(dt), which == "a")
    w = place(torch.randn((N, K), generator=gen, device="cuda").to(dt), which == "w")
    odd = which == "bias and out" and not bf16
    b = place(torch.randn(N, generator=gen, device="cuda"), odd)
    out = place(torch.zeros((M, N), dtype=dt, device="cuda"), odd)
    wm.wm_linear(M, N, K, wm.WM_BF16 if bf16 else wm.WM_F32, a, w, b, 0, out)
    ref = (a.double() @ w.double().T + b.double()).cpu().numpy()
    assert O.rel_l2(out.double().cpu().numpy(), ref) < (5e-3 if bf16 else 2 * (np.sqrt(K / 4) + 1) * 2.0 ** -24)
