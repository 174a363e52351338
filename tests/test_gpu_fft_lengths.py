"""Every grid length's compile-time FFT passes against the runtime-length ones.

For every 7-smooth length from 4 to 1024, on both axes: forward (zero-padded
rows and columns, odd and even image extents, the twice-padded column load),
adjoint with two coils (cropped passes, coil sum) and the one-call forward plus
omega-Jacobian layout.  The two sets of passes compute the same transforms
with other radices in FP32: relative L2 2e-6, the bound that FP32 storage, FFT
and accumulation are held to.
"""
import numpy as np
import pytest
import torch

from paper_2111_02912_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL_STEPS = 2e-6


def _smooth(k):
    for p in (2, 3, 5, 7):
        while k % p == 0:
            k //= p
    return k == 1


LENGTHS = [k for k in range(4, 1025) if _smooth(k)]


def _results(n, sigma, J, om, x, smaps, g):
    from paper_2111_02912_amd.nufft import KbNufft
    p = KbNufft((n, n), sigma=sigma, J=J, device=om.device)
    p.set_points(om)
    y, dom = p.forward_jac_omega(x, g, smaps)
    out = [p.forward(x, smaps), p.adjoint(g, smaps), p.jac_omega_fwd(x, g, smaps), y, dom]
    torch.cuda.synchronize()
    return p.K, [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("group", range(8))
def test_compile_time_passes_of_every_length(group, monkeypatch):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dev = torch.device("cuda", 0)
    for K in LENGTHS[group::8]:
        # N = K / 2 (even lengths), and an extent that is not half the length
        for n in {K // 2, max(2, (5 * K) // 9)}:
            sigma = K / n
            J = 6 if K >= 12 else 2
            print(f"FFT length K={K} N={n}", flush=True)
            om = torch.from_numpy(W.uniform_random(60, 2, seed=K)).to(dev)
            x = torch.from_numpy(W.complex_normal((1, n, n), K + 1)).to(dev)
            smaps = torch.from_numpy(W.complex_normal((2, n, n), K + 2)).to(dev)
            g = torch.from_numpy(W.complex_normal((1, 2, 60), K + 3)).to(dev)
            outs = []
            for generic in ("0", "1"):
                monkeypatch.setenv("KBN_GENERIC_FFT", generic)
                grid, o = _results(n, sigma, J, om, x, smaps, g)
                assert grid == (K, K)
                outs.append(o)
            for a, b in zip(*outs):
                assert np.linalg.norm(a - b) <= TOL_STEPS * np.linalg.norm(b), (K, n)
