"""The spread's owner lists where they change kernels: grids with more owner tiles
than one workgroup lists (12288), tiles around the entry counts at which a
tile is written by a whole workgroup (16 in 2D, 64 in 3D) and at which it is
split into work items (128, doubled until 256 slots hold them), tiles
without entries.  Adjoints against the exact NUDFT at a sample of pixels, and
against plans with larger owner tiles, whose cells add the same FP32 products
in another order (2e-6)."""
import numpy as np
import pytest
import torch

from oracle import ndft
from paper_2111_02912_amd import workloads as W

pytestmark = pytest.mark.gpu


def _samples(D, kind):
    if kind == "none":
        return np.zeros((0, D), np.float32)
    if kind == "one":
        return W.uniform_random(1, D, seed=21).astype(np.float32)
    om = [W.uniform_random(400, D, seed=22)]
    if kind == "counts":  # that many samples in one cell each
        at = W.uniform_random(16, D, seed=23)
        for k, n in enumerate((1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 256, 257)):
            om.append(np.repeat(at[k:k + 1], n, 0))
    if kind == "split":  # a few thousand in every cell near the corner of the grid, 60000 of them
        om.append(np.pi - 0.01 * np.abs(W.uniform_random(60000, D, seed=24)))
    return np.concatenate(om).astype(np.float32)


@pytest.mark.parametrize("N,big", [((512, 510), 12), ((96, 98, 97), 12), ((64, 60), 12), ((24, 20, 30), 12)])
@pytest.mark.parametrize("kind", ["none", "one", "counts", "split"])
def test_adjoint_of_owner_lists(N, big, kind):
    from paper_2111_02912_amd.nufft import KbNufft
    dev = torch.device("cuda", 0)
    D = len(N)
    om = _samples(D, kind)
    M = om.shape[0]
    print(f"owner lists N={N} {kind} M={M}", flush=True)
    y = W.complex_normal((1, 1, M), 25)
    out = []
    for kw in ({}, dict(spread_tile=big)):
        p = KbNufft(N, device=dev, **kw)
        for _ in range(2):  # the second pass finds the first one's counts and lists
            p.set_points(torch.from_numpy(om).to(dev))
        out.append(p.adjoint(torch.from_numpy(y).to(dev)).cpu().numpy())
        p.close()
    got, ref = out
    if M == 0:
        assert not got.any()
        return
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)
    pix = np.sort(W.rng(26).choice(int(np.prod(N)), 400, replace=False))
    assert ndft.rel_l2(got.reshape(1, -1)[:, pix], ndft.adjoint(om, y[:, 0], N, pix=pix)) < 2e-5
