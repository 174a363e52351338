"""The spread's owner lists where they change kernels: grids with more owner tiles
than one workgroup lists (12288), tiles around the entry counts at which a
tile is written by a whole workgroup (16 in 2D, 64 in 3D) and at which it is
split into work items (128, doubled until 256 slots hold them), tiles
without entries.  Adjoints against the exact NUDFT at a sample of pixels, and
against plans with larger owner tiles, whose cells add the same FP32 products
in another order (2e-6)."""
import os
import subprocess
import sys

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


# More owner tiles than a grid has rows: default 3D plans from K = 321 on (the
# matrix-core spread strides over its work items), and tiles of 9 cells, which
# become larger instead.  Samples at the ends of every axis reach the last items.
@pytest.mark.parametrize("nch", [1, 2, 3, 5])
def test_adjoint_of_more_tiles_than_grid_rows(nch):
    from paper_2111_02912_amd.nufft import KbNufft
    dev = torch.device("cuda", 0)
    N, M = (163, 162, 164), 3000
    print(f"more tiles than rows N={N} channels={nch}", flush=True)
    om = W.uniform_random(M, 3, seed=31)
    om[::7] = np.pi * np.sign(om[::7]) * (1 - 1e-3)
    y = W.complex_normal((nch, 1, M), 32)
    pix = np.sort(W.rng(33).choice(int(np.prod(N)), 300, replace=False))
    want = ndft.adjoint(om, y[:, 0], N, pix=pix)
    for kw in ({}, dict(spread_tile=9)):
        p = KbNufft(N, device=dev, **kw)
        p.set_points(torch.from_numpy(om).to(dev))
        got = p.adjoint(torch.from_numpy(y).to(dev)).cpu().numpy()
        p.close()
        assert ndft.rel_l2(got.reshape(nch, -1)[:, pix], want) < 2e-5


def test_scatter_spread_strides_over_work_items(tmp_path):
    """The scatter kernel (KBN_SPREAD_OS=0, read once per process) with more work
    items than a grid has rows."""
    print("scatter spread with more items than rows", flush=True)
    N, M = (163, 162, 164), 2000
    om = W.uniform_random(M, 3, seed=41)
    om[::5] = np.pi * np.sign(om[::5]) * (1 - 1e-3)
    y = W.complex_normal((2, 1, M), 42)
    np.savez(tmp_path / "in.npz", om=om, y=y)
    code = f"""
import numpy as np, torch
from paper_2111_02912_amd.nufft import KbNufft
d = np.load(r"{tmp_path / 'in.npz'}")
p = KbNufft({N}, device=torch.device("cuda", 0))
p.set_points(torch.from_numpy(d["om"]).cuda())
np.save(r"{tmp_path / 'out.npy'}", p.adjoint(torch.from_numpy(d["y"]).cuda()).cpu().numpy())
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    subprocess.run([sys.executable, "-c", code], check=True, timeout=100, cwd=root,
                   env=dict(os.environ, KBN_SPREAD_OS="0"))
    got = np.load(tmp_path / "out.npy")
    pix = np.sort(W.rng(43).choice(int(np.prod(N)), 300, replace=False))
    assert ndft.rel_l2(got.reshape(2, -1)[:, pix], ndft.adjoint(om, y[:, 0], N, pix=pix)) < 2e-5
