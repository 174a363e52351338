"""Each spread kernel by the owner tiles that select it, named and asserted
here from K, J and spread_tile, since even splits of an axis make a tile
smaller than the requested edge: the matrix-core kernels (2D / 3D, edges of at
most 8 cells), the output-stationary one (2D, at most 512 cells), the scatter
kernel (all else).  Adjoints against the exact NUDFT (2e-5) and across kernels,
which add the same FP32 products per grid cell in another order (2e-6)."""
import math

import numpy as np
import pytest
import torch

from oracle import ndft
from paper_2111_02912_amd import workloads as W

pytestmark = pytest.mark.gpu


def _edges(K, J, spread_tile):
    """Largest owner tile edge per axis."""
    want = (max(J, spread_tile) if spread_tile else 128) if len(K) == 1 else max(8, spread_tile)
    out = []
    for k in K:
        n = -(-k // want)
        while n > 1 and k // n < J - 1:
            n -= 1
        out.append(-(-k // n))
    return out


def _kernel(K, J, spread_tile):
    e = _edges(K, J, spread_tile)
    if len(K) >= 2 and max(e) <= 8:
        return "matrix"
    return "stationary" if len(K) == 2 and math.prod(e) <= 512 else "scatter"


def _plan(N, om, kernel, J=6, spread_tile=0):
    from paper_2111_02912_amd.nufft import KbNufft
    dev = torch.device("cuda", 0)
    p = KbNufft(N, device=dev, J=J, spread_tile=spread_tile)
    assert _kernel(p.K, J, spread_tile) == kernel, (p.K, _edges(p.K, J, spread_tile))
    p.set_points(torch.from_numpy(om).to(dev))
    return p


def _samples(M, D):
    """Half of them in a cluster around the grid's wrap-around, whose tiles' lists are split."""
    return np.concatenate([W.uniform_random(M - M // 2, D, seed=61),
                           np.pi - 0.02 * np.abs(W.uniform_random(M // 2, D, seed=62))]).astype(np.float32)


def _adjoint(p, y):
    return p.adjoint(torch.from_numpy(y).to(p.device)).cpu().numpy()


# 2D references whose tiles do exceed 512 cells
@pytest.mark.parametrize("N,M,nch,J", [((60, 52), 3000, 1, 6), ((45, 90), 3000, 9, 6), ((90, 45), 900, 17, 5),
                                       ((45, 75), 5000, 65, 4), ((32, 40), 4000, 5, 3), ((48, 40), 2500, 33, 8)])
def test_kernels_of_2d_owner_tiles_agree(N, M, nch, J):
    print(f"2D spread kernels N={N} M={M} channels={nch} J={J}", flush=True)
    om = _samples(M, 2)
    y = W.complex_normal((nch, 1, M), 63)
    ref = _adjoint(_plan(N, om, "scatter", J, 32), y)
    if J >= 6:
        assert ndft.rel_l2(ref, ndft.adjoint(om, y[:, 0], N)) < 2e-5
    for kernel, st in (("matrix", 0), ("stationary", 12), ("stationary", 20)):
        got = _adjoint(_plan(N, om, kernel, J, st), y)
        assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref), (kernel, st)


# the window of eight taps on grids that split into tiles of 7 and 8 cells, for
# every channel group of the kernel (1, 2, 4, 8 channels and a remainder)
@pytest.mark.parametrize("N,M", [((8, 12, 16), 700), ((11, 8, 14), 3), ((15, 22, 8), 2600)])
@pytest.mark.parametrize("nch", [1, 2, 3, 8, 11])
def test_matrix_core_spread_of_eight_taps(N, M, nch):
    print(f"3D spread J=8 N={N} M={M} channels={nch}", flush=True)
    om = _samples(M, 3)
    y = W.complex_normal((nch, 1, M), 64)
    p = _plan(N, om, "matrix", 8)
    got = _adjoint(p, y)
    assert ndft.rel_l2(got, ndft.adjoint(om, y[:, 0], N)) < 2e-5
    q = _plan(N, om, "scatter", 8, 12)
    ref = np.concatenate([_adjoint(q, y[c:c + 1]) for c in range(nch)])
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)
    for c in {0, nch - 1}:
        assert np.array_equal(got[c:c + 1], _adjoint(p, y[c:c + 1]))


# many values: copied in tile order first, on many tiles (256, and 32768 with the
# channels) from 3 x 2^20 of them, on fewer (25) from 2^22, and from 4 samples a tile;
# groups of 64 channels and a remainder
@pytest.mark.parametrize("N,M,nch", [((128, 100), 32767, 96), ((128, 100), 32768, 96), ((128, 100), 24198, 130),
                                     ((128, 100), 3199, 984), ((128, 100), 3200, 984), ((40, 36), 20971, 200),
                                     ((40, 36), 20972, 200), ((16, 20), 65536, 64), ((20, 20), 65536, 64)])
@pytest.mark.parametrize("along", [False, True])
def test_matrix_core_spread_of_many_channels(N, M, nch, along):
    """Samples in no order are copied, those along a trajectory are not."""
    from paper_2111_02912_amd.cg import cg_sense
    print(f"2D spread N={N} of {nch} channels, M={M} along a trajectory: {along}", flush=True)
    om = _samples(M, 2)
    if along:
        t = np.linspace(0, 1, M, endpoint=False)
        om = np.stack([3.1 * t * np.cos(80 * t), 3.1 * t * np.sin(80 * t)], 1).astype(np.float32)
    om[7::11, 0] = np.nan
    y = W.complex_normal((nch, 1, M), 67)
    p = _plan(N, om, "matrix")
    got = _adjoint(p, y)
    ref = _adjoint(_plan(N, om, "scatter" if N[0] > 20 else "stationary", 6, 32 if N[0] > 20 else 16), y)
    assert np.isfinite(got).all() and np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)
    ok = np.isfinite(om).all(1)
    pix = np.sort(W.rng(68).choice(int(np.prod(N)), 300, replace=False))
    want = ndft.adjoint(om[ok], np.ascontiguousarray(y[:, 0, ok]), N, pix=pix)
    assert ndft.rel_l2(got.reshape(nch, -1)[:, pix], want) < 2e-5
    x = cg_sense(p, torch.from_numpy(y).to(p.device), None, lam=float(M), iters=2)[0]  # E p in tile order
    for c in {0, 31, nch - 1}:
        assert np.array_equal(got[c:c + 1], _adjoint(p, y[c:c + 1]))
        assert torch.equal(x[c:c + 1], cg_sense(p, torch.from_numpy(y[c:c + 1]).to(p.device), None, lam=float(M), iters=2)[0])


def test_cg_and_jacobian_through_the_2d_scatter_kernel():
    """Flagged samples stay out of a solve, whose E p is in tile order, and the
    adjoint operator with coil maps and its Jacobian match the NUDFT."""
    from paper_2111_02912_amd.cg import cg_sense
    N, M, C = (60, 52), 3000, 3
    print(f"2D scatter kernel N={N}", flush=True)
    om = _samples(M, 2)
    smaps = W.sense_maps(C, N).astype(np.complex64)
    y = W.complex_normal((1, C, M), 65)
    gi = W.complex_normal((1,) + N, 66)
    p = _plan(N, om, "scatter", 6, 32)
    ts = torch.from_numpy(smaps).to(p.device)
    ty = torch.from_numpy(y).to(p.device)
    assert ndft.rel_l2(p.adjoint(ty, ts).cpu().numpy(), ndft.sense_adjoint(om, y, N, smaps)) < 2e-5
    dom = p.jac_omega_adj(ty, torch.from_numpy(gi).to(p.device), ts).cpu().numpy()
    assert ndft.rel_l2(dom, ndft.jac_omega_adj(om, y, gi, N, smaps)) < 1e-4
    bad = om.copy()
    bad[::7, 1] = np.nan
    keep = np.arange(M) % 7 != 0
    a = cg_sense(_plan(N, bad, "scatter", 6, 32), ty, ts, lam=float(M), iters=3)[0]
    b = cg_sense(_plan(N, om[keep], "scatter", 6, 32), ty[..., torch.from_numpy(keep)].contiguous(), ts, lam=float(M),
                 iters=3)[0]
    assert torch.isfinite(torch.view_as_real(a)).all() and torch.equal(a, b)


# fused batches whose adjoint-type tasks share launches: unequal grids with the
# same largest tile edges, one and several channel groups (32 channels each),
# split tiles, a coil sum, and a matrix-core plan that is issued whole
@pytest.mark.parametrize("spread_tile,nstreams", [(12, 1), (12, 3), (16, 3)])
def test_fused_batch_of_output_stationary_spreads(spread_tile, nstreams):
    from paper_2111_02912_amd import batch as KB
    print(f"fused spreads tile={spread_tile} streams={nstreams}", flush=True)
    dev = torch.device("cuda", 0)
    # (K / 12 and K / 16 leave edges of 12 x 12 and 16 x 16 for the first three)
    spec = [((48, 72), 6000, 1, 40, spread_tile), ((96, 48), 2500, 1, 33, spread_tile), ((72, 96), 900, 4, 9, spread_tile),
            ((50, 41), 5000, 1, 3, spread_tile), ((48, 48), 3000, 1, 2, 0)]
    tasks, outs, refs = [], [], []
    groups = set()
    for i, (N, M, C, B, st) in enumerate(spec):
        om = _samples(M, 2)
        p = _plan(N, om, "stationary" if st else "matrix", 6, st)
        if st:
            groups.add(tuple(_edges(p.K, 6, st)))
        s = torch.from_numpy(W.sense_maps(C, N).astype(np.complex64)).to(dev) if C > 1 else None
        k = torch.from_numpy(W.complex_normal((B, C, M), 70 + i)).to(dev)
        x = torch.from_numpy(W.complex_normal((B,) + N, 80 + i)).to(dev)
        o = [torch.full((B,) + N, float("nan"), dtype=torch.complex64, device=dev) for _ in range(2)]
        o.append(torch.full((B, C, M), float("nan"), dtype=torch.complex64, device=dev))
        tasks += [KB.Task(p, KB.ADJOINT, B, C, k, o[0], s), KB.Task(p, KB.JAC_X_FWD, B, C, k, o[1], s),
                  KB.Task(p, KB.FORWARD, B, C, x, o[2], s)]
        outs.append(o)
        refs.append([p.adjoint(k, s), p.adjoint(k, s), p.forward(x, s)])
    assert len(groups) < 4  # some of the adjoints do share a launch
    b = KB.KbnBatch(tasks, nstreams=nstreams, fuse=True)
    for _ in range(3):
        for o in outs:
            for t in o:
                t.fill_(float("nan"))
        torch.cuda.synchronize()
        b.run()
        torch.cuda.synchronize()
        for i, (o, r) in enumerate(zip(outs, refs)):
            for got, want in zip(o, r):
                assert torch.equal(got, want), i
    b.close()
