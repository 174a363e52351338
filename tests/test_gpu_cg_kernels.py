"""The CG iteration's vector kernels against the same iteration in FP64.

Both sides apply the library's operator to their own search directions, so
they differ by the FP32 rounding of x, r, p and q (6e-8 relative per update)
and of the operator on directions that differ by that much.  lambda is of
the size of the largest eigenvalues of E^H E, which keeps the growth over
three iterations well below 100 roundings: 6e-6.
"""
import numpy as np
import pytest
import torch

from paper_2111_02912_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 6e-6


# one block and several per image, a length past one pass of the grid's 1024
# blocks, one coil (no coil sum), coils and images in one run and in several
# (bytes of workspace), an axis of odd length
@pytest.mark.parametrize("N,M,B,C,reg,ws", [
    ((12,), 40, 1, 1, "identity", 0), ((15, 17), 400, 1, 2, "identity", 0), ((15, 17), 400, 3, 5, "finite_diff", 0),
    ((40, 36), 2000, 2, 3, "identity", 1), ((40, 36), 2000, 2, 3, "finite_diff", 200000),
    ((512, 512), 6000, 1, 2, "finite_diff", 0), ((100, 60, 50), 6000, 1, 2, "identity", 0), ((9, 12, 10), 900, 2, 4, "identity", 0),
])
def test_cg_iterations_match_fp64_vectors(N, M, B, C, reg, ws):
    from paper_2111_02912_amd.cg import cg_sense
    from paper_2111_02912_amd.nufft import KbNufft
    print(f"cg kernels N={N} M={M} B={B} C={C} {reg} workspace={ws}", flush=True)
    dev = torch.device("cuda", 0)
    plan = KbNufft(N, device=dev, max_workspace=ws)
    plan.set_points(torch.from_numpy(W.uniform_random(M, len(N), seed=51)).to(dev))
    smaps = torch.from_numpy(W.sense_maps(C, N)).to(dev) if C > 1 else None
    y = torch.from_numpy(W.complex_normal((B, C, M), 52)).to(dev)
    lam = float(max(M, np.prod(N)))
    x, rel = cg_sense(plan, y, smaps, lam=lam, iters=3, reg=reg)

    def lap(v):
        if reg == "identity":
            return v
        out = torch.zeros_like(v)
        for d in range(1, v.dim()):
            g = torch.diff(v, dim=d)
            n = v.shape[d]
            out.narrow(d, 1, n - 1).add_(g)
            out.narrow(d, 0, n - 1).sub_(g)
        return out

    def dot(a, b):
        return (a.conj() * b).real.flatten(1).sum(1).view(B, *[1] * len(N))

    r = plan.adjoint(y, smaps).to(torch.complex128)
    p, xr, bb = r.clone(), torch.zeros_like(r), dot(r, r)
    rr = bb
    for _ in range(3):
        q = plan.adjoint(plan.forward(p.to(torch.complex64), smaps), smaps).to(torch.complex128) + lam * lap(p)
        a = rr / dot(p, q)
        xr, r = xr + a * p, r - a * q
        rn = dot(r, r)
        p, rr = r + rn / rr * p, rn
    err = (x - xr).flatten(1).norm(dim=1) / xr.flatten(1).norm(dim=1)
    res = (rr / bb).sqrt().flatten()
    print("  ", err.max().item(), flush=True)
    assert err.max().item() < TOL
    assert torch.allclose(rel.double().cpu().flatten(), res.cpu(), rtol=100 * TOL, atol=TOL)


# E p in tile order through every spread kernel (matrix cores, output
# stationary, scatter), with and without samples whose location is not finite
@pytest.mark.parametrize("N,tile", [((40, 36), None), ((40, 36), 16), ((40, 36), 24), ((12, 14, 10), None),
                                    ((12, 14, 10), 10), ((300,), None)])
def test_cg_keeps_flagged_samples_out(N, tile):
    from paper_2111_02912_amd.cg import cg_sense
    from paper_2111_02912_amd.nufft import KbNufft
    print(f"cg flagged N={N} spread_tile={tile}", flush=True)
    dev = torch.device("cuda", 0)
    M, C = 3000, 3
    om = W.uniform_random(M, len(N), seed=53)
    smaps = torch.from_numpy(W.sense_maps(C, N)).to(dev) if len(N) > 1 else None
    y = W.complex_normal((1, C if len(N) > 1 else 1, M), 54)
    bad = om.copy()
    bad[::7, len(N) - 1] = np.nan
    keep = np.arange(M) % 7 != 0
    kw = {} if tile is None else {"spread_tile": tile}
    out = []
    for o, v in ((bad, y), (om[keep], np.ascontiguousarray(y[..., keep]))):
        plan = KbNufft(N, device=dev, **kw)
        plan.set_points(torch.from_numpy(o).to(dev))
        out.append(cg_sense(plan, torch.from_numpy(v).to(dev), smaps, lam=float(M), iters=3)[0])
    assert torch.isfinite(torch.view_as_real(out[0])).all()
    assert torch.equal(out[0], out[1])
