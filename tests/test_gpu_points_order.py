"""Calls issued right behind kbn_set_points, whose index pass is still
running beside them: the gathers start after its sort, the spreads after its
owner lists.  Every result has the bits of the same call on a plan whose pass
is known to have ended."""
import numpy as np
import pytest
import torch

from oracle import points_ref
from paper_2111_02912_amd import workloads as W

pytestmark = pytest.mark.gpu


# above and below the number of points from which the pass has its own stream
@pytest.mark.parametrize("N,Ms", [((96, 80), (8192, 60000, 500, 9000)), ((24, 30, 20), (30000, 8192, 100, 40000))])
@pytest.mark.parametrize("other_stream", [False, True])
def test_calls_behind_set_points(N, Ms, other_stream):
    from paper_2111_02912_amd.nufft import KbNufft
    dev = torch.device("cuda", 0)
    plan = KbNufft(N, device=dev)
    x = torch.from_numpy(W.complex_normal((1,) + tuple(N), 61)).to(dev)
    side = torch.cuda.Stream(dev)
    got, want, sets = [], [], []
    for k, M in enumerate(Ms):
        om = torch.from_numpy(W.uniform_random(M, len(N), seed=62 + k)).to(dev)
        y = torch.from_numpy(W.complex_normal((1, 1, M), 70 + k)).to(dev)
        sets.append((om, y))
    torch.cuda.synchronize()
    for om, y in sets:
        print(f"set points N={N} M={om.shape[0]} other_stream={other_stream}", flush=True)
        plan.set_points(om)
        f = plan.forward(x)
        if other_stream:
            side.wait_stream(torch.cuda.current_stream(dev))
            with torch.cuda.stream(side):
                a = plan.adjoint(y)
            torch.cuda.current_stream(dev).wait_stream(side)
        else:
            a = plan.adjoint(y)
        got.append((f, a, *plan.forward_jac_omega(x, y)))
    torch.cuda.synchronize()
    for om, y in sets:
        q = KbNufft(N, device=dev).set_points(om)
        q.check_error()
        want.append((q.forward(x), q.adjoint(y), *q.forward_jac_omega(x, y)))
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        assert all(torch.equal(a, b) for a, b in zip(g, w))


# sizes on both sides of the rules for the samples per histogram chunk (the
# one-workgroup scan, the larger scan at 256 samples and more per chunk, the
# larger scan at its limit of counts), with samples whose location is not finite
@pytest.mark.parametrize("N,M", [((48, 48, 48), 28672), ((48, 48, 48), 28673), ((48, 48, 48), 65536),
                                 ((75, 90, 64), 150001), ((30, 30, 30), 150000), ((256, 250), 300001)])
def test_sorted_order_for_every_chunking(N, M):
    from paper_2111_02912_amd.nufft import KbNufft
    print(f"sorted order N={N} M={M}", flush=True)
    om = W.uniform_random(M, len(N), seed=81)
    om[5::1000, 0] = np.inf
    p = KbNufft(N, device=torch.device("cuda", 0))
    p.set_points(torch.from_numpy(om).to(p.device))
    got = {k: v.cpu().numpy() for k, v in p.get_points().items()}
    cell, frac, bad = points_ref.cells(om, p.K)
    tid, nt = points_ref.tiles(cell, p.K, p.tile, bad)
    perm, off = points_ref.tile_order(tid, nt)
    assert np.array_equal(got["order"], perm)
    assert np.array_equal(got["offsets"], off)
    assert np.array_equal(got["cell"], cell[perm].T)
    assert np.array_equal(got["frac"].view(np.uint32), frac[perm].T.copy().view(np.uint32))


def test_capture_of_an_adjoint_behind_an_eager_forward():
    """A stream whose forward call already waited for the points may capture
    an adjoint on them; the replays give the eager call's bits."""
    from paper_2111_02912_amd.nufft import KbNufft
    print("capture behind an eager forward", flush=True)
    dev = torch.device("cuda", 0)
    N, M = (24, 30, 20), 40000
    plan = KbNufft(N, device=dev)
    om = torch.from_numpy(W.uniform_random(M, 3, seed=91)).to(dev)
    x = torch.from_numpy(W.complex_normal((1,) + N, 92)).to(dev)
    y = torch.from_numpy(W.complex_normal((1, 1, M), 93)).to(dev)
    plan.set_points(om)
    plan.check_error()
    want = plan.adjoint(y).clone()  # (and the workspace at its size)
    s = torch.cuda.Stream(dev)
    s.wait_stream(torch.cuda.current_stream(dev))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        plan.set_points(om)
        plan.forward(x)
        g.capture_begin()
        out = plan.adjoint(y)
        g.capture_end()
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        out.zero_()
        plan.forward(x)
        torch.cuda.synchronize()


def test_capture_behind_a_captured_batch_of_forward_calls():
    """Capturing a batch ends with its plans' index passes done, also where its
    tasks wait for the sorted samples only (the spread's lists of samples in a
    few cells take far longer than a forward call): any stream may then capture
    calls on the plan without kbn_check_error."""
    from paper_2111_02912_amd import batch as KB
    from paper_2111_02912_amd.nufft import KbNufft
    print("capture behind a captured batch", flush=True)
    dev = torch.device("cuda", 0)
    N, M = (24, 30, 20), 1500000
    plan = KbNufft(N, device=dev)
    om = torch.from_numpy((0.3 * W.uniform_random(M, 3, seed=94)).astype(np.float32)).to(dev)
    x = torch.from_numpy(W.complex_normal((1,) + N, 95)).to(dev)
    y = torch.empty((1, 1, M), dtype=torch.complex64, device=dev)
    plan.set_points(om)
    want = plan.forward(x).clone()
    plan.check_error()
    torch.cuda.synchronize()
    plan.set_points(om)
    b = KB.KbnBatch([KB.Task(plan, KB.FORWARD, 1, 1, x, y)], nstreams=1)
    b.capture()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = plan.forward(x)
    for _ in range(3):
        out.zero_()
        y.zero_()
        g.replay()
        b.launch()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(y, want)
        plan.forward(x)
        torch.cuda.synchronize()
    b.close()
