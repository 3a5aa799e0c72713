"""Graph-captured matvecs and the z-pass autotuner.  A captured matvec is
replayed several times with new input written in place and eager work and
synchronisations in between; every replay must equal the eager matvec
bit for bit (same kernels, same order).  The autotuner must keep the
results unchanged (the launch shape only moves work between workgroups) and
report a time for every candidate."""
import numpy as np
import pytest
import torch

import vie_inputs as vi
from gpu_common import library_operator, problem, rel, say, to_dev
from oracle import operator as opm
from paper_1811_00484_amd import vie

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dt", [((64, 20, 64), torch.complex64), ((12, 10, 9), torch.complex128)])
def test_graph_replays_equal_eager(n, dt):
    say("graph", n, dt)
    G, epsc, ref = problem(n, h=0.003)
    op = library_operator(n, h=0.003)
    e = to_dev(epsc, dt)
    x = torch.zeros((2, 3) + tuple(reversed(n)), dtype=dt, device=e.device)
    g = vie.MatvecGraph(op, x, e)
    try:
        for rep in range(4):
            u = vi.random_field(n, 40 + rep, nrhs=2)
            x.copy_(to_dev(u, dt))
            y_eager = vie.matvec(op, x, e)
            torch.cuda.synchronize()
            y = g.launch().clone()
            torch.cuda.synchronize()
            assert torch.equal(y, y_eager), rep
            err = rel(y.cpu().numpy()[1].astype(np.complex128), opm.matvec(ref, epsc, u[1], "A"))
            assert err <= (1e-5 if dt == torch.complex64 else 1e-11)
            _ = torch.linalg.vector_norm(y_eager)   # eager work between replays
    finally:
        g.close()


def test_graph_rejected_while_profiling():
    n = (12, 10, 9)
    G, epsc, ref = problem(n)
    op = library_operator(n)
    e = to_dev(epsc, torch.complex64)
    x = to_dev(vi.random_field(n, 3), torch.complex64)
    vie.profile_enable(True)
    try:
        with pytest.raises(RuntimeError):
            vie.MatvecGraph(op, x, e)
    finally:
        vie.profile_enable(False)
        vie.profile_collect()


@pytest.mark.parametrize("dt", [torch.complex64, torch.complex128])
def test_autotune_keeps_results(dt):
    n = (64, 48, 128)
    G, epsc, ref = problem(n, h=0.003)
    op = vie.compress(G, tol=1e-6)
    u = vi.random_field(n, 9)
    x = to_dev(u, dt)
    e = to_dev(epsc, dt)
    y0 = vie.matvec(op, x, e).cpu().numpy()
    chosen, ms = vie.autotune(op, dt, nrhs=1)
    say("   autotune", dt, chosen, ms)
    assert chosen in (4, 8, 16, 32)
    assert all(v > 0 for v in ms.values())
    assert ms[chosen] == min(ms.values())
    y1 = vie.matvec(op, x, e).cpu().numpy()
    # each quad is computed by the same code whatever the grouping: identical
    assert np.array_equal(y0, y1)


@pytest.mark.parametrize("dt", [torch.complex64, torch.complex128])
def test_autotune_candidates_reach_different_launches(dt):
    # 81 k1 quads of two k2: 3 workgroups a k2 of 32 quads or 21 of 4, one
    # after another in a workgroup, on 256 CUs: eight times the work per
    # workgroup, of which the z pass's other launch leaves more than half
    op = vie.compress(problem((80, 1, 64), h=0.003)[0], tol=1e-6)
    times = [vie.autotune(op, dt, nrhs=1)[1] for _ in range(3)]
    say("   autotune", dt, times)
    assert min(t[32] for t in times) >= 1.5 * min(t[4] for t in times)
