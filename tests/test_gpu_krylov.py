"""One GMRES cycle of the device solver against the same cycle in torch
(complex128, the library's own product): vectors short enough to take one,
two and four elements per thread of the Gram-Schmidt kernels and long enough
for eight, a ragged last workgroup, several right-hand sides, and a cycle
longer than one batch of 64 dots.

Tolerance: the minimiser over at most m directions, orthogonal to ~1e-13,
through a least-squares problem of condition below 1e3: 1e-10; complex64
(FP32 basis, unit roundoff 6e-8): 1e-3."""
import numpy as np
import pytest
import torch

import vie_inputs as vi
from gpu_common import F, device, say
from paper_1811_00484_amd import vie

pytestmark = pytest.mark.gpu


def _cycle(A, b, m):
    V = [b / torch.linalg.vector_norm(b)]
    H = np.zeros((m + 1, m), complex)
    for j in range(m):
        w = A(V[j])
        for _ in range(2):
            for i, v in enumerate(V):
                c = torch.vdot(v.reshape(-1), w.reshape(-1))
                H[i, j] += c.item()
                w = w - c * v
        H[j + 1, j] = torch.linalg.vector_norm(w).item()
        V.append(w / H[j + 1, j])
    e = np.zeros(m + 1)
    e[0] = torch.linalg.vector_norm(b).item()
    y = np.linalg.lstsq(H, e, rcond=None)[0]
    return sum(complex(y[i]) * V[i] for i in range(m))


@pytest.mark.parametrize("n,nrhs,m", [((9, 7, 5), 2, 8), ((60, 50, 49), 1, 6), ((75, 72, 70), 2, 5),
                                      ((98, 96, 90), 1, 4), ((8, 9, 10), 1, 70)])
@pytest.mark.parametrize("dt,bound", [(torch.complex128, 1e-10), (torch.complex64, 1e-3)])
def test_cycle_equals_torch(n, nrhs, m, dt, bound):
    from test_gpu_mix import _problem
    op, _ = _problem(n)
    er, sg, _ = vi.head_phantom(n, 0.004, seed=2)
    eps = torch.from_numpy(vi.complex_permittivity(er, sg, F)).to(device())
    rng = np.random.default_rng(4)
    shape = (nrhs, 3, n[2], n[1], n[0])
    b = torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).to(device())
    with pytest.warns(UserWarning) if m < 70 else _quiet():
        x, info, _ = vie.solve(op, b.to(dt), eps.to(dt), tol=1e-13, restart=m, max_outer=1)
    for s in range(nrhs):
        if m == 70:   # residuals of the two minimisers (far into convergence the minimiser itself is ill-defined)
            r = b[s] - vie.matvec(op, _cycle(lambda v: vie.matvec(op, v.contiguous(), eps), b[s], m), eps)
            rd = b[s] - vie.matvec(op, x[s].to(torch.complex128), eps)
            want, got = torch.linalg.vector_norm(r).item(), torch.linalg.vector_norm(rd).item()
            floor = 1e-5 if dt == torch.complex64 else 1e-11
            say("   cycle", n, dt, want, got)
            assert got <= 1.01 * want + floor * torch.linalg.vector_norm(b[s]).item()
            continue
        ref = _cycle(lambda v: vie.matvec(op, v.contiguous(), eps), b[s], m)
        err = (torch.linalg.vector_norm(x[s].to(torch.complex128) - ref) / torch.linalg.vector_norm(ref)).item()
        say("   cycle", n, nrhs, m, dt, "%.2e" % err)
        assert err <= bound


class _quiet:
    def __enter__(self):
        import warnings
        self._c = warnings.catch_warnings()
        self._c.__enter__()
        warnings.simplefilter("ignore")

    def __exit__(self, *a):
        return self._c.__exit__(*a)


# 3 n1 n2 n3 = 635040: two elements per thread of the Gram-Schmidt kernels (the
# grids above take one, four and eight), as a 64^3 solve does
@pytest.mark.parametrize("nrhs", [1, 2])
@pytest.mark.parametrize("dt,bound", [(torch.complex128, 1e-10), (torch.complex64, 1e-3)])
def test_cycle_with_two_elements_per_thread(nrhs, dt, bound):
    test_cycle_equals_torch((63, 60, 56), nrhs, 6, dt, bound)
