"""The piecewise-linear z pass at every launch shape it chooses between: mirror
groups of four, two and one pencils, all ten pairs' tables in LDS or batches
of them, one and two neighbouring groups per workgroup, and right-hand sides
that share a workgroup's tables.  Against the FP64 oracle on the same HOSVD
tensors, tolerances as in the parity tests of the same products (complex64
1e-5, complex128 1e-11)."""
import functools

import numpy as np
import pytest
import torch

from gpu_common import rel, say, to_dev
from oracle import pwl_k
from paper_1811_00484_amd import vie
from test_gpu_pwl import _device, _field, _reference, pwl_problem
from test_gpu_pwl_k import _device as _device_k, k_problem

pytestmark = pytest.mark.gpu

# z lengths whose pencils and tables fit as (group, pairs): complex64 (4, 5),
# (2, 10), (2, 5), (2, 2); complex128 (4, 5), (2, 10), (2, 5), (2, 2), (1, 5),
# (1, 2), (1, 1)
C64 = [(2, 3, 128), (3, 2, 150), (2, 2, 180), (1, 3, 250)]
C128 = [(3, 2, 64), (2, 3, 70), (2, 2, 100), (1, 2, 128), (2, 1, 150), (1, 2, 240), (2, 1, 250)]


@pytest.mark.parametrize("n", C64)
@pytest.mark.parametrize("mode", ["A", "AH"])
def test_c64_shapes(n, mode):
    G, epsc, kh, _ = pwl_problem(n)
    op = vie.compress_pwl(G, tol=1e-6)
    u = _field(n, 31)
    err = rel(_device(op, epsc, u, mode, torch.complex64), _reference(kh, epsc, u, mode))
    say("   pwl shape", n, mode, "%.2e" % err)
    assert err <= 1e-5


@pytest.mark.parametrize("n", C128)
@pytest.mark.parametrize("mode", ["A", "AH"])
def test_c128_shapes(n, mode):
    G, epsc, kh, _ = pwl_problem(n, tol=1e-8)
    op = vie.compress_pwl(G, tol=1e-8)
    u = _field(n, 32)
    err = rel(_device(op, epsc, u, mode, torch.complex128), _reference(kh, epsc, u, mode))
    say("   pwl shape", n, mode, "%.2e" % err)
    assert err <= 1e-11


@functools.lru_cache(maxsize=2)
def _wide(tol):
    # 41 x 25 groups: two a workgroup with one left over
    n = (40, 24, 7)
    G, epsc, kh, _ = pwl_problem(n, tol=tol)
    return n, vie.compress_pwl(G, tol=tol), epsc, kh


@pytest.mark.parametrize("dt,tol,bound", [(torch.complex64, 1e-6, 1e-5), (torch.complex128, 1e-8, 1e-11)])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_two_groups_and_shared_tables(dt, tol, bound, nrhs):
    n, op, epsc, kh = _wide(tol)
    for mode in ("A", "AH"):
        u = np.stack([_field(n, 33 + s) for s in range(nrhs)])
        x = to_dev(u.reshape(nrhs, 12, n[2], n[1], n[0]), dt)
        y = vie.matvec_pwl(op, x, to_dev(epsc, dt), adjoint=mode == "AH")
        y = y.cpu().numpy().astype(np.complex128).reshape(u.shape)
        for s in range(nrhs):
            err = rel(y[s], _reference(kh, epsc, u[s], mode))
            say("   pwl two groups", dt, mode, nrhs, s, "%.2e" % err)
            assert err <= bound


@pytest.mark.parametrize("n", [(40, 24, 7), (2, 2, 180), (2, 3, 128)])
def test_k_shapes(n):
    kt, kh, _ = k_problem(n)
    op = vie.compress_pwl_k(kt, tol=1e-6)
    u = _field(n, 35)
    err = rel(_device_k(op, u, torch.complex64), pwl_k.to_normalised_k(kh, u))
    say("   pwl k shape", n, "%.2e" % err)
    assert err <= 1e-5
