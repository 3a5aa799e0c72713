"""vie_tucker_hadamard where its kernels change: rows of i around the length
below which the (i, j) plane is walked flat, planes of 2^31 and more (j, k)
rows, few k under many j, and V of one to four columns.

Tolerance against numpy in 64 bits: three nested sums of at most 32 products,
relative to the sums of absolute values below 100 unit roundoffs."""
import numpy as np
import pytest
import torch

from gpu_common import device, say, to_dev
from paper_1811_00484_amd import vie

pytestmark = pytest.mark.gpu

U = {torch.complex64: 2.0 ** -24, torch.complex128: 2.0 ** -53}


def _cx(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _dense(core, F, cp):
    if cp:
        return np.einsum("l,il,jl,kl->kji", core, *F, optimize=True)
    return np.einsum("abc,ia,jb,kc->kji", core, *F, optimize=True)


def _check(n, r, cp, dt, inplace=False):
    rng = np.random.default_rng(sum(n) + sum(r))
    F = [_cx(rng, n[a], r[a]).astype(np.complex64) for a in range(3)]
    core = _cx(rng, *(r[:1] if cp else r)).astype(np.complex64)
    x = _cx(rng, n[2], n[1], n[0]).astype(np.complex64)
    xd = to_dev(x, dt)
    y = vie.tucker_hadamard(to_dev(core, dt), [to_dev(f, dt) for f in F], xd, cp=cp, out=xd if inplace else None)
    y = (xd if inplace else y).cpu().numpy().astype(np.complex128)
    core, F, x = core.astype(complex), [f.astype(complex) for f in F], x.astype(complex)
    want = _dense(core, F, cp) * x
    size = _dense(np.abs(core), [np.abs(f) for f in F], cp) * np.abs(x)
    err = float((np.abs(y - want) / size).max())
    say("   hadamard", n, r, cp, dt, "%.2e" % err)
    assert err <= 100 * U[dt]


@pytest.mark.parametrize("n1", [1, 2, 3, 5, 8, 12, 13, 15, 16, 17, 31, 64, 65])
@pytest.mark.parametrize("dt", list(U))
@pytest.mark.parametrize("cp", [False, True])
def test_rows_of_few_elements(n1, dt, cp):
    for n2, n3, r in ((37, 19, 7), (300, 5, 1), (20, 33, 32)):
        _check((n1, n2, n3), (r, r, r), cp, dt, inplace=r == 7)


@pytest.mark.parametrize("r", [1, 2])
def test_planes_of_more_than_2_31_rows(r):
    # one i: 17 GB of x, worked on in place, and V of as much per rank
    m = 46342
    assert m * m > 2 ** 31
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    F = [torch.view_as_complex(torch.randn(k, r, 2, generator=g, device="cuda")) for k in (1, m, m)]
    lam = torch.view_as_complex(torch.randn(r, 2, generator=g, device="cuda"))
    x = torch.view_as_complex(torch.randn(m, m, 1, 2, generator=g, device="cuda"))
    keep = {k: x[k].clone() for k in (0, 1, m // 2, m - 2, m - 1)}
    vie.tucker_hadamard(lam, F, x, cp=True, out=x)
    for k, row in keep.items():
        terms = (lam * F[0][0] * F[2][k]).to(torch.complex128) * F[1]
        want, size = terms.sum(1, keepdim=True) * row, terms.abs().sum(1, keepdim=True) * row.abs()
        assert float(((x[k] - want).abs() / size).max()) <= 20 * U[torch.complex64]


# rows of U2 split over workgroups (few k), with a remainder of a tile; V of
# one to three columns, whose workgroups take eight k, and of four
@pytest.mark.parametrize("n,r", [((70, 1000, 1), (9, 25, 1)), ((40, 577, 3), (25, 8, 3)), ((33, 65, 511), (6, 5, 7)),
                                 ((20, 64, 2), (4, 32, 2)), ((30, 300, 17), (1, 32, 16)), ((30, 256, 8), (2, 31, 5)),
                                 ((30, 257, 9), (3, 4, 9)), ((9, 1, 1), (3, 1, 1)), ((18, 5, 600), (32, 5, 32))])
@pytest.mark.parametrize("dt", list(U))
def test_v_of_few_k_and_few_columns(n, r, dt):
    _check(n, r, False, dt)


@pytest.mark.parametrize("n3,dt", [(1, torch.complex64), (2, torch.complex128)])
def test_few_k_leave_no_cu_idle(n3, dt):
    # 20000 rows of U2 to a k: in one workgroup each they take over a
    # millisecond; spread over the chip, the product is bound by its launches
    rng = np.random.default_rng(0)
    n, r = (64, 20000, n3), (25, 25, n3)
    F = [to_dev(_cx(rng, n[a], r[a]), dt) for a in range(3)]
    core, x = to_dev(_cx(rng, *r), dt), to_dev(_cx(rng, *reversed(n)), dt)
    best = 1e9
    for _ in range(5):
        s, e = torch.cuda.Event(True), torch.cuda.Event(True)
        s.record()
        vie.tucker_hadamard(core, F, x)
        e.record()
        e.synchronize()
        best = min(best, s.elapsed_time(e))
    say("   hadamard few k", n3, dt, best)
    assert best <= 0.5
