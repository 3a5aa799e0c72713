"""The piecewise-linear products in less workspace than all rows V_c(k1, k2, :)
take: slabs of k2, and of k1 within one k2, on thin grids (z ranks near n3),
at every mirror group that the z pass chooses between.

Workspace: the padded components after Y+ (48 n1 n2 n3 complex per vector) and
the larger of 24 n1 n2 n3 per vector and the rows, padded to whole fours;
accepted down to the former (and one row of every component).  Tolerances
against the FP64 oracle as in the parity tests of the same products
(complex64 1e-5, complex128 1e-11); the buffers start as NaN and end in a
guard."""
import ctypes
import functools

import numpy as np
import pytest
import torch

import vie_inputs as vi
from gpu_common import F, K0, device, rel, say, to_dev
from oracle import pwl, pwl_k
from paper_1811_00484_amd import vie
from test_gpu_pwl import _field

pytestmark = pytest.mark.gpu

BOUND = {torch.complex64: 1e-5, torch.complex128: 1e-11}
GUARD = 4096
H = 0.005


def _al(b):
    return (b + 255) // 256 * 256


@functools.lru_cache(maxsize=4)
def _problem(n, full_rank):
    G, kt = vi.green_pwl_tensor(n, H, K0), vi.green_pwl_k_tensor(n, H, K0)
    tol = 1e-8
    if full_rank:   # the zero planes of the parities stay; no rank is lost
        rng = np.random.default_rng(sum(n))
        G = G * rng.uniform(0.5, 1.5, G.shape)
        kt = kt * rng.uniform(0.5, 1.5, kt.shape)
        tol = 1e-13
    rng = np.random.default_rng(3)
    eps = 1 + rng.uniform(0, 50, (n[2], n[1], n[0])) - 1j * rng.uniform(0, 30, (n[2], n[1], n[0]))
    return (vie.compress_pwl(G, tol=tol), vie.compress_pwl_k(kt, tol=tol), pwl.tucker_kernels(G, tol)[0],
            pwl_k.tucker_kernels_k(kt, tol)[0], eps)


def _run(op, x, e, adjoint, nbytes, kind):
    lib = vie.load()
    buf = torch.full((nbytes + GUARD,), 255, dtype=torch.uint8, device=device())
    y = torch.empty_like(x)
    st = lib.vie_matvec_pwl(op.handle, vie.VIE_OP_A if kind == "A" else vie.VIE_OP_N, int(adjoint), vie._dt(x),
                            e.data_ptr() if kind == "A" else None, x.data_ptr(), y.data_ptr(), x.shape[0],
                            buf.data_ptr(), nbytes, vie._stream())
    torch.cuda.synchronize()
    assert bool((buf[nbytes:] == 255).all())
    return st, y


# (grid, full ranks): slabs of several k2; one k2 or part of its k1 at a time;
# no slab; and, at full ranks, groups of two pencils (complex64) and of two and
# of one (complex128)
GRIDS = [((30, 24, 1), False), ((25, 18, 3), False), ((40, 12, 8), False), ((20, 1, 1), False), ((14, 2, 2), False),
         ((3, 2, 1), False), ((12, 10, 9), False), ((8, 8, 90), True), ((8, 8, 150), True)]


@pytest.mark.parametrize("n,full_rank", GRIDS)
@pytest.mark.parametrize("dt", list(BOUND))
@pytest.mark.parametrize("nrhs", [1, 2])
def test_products_in_slabs(n, full_rank, dt, nrhs):
    opn, opk, khn, khk, eps = _problem(n, full_rank)
    lib = vie.load()
    u = np.stack([_field(n, 41 + s) for s in range(nrhs)])
    x, e = to_dev(u.reshape(nrhs, 12, n[2], n[1], n[0]), dt), to_dev(eps, dt)
    el = x.element_size()
    s1 = 24 * n[0] * n[1] * n[2] * nrhs
    for op, mode, ref, nc in ((opn, "A", khn, 6), (opn, "AH", khn, 6), (opk, "N", khk, 3)):
        want = np.stack([pwl_k.to_normalised_k(ref, v) if nc == 3 else
                         pwl.to_normalised(lambda w: pwl.matvec(ref, eps, w, mode), v) for v in u])
        asked = lib.vie_pwl_workspace_bytes(op.handle, vie._dt(x), nrhs)
        rs = int(op.ranks[:, 6 - nc:, 2].max())
        row = 10 * nc * ((rs + 3) // 4 * 4)
        rows = (n[0] + 1) * (n[1] + 1) * row + 12
        least = (2 * s1 + max(s1, row + 12)) * el
        assert asked == (2 * s1 + max(s1, rows)) * el
        for nbytes in (asked, least):
            st, y = _run(op, x, e, mode.endswith("H"), nbytes, mode[0])
            assert st == vie.VIE_OK, vie.load().vie_last_error()
            err = rel(y.cpu().numpy().astype(np.complex128).reshape(u.shape), want)
            say("   pwl slabs", n, dt, mode, nrhs, nbytes == least, rs, "%.2e" % err)
            assert err <= BOUND[dt], (mode, nbytes == least)
        assert _run(op, x, e, mode.endswith("H"), least - 1, mode[0])[0] == vie.VIE_E_ARG


# thin grids at full ranks: a slab of the small ones takes as long as the whole
# pass, so the workspace asked for holds the rows in one piece
@pytest.mark.parametrize("n", [(18, 24, 6), (25, 16, 9), (5, 56, 16), (10, 35, 5), (5, 5, 5), (60, 64, 1),
                               (140, 126, 1), (126, 128, 2)])
@pytest.mark.parametrize("dt", list(BOUND))
def test_the_workspace_asked_for_holds_all_rows(n, dt):
    rng = np.random.default_rng(sum(n))
    f = [rng.standard_normal((60, m, 16)) for m in n]   # sixteen terms: z ranks of min(n3, 16)
    G = np.einsum("bir,bjr,bkr->bkji", *f).reshape(10, 6, n[2], n[1], n[0])
    for b, pair in enumerate(pwl.PAIRS):
        for c, pq in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
            for a, odd in enumerate(pwl.odd_axes(*pair, *pq)):   # zero at offset 0
                if odd:
                    G[(b, c) + (slice(None),) * (2 - a) + (0,)] = 0
    op = vie.compress_pwl(G + 0j, tol=1e-13)
    x = to_dev(_field(n, 43).reshape(1, 12, n[2], n[1], n[0]), dt)
    s1, rs = 24 * n[0] * n[1] * n[2], int(op.ranks[:, :, 2].max())
    assert rs == min(n[2], 16)
    rows = (n[0] + 1) * (n[1] + 1) * 60 * ((rs + 3) // 4 * 4) + 12
    asked = vie.load().vie_pwl_workspace_bytes(op.handle, vie._dt(x), 1)
    say("   pwl asked", n, dt, rs, "%.2f" % (rows / s1))
    assert rows > s1 and asked >= (2 * s1 + rows) * x.element_size()
    st, y = _run(op, x, x[0, 0], False, asked, "N")
    assert st == vie.VIE_OK and bool(torch.isfinite(torch.view_as_real(y)).all())


@pytest.mark.parametrize("coupled", [False, True])
@pytest.mark.parametrize("dt,tol,refine", [(torch.complex64, 1e-5, 0), (torch.complex128, 1e-9, 1)])
def test_solves_with_the_least_product_workspace(coupled, dt, tol, refine):
    n = (20, 14, 1)
    opn, opk, _, _, eps = _problem(n, False)
    lib = vie.load()
    el = 16 if dt == torch.complex128 else 8
    d, cells = vie._dt(torch.empty(0, dtype=dt)), (n[2], n[1], n[0])
    e = to_dev(1 + 0.05 * (eps - 1), dt)
    b = to_dev(_field(n, 50).reshape((12,) + cells), dt)
    opts = vie.SolveOpts(tol, 30, 100, 0, refine, vie.VIE_RECON_FP32, 1e-4)
    o = ctypes.byref(opts)
    if coupled:
        b = torch.stack([b, 377.0 * b])
        m = to_dev(np.full(cells, 1.05 - 0.01j), dt)
        full = lib.vie_solve_jm_pwl_workspace_bytes(opn.handle, opk.handle, d, o)
        asked, least = lib.vie_jm_pwl_workspace_bytes(opn.handle, opk.handle, d), 72 * 2 * n[0] * n[1] * n[2] * el
        least += 2 * _al(b.numel() * el)
    else:
        full = lib.vie_solve_pwl_workspace_bytes(opn.handle, d, o)
        asked, least = lib.vie_pwl_workspace_bytes(opn.handle, d, 1), 72 * n[0] * n[1] * n[2] * el
    assert least < asked
    xs = []
    for nbytes in (full, full - _al(asked) + _al(least)):
        ws = torch.full((nbytes + GUARD,), 255, dtype=torch.uint8, device=device())
        x = torch.empty_like(b)
        if coupled:
            st = lib.vie_solve_jm_pwl(opn.handle, opk.handle, d, H, 2 * np.pi * F, e.data_ptr(), m.data_ptr(),
                                      b.data_ptr(), x.data_ptr(), o, None, ws.data_ptr(), nbytes, vie._stream())
        else:
            st = lib.vie_solve_pwl(opn.handle, d, e.data_ptr(), b.data_ptr(), x.data_ptr(), o, None, ws.data_ptr(),
                                   nbytes, vie._stream())
        torch.cuda.synchronize()
        assert st == vie.VIE_OK, lib.vie_last_error()
        assert bool((ws[nbytes:] == 255).all())
        xs.append(x.cpu().numpy().astype(np.complex128))
    # two solves to a residual of tol, well conditioned (low contrast)
    err = rel(xs[0], xs[1])
    say("   pwl solve", coupled, dt, "%.2e" % err)
    assert err <= 10 * tol
