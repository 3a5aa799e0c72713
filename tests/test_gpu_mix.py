"""The mixed-radix passes (every FFT length without a register-FFT kernel)
against the FP64 oracle on the same random Tucker form, at grids whose
transforms take each first, middle and last radix of the stage plans, one and
two k1 quads per z workgroup, an odd number of quads, and right-hand sides
that share a workgroup's tables.

Tolerances: ten transforms of at most nine radix-2-equivalent roundings each
and a table sum of a few terms, unit roundoff 6e-8 (1.1e-16): below 6e-6
(1e-14); 1e-13 in complex128 leaves room for the oracle's own rounding."""
import functools

import numpy as np
import pytest
import torch

from gpu_common import rel, say, to_dev
from oracle import circulant, operator as opm
from paper_1811_00484_amd import vie

pytestmark = pytest.mark.gpu

TOL = {torch.complex64: 6e-6, torch.complex128: 1e-13}


def _cx(rng, shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


@functools.lru_cache(maxsize=4)
def _problem(n, cp=False, rank=3):
    rng = np.random.default_rng(sum(n))
    cores, factors = [], []
    for c in range(6):
        signs = circulant.axis_signs(c)
        r = [1 if cp else min(n[a], rank) for a in range(3)]
        if cp:
            r = [min(min(n), 2)] * 3
        G = np.zeros(r, complex)
        if cp:
            for l in range(r[0]):
                G[l, l, l] = _cx(rng, ())
        else:
            G = _cx(rng, r)
        Us = []
        for a in range(3):
            U = _cx(rng, (n[a], r[a])) / np.sqrt(n[a])
            if signs[a] < 0:
                U[0, :] = 0
            Us.append(U)
        cores.append(G)
        factors.append(Us)
    nhat = [circulant.fourier_tensor_tucker(cores[c], factors[c], circulant.axis_signs(c)) for c in range(6)]
    return vie.from_tucker(n, cores, factors), opm.FourierOperator(n, nhat)


def _check(n, dt, nrhs=1, modes=("A", "AH"), **kw):
    op, ref = _problem(n, **kw)
    rng = np.random.default_rng(7)
    u = _cx(rng, (nrhs, 3, n[2], n[1], n[0]))
    eps = 1 + rng.uniform(0, 50, (n[2], n[1], n[0])) - 1j * rng.uniform(0, 30, (n[2], n[1], n[0]))
    x, e = to_dev(u, dt), to_dev(eps, dt)
    for mode in modes:
        y = vie.matvec(op, x, e, kind="N" if mode[0] == "N" else "A", adjoint=mode.endswith("H"))
        yo = np.stack([opm.matvec(ref, eps, v, mode) for v in u])
        err = rel(y.cpu().numpy().astype(np.complex128), yo)
        say("   mix", n, dt, mode, nrhs, "%.2e" % err)
        assert err <= TOL[dt], (n, mode)


# z lengths 2 .. 500: last radices 1..9, first radices 2..16, middle 4..10
Z = [1, 2, 3, 7, 9, 14, 16, 18, 21, 25, 27, 32, 35, 42, 45, 49, 54, 56, 63, 72, 81, 98, 105, 125, 147, 162, 180, 200,
     243, 245, 250]


@pytest.mark.parametrize("n3", Z)
@pytest.mark.parametrize("dt", list(TOL))
def test_z_lengths(n3, dt):
    _check((3, 5, n3), dt)


# x and y lengths: also the last radices 10, 12, 15 and 16 of the x and y
# passes, and pencil counts beside the tile width
@pytest.mark.parametrize("n1,n2", [(1, 50), (24, 45), (60, 75), (80, 90), (120, 7), (125, 18), (175, 16), (243, 15),
                                   (250, 35), (5, 245), (6, 160), (9, 250)])
@pytest.mark.parametrize("dt", list(TOL))
def test_xy_lengths(n1, n2, dt):
    _check((n1, n2, 3), dt)


@pytest.mark.parametrize("dt", list(TOL))
@pytest.mark.parametrize("nrhs", [1, 5])
def test_two_quads_a_workgroup_and_shared_tables(dt, nrhs):
    _check((40, 30, 35), dt, nrhs, modes=("A", "AH", "N", "NH"))


@pytest.mark.parametrize("dt", list(TOL))
def test_superdiagonal_core(dt):
    _check((36, 28, 15), dt, 2, cp=True)


@pytest.mark.parametrize("dt", list(TOL))
@pytest.mark.parametrize("n", [(70, 64, 3), (35, 20, 2), (9, 1, 3), (4, 1, 1), (2, 3, 64), (16, 16, 16)])
def test_v_rows_in_slabs(n, dt):
    # V rows larger than the intermediate they take the place of: in one piece
    # with the workspace that the library asks for, and with the least one in
    # several slabs of k2, one k2 at a time, or not at all
    _check(n, dt, 1, rank=64)
    op, ref = _problem(n, rank=64)
    rng = np.random.default_rng(9)
    u = _cx(rng, (3, n[2], n[1], n[0]))
    x = to_dev(u, dt)
    y = torch.empty_like(x)
    least = 18 * n[0] * n[1] * n[2] * x.element_size()
    ws = torch.empty(least, dtype=torch.uint8, device=x.device)
    lib = vie.load()
    st = lib.vie_matvec(op.handle, vie.VIE_OP_N, vie._dt(x), 0, None, x.data_ptr(), y.data_ptr(), 1, ws.data_ptr(),
                        least, vie._stream())
    assert st == vie.VIE_OK
    assert rel(y.cpu().numpy().astype(np.complex128), opm.matvec(ref, None, u, "N")) <= TOL[dt]
    assert lib.vie_matvec(op.handle, vie.VIE_OP_N, vie._dt(x), 0, None, x.data_ptr(), y.data_ptr(), 1, ws.data_ptr(),
                          least - 1, vie._stream()) == vie.VIE_E_ARG


@pytest.mark.parametrize("dt", list(TOL))
def test_dense_spectrum(dt):
    n = (36, 28, 15)
    op, _ = _problem(n)
    vie.densify(op, with_c128=True)
    vie.set_nhat(op, "dense")
    try:
        _check(n, dt, 2)
    finally:
        vie.set_nhat(op, "tucker")


# the register-FFT z pass on the same problems: an odd number of k1 quads, right-hand
# sides that share a workgroup's tables, and (complex128 at 512) a table in the
# place of the FFT slices
@pytest.mark.parametrize("n,nrhs", [((60, 40, 64), 5), ((42, 50, 128), 3), ((7, 6, 256), 2)])
@pytest.mark.parametrize("dt", list(TOL))
def test_register_z_pass_shares_tables(n, nrhs, dt):
    _check(n, dt, nrhs)


@pytest.mark.parametrize("n", [(60, 40, 64), (5, 6, 256)])
def test_register_z_pass_at_the_largest_rank(n):
    _check(n, torch.complex64, 1, rank=40)


def test_bf16_right_hand_sides_equal_single_calls():
    n = (60, 40, 64)
    op, _ = _problem(n)
    rng = np.random.default_rng(8)
    x = to_dev(_cx(rng, (5, 3, n[2], n[1], n[0])), torch.complex64)
    y = vie.matvec(op, x, kind="N", recon="bf16")
    for s in range(5):
        assert torch.equal(y[s], vie.matvec(op, x[s].contiguous(), kind="N", recon="bf16"))
