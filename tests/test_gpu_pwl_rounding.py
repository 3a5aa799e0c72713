"""Rounding of the piecewise-linear Fourier-domain sum in complex64: the twelve
products of an output are added as four sums of three (one per basis block),
not one after another.

Everything but that sum and the inverse transform's additions is exact here:
on a 2 x 2 x 2 grid the transforms' twiddles are +-1 and +-i, x holds integers
whose transform stays below 2^24, and every defining tensor has one entry (a
float), whose Fourier-domain values are that entry times 1, +-2 i, +-4 or
+-8 i.  Both orders are emulated with FP32 fused multiply-adds; the device
result has to be on the near side of the geometric mean of their errors."""
import numpy as np
import pytest
import torch

from gpu_common import say, to_dev
from oracle import pwl
from paper_1811_00484_amd import vie

pytestmark = pytest.mark.gpu

F32 = np.float32
R = 1024


def _tensors(rng):
    G = np.zeros((10, 6, 2, 2, 2), complex)
    for P, (l, lp) in enumerate(pwl.PAIRS):
        for c, (p, q) in enumerate(pwl.COMPONENTS):
            D = [int(o) for o in pwl.odd_axes(l, lp, p, q)]
            v = complex(*rng.standard_normal(2).astype(F32).astype(float))
            G[P, c, D[2], D[1], D[0]] = v / (np.sqrt(12.0) ** ((l > 0) + (lp > 0)))
    return G


def _matrices(G):
    """The 12 x 12 product of every frequency, normalised basis, with the
    inverse transform's 1 / 64"""
    k = pwl.dense_kernels(G)
    M = np.zeros((4, 4, 4, 12, 12), complex)
    for l in range(4):
        for lp in range(4):
            for p in range(3):
                for q in range(3):
                    M[..., 3 * l + p, 3 * lp + q] = pwl.SCALE[l] * pwl.SCALE[lp] * k[l][lp][p][q] / 64
    return M


def _fma(a, b, c):
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(F32)


def _mac(s, a, b):
    re = _fma(-a.imag, b.imag, _fma(a.real, b.real, s[0]))
    im = _fma(a.imag, b.real, _fma(a.real, b.imag, s[1]))
    return re, im


def _sums(M, X, by_block):
    zero = (np.zeros((R, 4, 4, 4), F32),) * 2
    acc = [zero] * 12
    for l, lp in pwl.PAIRS:
        for r0, c0 in [(l, lp)] if l == lp else [(l, lp), (lp, l)]:
            for p in range(3):
                r = 3 * r0 + p
                s = zero if by_block else acc[r]
                for q in range(3):
                    s = _mac(s, M[None, ..., r, 3 * c0 + q], X[:, 3 * c0 + q])
                acc[r] = (acc[r][0] + s[0], acc[r][1] + s[1]) if by_block else s
    return np.stack([a + 1j * b for a, b in acc], axis=1).astype(np.complex64)


def _inverse(Y):
    """The unnormalised inverse transform's first half along every axis, z
    first, each addition rounded to FP32 (radix 4)"""
    for ax in (4, 3, 2):
        a = [np.take(Y, i, ax) for i in range(4)]
        Y = np.stack([(a[0] + a[2]) + (a[1] + a[3]), (a[0] - a[2]) + np.complex64(1j) * (a[1] - a[3])], ax)
    return Y


def test_the_sum_over_blocks_rounds_like_sums_of_three():
    rng = np.random.default_rng(0)
    G = _tensors(rng)
    M = _matrices(G)
    M32 = M.astype(np.complex64)
    assert np.abs(M32 - M).max() <= 1e-15 * np.abs(M).max()   # the tables are floats
    x = rng.integers(-2 ** 18, 2 ** 18, (2, R, 12, 2, 2, 2)).astype(float)
    x = x[0] + 1j * x[1]                                      # (R, 12, x, y, z)
    pad = np.zeros((R, 12, 4, 4, 4), complex)
    pad[:, :, :2, :2, :2] = x
    X = np.fft.fftn(pad, axes=(2, 3, 4))
    X = np.round(X.real) + 1j * np.round(X.imag)
    X32 = X.astype(np.complex64)
    assert np.array_equal(X32, X)
    exact = np.moveaxis(np.matmul(M, np.moveaxis(X, 1, -1)[..., None])[..., 0], -1, 1)
    want = 64 * np.fft.ifftn(exact, axes=(2, 3, 4))[:, :, :2, :2, :2]

    def err(y):
        return float(np.sqrt(np.mean(np.abs(y - want) ** 2) / np.mean(np.abs(want) ** 2)))

    blocks, chain = (err(_inverse(_sums(M32, X32, b))) for b in (True, False))
    op = vie.compress_pwl(G, tol=1e-6)
    xd = to_dev(np.ascontiguousarray(np.transpose(x, (0, 1, 4, 3, 2))), torch.complex64)
    y = vie.matvec_pwl(op, xd, kind="N").cpu().numpy().astype(np.complex128)
    got = err(np.transpose(y, (0, 1, 4, 3, 2)))
    say("   rounding: by blocks %.3e, one chain %.3e, device %.3e" % (blocks, chain, got))
    assert blocks < 0.95 * chain
    assert got <= np.sqrt(blocks * chain)
