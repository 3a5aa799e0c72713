"""Every radix that a stage plan of the mixed-radix passes can hold, first,
middle or last, meets the FP64 oracle: the lengths here are those that the
lists of test_gpu_mix.py leave out (middle radices 4, 6 and 8 and last radices
4 and 6 of the z pass, middle 4, 6, 7, 8 and 10 and last 2 and 4 of the x and y
passes).  The plan search is repeated here, and a CPU test checks that both
lists together reach everything it can return; problems and tolerances are
those of test_gpu_mix.py."""
import numpy as np
import pytest
import torch

import test_gpu_mix as mix
from gpu_common import say, to_dev
from paper_1811_00484_amd import vie
from test_gpu_mix import TOL, Z, _check

# relative cost of a short transform, and of a third stage
COST = {1: 0, 2: 2, 3: 5.5, 4: 4, 5: 9, 6: 9, 7: 16, 8: 6.5, 9: 13, 10: 12, 12: 10, 14: 18, 15: 16, 16: 9.5}
MIDDLE_COST = 14
FIRST = (2, 4, 6, 8, 10, 12, 14, 16)
MIDDLE = (1, 4, 5, 6, 7, 8, 9, 10)
LAST = (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 15, 16)
REGISTER = {"z": (128, 256, 512), "xy": (128, 192, 224, 256, 512)}   # lengths with kernels of their own
LAST_MAX = {"z": 9, "xy": 16}

MORE_Z = [4, 24, 36, 96, 108, 144, 192]
MORE_XY = [(2, 8), (98, 108), (140, 144), (180, 126)]


def _plan(length, last_max):
    best = None
    for a in FIRST:
        for b in MIDDLE:
            for c in LAST:
                if a * b * c != length or c > last_max or (b > 1 and c == 1):
                    continue
                cost = COST[a] + COST[b] + COST[c] + (MIDDLE_COST if b > 1 else 0) + (0.01 if a == 10 else 0)
                if best is None or cost < best[0]:
                    best = (cost, (a, b, c))
    return best[1]


def _smooth(m):
    for p in (2, 3, 5, 7):
        while m % p == 0:
            m //= p
    return m == 1


def _reached(kind, sizes):
    return {(i, r) for m in sizes if 2 * m not in REGISTER[kind] for i, r in enumerate(_plan(2 * m, LAST_MAX[kind]))}


@pytest.mark.parametrize("kind", ["z", "xy"])
def test_the_lists_reach_every_radix(kind):
    every = _reached(kind, [m for m in range(1, 257) if _smooth(m)])
    if kind == "z":
        sizes = Z + MORE_Z
    else:
        pairs = [p for m in mix.test_xy_lengths.pytestmark if m.args[0] == "n1,n2" for p in m.args[1]] + MORE_XY
        sizes = [m for p in pairs for m in p]
    assert _reached(kind, sizes) == every


@pytest.mark.gpu
@pytest.mark.parametrize("n3", MORE_Z)
@pytest.mark.parametrize("dt", list(TOL))
def test_more_z_lengths(n3, dt):
    _check((3, 5, n3), dt)


@pytest.mark.gpu
@pytest.mark.parametrize("n1,n2", MORE_XY)
@pytest.mark.parametrize("dt", list(TOL))
def test_more_xy_lengths(n1, n2, dt):
    _check((n1, n2, 3), dt)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [60, 80, 120])
def test_the_round_trip_has_no_gain(n):
    # N^ = 1 (every diagonal tensor a unit entry at offset zero): the product is
    # the round trip alone.  A mean gain of the complex64 transforms comes from
    # their constants; three axes add it up.  Bound: half a unit roundoff, the
    # random part averages out over 3 n^3 values.
    U = np.zeros((n, 1), complex)
    U[0] = 1
    zero = np.zeros((n, 1), complex)
    cores = [np.full((1, 1, 1), c < 3, complex) for c in range(6)]
    factors = [[U if c < 3 else zero] * 3 for c in range(6)]
    op = vie.from_tucker((n, n, n), cores, factors)
    rng = np.random.default_rng(n)
    x = to_dev(rng.standard_normal((1, 3, n, n, n)) + 1j * rng.standard_normal((1, 3, n, n, n)), torch.complex64)
    y, x = vie.matvec(op, x, kind="N").to(torch.complex128), x.to(torch.complex128)
    gain = float((torch.vdot(x.reshape(-1), (y - x).reshape(-1)) / torch.vdot(x.reshape(-1), x.reshape(-1))).real)
    gain -= float(np.float32(1 / (8 * n ** 3))) * 8 * n ** 3 - 1   # the tables' one float, with the inverse's scaling
    say("   gain", n, "%.2e" % gain)
    assert abs(gain) <= 2.0 ** -25
