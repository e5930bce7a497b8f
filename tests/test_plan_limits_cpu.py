"""rc_correct takes every shape that a simpler tiling of it could run: rows so wide that a tile's
32-bit offsets bound its lines and threads, and so many rows of few detectors that narrow strips
would be more tiles than a launch holds. The plan it reports runs as it is too."""
import random

import pytest

from probe import ask

SHAPES = [(2, 20763, 146830, 365), (3, 16783, 133215, 227), (1, 8160, 170581, 256),
          (4, 17388, 65452, 1625), (3, 39486, 227728, 582), (3, 13148, 141648, 1024),
          (1, 14507, 131829, 2514),
          (614695, 2, 400, 152), (300441, 3, 592, 374), (1956311, 2, 112, 512), (738504, 1, 1266, 115)]


@pytest.mark.parametrize("dn,out", [(0, 0), (2, 0), (0, -1), (6, -1)])
def test_wide_rows_and_many_bands(dn, out):
    for shape, line in zip(SHAPES, ask(["plan %d %d %d %d %d %d" % (*s, dn, out) for s in SHAPES])):
        ok, pow2, even, as_it_is = line.split()
        assert ok == "1" or (pow2, even) == ("0", "0"), (shape, line)
        assert ok == as_it_is, (shape, line)


def test_random_shapes():
    rng = random.Random(7)

    def log(lo, hi):
        return max(1, round(lo * (hi / lo) ** rng.random()))

    shapes = []
    while len(shapes) < 20000:
        B, N, D, L = log(1, rng.choice([8, 1e8])), log(1, rng.choice([1e5, 1e9])), log(1, 1e9), log(2, 65536)
        if B * D * L < 1.2e11 and B * N * D < 6e10:
            D = max(1, D & rng.choice([-1, -4, -8, -32]))
            shapes.append((B, N, D, max(2, L), 2 * rng.choice([0, 0, 0, 1, 2, 4]), rng.choice([0, -1])))
    refused = []
    for shape, line in zip(shapes, ask(["plan %d %d %d %d %d %d" % s for s in shapes])):
        ok, pow2, even, as_it_is = line.split()
        if ok != as_it_is or ok == "0" and (pow2 == "1" or even == "1"):
            refused.append(shape)
    assert not refused, (len(refused), refused[:5])
