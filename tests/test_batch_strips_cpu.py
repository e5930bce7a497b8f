"""Strips of a batch request: together every detector once, at least 8 each where a lane takes 8, and
8 pixels per lane in place too, whatever the row's length leaves for the last strip."""
import pytest

from probe import ask

RAW, L2, PACKED, DENSE = 0, 1, 2, 3


@pytest.mark.parametrize("in_place", [0, 1])
@pytest.mark.parametrize("path,L,W", [(DENSE, 4096, 128), (DENSE, 8192, 64), (PACKED, 4096, 64),
                                      (PACKED, 1024, 256), (RAW, 300, 128), (RAW, 16, 1024),
                                      (RAW, 2048, 16), (L2, 60000, 64)])
def test_strips_of_any_row(path, L, W, in_place):
    dets = list(range(8, 300)) + [511, 513, 519, 520, 1023, 1025, 1031, 4096, 4098, 4100, 4103, 8199]
    for D, line in zip(dets, ask([f"strips {D} {L} {path} {W} {in_place}" for D in dets])):
        vec, *rest = map(int, line.split())
        assert vec == 8, D
        at = 0
        for d0, width in zip(rest[::2], rest[1::2]):
            assert d0 == at and 8 <= width <= W, (D, line)
            at = d0 + width
        assert at == D


def test_strips_of_8_overlap_but_not_in_place():
    apart, inside = ask(["strips 20 2048 0 8 0", "strips 20 2048 0 8 1"])
    assert apart == "8 0 8 8 8 12 8"
    assert inside == "1 0 8 8 8 16 4"
