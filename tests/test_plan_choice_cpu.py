"""Plans of scenes whose time is mostly the staging of LUT rows, and of images off 64-byte sectors:
the modes that were measured to take up to twice the time there are not chosen."""
import pytest

from probe import ask

RAW, L2, PACKED, DENSE = 0, 1, 2, 3


def choice(B, N, D, L, dn=0, out=0):
    names = ("path", "strip", "strips", "vec", "threads", "chunk_lines", "nontemporal")
    return dict(zip(names, map(int, ask([f"choice {B} {N} {D} {L} {dn} {out}"])[0].split())))


@pytest.mark.parametrize("shape", [(1, 773, 2860, 8192), (3, 739, 1004, 8192), (4, 656, 646, 8192),
                                   (1, 701, 4688, 8192), (3, 726, 1768, 8192)])
def test_few_lines_take_no_narrow_dense_strips(shape):
    p = choice(*shape)
    assert not (p["path"] == DENSE and p["strip"] <= 32), p


def test_rows_loaded_16_bits_at_a_time_take_no_raw_strips_of_many_tiles():
    assert choice(1, 575, 10688, 2050)["path"] == PACKED


@pytest.mark.parametrize("dn,in_place,nontemporal", [(0, True, 2), (8, True, 0), (2, True, 0),
                                                     (8, False, 2)])
def test_stores_in_place_off_sectors_are_cached(dn, in_place, nontemporal):
    p = choice(1, 5000, 2048, 1024, dn, -1 if in_place else 0)
    assert p["strip"] >= 32 and p["nontemporal"] == nontemporal, p


@pytest.mark.parametrize("shape,vec", [((4, 12000, 6001, 1024), 8), ((2, 20000, 2001, 512), 8),
                                       ((4, 470, 6807, 4096), 1)])
@pytest.mark.parametrize("out", [0, -1])
def test_odd_rows_run_wide_but_not_two_tiles_per_cu(shape, vec, out):
    assert ask(["launch %d %d %d %d 0 %d" % (*shape, out)]) == [str(vec)]
