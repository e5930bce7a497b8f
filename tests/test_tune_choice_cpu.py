"""rc_tune times no two candidates that run the same launch, and in place an entry of the plan cache
whose tiles were timed with 8 pixels per lane only serves rows that can have them."""
import json

import pytest

from probe import ask


@pytest.mark.parametrize("shape", ["2 4700 5122 4096 0", "3 5400 4093 1024 0", "1 3000 4096 1024 2",
                                   "1 1024 1024 1024 0", "1 200 33 300 0"])
def test_candidates_run_differently(shape):
    n, distinct = map(int, ask([f"tune {shape}"])[0].split())
    assert n == distinct > 10


@pytest.mark.parametrize("entry,apart,in_place", [
    (dict(path=2, strip=128, vec=1, threads=256, unroll=8, strips=33, lane_map=1), "1", "0"),
    (dict(path=0, strip=64, vec=1, threads=1024, unroll=8, strips=0, lane_map=1), "1", "0"),
    (dict(path=2, strip=128, vec=1, threads=256, unroll=8, strips=0, lane_map=0), "1", "1"),
    (dict(path=2, strip=64, vec=1, threads=512, unroll=8, strips=0, lane_map=1), "1", "1"),
    (dict(path=1, strip=64, vec=1, threads=256, unroll=8, strips=0, lane_map=0), "1", "1"),
])
def test_entries_in_place(tmp_path, entry, apart, in_place):
    cache = tmp_path / "cache.json"
    line = dict(arch="probe", cus=256, levels=1024, dclass=12, nclass=10, bands=2, vmax=1, chunks=1,
                xcd_remap=1, nontemporal=0, kind=0, us=1.0, **entry)
    cache.write_text(json.dumps(line, separators=(",", ":")) + "\n")
    assert ask(["tuned 2 1000 4093 1024 0 0", "tuned 2 1000 4093 1024 0 1",
                "tuned 2 1000 4093 2048 0 0"], plan_cache=cache) == [apart, in_place, "0"]
