"""Dense tiles with blocks the dense form cannot hold: a few (decoded tile, those levels from the
LUT row, staging threads streaming too) and many (every header checked), bit-exact against the
oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1505_05655_amd as rc  # noqa: E402
from gpu_util import Guarded, to_dev_u16  # noqa: E402

pytestmark = pytest.mark.gpu


def _lut(D, L, bad):
    """Identity-like rows (steps 0 and 1); bad = [(detector, block)] get steps 0 and 2."""
    v = np.arange(L)
    lut = np.stack([np.minimum(v + (v > (7 * d) % 50), L - 1) for d in range(D)]).astype(np.uint16)
    for d, blk in bad:
        e = lut[d, blk * 64:(blk + 1) * 64].astype(np.int64)
        e[20] = e[19]       # step 0, then 2
        lut[d, blk * 64:(blk + 1) * 64] = e
    return lut[None]


# bad blocks: the strip's first position and block (whose words carry the count), its last, the
# last block of the row, two in one row; more than one per block of a row.
BAD = {
    "first": lambda D, nb: [(0, 0)],
    "last": lambda D, nb: [(D - 1, nb - 1)],
    "two": lambda D, nb: [(5, 3), (5, nb - 1), (D // 2, 0)],
    "at_limit": lambda D, nb: [(d, 2) for d in range(nb)],
    "many": lambda D, nb: [(d, b) for d in range(D) for b in (1, 2)],
}


@pytest.mark.parametrize("kind", sorted(BAD))
@pytest.mark.parametrize("vec,threads,lines,chunk", [(8, 256, 1501, 1501), (8, 256, 997, 251),
                                                     (4, 512, 300, 300), (1, 256, 301, 100)])
def test_dense_tile_with_unencodable_blocks(kind, vec, threads, lines, chunk):
    D, L = 96, 2048
    lut = _lut(D, L, BAD[kind](D, L // 64))
    rng = np.random.default_rng(5)
    dn = rng.integers(0, L + 50, (1, lines, D)).astype(np.uint16)
    want = oracle.get().correct(dn, lut)
    out = Guarded((1, lines, D))
    plan = rc.Plan(path=rc.RC_PATH_DENSE, strip=128, vec=vec, threads=threads,
                   unroll=4 if vec == 8 else 8, chunk_lines=chunk, xcd_remap=1, nontemporal=0,
                   strips=0, lane_map=1)
    d_dn, d_lut = to_dev_u16(dn), to_dev_u16(lut)
    rc.rc_correct_plan(d_dn, d_lut, lines, D, 1, L, out.t, plan)
    torch.cuda.synchronize()
    out.check_pads()
    np.testing.assert_array_equal(out.host(), want)
    n = rc.rc_correct_ws_bytes(D, 1, L)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
    out.t.zero_()
    rc.rc_correct_ws(d_dn, d_lut, lines, D, 1, L, out.t, ws, n)
    torch.cuda.synchronize()
    out.check_pads()
    np.testing.assert_array_equal(out.host(), want)
