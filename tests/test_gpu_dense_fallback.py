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


# Rows that the encoder has to tell apart: saturated at either end (run lengths around a lane's 8
# and a block's 64 entries), constant, steps of 2 out of and into a saturated run, decreasing,
# entries above levels - 1 and wrapping around 65535, and levels that end inside a lane, a block
# and a pass of 512.
def _odd_rows(L, rng):
    v = np.arange(L)
    rows = [np.clip(v - z, 0, L - 1) for z in (0, 1, 7, 8, 9, 63, 64, 65, 130)]
    rows += [np.clip(v + z, 0, L - 1) for z in (1, 7, 8, 63, 64, 65, 200)]
    rows += [np.full(L, c) for c in (0, 1, 5, L - 2, L - 1)]
    rows += [np.where(v < 70, 0, np.minimum(v - 68, L - 1)), np.where(v < L - 70, v // 2, L - 1)]
    rows += [np.clip((1.07 * v).astype(int) - 40, 0, L - 1), (0.93 * v).astype(int)]
    rows += [L - 1 - v, np.where(v == 90, 3, v), np.where(v == L - 2, L - 5, v)]
    rows += [v + 3 * (v > 100), np.minimum(v + 50, L + 20), (v + 65500) % 65536, v + L]
    rows += [rng.integers(0, 65536, L), np.clip(2 * v - 31, 0, L - 1)]
    return np.stack(rows).astype(np.uint16)


@pytest.mark.parametrize("L", [2048, 2049, 2060, 2100, 2560, 3000, 4096, 8191])
def test_encoder_on_odd_rows(L):
    rng = np.random.default_rng(L)
    lut = _odd_rows(L, rng)[None]
    D = lut.shape[1]
    # Every level of every row, and saturating DN.
    dn = np.concatenate([np.arange(L + 3), rng.integers(0, 65536, 61)])[None, :, None]
    dn = np.ascontiguousarray(np.broadcast_to(dn, (1, dn.shape[1], D))).astype(np.uint16)
    want = oracle.get().correct(dn, lut)
    N = dn.shape[1]
    n = rc.rc_correct_ws_bytes(D, 1, L)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
    d_dn, d_lut = to_dev_u16(dn), to_dev_u16(lut)
    for call in ("ws", "tile", "plain"):
        out = Guarded((1, N, D))
        if call == "ws":
            rc.rc_correct_ws(d_dn, d_lut, N, D, 1, L, out.t, ws, n)
        elif call == "tile":
            plan = rc.Plan(path=rc.RC_PATH_DENSE, strip=64, vec=1, threads=256, unroll=8,
                           chunk_lines=N, xcd_remap=1, nontemporal=0, strips=0, lane_map=0)
            if 64 * ((L + 63) // 64) * 10 > 160 * 1024:
                continue
            rc.rc_correct_plan(d_dn, d_lut, N, D, 1, L, out.t, plan)
        else:
            rc.rc_correct(d_dn, d_lut, N, D, 1, L, out.t)
        torch.cuda.synchronize()
        out.check_pads()
        np.testing.assert_array_equal(out.host(), want, err_msg=call)
