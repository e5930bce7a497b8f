"""LUT rows with entries above levels - 1, which no row of rc_lut_build has but a caller's LUT may:
looked up as they are through the workspace and the plain correction, also where the only such entry
is among the row's last, fewer than 8. Bit-exact against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1505_05655_amd as rc  # noqa: E402
from gpu_util import Guarded, to_dev_u16  # noqa: E402

pytestmark = pytest.mark.gpu


def _rows(L):
    v = np.arange(L)
    rows = []
    for back in (1, 2, 3, 7, 8, 9, 15, 16, 17, 63, 64, 65, 127, 128, 129):
        up = v.copy()
        up[L - back:] += 1 + np.arange(back)     # steps of 2 past L - 1
        rows += [np.minimum(up, 65535), np.minimum(v + (v >= L - back), L)]
        rows.append(np.where(v >= L - back, np.minimum(v, L - 2) + 2 * (v == L - 1), np.minimum(v, L - 2)))
    return np.stack(rows).astype(np.uint16)


@pytest.mark.parametrize("L", [2048, 2049, 2050, 2051, 2052, 2055, 2111, 2113, 2500, 4090, 8191])
def test_entries_above_the_last_level(L):
    lut = _rows(L)[None]
    D = lut.shape[1]
    dn = np.ascontiguousarray(np.broadcast_to(np.arange(L + 2)[None, :, None], (1, L + 2, D))
                              ).astype(np.uint16)
    want = oracle.get().correct(dn, lut)
    assert want.max() >= L
    N = L + 2
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
            rc.rc_correct_plan(d_dn, d_lut, N, D, 1, L, out.t, plan)
        else:
            rc.rc_correct(d_dn, d_lut, N, D, 1, L, out.t)
        torch.cuda.synchronize()
        out.check_pads()
        np.testing.assert_array_equal(out.host(), want, err_msg=call)
