"""In place, with 8 pixels per lane on rows and images that allow fewer: the workspace corrections,
and tiles with blocks the dense form cannot hold. Bit-exact against the oracle, no write outside
the image."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1505_05655_amd as rc  # noqa: E402
import pins  # noqa: E402
from gpu_util import Guarded, to_dev_f64, to_dev_u16  # noqa: E402
from test_gpu_dense_fallback import BAD, _lut  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [9, 17, 33, 63, 65, 100, 129, 257, 511, 777, 1027])
@pytest.mark.parametrize("lines,L", [(300, 2048), (77, 4096), (40, 8192)])
def test_workspace_corrections(D, lines, L):
    B, o = 2, oracle.get()
    coeffs, dn = pins.tiny_case(D + lines, B, lines, D, L)
    coeffs[..., 1] = np.random.default_rng(D).uniform(0.9, 1.1, size=(B, D))
    lut = o.lut_build(coeffs, L)
    want = o.correct(dn, lut)
    n = rc.rc_correct_ws_bytes(D, B, L)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
    d_c, d_dn, d_lut = to_dev_f64(coeffs), to_dev_u16(dn).view(B, lines, D), to_dev_u16(lut)
    for call in ("ws", "pre"):
        img = Guarded((B, lines, D), offset=D % 5)
        img.t.copy_(d_dn)
        if call == "ws":
            rc.rc_correct_ws(img.t, d_lut, lines, D, B, L, img.t, ws, n)
        else:
            rc.rc_lut_build_ws(d_c, B, D, L, d_lut, ws, n)
            rc.rc_correct_pre(img.t, d_lut, lines, D, B, L, img.t, ws, n)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(img.host(), want, err_msg=call)
        img.check_pads()


@pytest.mark.parametrize("kind", ["two", "many"])
@pytest.mark.parametrize("D,lines", [(97, 1501), (257, 333), (203, 64)])
def test_blocks_that_do_not_fit(kind, D, lines):
    L = 2048
    lut = _lut(D, L, BAD[kind](D, L // 64))
    dn = np.random.default_rng(D).integers(0, L + 50, (1, lines, D)).astype(np.uint16)
    want = oracle.get().correct(dn, lut)
    n = rc.rc_correct_ws_bytes(D, 1, L)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
    img = Guarded((1, lines, D), offset=1)
    img.t.copy_(to_dev_u16(dn))
    rc.rc_correct_ws(img.t, to_dev_u16(lut), lines, D, 1, L, img.t, ws, n)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(img.host(), want)
    img.check_pads()
