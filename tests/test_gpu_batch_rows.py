"""Batch requests of any row length: strips whose rest is under 8 detectors, one detector, in
place, several line chunks, and coefficients whose LUT rows fit neither the packed nor the dense
form. Bit-exact against the oracle over two replays."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1505_05655_amd as rc  # noqa: E402
import pins  # noqa: E402
from gpu_util import Guarded, to_dev_f64, to_dev_u16  # noqa: E402

pytestmark = pytest.mark.gpu

# bands, lines, detectors (around 8, a dense strip of 128 and a packed one of 256), levels, offset
# of the images in elements, in place
SPECS = [(1, 40, 5, 1024, 0, False), (1, 40, 8, 4096, 1, False), (2, 300, 129, 4096, 0, False),
         (2, 300, 129, 4096, 3, True), (1, 500, 257, 1024, 0, False), (1, 500, 263, 1024, 1, True),
         (1, 500, 264, 1024, 0, True), (1, 9000, 70, 2048, 0, False), (1, 8500, 131, 1024, 5, True),
         (3, 64, 1029, 4096, 0, False), (1, 200, 100, 8192, 0, False), (1, 30, 33, 300, 7, True),
         (1, 20, 12, 16384, 0, False)]


@pytest.mark.parametrize("curve", ["calibration", "unfit"])
def test_batch_of_odd_rows(curve):
    o = oracle.get()
    reqs, keep = [], []
    for i, (B, N, D, L, off, inplace) in enumerate(SPECS):
        coeffs, dn = pins.tiny_case(100 + i, B, N, D, L)
        rng = np.random.default_rng(i)
        coeffs[..., 0] = rng.normal(0, L / 128, size=(B, D))
        coeffs[..., 1] = rng.uniform(0.9, 1.1, size=(B, D))
        coeffs[..., 2:] = 0.0
        if curve == "unfit":  # one row with steps 0 to 3, one decreasing
            coeffs[0, D // 2] = [0.0, 0.3, 1.2 / L, 0.0]
            coeffs[-1, D - 1] = [L - 1.0, -0.7, 0.0, 0.0]
        lut = o.lut_build(coeffs, L)
        want = o.correct(dn, lut)
        src = Guarded((B, N, D), offset=off)
        out = src if inplace else Guarded((B, N, D), offset=off)
        d_lut = torch.zeros((B, D, L), dtype=torch.int16, device="cuda:0")
        keep.append((to_dev_u16(dn).view(B, N, D), src, out, d_lut, lut, want))
        reqs.append((to_dev_f64(coeffs), src.t, d_lut, out.t))
    batch = rc.Batch(reqs)
    for replay in range(2):
        for dn, src, out, d_lut, _, _ in keep:
            src.t.copy_(dn)
            d_lut.zero_()
        torch.cuda.synchronize()
        batch.run()
        torch.cuda.synchronize()
        for spec, (dn, src, out, d_lut, lut, want) in zip(SPECS, keep):
            msg = f"{spec} replay {replay}"
            np.testing.assert_array_equal(d_lut.cpu().numpy().view(np.uint16), lut, err_msg=msg)
            np.testing.assert_array_equal(out.host(), want, err_msg=msg)
            out.check_pads()
    batch.close()
