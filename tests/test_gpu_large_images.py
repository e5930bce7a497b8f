"""Images whose plans or launches only large sizes reach, against torch on the same GPU or the
oracle: non-temporal loads (images of 256 MiB to 1 GiB in and out), rows too wide for tiles of many
lines, gradient demosaicing in bands of 10 to 32 rows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1505_05655_amd as rc  # noqa: E402

pytestmark = pytest.mark.gpu


def _check(B, N, D, L, in_place):
    g = torch.Generator(device="cuda:0").manual_seed(D)
    src = torch.randint(0, L + L // 8, (B, N, D), generator=g, device="cuda:0", dtype=torch.int16)
    lut = torch.randint(0, L, (B, D, L), generator=g, device="cuda:0", dtype=torch.int16)
    base = torch.arange(D, device="cuda:0") * L
    want = torch.empty_like(src)
    for b in range(B):
        for n0 in range(0, N, 512):
            at = src[b, n0:n0 + 512].long().clamp_(max=L - 1) + base
            want[b, n0:n0 + 512] = lut[b].view(-1)[at]
    out = src if in_place else torch.zeros_like(src)
    rc.rc_correct(src, lut, N, D, B, L, out)
    assert torch.equal(out, want)


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("shape", [(2, 8000, 6016, 1024), (1, 20000, 4096, 256)])
def test_non_temporal_loads(shape, in_place):
    B, N, D, L = shape
    assert rc.rc_plan_for(N, D, B, L)[0].as_dict()["nontemporal"] == 1
    _check(B, N, D, L, in_place)


@pytest.mark.parametrize("shape", [(1, 4000, 140001, 64), (1, 900, 200000, 300), (1, 64, 270000, 16)])
def test_very_wide_rows(shape):
    _check(*shape, False)


# Images, rows, columns and the band height each takes on 256 CUs (see
# test_demosaic_bands_cpu.py), the last band shorter.
GRADIENT = [((1, 1704, 1056), 10), ((2, 2134, 1056), 12), ((5, 500, 1056), 14), ((4, 1534, 1056), 16),
            ((5, 2134, 1056), 18), ((6, 1274, 1056), 20), ((6, 1532, 2048), 24),
            ((9, 1016, 2080), 28), ((9, 1790, 2048), 32), ((9, 2046, 2048), 10)]


@pytest.mark.parametrize("shape", [s for s, _ in GRADIENT], ids=str)
def test_gradient_bands(shape):
    rng = np.random.default_rng(shape[1])
    raw = rng.integers(0, 65536, shape).astype(np.uint16)
    raw[:, : shape[1] // 2] //= 64
    out = rc.demosaic(torch.from_numpy(raw.view(np.int16)).to("cuda:0"), method="gradient")
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint16), oracle.get().demosaic_gradient(raw))
