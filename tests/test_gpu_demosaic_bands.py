"""Demosaicing in short row bands: heights around every band length (2, 4, 8 rows bilinear; 6, 8,
10 gradient), rows on and off 64-byte sectors, an output that is only 8-byte aligned, and launches
large enough for the longest bands. Bit-exact against the oracle, no write outside the output."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1505_05655_amd as rc  # noqa: E402

pytestmark = pytest.mark.gpu

SENTINEL = 0x5A5A
SHAPES = [(1, h, w) for h in (4, 6, 8, 10, 12, 14, 18, 22, 26) for w in (32, 1028, 2048)]
SHAPES += [(4, 2046, 2048), (2, 2042, 2048), (3, 1546, 1612), (9, 700, 2336)]


@pytest.mark.parametrize("method", ["bilinear", "gradient"])
@pytest.mark.parametrize("off", [0, 4])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_bands(shape, off, method):
    I, H, W = shape
    rng = np.random.default_rng(I + H + W)
    raw = rng.integers(0, 65536, shape).astype(np.uint16)
    raw[:, : H // 2] //= 64  # small differences, ties
    o = oracle.get()
    want = o.demosaic(raw) if method == "bilinear" else o.demosaic_gradient(raw)
    n = 3 * raw.size
    buf = torch.full((n + 96,), SENTINEL, dtype=torch.int16, device="cuda:0")
    out = buf[32 + off:32 + off + n].view(I, 3, H, W)
    rc.demosaic(torch.from_numpy(raw.view(np.int16)).to("cuda:0"), method=method, out=out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint16), want)
    host = buf.cpu().numpy()
    assert np.all(host[:32 + off] == SENTINEL) and np.all(host[32 + off + n:] == SENTINEL)
