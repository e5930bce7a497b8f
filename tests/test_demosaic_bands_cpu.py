"""Rows per band of the demosaicing launches for very many images: whole Bayer rows, at least one
band, and fewer than 2^25 waves wherever the images alone do not take as many."""
import pytest

from probe import ask


@pytest.mark.parametrize("method,rows", [("bilinear", 2), ("gradient", 4)])
@pytest.mark.parametrize("sectors", [0, 1])
def test_band_ends_for_any_number_of_images(method, rows, sectors):
    cases = [(images, H, W) for images in (1, 1000, (1 << 24) - 1, 1 << 24, (1 << 25) - 1, 1 << 25,
                                           (1 << 26) - 1)
             for H in (rows, 8, 4096) for W in (4, 256, 260, 1024)
             if images * H * W < 1 << 34]
    got = ask([f"demosaic {method} {i} {h} {w} {sectors}" for i, h, w in cases])
    for (images, H, W), line in zip(cases, got):
        band = int(line)
        waves = images * -(-(W // 4) // 64) * -(-H // band) if band > 0 else 0
        assert band >= 2 and band % 2 == 0, (images, H, W, band)
        assert band < 2 * max(H, 32), (images, H, W, band)
        assert waves < 1 << 25 or band >= H, (images, H, W, band)


def test_gradient_band_heights():
    pytest.importorskip("torch")
    from test_gpu_large_images import GRADIENT
    got = ask(["demosaic gradient %d %d %d 1" % s for s, _ in GRADIENT])
    assert [int(x) for x in got] == [band for _, band in GRADIENT]
    assert all(s[1] % band for s, band in GRADIENT)
