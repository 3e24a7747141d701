"""Stores past the caches (pixels_past, rows_past, fill_past): which calls take them, and that the pixels are the same either way -- colour at half and full
chroma resolution, gray, rows that end inside a chunk, DC-only decodes -- and the same as the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen

pytestmark = pytest.mark.gpu


def _same_pixels(data, n, w, h, c, k, taken):
    """The decode of k with no more than three records open, then with four: the first takes the stores past the caches where `taken` says so."""
    with pkg.pcr_open(data, 0) as r:
        a = r.decode_batch(k)
        assert r.last_past_stores() == taken, k
        others = [pkg.pcr_open(pcrgen.write_record([pcrgen.make_jpeg(1, 1, 8, 8, 1, 1.0, 1, 1, 90)]), 0) for _ in range(3)]
        b = r.decode_batch(k, torch.full_like(a, 7))
        assert not r.last_past_stores() and torch.equal(a, b), k
        for o in others:
            o.close()
        per = a.view(n, h, w, c)
        assert bool((per == per[0]).all()), k
        want = oracle.decode_record_image(data, 0, k)[1]
        assert np.abs(per[0].cpu().numpy().astype(int) - want.reshape(h, w, c)).max() <= 1, k


@pytest.mark.parametrize("n,w,h,c,sub,taken", [
    (12, 512, 512, 3, 2, {5: 0}),                              # 9 + 9 MB of planes and pixels
    (46, 1021, 1024, 3, 2, {5: 0}),                            # 138 + 138: nearly all of it fits
    (60, 1021, 1024, 3, 2, {1: 0, 5: 1, 10: 0}),               # 180 + 180: the planes fit, the pixels not beside them; DC alone, with refinement
    (35, 1024, 1021, 3, 1, {5: 1}),                            # 210 + 105
    (115, 1021, 1024, 1, 1, {3: 1, 6: 0}),                     # 230 + 115
    (90, 1024, 1021, 3, 2, {5: 0}),                            # 270 + 270: the planes do not fit either
])
def test_pixels(n, w, h, c, sub, taken):
    data = pcrgen.write_record([pcrgen.make_jpeg(40 + w + h, 2, w, h, c, 9.0, sub, sub, 88, restart=1)] * n)
    for k, t in taken.items():
        _same_pixels(data, n, w, h, c, k, bool(t))


def test_pixels_for_the_training_tail_stay_in_the_caches():
    n, w, h = 60, 1024, 1024
    data = pcrgen.write_record([pcrgen.make_jpeg(7, 2, w, h, 3, 9.0, 2, 2, 88, restart=1)] * n)
    with pkg.pcr_open(data, 0) as r:
        whole = r.decode_batch(5)
        assert r.last_past_stores()
        boxes = torch.tensor([[0, 0, w, h, 0]] * n, dtype=torch.int32, device="cuda")
        pixels = torch.full_like(whole, 3)
        r.decode_crop_batch(5, boxes, 96, 96, (0.5,) * 3, (2.0,) * 3, pixels)
        assert not r.last_past_stores() and torch.equal(pixels, whole)


@pytest.mark.parametrize("n,k,rows,fills", [(80, 1, False, False), (90, 1, True, False), (130, 5, False, False), (140, 5, False, True), (140, 10, False, True)])
def test_pixel_rows_and_the_zero_fill_beside_other_records(n, k, rows, fills):
    """Either side of 256 MB of pixels and of 400 MB of planes, alone and with three other records open."""
    w, h = 1021, 1024
    data = pcrgen.write_record([pcrgen.make_jpeg(9, 2, w, h, 3, 9.0, 2, 2, 88, restart=1)] * n)
    with pkg.pcr_open(data, 0) as r:
        a = r.decode_batch(k)
        assert not r.last_past_stores() and not r.last_past_fills()
        others = [pkg.pcr_open(pcrgen.write_record([pcrgen.make_jpeg(1, 1, 8, 8, 1, 1.0, 1, 1, 90)]), 0) for _ in range(3)]
        out = torch.full_like(a, 7)
        for _ in range(2):                                   # (planes that hold the last call's coefficients are cleared again)
            r.decode_batch(k, out)
            assert (r.last_past_stores(), r.last_past_fills()) == (rows, fills)
            assert torch.equal(a, out)
        for o in others:
            o.close()
