"""The strips of k_ssim_tiles at their edges: pictures one column and one row short of, at and beyond a strip (54 window
positions across, 32, 64 or 128 down, groups of four rows), and a record large enough for the tallest strips."""
import numpy as np
import pytest

import oracle
import pcrgen
import paper_1911_00472_amd as pkg

pytestmark = pytest.mark.gpu
TOL = 3e-4                                       # as derived in test_gpu_similarity.py

EDGES = [(63, 41), (64, 42), (65, 43), (66, 44), (118, 13), (119, 73), (11, 107), (12, 75), (175, 176), (177, 352)]


@pytest.mark.parametrize("C,copies", [(3, 1), (1, 1), (3, 120), (3, 400)])
def test_strip_edges(C, copies):
    import torch
    sub = 2 if C == 3 else 1
    files = [pcrgen.make_jpeg(700 + i, 1, w, h, C, 7.0, sub, sub, 85) for i, (w, h) in enumerate(EDGES)]
    rec = pcrgen.write_record(files * copies)
    want = []
    for i in range(len(EDGES)):
        a, b = (oracle.decode_record_image(rec, i, k)[1] for k in (2, oracle.record_header(rec)["G"]))
        want.append(oracle.msssim(a, b))
    with pkg.Record(rec) as r:
        got = r.msssim_batch(r.decode_batch(2), r.decode_batch(r.G)).cpu().numpy().reshape(copies, -1)
    assert np.array_equal(got, np.broadcast_to(got[0], got.shape))
    assert np.abs(got[0] - np.array(want)).max() <= TOL, (got[0], want)


@pytest.mark.parametrize("w,h,C,sub,copies", [(11, 11, 3, 1, 1), (12, 11, 3, 2, 1), (22, 22, 3, 1, 1), (23, 24, 3, 2, 1), (11, 12, 1, 1, 1), (64, 137, 3, 2, 1),
                                              (65, 138, 3, 2, 5600), (64, 139, 3, 2, 5600), (23, 149, 3, 1, 8200)])
def test_blocks_at_both_ends_of_the_buffer(w, h, C, sub, copies):
    """Three and six bytes are loaded with the byte or two ahead of them, except at the buffer's first block; two rows of
    pixels are in flight; strips of 128 rows (many pictures) end one row short of, at and beyond a picture."""
    import torch
    rec = pcrgen.write_record([pcrgen.make_jpeg(811, 2, w, h, C, 11.0, sub, sub, 88)] * copies)
    a, b = (oracle.decode_record_image(rec, 0, k)[1] for k in (2, oracle.record_header(rec)["G"]))
    with pkg.Record(rec) as r:
        got = r.msssim_batch(r.decode_batch(2), r.decode_batch(r.G)).cpu().numpy()
    assert np.array_equal(got, np.broadcast_to(got[0], got.shape))
    assert abs(got[0] - oracle.msssim(a, b)) <= TOL


@pytest.mark.parametrize("w,h,C,copies", [(40, 40, 3, 3), (64, 64, 3, 3), (65, 64, 1, 3), (128, 128, 3, 5), (200, 200, 1, 5), (220, 220, 3, 5), (65, 64, 1, 1100)])
def test_workgroups_without_a_tile(w, h, C, copies):
    """2, 4, 6, 16, 34 and 40 tiles of 32 rows a picture, and 4 of 128: a multiple of four has a workgroup more than tiles."""
    sub = 2 if C == 3 else 1
    files = [pcrgen.make_jpeg(820 + i, 1, w, h, C, 9.0, sub, sub, 85) for i in range(2)]
    rec = pcrgen.write_record(files * copies)
    want = [oracle.msssim(*(oracle.decode_record_image(rec, i, k)[1] for k in (2, oracle.record_header(rec)["G"]))) for i in range(2)]
    with pkg.Record(rec) as r:
        a, b = r.decode_batch(2), r.decode_batch(r.G)
        got = r.msssim_batch(a, b).cpu().numpy().reshape(copies, 2)
        assert np.array_equal(got, np.broadcast_to(got[0], got.shape))
        assert np.abs(got[0] - np.array(want)).max() <= TOL
