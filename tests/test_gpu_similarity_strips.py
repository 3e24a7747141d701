"""The strips of k_ssim_tiles at their edges: pictures one column and one row short of, at and beyond a strip (54 window
positions across, 32, 64 or 96 down, groups of four rows), and a record large enough for the tallest strips."""
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
