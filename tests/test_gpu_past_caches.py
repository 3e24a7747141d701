"""Stores past the caches (CacheRule): the pixels are the same on either side of every line, whichever kernels take it -- colour at half and
full chroma resolution, gray, rows that end inside a chunk, DC-only decodes -- and the same as the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,w,h,c,sub,ks", [(12, 512, 512, 3, 2, (5, 10)), (23, 517, 509, 3, 2, (4, 10)), (60, 517, 509, 1, 1, (3, 6)), (34, 1021, 1024, 3, 1, (10,)),
                                            (75, 1024, 1021, 3, 2, (1, 5)), (100, 1021, 1024, 3, 2, (1, 10))])
def test_the_same_on_both_sides(n, w, h, c, sub, ks):
    """9 to 300 MB of planes, calls on one stream and on four in turn: each rule is taken and left."""
    data = pcrgen.write_record([pcrgen.make_jpeg(40 + w + h, 2, w, h, c, 9.0, sub, sub, 88, restart=1)] * n)
    with pkg.pcr_open(data, 0) as r:
        alone = [r.decode_batch(k) for k in ks]
        streams = [torch.cuda.Stream() for _ in range(3)]
        others = [pkg.pcr_open(pcrgen.write_record([pcrgen.make_jpeg(1, 1, 8, 8, 1, 1.0, 1, 1, 90)]), 0) for _ in range(3)]
        for k, a in zip(ks, alone):
            out = torch.full_like(a, 7)
            for o, s in zip(others, streams):
                o.decode_batch(1, stream=s.cuda_stream)
            assert torch.equal(r.decode_batch(k, out), a), k
            torch.cuda.synchronize()
            per = a.view(n, h, w, c)
            assert bool((per == per[0]).all()), k
            want = oracle.decode_record_image(data, 0, k)[1]
            assert np.abs(per[0].cpu().numpy().astype(int) - want.reshape(h, w, c)).max() <= 1, k
        for o in others:
            o.close()
