"""First scans over coefficients that an earlier scan of the component already holds (no encoder should write them, the
parser takes them): decoded in file order, so that the coefficients are the oracle's, alone and among usual images."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen

pytestmark = pytest.mark.gpu

DC = (1, 0, 0, 0, 0, 0, 0, 0)
USUAL = [DC, (1, 0, 0, 0, 1, 5, 0, 2), (1, 0, 0, 0, 6, 63, 0, 2), (1, 0, 0, 0, 1, 63, 2, 1), (1, 0, 0, 0, 1, 63, 1, 0)]
SCRIPTS = {
    "ac first twice": [DC, (1, 0, 0, 0, 1, 63, 0, 1), (1, 0, 0, 0, 1, 63, 0, 0)],
    "ac first over a part": [DC, (1, 0, 0, 0, 1, 20, 0, 1), (1, 0, 0, 0, 10, 63, 0, 0), (1, 0, 0, 0, 1, 9, 1, 0)],
    "dc first twice": [(1, 0, 0, 0, 0, 0, 0, 1), DC, (1, 0, 0, 0, 1, 63, 0, 1), (1, 0, 0, 0, 1, 63, 1, 0)],
    # (the refinement is replayed on the final coefficients, which is not what the oracle does with such a file: the same
    # result launch by launch is what can be asked for)
    "ac first after a refinement": [DC, (1, 0, 0, 0, 1, 63, 0, 2), (1, 0, 0, 0, 1, 63, 2, 1), (1, 0, 0, 0, 1, 20, 0, 1)],
}


def _coefficients(rec, k, lanes, timing):
    with pkg.pcr_open(rec, 0) as r:
        r.set_lane_decoders(lanes)
        r.enable_stage_timing(timing)
        status = torch.empty(r.n, dtype=torch.int32, device="cuda")
        pix = r.decode_batch(k, status=status).cpu().numpy()
        assert (status.cpu().numpy() == 0).all()
        return r.decode_coefficients(k).cpu().numpy(), pix, r.coef_layout()


@pytest.mark.parametrize("restart", [0, 2])
@pytest.mark.parametrize("name", sorted(SCRIPTS))
def test_first_scans_over_earlier_ones(name, restart):
    script = SCRIPTS[name]
    sizes = [(8, 8), (203, 95), (120, 333)]
    files = [pcrgen.encode_pixels(pcrgen.synth(10 + i, 1 + i % 2, w, h, 1, 14.0), 1, 1, 93, script, restart=restart) for i, (w, h) in enumerate(sizes)]
    files.insert(1, pcrgen.encode_pixels(pcrgen.synth(20, 1, 150, 111, 1, 14.0), 1, 1, 93, USUAL, restart=restart))
    rec = pcrgen.write_record(files)
    for k in range(1, len(script) + 1):
        for lanes in (0, 1):
            coef, pix, lay = _coefficients(rec, k, lanes, False)
            by_launch = _coefficients(rec, k, lanes, True)
            assert np.array_equal(coef, by_launch[0]) and np.array_equal(pix, by_launch[1]), (k, lanes)
            if "refinement" in name and k == len(script):
                continue
            for i in range(len(files)):
                want, _, _ = oracle.decode_record_image(rec, i, k)
                assert np.array_equal(coef[int(lay[i]):int(lay[i + 1])], want), (i, k, lanes)
