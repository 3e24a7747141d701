"""The runs of MCUs of k_pixel at their edges: pictures one MCU short of, at and beyond what a workgroup holds (121 gray
MCUs, 42 of 4:4:4, 30 of 4:2:2, 32 of 4:4:0, 21 of 4:2:0), in one row, in one column and in rows a run ends inside of, with
every refinement script a pass can be made alone or together with the one before it."""
import numpy as np
import pytest

import oracle
import paper_1911_00472_amd as pkg
import pcrgen

pytestmark = pytest.mark.gpu

RUNS = {"gray": (1, 1, 1, 121), "444": (3, 1, 1, 42), "422": (3, 2, 1, 30), "440": (3, 1, 2, 32), "420": (3, 2, 2, 21)}
PIXEL_TOL = 1                                    # LSB: fp32 against the oracle's fp64, one rounding on both sides


def _script(nc):
    """Three bits of refinement, the bands cut differently in each: passes that join the one before (luma, both last bits),
    passes of one bit after another of the same bit, a DC refinement between them."""
    dc = [(nc,) + tuple(range(nc)) + (0,) * (3 - nc) + (0, 0, 0, 1)]
    ac = []
    for c in range(nc):
        ac += [(1, c, 0, 0, 1, 9, 0, 3), (1, c, 0, 0, 10, 63, 0, 2), (1, c, 0, 0, 1, 9, 3, 2), (1, c, 0, 0, 1, 63, 2, 1)]
    ac += [(nc,) + tuple(range(nc)) + (0,) * (3 - nc) + (0, 0, 1, 0)]
    for c in range(nc):
        ac += [(1, c, 0, 0, 1, 31, 1, 0), (1, c, 0, 0, 32, 63, 1, 0)] if c == 1 else [(1, c, 0, 0, 1, 63, 1, 0)]
    return dc + ac


@pytest.mark.parametrize("kind", sorted(RUNS))
def test_run_edges(kind):
    C, hs, vs, per = RUNS[kind]
    grids = [(1, 1), (per - 1, 1), (per, 1), (per + 1, 1), (1, per + 1), (7, (2 * per) // 7 + 1), (per // 2 + 1, 3)]
    script = _script(C)
    files = []
    for i, (mx, my) in enumerate(grids):
        w, h = 8 * hs * mx - (i % 3), 8 * vs * my - (i % 4)          # (the last MCU's columns and rows are not all there)
        files.append(pcrgen.encode_pixels(pcrgen.synth(900 + i, i % 3, w, h, C, 14.0), hs, vs, 93, script, restart=0))
    rec = pcrgen.write_record(files)
    with pkg.pcr_open(rec, 0) as r:
        lay = r.output_layout()
        for k in (1, 2, len(script) // 2, len(script)):
            out = r.decode_batch(k).cpu().numpy()
            for i, (_, want, info) in enumerate(oracle.decode_record(rec, k, threads=8)):
                got = out[int(lay[i]):int(lay[i + 1])].reshape(want.shape).astype(int)
                assert np.abs(got - want).max() <= PIXEL_TOL, (kind, i, k)
