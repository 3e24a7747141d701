"""k_unstuff at the edges of its lanes (16 bytes), steps (1024 bytes; 4096 where a workgroup shares a scan) and of the line
between the two ways (scans of 6144 bytes on average): stuffed zeros, restart markers and fill bytes fall on every phase
of a lane, and the last scan ends with the record."""
import numpy as np
import pytest

import oracle
import paper_1911_00472_amd as pkg
import pcrgen
from jpeg_files import with_fill_bytes

pytestmark = pytest.mark.gpu


def _noise(seed, side):
    return np.random.default_rng(seed).integers(0, 256, (side, side, 1), dtype=np.uint8)


@pytest.mark.parametrize("restart", [0, 1, 5])
@pytest.mark.parametrize("side", [8, 24, 32, 56, 64, 72, 80, 88, 120])           # about 80, 530, 1000, 2800, 3700, 4600, 5700, 6800, 13000 bytes
def test_scan_lengths_restarts_and_fill(side, restart):
    files = [pcrgen.encode_pixels(_noise(100 * side + i, side), 1, 1, 97 - (i % 3), "sequential", restart=restart) for i in range(5)]
    files += [with_fill_bytes(f) for f in files]
    files.insert(3, pcrgen.encode_pixels(_noise(side, 9), 1, 1, 50, "sequential", restart=restart))      # (one short scan among them)
    rec = pcrgen.write_record(files)
    with pkg.pcr_open(rec, 0) as r:
        lay = r.coef_layout()
        got = r.decode_coefficients(r.G).cpu().numpy()
        for i in range(r.n):
            want, _, _ = oracle.decode_record_image(rec, i, r.G)
            assert np.array_equal(got[int(lay[i]):int(lay[i + 1])], want), i


@pytest.mark.parametrize("restart", [0, 3])
@pytest.mark.parametrize("side,count", [(128, 3), (136, 3), (144, 3), (200, 3), (264, 2), (136, 170), (136, 171), (136, 520)])
def test_many_wavefronts_per_scan(side, count, restart):
    """Few long scans: sixteen wavefronts each, steps of 16384 bytes, scans that end short of, at and beyond one; short scans
    beside them; as many scans as still go that way, and more."""
    files = [pcrgen.encode_pixels(_noise(300 * side + i, side), 1, 1, 98 - (i % 3), "sequential", restart=restart) for i in range(3)]
    files = (files * (count // 3 + 1))[:count]
    files[1] = pcrgen.encode_pixels(_noise(side, 11), 1, 1, 50, "sequential", restart=restart)
    files[-1] = with_fill_bytes(files[-1])
    rec = pcrgen.write_record(files)
    with pkg.pcr_open(rec, 0) as r:
        lay = r.coef_layout()
        got = r.decode_coefficients(r.G).cpu().numpy()
        for i in list(range(min(4, r.n))) + [r.n - 1]:
            want, _, _ = oracle.decode_record_image(rec, i, r.G)
            assert np.array_equal(got[int(lay[i]):int(lay[i + 1])], want), i
