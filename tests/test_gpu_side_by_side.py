"""Scans decoded side by side in one launch (plain records, restart intervals) against the oracle and against the same
scans decoded launch by launch (stage timing on): chains from one scan to more than a workgroup takes, one block to many,
upgrades that find some of the scans done, a damaged scan in the middle of a chain."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen

pytestmark = pytest.mark.gpu

DC = (1, 0, 0, 0, 0, 0, 0, 0)
# AC scans of one component: (first bands with bits 2.., then refinements of overlapping bands)
CHAINS = {
    1: [(1, 63, 0, 0)],
    2: [(1, 63, 0, 1), (1, 63, 1, 0)],
    4: [(1, 5, 0, 2), (6, 63, 0, 2), (1, 63, 2, 1), (1, 63, 1, 0)],
    8: [(1, 5, 0, 2), (6, 20, 0, 2), (21, 63, 0, 2), (1, 5, 2, 1), (6, 63, 2, 1), (1, 20, 1, 0), (21, 40, 1, 0), (41, 63, 1, 0)],
    9: [(1, 5, 0, 2), (6, 20, 0, 2), (21, 63, 0, 2), (1, 5, 2, 1), (6, 63, 2, 1), (1, 9, 1, 0), (10, 20, 1, 0), (21, 40, 1, 0), (41, 63, 1, 0)],
}


def _image(seed, w, h, script, restart):
    return pcrgen.encode_pixels(pcrgen.synth(seed, 1 + seed % 2, w, h, 1, 14.0), 1, 1, 93, script, restart=restart)


def _decode(rec, k, timing, k0=0):
    with pkg.pcr_open(rec, 0) as r:
        if timing:
            r.enable_stage_timing(True)
        status = torch.empty(r.n, dtype=torch.int32, device="cuda")
        if k0:
            r.decode_batch(k0)
            pix = r.upgrade_batch(k, status=status)
            return pix.cpu().numpy(), None, status.cpu().numpy(), None
        pix = r.decode_batch(k, status=status).clone()
        coef = r.decode_coefficients(k)
        return pix.cpu().numpy(), coef.cpu().numpy(), status.cpu().numpy(), r.coef_layout()


@pytest.mark.parametrize("restart", [0, 2])
@pytest.mark.parametrize("length", sorted(CHAINS))
def test_chain_lengths_and_sizes(length, restart):
    script = [DC] + [(1, 0, 0, 0) + s for s in CHAINS[length]]
    files = [_image(10 * length + i, w, h, script, restart) for i, (w, h) in enumerate([(8, 8), (9, 17), (40, 8), (203, 95), (120, 333)])]
    rec = pcrgen.write_record(files)
    for k in range(1, len(script) + 1):
        pix, coef, status, lay = _decode(rec, k, False)
        pix1, coef1, status1, _ = _decode(rec, k, True)
        assert (status == 0).all() and (status1 == 0).all()
        assert np.array_equal(coef, coef1) and np.array_equal(pix, pix1), k
        for i in range(len(files)):
            want, _, _ = oracle.decode_record_image(rec, i, k)
            assert np.array_equal(coef[int(lay[i]):int(lay[i + 1])], want), (i, k)
        if k > 1:
            for k0 in {1, k - 1}:
                assert np.array_equal(_decode(rec, k, False, k0)[0], pix), (k0, k)


def test_a_damaged_scan_in_a_chain_flags_its_image_only():
    script = [DC] + [(1, 0, 0, 0) + s for s in CHAINS[4]]
    files = [_image(500 + i, 150, 111, script, 0) for i in range(4)]
    rec = pcrgen.write_record(files)
    good = _decode(rec, len(script), False)
    with pkg.pcr_open(rec, 0) as r:
        off, length = r.index()
    for g in range(1, len(script)):
        bad = bytearray(rec)
        at = int(np.asarray(off).reshape(len(script), -1)[g][1]) + int(np.asarray(length).reshape(len(script), -1)[g][1])
        bad[at - 60:at - 2] = bytes(b & 0x7F for b in np.random.default_rng(g).integers(0, 256, 58, dtype=np.uint8))
        a, b = _decode(bytes(bad), len(script), False), _decode(bytes(bad), len(script), True)
        assert np.array_equal(a[2], b[2]) and (np.delete(a[2], 1) == 0).all()
        if a[2][1] == 0:                                      # (the damage happened to be a valid stream)
            assert np.array_equal(a[1], b[1])
        lay = a[3]
        for i in (0, 2, 3):
            assert np.array_equal(a[1][int(lay[i]):int(lay[i + 1])], good[1][int(lay[i]):int(lay[i + 1])])
