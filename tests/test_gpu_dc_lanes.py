"""DC first scans with a lane per unit where the lanes of a wavefront differ or run out: MCUs of every shape in one
wavefront, units of one block, tables that end where the record ends (their 32 bytes are then read from ahead of them), sixteen
codes and one; alone and in the launch of the AC first scans."""
import contextlib

import numpy as np
import pytest

import oracle
import paper_1911_00472_amd as pkg
import pcrgen
from jpeg_files import DC_TABLES, dc_table_file

pytestmark = pytest.mark.gpu


def _check(rec, k, lanes=1):
    with pkg.pcr_open(rec, 0) as r:
        r.set_lane_decoders(lanes)
        got, lay = r.decode_coefficients(k).cpu().numpy(), r.coef_layout()
        pix, play = r.decode_batch(k).cpu().numpy(), r.output_layout()
        for i in range(r.n):
            want, p, _ = oracle.decode_record_image(rec, i, k)
            assert np.array_equal(got[int(lay[i]):int(lay[i + 1])], want), (i, k)
            assert np.abs(pix[int(play[i]):int(play[i + 1])].reshape(p.shape).astype(int) - p).max() <= 1, (i, k)


@pytest.mark.parametrize("interval", [1, 5, 64])
@pytest.mark.parametrize("k", [1, 2, 5])
def test_every_shape_in_one_wavefront(interval, k):
    files = []
    for i in range(24):
        hs, vs = ((2, 2), (1, 1), (2, 1), (1, 2))[i % 4]
        w, h = 8 + 23 * (i % 5), 9 + 17 * (i % 7)
        files.append(pcrgen.encode_pixels(pcrgen.synth(60 + i, i % 3, w, h, 3, 4.0 + i), hs, vs, 70 + i))
    _check(pkg.record_write_indexed(files, None, interval), k)


def test_wavefronts_of_one_shape_and_some_of_several():
    """More than sixty-four units of each shape, and some left over of each; the order is the wavefront decoders' too."""
    files = []
    for i in range(75):
        hs, vs = ((2, 2), (1, 1), (2, 1), (1, 2))[i % 4]
        files.append(pcrgen.encode_pixels(pcrgen.synth(90 + i, i % 3, 30 + 5 * (i % 9), 20 + 9 * (i % 6), 3, 3.0 + i % 7), hs, vs, 70 + i % 20))
    rec = pkg.record_write_indexed(files, None, 2)
    for k in (1, 2):
        _check(rec, k)
    _check(rec, 1, lanes=-1)


@pytest.mark.parametrize("count", [64, 65, 127, 200])
def test_tables_at_the_very_end_of_the_record(count):
    """Gray pictures of one block, the record cut behind its first scan group: the last table has fewer than 32 bytes."""
    files = [pcrgen.encode_pixels(pcrgen.synth(9 + i, i % 3, 8, 8, 1, 2.0), 1, 1, 60) for i in range(count)]
    rec = pcrgen.write_record(files)
    ends = oracle.record_index(rec)[4]
    _check(rec[:int(ends[0])], 1)


def test_many_categories():
    """Differences of every size: tables of all the codes a picture can need, beside tables of a single one."""
    q = np.ones((2, 64), np.uint16)
    rng = np.random.default_rng(3)
    files = []
    for i in range(80):
        c = np.zeros((pcrgen.plane_blocks(64, 56, 1, 1, 1)[0], 64), np.int16)
        if i % 3:
            c[:, 0] = rng.choice([-1023, -512, -255, -128, -60, -30, -9, -4, -2, 0, 1, 3, 7, 15, 31, 100, 500, 1000], len(c))
        files.append(pcrgen.encode_coefs(c.reshape(-1), 64, 56, 1, 1, 1, q, [(1, 0, 0, 0, 0, 0, 0, 0), (1, 0, 0, 0, 1, 63, 0, 0)], 0))
    _check(pkg.record_write_indexed(files, None, 7), 1)
    _check(pkg.record_write_indexed(files, None, 7), 2)


@pytest.mark.parametrize("name", DC_TABLES)
def test_tables_whose_last_code_is_all_ones(name):
    """Both decoders take the same tables."""
    files = [dc_table_file(name, seed, blocks) for seed in range(22) for blocks in ((7, 5), (1, 1), (2, 40))]
    rec = pcrgen.write_record(files)
    _check(rec, 1, lanes=1)
    _check(rec, 1, lanes=-1)


@pytest.mark.parametrize("side, interval, pictures, k, others", [
    (64, 0, 3583, 1, 0), (64, 0, 3584, 1, 0),          # whole scans of 96 blocks: to the lanes from 3584 on
    (24, 1, 1535, 1, 0), (24, 1, 1536, 1, 0),          # four units a scan: from 6144 on
    (24, 1, 1023, 1, 1), (24, 1, 1024, 1, 1),          # with a second record open: from 4096 on
    (24, 1, 2047, 2, 0), (24, 1, 2048, 2, 0),          # where they could be beside AC scans by wavefronts: from 8192 on
    (176, 0, 70, 1, 0)])                               # whole scans of 726 blocks: to the wavefronts
def test_either_side_of_the_line_between_wavefronts_and_lanes(side, interval, pictures, k, others):
    few = [pcrgen.make_jpeg(70 + i, i % 3, side, side, 3, 6.0, 2, 2, 80) for i in range(5)]
    files = [few[i % 5] for i in range(pictures)]
    rec = pkg.record_write_indexed(files, None, interval) if interval else pcrgen.write_record(files)
    with contextlib.ExitStack() as open_too, pkg.pcr_open(rec, 0) as r:
        for _ in range(others):
            open_too.enter_context(pkg.pcr_open(pcrgen.write_record(few[:1]), 0))
        by_rule = [r.decode_coefficients(k).cpu().numpy(), r.decode_batch(k).cpu().numpy()]
        lay = r.coef_layout()
        for i in (0, 1, 2, 3, 4, pictures - 1):
            want = oracle.decode_record_image(rec, i, k)[0]
            assert np.array_equal(by_rule[0][int(lay[i]):int(lay[i + 1])], want), i
        for lanes in (1, -1):
            r.set_lane_decoders(lanes)
            assert np.array_equal(r.decode_coefficients(k).cpu().numpy(), by_rule[0]) and np.array_equal(r.decode_batch(k).cpu().numpy(), by_rule[1]), lanes
