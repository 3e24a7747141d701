"""Long first scans decoded by many lanes each (k_first_split) against the oracle and the wavefront decoders (which
set_lane_decoders(-1) keeps to): every sampling, scans of one piece and of thousands, streams that hardly fall into step (smooth pictures,
one colour) and are left to the wavefronts, codes and runs of every length, restart intervals and entry points far apart, upgrades, damaged data."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen
from test_record_entry_points import _entry_at

pytestmark = pytest.mark.gpu


NO, YES, WIDE = (0, 0), (1, 0), (1, 1)                       # launches of many lanes a scan; those of them of a thousand lanes


def _both(rec, splits, check=()):
    """Coefficients, pixels and status of the decoder the rule picks and of the wavefront decoders are the same; some images, the oracle's.
    splits: {k: the launches of many lanes a scan there are}."""
    ks = sorted(splits)
    with pkg.pcr_open(rec, 0) as r:
        clay = r.coef_layout()
        for k in ks:
            got = []
            for mode in (0, -1):
                r.set_lane_decoders(mode)
                st = torch.full((r.n,), 77, dtype=torch.int32, device="cuda")
                pix = r.decode_batch(k, status=st).cpu().numpy().copy()
                took = r.last_first_splits()
                assert took == ((0, 0) if mode else splits[k]), (k, mode, took)
                got.append((r.decode_coefficients(k).cpu().numpy().copy(), pix, st.cpu().numpy().copy()))
            good = got[0][2] == 0
            assert np.array_equal(got[0][2], got[1][2]), (k, got[0][2], got[1][2])
            for i in np.flatnonzero(good):
                a, b = int(clay[i]), int(clay[i + 1])
                assert np.array_equal(got[0][0][a:b], got[1][0][a:b]), (k, i)
            if good.all():
                assert np.array_equal(got[0][1], got[1][1]), k
            for i in check:
                want, _, _ = oracle.decode_record_image(rec, i, k)
                assert np.array_equal(got[0][0][int(clay[i]):int(clay[i + 1])], want), (k, i)
        return got[0][2]


SAMPLINGS = [(1, 1, 1), (3, 1, 1), (3, 2, 1), (3, 1, 2), (3, 2, 2)]
# by side, in the order of SAMPLINGS: at 1, 2, 3 (and 5)
SIZES = {40: ["nnn", "nnnn", "nnnn", "nnnn", "nnnn"], 100: ["nyy", "nnyy", "nnny", "nnny", "nnny"], 257: ["yyy", "yyyy", "nnyy", "nnyy", "nyyy"],
         640: ["yww", "ywww", "ywww", "ywww", "ywww"]}


def size_record(C, hs, vs, side):
    """A record of three pictures and the launches a decode of it makes."""
    files = [pcrgen.make_jpeg(30 + side + i, i % 3, side, side + 7 * i, C, 3.0 + 12 * i, hs, vs, 80 + 6 * i) for i in range(3)]
    takes = SIZES[side][SAMPLINGS.index((C, hs, vs))]
    return pcrgen.write_record(files), {k: {"n": NO, "y": YES, "w": WIDE}[t] for k, t in zip((1, 2, 3, 5), takes)}


@pytest.mark.parametrize("C,hs,vs", SAMPLINGS)
@pytest.mark.parametrize("side", sorted(SIZES))
def test_every_sampling_and_size(C, hs, vs, side):
    rec, splits = size_record(C, hs, vs, side)
    assert (_both(rec, splits, check=(0, 2)) == 0).all()


def mixed_record():
    """A picture that is worth many lanes beside pictures of a few blocks."""
    small = [(8, 8, 1, 1), (17, 9, 2, 2), (40, 33, 2, 1), (24, 40, 1, 2), (60, 50, 1, 1), (100, 90, 2, 2), (9, 120, 2, 1)]
    return pcrgen.write_record([pcrgen.make_jpeg(400 + i, 1, w, h, 3, 20.0, hs, vs, 92) for i, (w, h, hs, vs) in enumerate([(900, 700, 2, 2)] + small)])


def test_scans_of_one_piece_beside_scans_of_thousands():
    assert (_both(mixed_record(), {1: YES, 2: WIDE, 3: WIDE, 5: WIDE}, check=range(8)) == 0).all()


def test_streams_that_hardly_fall_into_step():
    flat = np.full((900, 900, 3), 90, np.uint8)
    ramp = np.broadcast_to((np.arange(900, dtype=np.uint16)[:, None, None] // 4).astype(np.uint8), (900, 900, 3)).copy()
    half = flat.copy()
    half[:450] = np.random.default_rng(3).integers(0, 256, (450, 900, 3), dtype=np.uint8)
    files = [pcrgen.encode_pixels(a, hs, hs, q) for a in (flat, ramp, half) for hs, q in ((2, 75), (1, 95))]
    assert (_both(pcrgen.write_record(files), {1: YES, 2: WIDE, 5: WIDE}, check=(2, 5)) == 0).all()


@pytest.mark.parametrize("n,side,splits", [(70, 500, {1: YES, 5: WIDE}), (300, 200, {1: NO, 5: NO}), (300, 400, {1: YES, 2: YES, 5: YES}), (600, 300, {1: NO, 5: YES})])
def test_more_units_than_find_room_at_once(n, side, splits):
    files = [pcrgen.make_jpeg(500 + i, 1, side - 7 * i, side + i, 3, 20.0, 2 - i % 2, 2 - i % 2, 90) for i in range(5)]
    assert (_both(pcrgen.write_record((files * n)[:n]), splits, check=(0, 1)) == 0).all()


def test_restart_intervals_and_entry_points_far_apart():
    files = [pcrgen.make_jpeg(610 + i, 1, 700, 500, 3, 15.0, 2, 2, 90, restart=12 if i % 2 else 0) for i in range(4)]
    assert (_both(pcrgen.write_record(files), {1: YES, 5: YES}, check=(0, 1)) == 0).all()
    assert (_both(pkg.record_write_indexed(files, None, 4096), {1: YES, 2: YES, 5: YES}, check=(0, 1)) == 0).all()


def test_one_long_scan_takes_a_thousand_lanes():
    files = [pcrgen.make_jpeg(640, 2, 1100, 1000, 3, 30.0, 1, 1, 97)]
    assert (_both(pcrgen.write_record(files), {1: YES, 4: WIDE, 5: WIDE}, check=(0,)) == 0).all()


def test_upgrades_start_from_what_it_left():
    rec = pcrgen.write_record([pcrgen.make_jpeg(660 + i, 1, 300 + 20 * i, 280, 3, 18.0, 2, 2, 90) for i in range(3)])
    with pkg.pcr_open(rec, 0) as r:
        for k0, k, took in ((1, 2, [NO, YES]), (1, 5, [NO, YES]), (2, 5, [NO, YES]), (3, 10, [NO, NO]), (5, 7, [YES, NO])):
            r.decode_batch(k0)
            assert r.last_first_splits() == took[0], k0
            got = r.upgrade_batch(k).cpu().numpy().copy()
            assert r.last_first_splits() == took[1], (k0, k)
            assert np.array_equal(got, r.decode_batch(k).cpu().numpy()), (k0, k)


@pytest.mark.parametrize("seed", range(4))
def test_damaged_data_flag_the_same_images(seed):
    """Bytes changed, dropped and put in behind the first scans' headers; scans cut short; both decoders flag the same images and
    agree on the others."""
    rng = np.random.default_rng(70 + seed)
    files = []
    for i in range(8):
        f = bytearray(pcrgen.make_jpeg(680 + i, 1, 260, 200 + 11 * i, 3, 20.0, 2 - i % 2, 2 - i % 2, 90))
        ends = pcrgen.split_scans(bytes(f))
        g = int(rng.integers(0, 5))
        at = int(rng.integers(ends[g] - (ends[g] - (ends[g - 1] if g else 0)) // 3, ends[g] - 4))
        kind = (i + seed) % 4
        if kind == 0:
            f[at] = f[at] ^ 0x55 if f[at] not in (0xFF, 0xAA) and f[at - 1] != 0xFF else f[at]
        elif kind == 1:
            del f[at:ends[g]]
        elif kind == 2:
            f[at:at] = bytes(rng.integers(0, 255, 9, dtype=np.uint8))
        files.append(bytes(f))
    _both(pcrgen.write_record(files), {1: NO, 2: NO, 5: YES})


def test_entries_out_of_order_flag_their_images_only():
    """An entry that lies beyond its scan flags its image while other workgroups of the launch begin with the image's other units: both
    decoders flag the same images, blank them and agree on the others."""
    files = [pcrgen.make_jpeg(700 + i, 1, 600 - 9 * i, 480 + 7 * i, 3, 18.0, 2, 2, 90) for i in range(12)]
    good = pkg.record_write_indexed(files, None, 1024)
    bad = bytearray(good)
    hit = {1: 0, 4: 1, 5: 4, 8: 1, 11: 4}                      # image: the scan whose entry is moved
    for i, g in hit.items():
        at, _ = _entry_at(good, g, i, 1)
        bad[at:at + 4] = (10 ** 9).to_bytes(4, "little")
    for k in (1, 2, 5):
        st = _both(bytes(bad), {k: YES})
        assert sorted(np.flatnonzero(st)) == sorted(i for i, g in hit.items() if g < k), k
    with pkg.pcr_open(bytes(bad), 0) as b, pkg.pcr_open(good, 0) as r:
        lay, want, got = r.output_layout(), r.decode_batch(5).cpu().numpy(), b.decode_batch(5).cpu().numpy()
        for i in range(len(files)):
            a, e = int(lay[i]), int(lay[i + 1])
            assert not got[a:e].any() if i in hit else np.array_equal(got[a:e], want[a:e]), i


@pytest.mark.parametrize("contrast", [1, 8])
def test_dc_scans_of_many_bits_a_block(contrast):
    """DC scans that fall into step and DC scans that do not (the wavefronts decode those), with and without AC scans beside them: the
    bytes of the wavefront decoders."""
    rng = np.random.default_rng(31)
    base = [np.kron(rng.integers(0, 256, (40, 50, 3)), np.ones((8, 8, 1))) for _ in range(2)]
    files = [pcrgen.encode_pixels(np.clip((b - 128) * contrast / 8 + 128, 0, 255).astype(np.uint8), 2, 2, 90) for b in base] * 12
    with pkg.pcr_open(pkg.record_write(files), 0) as r:
        for k in (1, 2, 5):
            out = []
            for mode in (0, -1):
                r.set_lane_decoders(mode)
                st = torch.full((r.n,), 77, dtype=torch.int32, device="cuda")
                out.append(r.decode_batch(k, status=st).clone())
                assert (st.cpu().numpy() == 0).all()
                assert r.last_first_splits() == (YES if mode == 0 and (contrast == 1 or k == 5) else NO), (k, mode)
            assert torch.equal(*out), k
