"""Long sequential scans, decoded by many lanes per scan -- in steps (k_sequential_split) and by tries (k_split_tries and what follows) -- and by one
wavefront, against the oracle: around the length many lanes are taken from, gray and every sampling layout, several scans per file, streams that
never fall into step (left to the one-wavefront decoder), codes of the greatest lengths, damaged and truncated data."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen
from jpeg_files import planar_sequential

pytestmark = pytest.mark.gpu


def _noise(seed, w, h, c, low=0, high=256):
    return np.random.default_rng(seed).integers(low, high, (h, w, c), dtype=np.uint8)


AUTO, ONE, STEPS, TRIES = 0, 1, 2, 3


def _coefficients(rec, mode=AUTO, took=None):
    """took(by, tries, steps, left, rounds by tries, rounds in steps): what is to be said of the decode's route."""
    with pkg.pcr_open(rec, 0) as r:
        r.set_sequential_decoders(mode)
        st = torch.empty(r.n, dtype=torch.int32, device="cuda")
        pix = r.decode_batch(r.G, status=st).cpu().numpy()
        route = r.last_sequential_decoders()
        assert mode == AUTO or route[0] == (mode if sum(route[1:4]) else ONE), (mode, route)
        assert took is None or took(*route), route
        return r.decode_coefficients(r.G).cpu().numpy(), r.coef_layout(), st.cpu().numpy(), pix, r.output_layout()


def _check(files, **took):
    """Every decoder, whatever would be chosen; took: by the name of the mode, what is to be said of its route."""
    rec = pcrgen.write_record(files)
    want = [oracle.decode_record_image(rec, i, oracle.record_header(rec)["G"])[0] for i in range(len(files))]
    for mode, name in enumerate(("auto", "one", "steps", "tries")):
        coef, lay, st, _, _ = _coefficients(rec, mode, took.get(name))
        assert (st == 0).all(), name
        for i in range(len(files)):
            assert np.array_equal(coef[int(lay[i]):int(lay[i + 1])], want[i]), (name, i)


@pytest.mark.parametrize("c,hs,vs", [(1, 1, 1), (3, 1, 1), (3, 2, 1), (3, 1, 2), (3, 2, 2)])
def test_sizes_around_the_line_and_every_layout(c, hs, vs):
    files = [pcrgen.encode_pixels(_noise(10 * s + c, s, s + 3, c), hs, vs, q, "sequential", restart=0)
             for s, q in [(8, 90), (40, 60), (45, 90), (52, 92), (61, 96), (150, 75), (233, 97)]]
    files += [pcrgen.encode_pixels(pcrgen.synth(77 + i, 1 + i % 2, 300 + 37 * i, 280, c, 4.0 + 9 * i), hs, vs, 85, "sequential", restart=0) for i in range(3)]
    assert min(map(len, files)) < 1500 and sum(len(f) > 2600 for f in files) >= 5
    _check(files)


def test_streams_that_do_not_fall_into_step_and_several_scans():
    flat = np.full((1024, 1024, 3), 90, np.uint8)
    half = flat.copy()
    half[:500] = _noise(1, 1024, 500, 3)
    stripes = np.tile(np.arange(64, dtype=np.uint8)[None, :, None] * 3, (640, 10, 1))
    files = [pcrgen.encode_pixels(flat, 2, 2, 90, "sequential", restart=0), pcrgen.encode_pixels(half, 2, 2, 60, "sequential", restart=0),
             pcrgen.encode_pixels(stripes, 1, 1, 95, "sequential", restart=0), pcrgen.encode_pixels(_noise(5, 250, 250, 3), 2, 2, 100, "sequential", restart=40)]
    _check(files)
    _check([planar_sequential(5, 200, 170, 95), planar_sequential(6, 64, 64, 90)])


def test_who_decodes_what():
    """Streams that fall into step with no more than the tries, with pieces decoded on, in some rounds of steps; that steps give up early and that use up the
    room of the tries."""
    photo = pcrgen.synth(3, 2, 500, 440, 3, 26.0)
    flat = np.full((2048, 2048, 3), 90, np.uint8)
    _check([pcrgen.encode_pixels(photo, 2, 2, 90, "sequential")], auto=lambda by, t, s, left, rt, rs: by == TRIES and (t, left) == (1, 0) and rt >= 1,
           steps=lambda by, t, s, left, rt, rs: (s, left) == (1, 0) and rs >= 8, one=lambda by, *n: by == ONE and sum(n) == 0)
    _check([pcrgen.encode_pixels(flat, 2, 2, 90, "sequential")], tries=lambda by, t, s, left, rt, rs: (t, left, rt) == (1, 0, 0), steps=lambda by, t, s, left, *r: (s, left) == (0, 1))
    _check([pcrgen.encode_pixels(pcrgen.synth(3, 2, 500, 440, 1, 26.0), 1, 1, 90, "sequential")], auto=lambda by, t, s, left, *r: by == STEPS and (s, left) == (1, 0))
    _check([pcrgen.encode_pixels(_noise(5, 250, 250, 3), 2, 2, 100, "sequential")], steps=lambda by, t, s, left, *r: (s, left) == (0, 1), tries=lambda by, t, s, left, *r: (t, s, left) == (0, 0, 1))
    _check([planar_sequential(5, 200, 170, 95)], auto=lambda by, t, s, left, *r: by == STEPS and (s, left) == (3, 0), tries=lambda by, t, s, left, *r: (t, left) == (3, 0))


@pytest.mark.parametrize("hs,vs,quality,noise,side,by", [(2, 2, 75, 8.0, 600, {16: TRIES, 200: STEPS}), (2, 1, 90, 20.0, 325, {64: TRIES, 300: STEPS}), (2, 2, 90, 26.0, 255, {64: TRIES, 300: TRIES})])
def test_many_scans_of_few_bits_a_block_go_in_steps(hs, vs, quality, noise, side, by):
    """Where the steps were measured to be faster, and where not."""
    files = [pcrgen.encode_pixels(pcrgen.synth(3 + i, 2, side, side - 5, 3, noise), hs, vs, quality, "sequential", restart=0) for i in range(8)]
    for n, want in by.items():
        with pkg.pcr_open(pcrgen.write_record([files[i % 8] for i in range(n)]), 0) as r:
            st = torch.empty(n, dtype=torch.int32, device="cuda")
            a = r.decode_coefficients(r.G) if n == min(by) else None
            r.decode_batch(r.G, status=st)
            route = r.last_sequential_decoders()
            assert route[0] == want and route[3] == 0 and not st.any(), (n, route)
            if a is not None:
                r.set_sequential_decoders(ONE)
                assert torch.equal(a, r.decode_coefficients(r.G))


@pytest.mark.parametrize("sub", [1, 2])
def test_blocks_of_very_many_bits_go_in_steps(sub):
    """Noise at quality 100: what is to be decoded on outgrows the room of the tries, and one wavefront takes four times as long as the steps.  Alone; asked to go by
    tries all the same; beside pictures that do."""
    dense = pcrgen.encode_pixels(pcrgen.synth(3, 2, 800, 800, 3, 10.0), sub, sub, 100, "sequential")
    usual = [pcrgen.encode_pixels(pcrgen.synth(9 + i, 2, 500, 440, 3, 26.0), sub, sub, 90, "sequential") for i in range(3)]
    assert len(dense) > 800000
    _check([dense], auto=lambda by, t, s, left, *r: by == STEPS and (t, s, left) == (0, 1, 0), tries=lambda by, t, s, left, *r: (t, s, left) == (0, 1, 0))
    _check(usual[:2] + [dense] + usual[2:], auto=lambda by, t, s, left, *r: by != ONE and left == 0, tries=lambda by, t, s, left, *r: (t, s, left) == (3, 1, 0))


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("n,w,h,restart", [(300, 260, 250, 0), (40, 700, 640, 900)])
def test_the_tries_work_in_memory_the_record_was_opened_with(n, w, h, restart):
    files = [pcrgen.encode_pixels(pcrgen.synth(60 + i, 2, w, h, 3, 18.0), 2, 2, 92, "sequential", restart=restart) for i in range(4)]
    rec = pcrgen.write_record([files[i % 4] for i in range(n)])
    for _ in range(2):                                       # (the first time round the kernels are loaded)
        with pkg.pcr_open(rec, 0) as r:
            out, st = torch.empty(int(r.output_layout()[-1]), dtype=torch.uint8, device="cuda"), torch.empty(r.n, dtype=torch.int32, device="cuda")
            before = _free()
            r.decode_batch(1, out, st)
            after = _free()
            by, tries, steps, left, _, _ = r.last_sequential_decoders()
            assert by == TRIES and tries >= n and not steps and not left and not st.any()
    assert after == before


@pytest.mark.parametrize("mode", [ONE, STEPS, TRIES])
def test_damaged_data_flag_their_image_only(mode):
    files = [pcrgen.encode_pixels(_noise(900 + i, 150, 141, 3), 2, 2, 90, "sequential", restart=0) for i in range(4)]
    rec = pcrgen.write_record(files)
    _, _, st, pix, lay = _coefficients(rec, mode)
    assert (st == 0).all()
    with pkg.pcr_open(rec, 0) as r:
        off, length = r.index()
    o, n = int(np.asarray(off).reshape(-1)[2]), int(np.asarray(length).reshape(-1)[2])
    flagged = 0
    for name, at, fill in [("cut", n - 400, b"\xff\xd9" + bytes(398)), ("ones", n // 2, b"\xff\x00" * 100), ("zeros", n // 2, bytes(200)), ("noise", n // 3, None)]:
        bad = bytearray(rec)
        data = fill if fill is not None else bytes(x & 0x7F for x in np.random.default_rng(3).integers(0, 256, 200, dtype=np.uint8))
        bad[o + at:o + at + len(data)] = data
        coef, clay, st, p, _ = _coefficients(bytes(bad), mode)
        _, _, one, _, _ = _coefficients(bytes(bad), ONE)
        assert np.array_equal(st != 0, one != 0), name
        assert (np.delete(st, 2) == 0).all(), name
        flagged += int(st[2] != 0)
        for i in (0, 1, 3):
            assert np.array_equal(p[int(lay[i]):int(lay[i + 1])], pix[int(lay[i]):int(lay[i + 1])]), (name, i)
        if st[2] == 0:
            want, _, _ = oracle.decode_record_image(bytes(bad), 2, 1)
            assert np.array_equal(coef[int(clay[2]):int(clay[3])], want), name
    assert flagged >= 2


@pytest.mark.parametrize("mode", [ONE, STEPS, TRIES])
@pytest.mark.parametrize("scan", [0, 1, 2])
def test_one_damaged_scan_of_several(scan, mode):
    """Workgroups that decode an image's other scans begin and end around the one that flags it: that image is flagged and blank,
    the others are as they were."""
    files = [planar_sequential(20 + i, 420, 333, 95) for i in range(6)]
    rec = pcrgen.write_record(files)
    with pkg.pcr_open(rec, 0) as r:
        G, (off, length) = r.G, r.index()
    _, _, st, pix, lay = _coefficients(rec, mode)
    assert G == 3 and (st == 0).all() and int(np.asarray(length).min()) * 8 > 65536
    bad = bytearray(rec)
    for i in (1, 3, 4):
        at = int(np.asarray(off).reshape(G, -1)[scan][i]) + int(np.asarray(length).reshape(G, -1)[scan][i]) - 3000
        bad[at:at + 2998] = b"\xff\xd9" + bytes(2996)           # (the data end early)
    # (the streams but for their ends are whole: they fall into step, and it is the lanes that store that see the data end)
    _, _, st, p, _ = _coefficients(bytes(bad), mode, lambda by, t, s, left, *r: left == 0)
    assert [int(v != 0) for v in st] == [0, 1, 0, 1, 1, 0]
    for i in range(6):
        got, want = p[int(lay[i]):int(lay[i + 1])], pix[int(lay[i]):int(lay[i + 1])]
        assert not got.any() if st[i] else np.array_equal(got, want), i


@pytest.mark.parametrize("quality,noise,sub,side", [(97, 16.0, 2, 240), (100, 40.0, 1, 240), (100, 8.0, 2, 120), (100, 40.0, 2, 800), (97, 16.0, 1, 120)])
def test_high_qualities_at_which_the_rounds_are_given_up_early_or_go_on_to_the_end(quality, noise, sub, side):
    _check([pcrgen.encode_pixels(pcrgen.synth(3 + i, 2, side, side, 3, noise), sub, sub, quality, "sequential") for i in range(2)])


@pytest.mark.parametrize("others", [0, 3])
def test_more_long_scans_than_the_split_pays_for(others):
    """Too many files at a time for a workgroup each (alone from some 700 of this size on, sooner beside other records that
    are open): the one-wavefront decoder takes them all, with the same coefficients."""
    distinct = [pcrgen.encode_pixels(pcrgen.synth(60 + i, 2, 130 + i, 121, 3, 18.0), 2, 2, 92, "sequential", restart=0) for i in range(8)]
    assert min(map(len, distinct)) * 8 > 65536
    open_beside = [pkg.pcr_open(pcrgen.write_record(distinct), 0) for _ in range(others)]
    for n in (8, 250, 1100):
        rec = pcrgen.write_record([distinct[i % 8] for i in range(n)])
        coef, lay, st, _, _ = _coefficients(rec, took=lambda by, *r: by == (TRIES if n * (1 + others) <= 250 else ONE))
        assert (st == 0).all()
        want = [oracle.decode_record_image(rec, i, 1)[0] for i in range(8)]
        for i in range(n):
            assert np.array_equal(coef[int(lay[i]):int(lay[i + 1])], want[i % 8]), (n, i)
    for r in open_beside:
        r.close()


@pytest.mark.parametrize("n,w,h,c,hs,vs,quality,noise,restart", [
    (3, 97, 90, 3, 2, 2, 95, 20.0, 0), (2, 640, 600, 3, 2, 1, 90, 14.0, 0), (1, 2000, 1500, 3, 2, 2, 92, 20.0, 0), (2, 900, 700, 3, 1, 1, 97, 30.0, 0),
    (2, 700, 640, 3, 1, 2, 90, 18.0, 900), (2, 1024, 1024, 3, 2, 2, 90, 0.0, 0), (1, 300, 300, 3, 2, 2, 97, 40.0, 0), (2, 500, 500, 1, 1, 1, 92, 26.0, 0)])
def test_few_scans_by_tries(n, w, h, c, hs, vs, quality, noise, restart):
    """Few scans, which go by tries: from a few pieces to as many as a scan is cut into, pieces of several workgroups, units between
    restart markers, every sampling layout; noise at a high quality, of which most pieces fall in with no try; pictures that hold next to nothing."""
    _check([pcrgen.encode_pixels(pcrgen.synth(31 + i, 2, w + 16 * i, h - 9 * i, c, noise), hs, vs, quality, "sequential", restart=restart) for i in range(n)],
           auto=lambda by, *r: by == (TRIES if c == 3 else STEPS), tries=lambda by, t, s, left, *r: t >= n and left == 0)
