"""The three decoders of long sequential scans -- in steps (k_sequential_split), by tries (k_split_tries and what follows), by one wavefront -- each asked
for and each chosen: the same coefficients and the same status whichever takes a scan, which of them takes what, and what is left by one to
the next."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen
import test_gpu_sequential_split as split
from jpeg_files import planar_sequential
from test_gpu_sequential_split import _noise

pytestmark = pytest.mark.gpu

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


def _cases(test):
    """What a test of the other file is parametrised with."""
    return next(m for m in test.pytestmark if m.name == "parametrize").args


@pytest.fixture(params=[ONE, STEPS, TRIES])
def one_decoder(request, monkeypatch):
    """The tests of the other file with one decoder, and with the status that one wavefront gives."""
    def decode(rec, status=False):
        got = _coefficients(rec, request.param, decode.took)
        assert np.array_equal(got[2] != 0, _coefficients(rec, ONE)[2] != 0)
        return got
    decode.took = None
    monkeypatch.setattr(split, "_coefficients", decode)
    return decode


@pytest.mark.parametrize(*_cases(split.test_sizes_around_the_line_and_every_layout))
def test_every_layout(one_decoder, c, hs, vs):
    split.test_sizes_around_the_line_and_every_layout(c, hs, vs)


def test_streams_that_do_not_fall_into_step(one_decoder):
    split.test_streams_that_do_not_fall_into_step_and_several_scans()


def test_damaged_data(one_decoder):
    split.test_damaged_data_flag_their_image_only()


@pytest.mark.parametrize(*_cases(split.test_one_damaged_scan_of_several))
def test_one_damaged_scan(one_decoder, scan):
    # (the streams but for their ends are whole: they fall into step, and it is the lanes that store that see the data end)
    one_decoder.took = lambda by, t, s, left, *r: left == 0
    split.test_one_damaged_scan_of_several(scan)


@pytest.mark.parametrize(*_cases(split.test_high_qualities_at_which_the_rounds_are_given_up_early_or_go_on_to_the_end))
def test_high_qualities(one_decoder, quality, noise, sub, side):
    split.test_high_qualities_at_which_the_rounds_are_given_up_early_or_go_on_to_the_end(quality, noise, sub, side)


@pytest.mark.parametrize(*_cases(split.test_few_scans_by_tries))
def test_few_scans(n, w, h, c, hs, vs, quality, noise, restart):
    _check([pcrgen.encode_pixels(pcrgen.synth(31 + i, 2, w + 16 * i, h - 9 * i, c, noise), hs, vs, quality, "sequential", restart=restart) for i in range(n)],
           auto=lambda by, *r: by == (TRIES if c == 3 else STEPS), tries=lambda by, t, s, left, *r: t >= n and left == 0)


@pytest.mark.parametrize("others", [0, 3])
def test_more_long_scans_than_many_lanes_pay_for(others):
    distinct = [pcrgen.encode_pixels(pcrgen.synth(60 + i, 2, 130 + i, 121, 3, 18.0), 2, 2, 92, "sequential", restart=0) for i in range(8)]
    open_beside = [pkg.pcr_open(pcrgen.write_record(distinct), 0) for _ in range(others)]
    for n in (8, 250, 1100):
        _coefficients(pcrgen.write_record([distinct[i % 8] for i in range(n)]), took=lambda by, *r: by == (TRIES if n * (1 + others) <= 250 else ONE))
    for r in open_beside:
        r.close()


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
