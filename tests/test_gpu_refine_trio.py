"""Refinement scans with three wavefronts a unit (k_decode_trios) against the oracle and against one wavefront a unit, which
set_lane_decoders(-1) keeps to: fewer blocks than a ring holds and many times as many, chains that wait for each other, units cut by
markers and entry points, upgrades, blocks longer than the ring of windows, damaged data; and on both sides of the line
between the two."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen
from test_gpu_wave_symbols import KINDS, _blocks

pytestmark = pytest.mark.gpu

REFINE_ONLY = [(1, 0, 0, 0, 0, 0, 0, 0), (1, 0, 0, 0, 1, 63, 0, 3), (1, 0, 0, 0, 1, 63, 3, 2), (1, 0, 0, 0, 1, 63, 2, 1), (1, 0, 0, 0, 1, 63, 1, 0)]


def _decode(r, k, mode, k0=0):
    r.set_lane_decoders(mode)
    st = torch.full((r.n,), 77, dtype=torch.int32, device="cuda")
    if k0:
        r.decode_batch(k0)
        pix = r.upgrade_batch(k, status=st)
    else:
        pix = r.decode_batch(k, status=st)
    took = r.last_refine_trios()
    return pix.cpu().numpy().copy(), st.cpu().numpy().copy(), took


def _same(rec, ks, check, k0s=(0,), trios=True):
    with pkg.pcr_open(rec, 0) as r:
        lay = r.coef_layout()
        for k in ks:
            for k0 in k0s:
                if k0 >= k:
                    continue
                a, b = _decode(r, k, 0, k0), _decode(r, k, -1, k0)
                assert (a[2] > 0) == trios and b[2] == 0, (k, k0, a[2], b[2])
                assert (a[1] == 0).all() and (b[1] == 0).all() and np.array_equal(a[0], b[0]), (k, k0)
            r.set_lane_decoders(0)
            got = r.decode_coefficients(k).cpu().numpy()
            for i in check:
                want, _, _ = oracle.decode_record_image(rec, i, k)
                assert np.array_equal(got[int(lay[i]):int(lay[i + 1])], want), (k, i)


@pytest.mark.parametrize("size", [(8, 8), (16, 8), (56, 8), (64, 8), (72, 8), (9, 130), (232, 121)])
@pytest.mark.parametrize("cut", [0, 1, -7])                  # a marker every so many MCU rows, or an entry point every so many MCUs
def test_rings_and_units(size, cut):
    """1, 2, 7, 8, 9, 34 and 464 blocks: rings that never fill, that just do, that go round; four scans in a row that wait for each other."""
    w, h = size
    q, rng = np.ones((2, 64), np.uint16), np.random.default_rng(w * h)
    n = pcrgen.plane_blocks(w, h, 1, 1, 1)[0]
    files = [pcrgen.encode_coefs(_blocks(kind, rng, n).reshape(-1), w, h, 1, 1, 1, q, REFINE_ONLY, max(cut, 0)) for kind in KINDS]
    rec = pkg.record_write_indexed(files, None, -cut) if cut < 0 else pcrgen.write_record(files)
    _same(rec, [3, 4, 5], range(len(files)), (0, 2, 4))


def test_color_and_blocks_longer_than_the_ring_of_windows():
    """Sixty-three new coefficients a block with codes of nine bits and more: some twenty windows between two blocks."""
    q, rng = np.ones((2, 64), np.uint16), np.random.default_rng(9)
    nb = pcrgen.plane_blocks(144, 80, 3, 2, 2)
    files = []
    for kind in ("all new", "every symbol", "sixteen"):
        c = np.concatenate([_blocks(kind, rng, n) for n in nb])
        if kind == "all new":                                # codes of run 0, size 1 made rare: half of the blocks hold every other symbol instead
            c[::2] = np.concatenate([_blocks("every symbol", rng, n) for n in nb])[::2]
        files.append(pcrgen.encode_coefs(c.reshape(-1), 144, 80, 3, 2, 2, q, None, 0))
    _same(pcrgen.write_record(files), range(6, 11), range(len(files)), (0, 5, 9))


@pytest.mark.parametrize("firsts,refines,trios", [(4, 4, True), (3, 4, True), (3, 5, False)])
def test_the_widest_chains(firsts, refines, trios):
    """Eight scans of a component, four of them refinement scans: sixteen wavefronts, as many as a workgroup has; with five the chains keep one wavefront a unit."""
    cuts = [1, 6, 21, 41][:firsts] + [64]
    script = [(1, 0, 0, 0, 0, 0, 0, 0)] + [(1, 0, 0, 0, a, b - 1, 0, refines) for a, b in zip(cuts, cuts[1:])] + [(1, 0, 0, 0, 1, 63, l, l - 1) for l in range(refines, 0, -1)]
    q, rng = np.ones((2, 64), np.uint16), np.random.default_rng(firsts)
    n = pcrgen.plane_blocks(120, 72, 1, 1, 1)[0]
    files = [pcrgen.encode_coefs((_blocks(kind, rng, n) * rng.choice([1, 1, 3, 7], (n, 1))).reshape(-1), 120, 72, 1, 1, 1, q, script, r) for kind in KINDS for r in (0, 2)]
    rec = pcrgen.write_record(files)
    G = len(script)
    _same(rec, [G], range(len(files)), trios=trios)
    _same(rec, [G], (0, 3), (1 + firsts,))                    # (an upgrade: the refinement scans alone)
    _same(rec, [G - 1], (0, 3), trios=True)


@pytest.mark.parametrize("entry", [0, 16])
def test_both_sides_of_the_line(entry):
    files = [pcrgen.make_jpeg(40 + i, 1, 72, 56, 1, 8.0, 1, 1, 92) for i in range(8)]
    write = (lambda f: pkg.record_write_indexed(f, None, entry)) if entry else pcrgen.write_record
    _same(write(files * 8), [6], range(8))
    _same(write(files * 256), [6], (0, 1000, 2047), trios=False)


def test_records_open_beside_move_the_line():
    files = [pcrgen.make_jpeg(40 + i, 1, 72, 56, 1, 8.0, 1, 1, 92) for i in range(8)]
    rec = pcrgen.write_record(files * 60)
    _same(rec, [6], range(8))
    others = [pkg.pcr_open(pcrgen.write_record(files[:1]), 0) for _ in range(3)]
    _same(rec, [6], range(8), trios=False)
    for o in others:
        o.close()


def test_damage_is_seen_alike():
    """Streams cut short, overwritten and with bits flipped: the same images are flagged, the others are what they were."""
    rng = np.random.default_rng(3)
    files = [pcrgen.make_jpeg(70 + i, 1, 120, 88, 1, 10.0, 1, 1, 93) for i in range(6)]
    rec = pcrgen.write_record(files)
    with pkg.pcr_open(rec, 0) as r:
        G, lay = r.G, r.output_layout()
        off, length = (np.asarray(v).reshape(G, -1) for v in r.index())
        good = _decode(r, G, 0)
    assert good[2] == 1 and (good[1] == 0).all()
    flagged = 0
    for trial in range(24):
        bad = bytearray(rec)
        i = int(rng.integers(6))
        g = int(rng.choice([g for g in range(1, G) if length[g][i] > 400]))       # (its headers stay whole)
        a, b = int(off[g][i]), int(off[g][i] + length[g][i])
        if trial % 3 == 0:
            at = int(rng.integers(b - (b - a) // 2, b - 3))
            bad[at] ^= 1 << int(rng.integers(7))
            if bad[at] == 0xFF:
                bad[at] = 0x7F
        elif trial % 3 == 1:
            bad[b - 40:b - 2] = bytes([0x55 if trial % 2 else 0x00] * 38)
        else:
            bad[b - 60:b - 2] = bytes(v & 0x7F for v in rng.integers(0, 256, 58, dtype=np.uint8))
        with pkg.pcr_open(bytes(bad), 0) as r:
            x, y = _decode(r, G, 0), _decode(r, G, -1)
        assert np.array_equal(x[1], y[1]), (trial, g, i, x[1], y[1])
        flagged += int(x[1][i] != 0)
        for j in range(6):
            if x[1][j] == 0:
                want = y[0] if j == i else good[0]
                assert np.array_equal(x[0][int(lay[j]):int(lay[j + 1])], want[int(lay[j]):int(lay[j + 1])]), (trial, j)
    assert flagged
