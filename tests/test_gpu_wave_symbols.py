"""The wavefront decoders' symbol loops where they can go wrong: runs that end on the band's last zero, on its last position, on the
sixty-third table entry; sixteen zeros and more; end-of-band runs; blocks with no zero left; codes of every length up to the
ones neither look-up resolves; bands of one position.  Coefficients against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1911_00472_amd as pkg
import pcrgen

pytestmark = pytest.mark.gpu

W, H = 152, 120
BANDS = {"whole": [(1, 63)], "first two": [(1, 2), (3, 63)], "last two": [(1, 61), (62, 63)], "one": [(1, 4), (5, 5), (6, 63)]}
ZZ = np.array([0, 1, 8, 16, 9, 2, 3, 10, 17, 24, 32, 25, 18, 11, 4, 5, 12, 19, 26, 33, 40, 48, 41, 34, 27, 20, 13, 6, 7, 14, 21, 28, 35, 42, 49,
               56, 57, 50, 43, 36, 29, 22, 15, 23, 30, 37, 44, 51, 58, 59, 52, 45, 38, 31, 39, 46, 53, 60, 61, 54, 47, 55, 62, 63])


def _blocks(kind, rng, n):
    c = np.zeros((n, 64), np.int64)
    if kind == "one position":                                # every run length, up to the last position
        c[np.arange(n), 1 + np.arange(n) % 63] = rng.choice([-5, -3, -2, -1, 1, 2, 3, 4], n)
    elif kind == "all but one":                               # history almost everywhere; the one zero left moves through the band
        c[:, 1:] = rng.choice([-6, -4, 4, 7], (n, 63))
        c[np.arange(n), 1 + np.arange(n) % 63] = rng.choice([-1, 0, 1], n)
    elif kind == "no zero":
        c[:, 1:] = rng.choice([-7, -5, 4, 9], (n, 63))
    elif kind == "all new":                                   # sixty-three coefficients of one, table entries 1 .. 63
        c[:, 1:] = rng.choice([-1, 1], (n, 63))
    elif kind == "sixteen":                                   # runs of 15, 16, 17, 32, 48 zeros, with and without history inside
        for i, p in enumerate(rng.choice([16, 17, 18, 33, 34, 49, 50, 63], (n, 2))):
            c[i, p] = rng.choice([-1, 1])
            if i % 2:
                c[i, 1 + rng.integers(0, 63)] = 4
    elif kind == "mostly nothing":
        c[::7, 1 + rng.integers(0, 63)] = rng.choice([-2, -1, 1, 2], len(c[::7]))
    else:                                                     # "every symbol": sizes and runs of falling frequency, codes of up to 16 bits
        for i in range(n):
            p = 0
            while True:
                p += 1 + min(int(rng.geometric(0.35)) - 1, 40)
                if p > 63:
                    break
                s = min(int(rng.geometric(0.45)), 10)
                c[i, p] = int(rng.integers(1 << (s - 1), 1 << s)) * int(rng.choice([-1, 1]))
    c[:, 0] = rng.integers(-200, 200, n)
    out = np.zeros_like(c)
    out[:, ZZ] = c
    return out.astype(np.int16)


KINDS = ["one position", "all but one", "no zero", "all new", "sixteen", "mostly nothing", "every symbol"]


def _check(files, ks, lanes):
    rec = pcrgen.write_record(files)
    with pkg.pcr_open(rec, 0) as r:
        r.set_lane_decoders(lanes)
        for k in ks:
            got, lay = r.decode_coefficients(k).cpu().numpy(), r.coef_layout()
            for i in range(r.n):
                want, _, _ = oracle.decode_record_image(rec, i, k)
                assert np.array_equal(got[int(lay[i]):int(lay[i + 1])], want), (KINDS[i % len(KINDS)], k)


@pytest.mark.parametrize("band", sorted(BANDS))
@pytest.mark.parametrize("restart", [0, 3])
def test_progressive(band, restart):
    q, rng = np.ones((2, 64), np.uint16), np.random.default_rng(len(band))
    script = [(1, 0, 0, 0, 0, 0, 0, 0)] + [(1, 0, 0, 0, a, b, 0, 2) for a, b in BANDS[band]]
    script += [(1, 0, 0, 0, a, b, h, h - 1) for h in (2, 1) for a, b in BANDS[band]]
    n = pcrgen.plane_blocks(W, H, 1, 1, 1)[0]
    files = [pcrgen.encode_coefs(_blocks(kind, rng, n).reshape(-1), W, H, 1, 1, 1, q, script, restart) for kind in KINDS]
    _check(files, [2, len(BANDS[band]) + 1, len(script) - 1, len(script)], 0)


@pytest.mark.parametrize("restart", [0, 3])
def test_sequential(restart):
    """Tables that differ between the components of an MCU: the words of a window are looked up again inside it."""
    q, rng = np.ones((2, 64), np.uint16), np.random.default_rng(4)
    n = pcrgen.plane_blocks(W, H, 3, 2, 1)
    files = [pcrgen.encode_coefs(np.concatenate([_blocks(KINDS[(i + j) % len(KINDS)], rng, m).reshape(-1) for j, m in enumerate(n)]), W, H, 3, 2, 1, q, "sequential", restart)
             for i in range(len(KINDS))]
    _check(files, [1], 0)
