"""The paper's encoding step end to end (Section 5, "Encoding"): baseline files -> coefficients decoded on the
device -> progressive files -> one record; the record then decodes, on the device, to the pictures of the
baseline files, and at every scan group to what the oracle makes of it."""
import numpy as np
import pytest

import oracle
import paper_1911_00472_amd as pkg
from test_gpu_parity import _check_record, _sequential_files

pytestmark = pytest.mark.gpu


def test_baseline_files_become_a_progressive_record():
    import torch
    assert torch.cuda.is_available()
    files = _sequential_files()
    prog = pkg.transcode_files(files)
    labels = list(range(len(files)))
    rec_b, rec_p = pkg.record_write(files, labels), pkg.record_write(prog, labels)
    assert oracle.record_header(rec_b)["G"] == 1 and oracle.record_header(rec_p)["G"] == 10
    with pkg.pcr_open(rec_b, 0) as rb, pkg.pcr_open(rec_p, 0) as rp:
        assert [rb.image_info(i) for i in range(rb.n)] == [rp.image_info(i) for i in range(rp.n)]
        a = rb.decode_batch(1).cpu().numpy()
        b = rp.decode_batch(10).cpu().numpy()
        assert np.array_equal(a, b)                               # lossless: the same coefficients give the same pixels
    _check_record(rec_p, (1, 2, 5, 7, 10))
    # a progressive source goes through unchanged in content as well
    again = pkg.transcode_files(prog[:3])
    for f0, f1 in zip(prog[:3], again):
        assert f0 == f1


def test_restart_intervals_written_by_the_transcoder_decode_the_same():
    """The transcoder's restart markers split every scan into streams of their own; the pictures do not change."""
    import torch
    assert torch.cuda.is_available()
    files = _sequential_files()
    rec_b = pkg.record_write(files)
    with pkg.pcr_open(rec_b, 0) as rb:
        want = rb.decode_batch(1).cpu().numpy()
    for ri in (5, 64):
        prog = pkg.transcode_files(files, restart_interval=ri)
        rec_p = pkg.record_write(prog)
        with pkg.pcr_open(rec_p, 0) as rp:
            assert np.array_equal(rp.decode_batch(10).cpu().numpy(), want)
        _check_record(rec_p, (1, 6, 10), check_bytes=False)


def test_symbol_histograms_on_the_device(rgb_small, gray64, extreme_record):
    """pcr_symbol_histograms against the host coder's own counts, symbol by symbol: 4:2:0 with odd sizes, gray, 4:4:4 and
    4:2:2, baseline sources, the hand-made extreme planes (dense blocks, zero runs inside refinement scans, end-of-band
    runs over hundreds of blocks), a run of more than 32767 empty blocks, with and without restart intervals; and the
    files written from the device's counts are the files written without them."""
    import pcrgen
    import torch
    assert torch.cuda.is_available()
    pix = np.full((1456, 1464, 1), 97, np.uint8)
    pix[:8, :8, 0] = np.arange(64, dtype=np.uint8).reshape(8, 8) * 3
    long_run = pcrgen.encode_pixels(pix, 1, 1, 90, "sequential")
    shapes = [(33, 17), (64, 64), (100, 9)]
    sets = [list(rgb_small[1][:10]), None, list(extreme_record[1]), _sequential_files()[:6], [long_run],
            [pcrgen.make_jpeg(700 + i, 1, w, h, 3, 6.0, hs, vs, 90) for i, (w, h) in enumerate(shapes) for (hs, vs) in ((1, 1), (2, 1))]]
    for si, files in enumerate(sets):
        rec = gray64[0] if files is None else pkg.record_write(files)
        with pkg.pcr_open(rec, 0) as r:
            if files is None:
                files = [r.reassemble(i, r.G) for i in range(r.n)]
            lay = r.coef_layout()
            coef = r.decode_coefficients(r.G).cpu().numpy()
            for ri in ((0, 7) if si != 4 else (0,)):
                got = r.symbol_histograms(ri).cpu().numpy().astype(np.uint32)
                assert got.shape == (r.n, 10, 2, 256)
                for i in range(r.n):
                    want = pkg.transcode_symbol_counts(files[i], coef[int(lay[i]):int(lay[i + 1])], ri)
                    assert np.array_equal(got[i], want), (si, i, ri, np.argwhere(got[i] != want)[:5])
            assert r.resident_scan_group() == 0
    files = _sequential_files()[:5] + list(rgb_small[1][:3])
    for ri in (0, 9):
        assert pkg.transcode_files(files, restart_interval=ri) == pkg.transcode_files(files, restart_interval=ri, device_counts=False)


@pytest.mark.parametrize("name", ["tiny", "edges", "dense", "runs", "mixed"])
def test_device_coder_writes_the_host_coders_files(name, extreme_record):
    """pcr_coder.h against pcr_encode.h, byte for byte: pictures of one block, of 512 blocks and one more or fewer (a workgroup's
    turn), noise at quality 100 (more bits per turn than its words in LDS hold), end-of-band runs over several turns and beyond
    32767 blocks, and planes of every kind in one batch."""
    import pcrgen
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(5)

    def noise(w, h, nc, quality=100):
        return pcrgen.encode_pixels(rng.integers(0, 256, (h, w, nc)).astype(np.uint8), 1, 1, quality, "sequential")

    def spot(w, h, *at):                                    # flat but for a few blocks
        pix = np.full((h, w, 1), 120, np.uint8)
        for x, y in at:
            pix[y:y + 8, x:x + 8, 0] = np.arange(64, dtype=np.uint8).reshape(8, 8) * 3
        return pcrgen.encode_pixels(pix, 1, 1, 90, "sequential")

    if name == "tiny":
        files = [noise(1, 1, 1), noise(1, 1, 3), noise(8, 8, 3), noise(9, 7, 1), spot(8, 8)]
    elif name == "edges":
        files = [pcrgen.make_jpeg(40 + i, 1, w, h, nc, 9.0, s, s, 90) for i, (w, h, nc, s) in enumerate(
            [(512, 64, 1, 1), (504, 64, 1, 1), (520, 64, 1, 1), (512, 64, 3, 1), (513, 65, 3, 2), (1024, 64, 3, 2), (4104, 8, 1, 1), (8, 4104, 3, 1)])]
    elif name == "dense":
        files = [noise(256, 256, 1), noise(200, 190, 3), noise(512, 72, 3, 97)]
    elif name == "runs":
        files = [spot(1464, 1456, (0, 0)), spot(1464, 1456), spot(1464, 1456, (800, 0), (1456, 1448)), spot(1472, 2960, (0, 0), (1464, 2952)), spot(512, 128, (504, 56), (0, 64))]
    else:
        files = _sequential_files()[:4] + list(extreme_record[1])[:4] + [noise(40, 30, 3), spot(640, 64, (632, 56))]
    got, want = pkg.transcode_files(files), pkg.transcode_files(files, device_counts=False)
    for i, (a, b) in enumerate(zip(got, want)):
        assert a == b, (name, i, len(a), len(b))


@pytest.mark.parametrize("device_counts", [1, 0])
def test_files_there_is_no_room_for_are_not_written(device_counts):
    """Room of exactly a file's size, one byte less, hardly any and none: what fits is whole, of the rest nothing is written, and the sizes
    of all come back."""
    import ctypes
    import pcrgen
    from paper_1911_00472_amd import binding as B
    files = [pcrgen.make_jpeg(80 + i, i % 3, 90 + 7 * i, 60, 3 if i % 4 else 1, 14.0, 1, 1, 92) for i in range(8)]
    want = pkg.transcode_files(files)
    short = [0, 1, 0, len(want[3]) - 20, 0, 2, len(want[6]), 700]
    room = [len(w) - s for w, s in zip(want, short)]
    off = np.concatenate([[0], np.cumsum(room)]).astype(np.uint64)
    out = np.full(int(off[-1]), 0xA5, np.uint8)
    written = np.zeros(len(files), np.uint64)
    bufs, ptrs, sizes = B._file_table(files)
    with pkg.pcr_open(pkg.record_write(files), 0) as r:
        rc = B.lib().pcr_transcode_batch(r._h, ptrs, sizes, len(files), 0, device_counts, 4, out.ctypes.data_as(ctypes.c_void_p), off.ctypes.data_as(ctypes.c_void_p),
                                         written.ctypes.data_as(ctypes.c_void_p), None)
    assert rc == pkg.E_RANGE and written.tolist() == [len(w) for w in want]
    for i, w in enumerate(want):
        got = out[int(off[i]):int(off[i + 1])].tobytes()
        assert got == (w if short[i] == 0 else b"\xa5" * room[i]), i
