"""The device's marker parser and table builder (k_headers) against the host's parser (pcr_open) and the oracle: header
variants, long segments ahead of the tables, tables taken over from earlier regions, many scans, small and large records
(the offsets of the regions come from the same kernel or from k_index), damaged headers."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_00472_amd as pkg
import pcrgen

pytestmark = pytest.mark.gpu


def _device_record(rec):
    a = np.frombuffer(rec, np.uint8)
    return torch.from_numpy(np.concatenate([a, np.zeros((-len(a)) % 64, np.uint8)])).cuda()[:len(a)]


def _same(rec, images=None):
    """Every scan group of the record opened both ways, against each other and the oracle."""
    with pkg.pcr_open(rec, 0) as a, pkg.pcr_open_device(_device_record(rec)) as b:
        assert np.array_equal(a.output_layout(), b.output_layout()) and np.array_equal(a.coef_layout(), b.coef_layout())
        lay, clay = a.output_layout(), a.coef_layout()
        for k in range(1, a.G + 1):
            ca, cb = a.decode_coefficients(k).cpu().numpy(), b.decode_coefficients(k).cpu().numpy()
            pa, pb = a.decode_batch(k).cpu().numpy(), b.decode_batch(k).cpu().numpy()
            assert np.array_equal(ca, cb) and np.array_equal(pa, pb), k
            for i in (range(a.n) if images is None else images):
                c0, p0, info = oracle.decode_record_image(rec, i, k)
                assert np.array_equal(ca[int(clay[i]):int(clay[i + 1])], c0), (i, k)
                assert np.abs(pa[int(lay[i]):int(lay[i + 1])].astype(int) - p0.reshape(-1)).max() <= 1, (i, k)


@pytest.mark.parametrize("comment", [1, 900, 1023, 5000])
def test_segments_longer_than_the_staged_window(comment):
    """A comment ahead of the tables pushes them across, or wholly past, the bytes staged on the chip."""
    base = pcrgen.make_jpeg(3, 1, 57, 41, 3, 8.0, 2, 2, 90)
    seg = b"\xff\xfe" + (comment + 2).to_bytes(2, "big") + bytes((7 * j) & 0x7F for j in range(comment))
    ends = pcrgen.split_scans(base)
    first = base[:2] + seg + base[2:]
    later = base[:ends[3]] + seg + base[ends[3]:]
    _same(pcrgen.write_record([first, later, base]))


def _table_moved_to_the_front(f, scan, slot):
    """The AC table definition of a one-component scan, moved ahead of the frame header under table id `slot`."""
    ends = pcrgen.split_scans(f)
    region = bytearray(f[ends[scan - 1]:ends[scan]])
    assert region[:2] == b"\xff\xc4" and region[4] >> 4 == 1
    size = 2 + int.from_bytes(region[2:4], "big")
    table, rest = bytearray(region[:size]), region[size:]
    assert rest[:2] == b"\xff\xda" and rest[4] == 1
    table[4] = 0x10 | slot
    rest[6] = slot
    return f[:2] + bytes(table) + f[2:ends[scan - 1]] + bytes(rest) + f[ends[scan]:]


def test_tables_defined_in_an_earlier_region():
    """A later scan's table comes from bytes outside its own region (and the ballots find the region that defined it)."""
    files = []
    for i in range(3):
        f = pcrgen.make_jpeg(11 + i, 1, 64 + 9 * i, 40, 3, 6.0, 2, 2, 85)
        files += [_table_moved_to_the_front(f, 4, 2), _table_moved_to_the_front(_table_moved_to_the_front(f, 9, 3), 5, 2)]
    _same(pcrgen.write_record(files))


@pytest.mark.parametrize("n", [1, 512, 513])
def test_region_offsets_of_small_and_large_records(n):
    few = [pcrgen.make_jpeg(40 + i, 1, 9 + i, 17, 3, 6.0, 2, 2, 90) for i in range(5)]
    _same(pcrgen.write_record([few[i % 5] for i in range(n)]), images=sorted({0, 1 % n, n // 2, n - 1}))


def test_damaged_headers_flag_their_image_only():
    """Bytes damaged after the record was opened: the decode's own parse must notice, and touch no other image."""
    files = [pcrgen.make_jpeg(70 + i, 1, 50, 50, 3, 6.0, 2, 2, 90) for i in range(4)]
    rec = pcrgen.write_record(files)
    with pkg.pcr_open(rec, 0) as r:
        offsets, _ = r.index()
        want = r.decode_batch(r.G).cpu().numpy()
        lay = r.output_layout()
    for g, at, value in ((0, 0, 0x00), (0, 2, 0x12), (3, 1, 0xC0), (9, 2, 0xFF)):
        t = _device_record(rec).clone()
        with pkg.pcr_open_device(t) as r:
            t[int(offsets[g, 2]) + at] = value
            status = torch.full((4,), 77, dtype=torch.int32, device="cuda")
            got = r.decode_batch(r.G, status=status).cpu().numpy()
            st = status.cpu().tolist()
        assert st[2] != 0 and st[0] == st[1] == st[3] == 0, (g, at, st)
        for i in range(4):
            part = got[int(lay[i]):int(lay[i + 1])]
            if i != 2:
                assert np.array_equal(part, want[int(lay[i]):int(lay[i + 1])]), (g, at, i)
            elif g > 0:                                        # (without a frame header there is nothing to fill)
                assert not part.any(), (g, at)


@pytest.mark.parametrize("start", [936, 952, 968, 984, 1000])
def test_segments_across_the_end_of_the_staged_window(start):
    """Comments of sixteen lengths in a row ahead of the tables and ahead of a later scan: every segment behind them begins at every
    offset from the end of the staged bytes, and is read half from them and half from memory."""
    files = []
    for comment in range(start, start + 16):
        base = pcrgen.make_jpeg(5, 1, 23, 17, 3, 8.0, 2, 1, 90)
        seg = b"\xff\xfe" + (comment + 2).to_bytes(2, "big") + bytes((5 * j) & 0x7F for j in range(comment))
        ends = pcrgen.split_scans(base)
        at = base.index(b"\xff\xc2")
        files.append(base[:at] + seg + base[at:])
        files.append(base[:ends[2]] + seg + base[ends[2]:])
    _same(pcrgen.write_record(files))


def test_a_refinement_that_builds_on_as_many_scans_as_can_be():
    """Six earlier refinements of a band, the most a scan may build on, and bands that overlap some of them."""
    dc, whole = (1, 0, 0, 0, 0, 0, 0, 0), [(1, 0, 0, 0, 1, 63, 0, 7)] + [(1, 0, 0, 0, 1, 63, a, a - 1) for a in range(7, 0, -1)]
    parts = [(1, 0, 0, 0, 1, 20, 0, 3), (1, 0, 0, 0, 21, 63, 0, 3)] + [(1, 0, 0, 0, lo, hi, a, a - 1) for a in (3, 2) for lo, hi in ((1, 9), (10, 30), (31, 63))]
    parts += [(1, 0, 0, 0, 1, 63, 1, 0)]
    files = [pcrgen.encode_pixels(pcrgen.synth(7 + i, 1, 40 + i, 33, 1, 25.0), 1, 1, 95, [dc] + s) for i, s in enumerate((whole, parts))]
    for f in files:
        _same(pcrgen.write_record([f]))


@pytest.mark.parametrize("n", [1024, 1025, 2048, 2049])
def test_region_offsets_where_the_parser_sums_them_itself(n):
    """The lengths ahead of a region are summed by the parser up to 2048 images for scan groups 1 .. 8 and up to 1024 beyond; else by k_index."""
    few = [pcrgen.make_jpeg(90 + i, 1, 8 + i, 9, 3, 6.0, 1, 1, 80) for i in range(5)]
    _same(pcrgen.write_record([few[i % 5] for i in range(n)]), images=sorted({0, 63, 64, 511, 512, 513, 1023, n // 2, n - 1}))


@pytest.mark.parametrize("n", [1024, 1025, 2048, 2049])
def test_many_small_images(n):
    """Workgroups of eight wavefronts and of four, offsets summed in the kernel and by k_index, at scan groups that need little
    room on the chip and more."""
    sizes = [(8, 8), (17, 9), (24, 30), (9, 33)]
    files = [pcrgen.make_jpeg(60 + i, 1, w, h, 3, 12.0, 2 - i % 2, 2 - i % 2, 88) for i, (w, h) in enumerate(sizes)]
    rec = pcrgen.write_record((files * (n // len(files) + 1))[:n])
    images = [0, 1, 2, 3, n // 2, n - 2, n - 1]
    with pkg.pcr_open(rec, 0) as r:
        lay = r.output_layout()
        for k in (1, 3, 5, 8, 9, 10):
            status = torch.full((n,), 77, dtype=torch.int32, device="cuda")
            got = r.decode_batch(k, status=status).cpu().numpy()
            assert (status.cpu().numpy() == 0).all()
            for i in images:
                _, want, _ = oracle.decode_record_image(rec, i, k)
                assert np.abs(got[int(lay[i]):int(lay[i + 1])].astype(int) - want.reshape(-1)).max() <= 1, (i, k)
            for i in range(n):
                assert np.array_equal(got[int(lay[i]):int(lay[i + 1])], got[int(lay[i % 4]):int(lay[i % 4 + 1])]), (i, k)
