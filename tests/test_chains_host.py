"""Which scans one launch decodes side by side (pcr_chains.h, compiled for the CPU): two scans of a component whose bands
overlap are never decoded at the same time, unless the later one is a refinement scan of the same chain that waits for the
earlier one -- the symbol loops of first scans wait for nothing."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("chains") / "libchains.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-o", so, os.path.join(HERE, "host_emul", "chains.cpp")])
    lib = ctypes.CDLL(so)

    def run(scans, k0=0, k=None):
        a = np.ascontiguousarray(scans, np.int32).reshape(-1, 8)
        out = np.zeros((len(a), 4), np.int32)
        step = lib.chain_plan(a.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), len(a), k0, len(a) if k is None else k, out.ctypes.data_as(ctypes.POINTER(ctypes.c_int)))
        assert step >= 0
        return bool(step), out
    run.lib = lib
    return run


def _scan(comps, Ss, Se, Ah, Al, ri=0, units=1, entries=0):
    return (comps, Ss, Se, Ah, Al, ri, units, entries)


def _check(scans, out, k0, k):
    for g in range(k0, k):
        for q in range(k0, g):
            a, b = scans[q], scans[g]
            if not (a[0] & b[0]) or a[1] > b[2] or b[1] > a[2] or out[g][0] < 0 or out[q][0] < 0:
                continue
            if out[g][0] != out[q][0]:
                assert out[q][0] < out[g][0], ("the later launch has the earlier scan", q, g)
                continue
            assert out[g][0] == 0 and out[g][1] == out[q][1], ("decoded at the same time", q, g)
            assert b[3] > 0 and b[1] > 0, ("a scan that waits for nothing follows another", q, g)
            assert out[q][2] < out[g][2] and out[g][3] >> out[q][2] & 1, ("does not wait", q, g)


DC, LUMA = _scan(1, 0, 0, 0, 0), [_scan(1, 1, 5, 0, 2), _scan(1, 6, 63, 0, 2), _scan(1, 1, 63, 2, 1), _scan(1, 1, 63, 1, 0)]
FILES = {
    "usual": ([DC] + LUMA, True),
    "interleaved": ([_scan(7, 0, 0, 0, 1), _scan(1, 1, 5, 0, 2), _scan(4, 1, 63, 0, 1), _scan(2, 1, 63, 0, 1), _scan(1, 6, 63, 0, 2), _scan(1, 1, 63, 2, 1),
                     _scan(7, 0, 0, 1, 0), _scan(4, 1, 63, 1, 0), _scan(2, 1, 63, 1, 0), _scan(1, 1, 63, 1, 0)], True),
    "ac first twice": ([DC, _scan(1, 1, 63, 0, 1), _scan(1, 1, 63, 0, 0)], False),
    "ac first over a part": ([DC, _scan(1, 1, 20, 0, 1), _scan(1, 10, 63, 0, 1), _scan(1, 1, 63, 1, 0)], False),
    "ac first after a refinement": ([DC, _scan(1, 1, 63, 0, 2), _scan(1, 1, 63, 2, 1), _scan(1, 1, 20, 0, 1)], False),
    "dc first twice": ([_scan(1, 0, 0, 0, 1), _scan(1, 0, 0, 0, 0)] + LUMA, False),
    "dc first of all, then of one": ([_scan(7, 0, 0, 0, 1), _scan(2, 0, 0, 0, 0), _scan(2, 1, 63, 0, 0)], False),
}


@pytest.mark.parametrize("restart", [0, 3])
@pytest.mark.parametrize("name", sorted(FILES))
def test_scans_that_overlap_are_ordered(plan, name, restart):
    scans, step = FILES[name]
    scans = [s[:5] + (restart, 4 if restart else 1, 0) for s in scans]
    assert plan(scans)[0] == step
    for k0 in range(len(scans)):
        for k in range(k0 + 1, len(scans) + 1):
            _check(scans, plan(scans, k0, k)[1], k0, k)


def test_any_sequence_of_scans_is_ordered(plan):
    """Random scans, most of which no encoder would write."""
    rng = random.Random(4)
    for _ in range(3000):
        scans = []
        for _ in range(rng.randint(1, 12)):
            ah = rng.choice([0, 0, 1])
            if rng.random() < 0.3:
                scans.append(_scan(rng.choice([1, 2, 4, 7]), 0, 0, ah, 0))
            else:
                a, b = sorted((rng.randint(1, 63), rng.randint(1, 63)))
                scans.append(_scan(rng.choice([1, 2, 4]), a, b, ah, 0, rng.choice([0, 0, 0, 5]), rng.choice([1, 1, 1, 3]), rng.choice([0, 0, 0, 64])))
        k0 = rng.randrange(len(scans))
        k = rng.randint(k0 + 1, len(scans))
        _check(scans, plan(scans, k0, k)[1], k0, k)


@pytest.mark.parametrize("size, sub, interval, units, blocks, longest", [
    ((256, 256), 2, 64, 8, 1536, 192), ((256, 256), 2, 128, 4, 1536, 384), ((600, 450), 1, 64, 134, 4275 * 3, 96), ((256, 256), 2, 0, 1, 1536, 1536), ((45, 30), 2, 1, 6, 36, 6),
    ((200, 136), 2, 32, 8, 117 * 6, 90)])
def test_dc_units_of_a_written_record(plan, size, sub, interval, units, blocks, longest):
    """What the choice of decoder for DC first scans goes by: their entry points are twice as many as the interval says.  (The
    longest unit is taken from the mean of its scan, 117 / 8 MCUs in the last row.)"""
    import paper_1911_00472_amd as pkg
    import pcrgen
    files = [pcrgen.make_jpeg(40 + i, 1, size[0], size[1], 3, 6.0, sub, sub, 80) for i in range(2)]
    rec = np.frombuffer(pkg.record_write_indexed(files, None, interval) if interval else pcrgen.write_record(files), np.uint8)
    out = np.zeros(4, np.uint32)
    u32p, u8p = ctypes.POINTER(ctypes.c_uint32), ctypes.POINTER(ctypes.c_uint8)
    plan.lib.dc_launch_of.argtypes = [u8p, ctypes.c_size_t, ctypes.c_uint32, u32p]
    assert plan.lib.dc_launch_of(rec.ctypes.data_as(u8p), len(rec), 2, out.ctypes.data_as(u32p)) == 0
    assert tuple(out) == (2 * units, 2, 2 * blocks, longest)


# us a call by wavefronts and by lanes: several records open, beside AC scans by wavefronts, whole scans, blocks of the longest
# unit, mean over longest, {units of a launch: (wavefronts, lanes)}
DC_TIMES = [
    (0, 0, 0, 32, 1, {2048: (61, 69), 4096: (67, 71), 8192: (72, 66)}), (0, 0, 0, 96, 1, {2144: (78, 91), 4288: (88, 92), 8576: (106, 93)}),
    (0, 0, 0, 192, 1, {2048: (89, 110), 4096: (112, 118), 6144: (131, 127), 8192: (151, 134)}),
    (0, 0, 0, 384, 1, {2048: (124, 155), 4096: (161, 171), 6144: (224, 214), 8192: (271, 237)}),
    (0, 0, 0, 3072, 1, {4096: (908, 991), 6144: (1180, 1175), 8192: (1504, 1333)}),
    (0, 0, 1, 9, 1, {2048: (81, 96), 4096: (112, 117), 6144: (149, 148), 8192: (190, 177)}),
    (0, 0, 1, 216, 1, {2048: (129, 140), 4096: (208, 196), 6144: (261, 233), 8192: (341, 289)}),
    (0, 0, 1, 384, 1, {2048: (165, 189), 3072: (201, 209), 4096: (235, 226), 6144: (331, 303), 8192: (444, 379)}),
    (0, 0, 1, 864, 1, {2048: (230, 289), 4096: (401, 405), 6144: (535, 507), 8192: (695, 609)}),
    (0, 0, 1, 3750, 1, {2048: (743, 1031), 4096: (1178, 1274), 6144: (1539, 1528), 8192: (2006, 1787)}),
    (0, 0, 1, 216, 130 / 216, {4096: (158, 161), 6144: (208, 195), 8192: (267, 233), 12288: (377, 307)}),
    (0, 0, 1, 384, 188 / 384, {4096: (174, 199), 6144: (227, 235), 8192: (288, 276), 12288: (422, 364)}),
    (0, 0, 1, 726, 470 / 726, {4096: (243, 281), 6144: (349, 359), 8192: (462, 440), 12288: (682, 590)}),
    (0, 0, 1, 1536, 698 / 1536, {4096: (341, 489), 8192: (588, 675), 12288: (849, 851)}), (0, 0, 1, 2790, 979 / 2790, {8192: (721, 999), 12288: (984, 1175)}),
    (1, 0, 0, 192, 1, {2048: (214, 233), 4096: (286, 229), 6144: (366, 273)}), (1, 0, 1, 384, 1, {2048: (453, 472), 4096: (823, 724)}),
    (1, 0, 1, 1536, 1, {2048: (1043, 1238), 3072: (1478, 1506), 4096: (1912, 1785)}),
    (1, 0, 1, 384, 188.5 / 384, {1024: (196, 279), 2048: (295, 348), 4096: (547, 478), 6144: (767, 648)}),
    (1, 0, 1, 720, 258 / 720, {2048: (360, 513), 4096: (556, 659), 6144: (852, 795)}), (1, 0, 1, 1260, 653 / 1260, {2048: (536, 826), 4096: (847, 1058), 6144: (1339, 1294)}),
    (1, 0, 1, 1944, 1324 / 1944, {2048: (875, 1261), 4096: (1576, 1712)}),
    (0, 1, 0, 192, 1, {2048: (134, 177), 4096: (182, 210), 8192: (328, 325)}), (0, 1, 0, 96, 1, {2144: (105, 133), 4288: (126, 147), 8576: (178, 183), 12864: (223, 218)}),
    (0, 1, 1, 384, 1, {4096: (416, 465), 8192: (737, 735), 12288: (1062, 1017)}), (0, 1, 1, 726, 470 / 726, {6144: (624, 704), 12288: (1154, 1152)}),
    (1, 1, 1, 384, 1, {2048: (774, 863), 4096: (1402, 1361), 8192: (2647, 2403)}), (1, 1, 0, 96, 1, {2144: (224, 272), 4288: (337, 336), 8576: (535, 472)}),
    (1, 1, 1, 1260, 653 / 1260, {4096: (1789, 1937), 6144: (2576, 2562)}),
]


# bits of a launch's refinement scans, of their longest unit, of the first scans beside them (14 a block added), workgroups, and us a call by one
# wavefront a unit and by three with 1, 2 and 4 records of it at a time
TRIO_TIMES = [
    (220979340, 390258, 103456860, 1600, {1: (5716, 4123), 2: (7412, 5881), 4: (14404, 12175)}), (283259540, 390258, 132854292, 2048, {1: (5860, 4256), 2: (7703, 6954), 4: (14917, 14470)}),
    (353493736, 390258, 165346008, 2560, {1: (6038, 4394), 2: (8332, 8474), 4: (15914, 16912)}), (441337496, 390258, 206327024, 3200, {1: (6223, 4906), 2: (9053, 10544)}),
    (565408820, 390258, 264644940, 4096, {1: (6456, 6344), 2: (10218, 13394)}), (202014542, 322898, 264644940, 4096, {1: (5166, 4024), 2: (7427, 7364)}),
    (5556344, 11408, 13242080, 2800, {1: (304, 285), 4: (825, 899)}), (9463472, 11448, 22513536, 4800, {1: (349, 396), 2: (543, 687), 4: (1116, 1420)}),
    (9463472, 11448, 12151960, 4800, {1: (316, 326), 2: (449, 522), 4: (891, 1028)}), (21930696, 45808, 51212232, 2800, {1: (897, 798), 2: (1377, 1430), 4: (2071, 2709)}),
    (23527744, 26456, 10150128, 1100, {1: (496, 400), 2: (726, 742), 4: (1431, 1468)}), (38208872, 26480, 16433400, 1800, {1: (571, 650), 2: (919, 1095), 4: (1562, 1981)}),
    (4448712, 6672, 1866288, 1600, {1: (213, 188), 2: (265, 274), 4: (525, 544)}), (635104, 758, 696856, 3600, {1: (121, 137), 2: (161, 192), 4: (324, 389)}),
    (120226024, 105552, 48068928, 2800, {1: (1839, 1674), 2: (3131, 3495), 4: (4935, 6782)}), (49392072, 80624, 61699024, 3600, {1: (1441, 1130), 4: (4167, 4335)}),
    (2433792, 3314, 1065960, 1280, {1: (160, 150), 2: (187, 206), 4: (334, 373)}), (5118056, 3314, 2192920, 2560, {1: (170, 208), 2: (232, 312), 4: (444, 617)}),
    (690128, 848, 317216, 1280, {1: (112, 114), 2: (126, 140), 4: (169, 210)}), (1306186, 3281, 0, 476, {1: (227, 210), 2: (443, 412), 4: (500, 464)}),
    (3082852, 3291, 0, 1083, {1: (243, 228), 2: (284, 284), 4: (520, 529)}), (5462106, 3301, 0, 1851, {1: (271, 280), 2: (335, 364), 4: (649, 739)}),
]


@pytest.mark.parametrize("work, longest, beside, groups, times", TRIO_TIMES)
def test_refinement_scans_go_where_they_were_measured_to_be_faster(plan, work, longest, beside, groups, times):
    """With the records that are decoded at a time, three wavefronts a unit are nowhere taken where they are 4 % slower than one; nor is one where three gain a
    tenth, or, close to the line (seven ninths of the launch would go to three), a fifth."""
    lib = plan.lib
    lib.trio_pays.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int]
    for open_records, (one, three) in times.items():
        if lib.trio_pays(work, longest, beside, groups, open_records):
            assert three <= 1.04 * one, open_records
        else:
            near = lib.trio_pays(work * 7 // 9, longest, beside * 7 // 9, groups * 7 // 9, open_records)
            assert three >= (0.8 if near else 0.9) * one, open_records
    assert not any(lib.trio_pays(work, longest, beside, groups, n + 1) and not lib.trio_pays(work, longest, beside, groups, n) for n in range(0, 6))


@pytest.mark.parametrize("several, beside, whole, longest, mean, times", DC_TIMES)
def test_dc_scans_go_where_they_were_measured_to_be_faster(plan, several, beside, whole, longest, mean, times):
    for units, (wavefronts, lanes) in times.items():
        by_lanes = plan.lib.dc_by_lanes(units if whole else units // 4, units, round(units * longest * mean), longest, several, beside)
        assert (lanes if by_lanes else wavefronts) <= 1.05 * min(lanes, wavefronts), units


@pytest.mark.parametrize("shapes, most", [(1, 9), (2, 1), (3, 200), (4, 9)])
def test_no_wavefront_has_dc_units_of_several_shapes(plan, shapes, most):
    """Sixty-four units to a wavefront, but for the last of each shape; units of a shape keep their order."""
    rng = np.random.default_rng(shapes)
    shape, count = rng.integers(0, shapes, 300, dtype=np.uint32), rng.integers(1, most + 1, 300, dtype=np.uint32)
    total = int(count.sum())
    out, starts = np.zeros((total, 2), np.uint32), np.zeros(total + 1, np.uint32)
    u32p = ctypes.POINTER(ctypes.c_uint32)
    waves = plan.lib.dc_order(shape.ctypes.data_as(u32p), count.ctypes.data_as(u32p), len(shape), 64, out.ctypes.data_as(u32p), starts.ctypes.data_as(u32p))
    want = [(e, j) for e in range(len(shape)) for j in range(count[e])]
    if shapes == 1:
        assert waves == -1 and [tuple(u) for u in out] == want
        return
    assert sorted(map(tuple, out)) == want
    for v in range(shapes):
        assert [tuple(u) for u in out if shape[u[0]] == v] == [u for u in want if shape[u[0]] == v]
    assert starts[0] == 0 and starts[waves] == total and waves <= total // 64 + shapes
    for a, b in zip(starts[:waves], starts[1:waves + 1]):
        assert a < b <= a + 64 and len(set(shape[out[a:b, 0]])) == 1


def test_a_dc_scan_s_shape_is_of_its_own_components(plan):
    """Two files whose scan of two components is decoded alike have the same shape, whatever the third component is."""
    def of(ns, comp, hs, vs):
        a = [np.array(v, np.uint32) for v in (comp, hs, vs)]
        return plan.lib.dc_shape_of(ns, *[v.ctypes.data_as(ctypes.POINTER(ctypes.c_uint32)) for v in a])
    assert of(2, (1, 2, 0), (2, 1, 1), (2, 1, 1)) == of(2, (1, 2, 0), (1, 1, 1), (1, 1, 1))
    assert of(1, (0, 0, 0), (2, 1, 1), (2, 1, 1)) == of(1, (2, 0, 0), (1, 1, 1), (1, 1, 1))
    assert of(3, (0, 1, 2), (2, 1, 1), (2, 1, 1)) != of(3, (0, 1, 2), (2, 1, 1), (1, 1, 1))
    assert of(2, (0, 1, 0), (2, 1, 1), (2, 1, 1)) != of(2, (0, 1, 0), (1, 1, 1), (1, 1, 1))


def _asked(plan, name, rec, *args):
    u32p, u8p = ctypes.POINTER(ctypes.c_uint32), ctypes.POINTER(ctypes.c_uint8)
    a, out = np.frombuffer(rec, np.uint8), np.zeros(4, np.uint32)
    f = getattr(plan.lib, name)
    f.argtypes = [u8p, ctypes.c_size_t] + [ctypes.c_uint32] * len(args) + [u32p]
    assert f(a.ctypes.data_as(u8p), a.size, *args, out.ctypes.data_as(u32p)) == 0
    return [int(v) for v in out]


def test_first_scans_the_gpu_tests_give_many_lanes(plan):
    """The rule says of the records of the GPU tests of first scans by many lanes what those say that the launches were."""
    import test_gpu_first_split as gpu
    records = [gpu.size_record(*s, side) for side in gpu.SIZES for s in gpu.SAMPLINGS] + [(gpu.mixed_record(), {1: gpu.YES, 2: gpu.WIDE, 5: gpu.WIDE})]
    for rec, splits in records:
        for k, want in splits.items():
            assert tuple(_asked(plan, "first_split_of", rec, k, 1)[:2]) == want, k


def test_ac_launches_the_gpu_tests_send_to_the_lanes(plan):
    """The same of the launches of first scans that go to the lanes by themselves (a job: sixty units of scans that share its tables); one
    record's are by lanes for their bits and blocks, and would not be by their number."""
    import paper_1911_00472_amd as pkg
    import pcrgen
    import test_gpu_lane_decoders as gpu
    below = 0
    for side, n, entry, restart, shapes in gpu.BY_THEMSELVES:
        some = [pcrgen.make_jpeg(60 + i, 1 + (i % 2), side - 3 * i, side + i, 3, 12.0, 2, 2, 80, restart=restart) for i in range(6)]
        files = [some[i % 6] for i in range(n)]
        rec = pkg.record_write_indexed(files, None, entry) if entry else pcrgen.write_record(files)
        for k, (lanes, _) in zip((2, 5), shapes):
            units = _asked(plan, "lanes_launch_of", rec, k, 0, 1, 0)[2]
            got, many, _, _ = _asked(plan, "lanes_launch_of", rec, k, 0, units // 60, 0)
            assert got == lanes, (side, n, k)
            below += got and not many
    assert below >= 3
