// CPU build of the planning of launches that decode several scans side by side, and of the choice of decoder for DC first
// scans (pcr_chains.h).  Test-only.
#include <cstring>
#include <vector>
#include "../../paper_1911_00472_amd/csrc/pcr_chains.h"

using namespace pcr;

// Scans k0 .. k - 1 of an image, `count` scans in all; row g of scans: components (a bit each), Ss, Se, Ah, Al, restart
// interval, units, entry points.  Row g of out: the launch that decodes the scan (0: the chains, 1 + level: a launch of
// its level after them, -1: none), its chain (AC: from 0 on, DC: from 1000 on), its place in the chain, the places of the
// scans of the chain that it waits for (a bit each).  Returns whether all scans of the call keep in step (-1: a chain is wrong about which of its scans
// are refinement scans).
extern "C" int chain_plan(const int* scans, int count, int k0, int k, int* out) {
    std::vector<ScanDesc> s((size_t)count);
    std::vector<uint32_t> units((size_t)count), entries((size_t)count);
    for (int g = 0; g < count; g++) {
        const int* p = scans + 8 * g;
        memset(&s[g], 0, sizeof(ScanDesc));
        for (int c = 0; c < kMaxComp; c++) if (p[0] >> c & 1) s[g].comp[s[g].ns++] = (uint8_t)c;
        s[g].Ss = (uint8_t)p[1]; s[g].Se = (uint8_t)p[2]; s[g].Ah = (uint8_t)p[3]; s[g].Al = (uint8_t)p[4]; s[g].ri = (uint16_t)p[5];
        s[g].data_len = 1000u + 10u * (uint32_t)g;
        units[g] = (uint32_t)p[6]; entries[g] = (uint32_t)p[7];
    }
    std::vector<uint8_t> level((size_t)count);
    scan_levels(s.data(), (uint32_t)count, level.data());
    ChainSet set;
    set.add(0, s.data(), units.data(), entries.data(), (uint32_t)k0, (uint32_t)k);
    const int in_step = set.possible;
    if (!in_step) { set = ChainSet(); set.add_level_one(0, s.data(), level.data(), units.data(), (uint32_t)k0, (uint32_t)k); }
    for (int g = 0; g < count; g++) {
        const bool serial = g >= k0 && g < k && !(s[g].Ss == 0 && s[g].Ah > 0);       // (DC refinement scans are read in place)
        out[4 * g] = serial ? 1 + level[g] : -1; out[4 * g + 1] = out[4 * g + 2] = -1; out[4 * g + 3] = 0;
    }
    for (int kind = 0; kind < 2; kind++) {
        const auto& list = kind ? set.dc : set.ac;
        for (size_t c = 0; c < list.size(); c++)
            for (uint32_t a = 0; a < list[c].count; a++) {
                if ((list[c].refines >> a & 1u) != (s[list[c].scan[a]].Ah > 0 ? 1u : 0u)) return -1;
                int* o = out + 4 * list[c].scan[a];
                o[0] = 0; o[1] = (int)c + 1000 * kind; o[2] = (int)a; o[3] = (int)(list[c].waits >> (8 * a) & 255u);
            }
    }
    return in_step;
}

// The scans of scan groups 1 .. k of a record: each(image, its scans, number of the scan, its units).
template <class Each> static int each_scan(const uint8_t* rec, size_t nbytes, uint32_t k, const Each& each) {
    RecordHeader h;
    const int rc = parse_record_header(rec, nbytes, &h);
    if (rc) return rc;
    const uint32_t n = h.n, G = h.G;
    std::vector<uint32_t> off((size_t)G * n), len((size_t)G * n);
    uint64_t pos = h.header_bytes;
    for (uint32_t g = 0; g < h.k_avail; g++) {
        for (uint32_t i = 0; i < n; i++) { off[(size_t)g * n + i] = (uint32_t)pos; pos += len[(size_t)g * n + i] = ld_le32(rec + hdr_len_pos(n, G, g, i)); }
        pos = ld_le64(rec + hdr_group_end_pos(g));
    }
    for (uint32_t i = 0; i < n; i++) {
        ImgDesc img; std::vector<ScanDesc> sc(G);
        memset(&img, 0, sizeof img);
        parse_image(rec, off.data(), len.data(), n, i, ld_le32(rec + hdr_nscans_pos(n, G, i)), k, &img, sc.data());
        if (img.status) return img.status;
        for (uint32_t g = 0; g < img.nscans; g++) {
            const ScanDesc& sd = sc[g];
            const uint32_t entries = h.version == 2 && sd.ri == 0 ? entry_count(ld_le16(rec + hdr_ecount_pos(n, G, g, i))) : 0;
            each(img, sc.data(), g, sd.ri ? (sd.mcus + sd.ri - 1) / sd.ri : 1 + entries);
        }
    }
    return 0;
}
// The DC first scans, as one launch: units, scans, blocks.
static int dc_launch(const uint8_t* rec, size_t nbytes, uint32_t k, DcLaunch* L) {
    return each_scan(rec, nbytes, k, [&](const ImgDesc& img, const ScanDesc* sc, uint32_t g, uint32_t units) {
        if (sc[g].Ss == 0 && sc[g].Ah == 0 && !is_sequential_scan(sc[g])) L->add(img, sc[g], units);
    });
}
// The first scans: out: whether many lanes a scan pay, and a thousand of them.
extern "C" int first_split_of(const uint8_t* rec, size_t nbytes, uint32_t k, int with_dc, uint32_t* out) {
    FirstSplitLaunch L;
    const int rc = each_scan(rec, nbytes, k, [&](const ImgDesc& img, const ScanDesc* sc, uint32_t g, uint32_t units) { L.add(img, sc[g], units); });
    out[0] = L.pays(with_dc != 0); out[1] = out[0] && L.wide(with_dc != 0); out[2] = L.units; out[3] = L.dc_units;
    return rc;
}
// The AC scans of one level (0: the first scans), as one launch of so many jobs: out: whether it goes to the lanes, whether it would by the
// number of its units, that number, blocks of the longest.
extern "C" int lanes_launch_of(const uint8_t* rec, size_t nbytes, uint32_t k, uint32_t level, uint32_t jobs, int several, uint32_t* out) {
    LanesLaunch L;
    const int rc = each_scan(rec, nbytes, k, [&](const ImgDesc&, const ScanDesc* sc, uint32_t g, uint32_t units) {
        std::vector<uint8_t> at(g + 1);
        scan_levels(sc, g + 1, at.data());
        if (sc[g].Ss > 0 && !is_sequential_scan(sc[g]) && at[g] == level + 1) L.add(sc[g], units);
    });
    L.jobs = jobs;
    out[0] = L.by_lanes(level > 0, several != 0); out[1] = L.many(several != 0); out[2] = L.units; out[3] = L.longest_blocks;
    return rc;
}
// does a launch of refinement scans of so much work, the longest unit of so much, beside so much of first scans (then it is one of chains), go to three wavefronts a unit?
extern "C" int trio_pays(uint64_t work, uint32_t longest, uint64_t beside, uint32_t groups, int open_records) {
    TrioLaunch t;
    t.work = work; t.longest = longest; t.beside = beside; t.groups = groups; t.chains = beside > 0;
    return t.pays(open_records);
}
extern "C" int dc_launch_of(const uint8_t* rec, size_t nbytes, uint32_t k, uint32_t* out) {
    DcLaunch L;
    const int rc = dc_launch(rec, nbytes, k, &L);
    out[0] = L.units; out[1] = L.scans; out[2] = (uint32_t)L.blocks; out[3] = L.longest;
    return rc;
}
// does a launch of so many scans, cut into so many units of so many blocks in all, the longest of so many, go to the lanes?
extern "C" int dc_by_lanes(uint32_t scans, uint32_t units, uint32_t blocks, uint32_t longest, int several, int beside) {
    DcLaunch L;
    L.scans = scans; L.units = units; L.blocks = blocks; L.longest = longest;
    return L.by_lanes(several != 0, beside != 0);
}

// order of the units of n runs: out[2 i], out[2 i + 1] = run and number of the i-th; starts: where wavefronts begin; returns how many
extern "C" int dc_order(const uint32_t* shape, const uint32_t* count, uint32_t n, uint32_t lanes, uint32_t* out, uint32_t* starts) {
    size_t at = 0;
    struct Run { uint32_t shape, count; };
    const auto v = dc_units_by_shape(n, [&](uint32_t e) { return Run{shape[e], count[e]}; }, lanes, [&](uint32_t e, uint32_t j) { out[at++] = e; out[at++] = j; });
    std::copy(v.begin(), v.end(), starts);
    return (int)v.size() - 1;
}
extern "C" uint32_t dc_shape_of(uint32_t ns, const uint32_t* comp, const uint32_t* hs, const uint32_t* vs) {
    ImgDesc img; ScanDesc sd;
    memset(&img, 0, sizeof img); memset(&sd, 0, sizeof sd);
    sd.ns = (uint8_t)ns;
    for (uint32_t c = 0; c < (uint32_t)kMaxComp; c++) { sd.comp[c] = (uint8_t)comp[c]; img.hs[c] = (uint8_t)hs[c]; img.vs[c] = (uint8_t)vs[c]; }
    return dc_mcu_shape(img, sd);
}
