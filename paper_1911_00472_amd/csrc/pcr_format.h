// Record header and JPEG marker parsing, compiled for host and device.
//
// Record layout (paper Section 3, record figure: metadata first, then the scan groups in
// order of fidelity; raw struct serialisation, Section 5 "Loader"), little endian:
//   "PCR1" | u32 version | u32 n | u32 G | u64 header_bytes | u64 group_end[G] | i32 label[n]
//   | u32 n_scans[n] | u32 len[G][n] | padding | group 1 | group 2 | ...
// Group g holds the g-th scan region of every image back to back.  A region is the slice of
// the image's progressive JPEG file between the ends of two consecutive scans (Section 5,
// "Encoding"): region 1 starts with SOI and carries the frame header and tables, every
// later region carries the tables and the SOS header of its one scan followed by the
// entropy-coded data.
//
// Version 2 adds entry points, an index INTO the scans (the paper's metadata only says where each scan group
// starts; Section 4.2 names the decode of a scan as the bottleneck, and a scan of a stock file is one serial
// stream): after len[G][n] the header carries
//   u32 entry_interval | u32 0 | u16 ecount[G][n]
// and group g ends with the entries of its scans, image after image, ecount[g][i] entries of 16 bytes each:
//   u32 mcu | u32 bit | i16 pred[3] | u16 0
// "decoding of this scan may start at MCU `mcu` of the scan (block `mcu` of a scan of one component), at bit `bit`
// of its entropy-coded data counted without the stuffed zero bytes, with the DC predictions `pred` of the scan's
// components (scans that code DC differences), and no end-of-band run is pending there".  Entries are in
// increasing order; scans with restart markers and DC refinement scans have none.  The image bytes are exactly
// those of version 1: region lengths and offsets do not change, group_end[g] includes the group's entries.
#pragma once
#include "pcr_common.h"

namespace pcr {

struct RecordHeader {
    uint32_t n, G;
    uint64_t header_bytes;
    uint32_t k_avail;                      // scan groups wholly inside the bytes given
    uint32_t version;                      // 1, or 2: with entry points
    uint32_t entry_interval;               // version 2: MCUs between entry points the writer aimed at (informative)
};
// Version 2: an entry point is 16 bytes (MCU, bit offset, three DC predictions, two reserved bytes), or 8 (MCU and bit
// offset only) where the scan has no DC predictions to resume -- the AC scans, nearly all entries of a record.  The
// header's 16-bit entry count of an (image, scan) carries the form in its top bit.
constexpr uint32_t kEntryBytes = 16, kEntryBytesShort = 8, kEntryShortFlag = 0x8000u, kMaxEntriesPerScan = 0x7FFFu;

PCR_HD uint64_t hdr_group_end_pos(uint32_t g) { return 24 + 8ull * g; }
PCR_HD uint64_t hdr_label_pos(uint32_t G, uint32_t i) { return 24 + 8ull * G + 4ull * i; }
PCR_HD uint64_t hdr_nscans_pos(uint32_t n, uint32_t G, uint32_t i) { return 24 + 8ull * G + 4ull * n + 4ull * i; }
PCR_HD uint64_t hdr_len_pos(uint32_t n, uint32_t G, uint32_t g, uint32_t i) { return 24 + 8ull * G + 8ull * n + 4ull * ((uint64_t)g * n + i); }
PCR_HD uint64_t hdr_entry_interval_pos(uint32_t n, uint32_t G) { return hdr_len_pos(n, G, G, 0); }                  // version 2
PCR_HD uint64_t hdr_ecount_pos(uint32_t n, uint32_t G, uint32_t g, uint32_t i) { return hdr_len_pos(n, G, G, 0) + 8 + 2ull * ((uint64_t)g * n + i); }
PCR_HD uint32_t ld_le16(const uint8_t* p) { return (uint32_t)p[0] | ((uint32_t)p[1] << 8); }
// the entry-count field of the header taken apart
PCR_HD uint32_t entry_count(uint32_t field) { return field & kMaxEntriesPerScan; }
PCR_HD uint32_t entry_stride(uint32_t field) { return (field & kEntryShortFlag) ? kEntryBytesShort : kEntryBytes; }
PCR_HD uint64_t entry_bytes(uint32_t field) { return (uint64_t)entry_count(field) * entry_stride(field); }

// Validate the fixed part of the header.  `bytes` must hold at least min(nbytes, header).
PCR_HD int parse_record_header(const uint8_t* bytes, uint64_t nbytes, RecordHeader* h) {
    if (nbytes < 24) return kETruncated;
    if (bytes[0] != 'P' || bytes[1] != 'C' || bytes[2] != 'R' || bytes[3] != '1') return kEFormat;
    h->version = ld_le32(bytes + 4);
    if (h->version != 1 && h->version != 2) return kEUnsupported;
    h->n = ld_le32(bytes + 8); h->G = ld_le32(bytes + 12); h->header_bytes = ld_le64(bytes + 16);
    if (h->n == 0 || h->G == 0 || h->G > 64 || h->n > (1u << 24)) return kEFormat;
    uint64_t need = h->version == 2 ? hdr_ecount_pos(h->n, h->G, h->G, 0) : hdr_len_pos(h->n, h->G, h->G, 0);
    if (h->header_bytes < need) return kEFormat;
    if (nbytes < h->header_bytes) return kETruncated;
    h->entry_interval = h->version == 2 ? ld_le32(bytes + hdr_entry_interval_pos(h->n, h->G)) : 0;
    uint64_t prev = h->header_bytes; uint32_t k = 0;
    for (uint32_t g = 0; g < h->G; g++) {
        uint64_t e = ld_le64(bytes + hdr_group_end_pos(g));
        if (e < prev) return kEFormat;
        if (e <= nbytes && k == g) k = g + 1;
        prev = e;
    }
    h->k_avail = k;
    return kOk;
}

// ---------------------------------------------------------------------------------------
// Marker parsing of one image: walks the headers of regions 0..kmax-1 (never the
// entropy-coded data) and fills the image and scan descriptors.
//   rec      record bytes: a pointer, or on the device anything indexed by record offset (HeaderBytes)
//   off,len  index tables [G][n] (absolute offsets / lengths of the regions)
// Every read is bounds-checked against the region it belongs to.  On the device bytes are taken twenty-four at a time (head_at),
// enough for a segment's marker and length with what is looked at of its payload, at one place in the code: code that runs once
// costs what it takes to fetch it, and a chain of byte reads would be as slow.  The host reads them where they are (through the
// same twenty-four bytes its parse of 2048 small 4:4:4 pictures, three regions each, took 383 us; byte reads and selects
// before 336; now 301).
// The walk over a region's segments (walk_region) needs nothing from other regions; what a scan takes over from
// earlier ones -- tables in force, restart interval, the scans it refines -- is put together afterwards
// (resolve_scan, scan_history).  The host goes through an image's regions one by one (parse_image), the device
// walks all of them at once, a wavefront each (k_headers).
// ---------------------------------------------------------------------------------------
struct RegionWalk {
    uint32_t dht[8];                       // offset of BITS of the table this region last defines for class * 4 + id (0: none)
    uint32_t qoff[4]; uint8_t qprec[4];    // the same for quantisation tables
    uint32_t sos, sos_end;                 // payload of the scan header; entropy-coded data starts at sos_end
    uint64_t sos_head[2];                  // its first sixteen bytes
    int32_t ri;                            // restart interval defined here, -1: none
};

PCR_HD uint32_t byte_of(uint64_t v, uint32_t b) { return (uint32_t)(v >> (8 * b)) & 255u; }
// What walk_region sees of a segment, or of a table in one: its first bytes.  Host: where they are (walk_region has looked at the
// bounds before it asks).  Device: twenty-four of them in scalar registers (head_at for HeaderBytes, pcr_kernels.h).
struct HostHead {
    const uint8_t* q; uint32_t there;
    PCR_HD uint32_t byte(uint32_t i) const { return q[i]; }
    PCR_HD void skip_marker() { q += 4; there -= 4; }
    PCR_HD uint32_t counts() const { uint32_t t = 0; for (uint32_t i = 1; i <= 16; i++) t += q[i]; return t; }        // of a Huffman table
    PCR_HD void first16(uint64_t h[2]) const {                      // (what is not there: zeros)
        h[0] = h[1] = 0;
        if (there >= 16) { __builtin_memcpy(h, q, 16); return; }
        for (uint32_t i = 0; i < there; i++) h[i >> 3] |= (uint64_t)q[i] << (8 * (i & 7));
    }
};
PCR_HD HostHead head_at(const uint8_t* rec, uint32_t p, uint32_t end) { return HostHead{rec + p, end - p}; }

// a[i] = v, i < N.  (Device: one store to LDS.  Host: a select per entry, because what one entry was stored to is read as a whole
// right after, and a wide load waits for a narrow store it overlaps.)
template <int N, class T>
PCR_HD void set_entry(T* a, uint32_t i, T v) {
#if defined(__HIP_DEVICE_COMPILE__)
    a[i] = v;
#else
    for (uint32_t t = 0; t < (uint32_t)N; t++) a[t] = t == i ? v : a[t];
#endif
}

PCR_HD void setup_geometry(ImgDesc* d) {
    const int nc = uni((int)d->nc);
    d->hmax = 1; d->vmax = 1;
    for (int c = 0; c < nc; c++) { if (d->hs[c] > d->hmax) d->hmax = d->hs[c]; if (d->vs[c] > d->vmax) d->vmax = d->vs[c]; }
    const uint32_t hsh = d->hmax - 1u, vsh = d->vmax - 1u;     // (factors are 1 or 2: shifts)
    d->mcux = (uint16_t)((d->W + (8u << hsh) - 1) >> (3 + hsh));
    d->mcuy = (uint16_t)((d->H + (8u << vsh) - 1) >> (3 + vsh));
    for (int c = 0; c < nc; c++) {
        d->bw[c] = (uint16_t)(d->mcux * d->hs[c]); d->bh[c] = (uint16_t)(d->mcuy * d->vs[c]);
        uint32_t xc = ((uint32_t)d->W * d->hs[c] + hsh) >> hsh, yc = ((uint32_t)d->H * d->vs[c] + vsh) >> vsh;
        d->cw[c] = (uint16_t)((xc + 7) / 8); d->ch[c] = (uint16_t)((yc + 7) / 8);
    }
}

// The segments of region g up to its scan header.  The frame header goes into *img (region 0 must hold it, later
// regions must not).  On the device a wavefront walks a region: what head_at returns is the same in all lanes and known to
// be (uni), so that all of this is scalar code, and *w and *img lie in LDS.
template <class Bytes>
PCR_HD int walk_region(const Bytes& rec, uint32_t p, uint32_t end, uint32_t g, RegionWalk* w, ImgDesc* img) {
    for (int t = 0; t < 8; t++) w->dht[t] = 0;
    for (int t = 0; t < 4; t++) { w->qoff[t] = 0; w->qprec[t] = 0; }
    w->ri = -1; w->sos = w->sos_end = 0;
    bool have_frame = g > 0;
    if (g == 0) {
        if (end - p < 2 || rec[p] != 0xFF || rec[p + 1] != 0xD8) return kEFormat;
        p += 2;
    }
    uint32_t m = 0, s = 0, se = 0;                           // the segment's marker, what is left of its payload
    while (true) {                                           // one turn per segment, or per table of a segment that holds several
        const bool fresh = s >= se;
        if (fresh && end - p < 4) return kEFormat;
        auto h = head_at(rec, fresh ? p : s, end);
        if (fresh) {
            if (h.byte(0) != 0xFF) return kEFormat;
            m = h.byte(1);
            if (m == 0xFF) { p++; continue; }
            const uint32_t L = (h.byte(2) << 8) | h.byte(3);
            if (L < 2 || L + 2 > end - p) return kEFormat;
            s = p + 4; se = p + 2 + L;
            p = se;
            h.skip_marker();
        }
        const uint32_t left = se - s, first = left ? h.byte(0) : 0u;
        if (m == 0xDB) {
            if (left == 0) continue;
            const uint32_t pq = first >> 4, tq = first & 15;
            if (tq > 3 || pq > 1 || left - 1 < 64 * (pq + 1)) return kEFormat;
            set_entry<4>(w->qoff, tq, s + 1); set_entry<4>(w->qprec, tq, (uint8_t)pq);
            s += 1 + 64 * (pq + 1);
        } else if (m == 0xC4) {
            if (left == 0) continue;
            const uint32_t tc = first >> 4, th = first & 15;
            if (tc > 1 || th > 3 || left < 17) return kEFormat;
            const uint32_t nv = h.counts();
            if (nv > 256 || left - 17 < nv) return kEFormat;
            set_entry<8>(w->dht, tc * 4 + th, s + 1);
            s += 17 + nv;
        } else if (m == 0xC0 || m == 0xC1 || m == 0xC2) {
            if (have_frame || left < 6) return kEFormat;
            if (first != 8) return kEUnsupported;
            const uint32_t nc = h.byte(5);
            img->progressive = (m == 0xC2);
            img->H = (uint16_t)((h.byte(1) << 8) | h.byte(2)); img->W = (uint16_t)((h.byte(3) << 8) | h.byte(4)); img->nc = (uint8_t)nc;
            if (img->H == 0 || img->W == 0) return kEUnsupported;
            if (nc != 1 && nc != 3) return kEUnsupported;
            if (left < 6u + 3u * nc) return kEFormat;
            for (uint32_t c = 0; c < (uint32_t)kMaxComp; c++) {
                if (c >= nc) continue;
                const uint32_t hs = h.byte(7 + 3 * c) >> 4, vs = h.byte(7 + 3 * c) & 15, tq = h.byte(8 + 3 * c);
                img->cid[c] = (uint8_t)h.byte(6 + 3 * c); img->hs[c] = (uint8_t)hs; img->vs[c] = (uint8_t)vs; img->tq[c] = (uint8_t)tq;
                if (hs < 1 || hs > 2 || vs < 1 || vs > 2 || tq > 3) return kEUnsupported;
            }
            if (nc == 1) { img->hs[0] = 1; img->vs[0] = 1; }
            setup_geometry(img);
            have_frame = true;
            s = se;
        } else if ((m >= 0xC3 && m <= 0xCF && m != 0xC8 && m != 0xCC) || m == 0xDC) {
            return kEUnsupported;                  // lossless, hierarchical, arithmetic coding, DNL
        } else if (m == 0xDD) {
            if (left < 2) return kEFormat;
            w->ri = (int32_t)((first << 8) | h.byte(1));
            s = se;
        } else if (m == 0xDA) {
            if (!have_frame || left < 1) return kEFormat;
            w->sos = s; w->sos_end = se;
            h.first16(w->sos_head);
            return kOk;
        } else {
            s = se;                                // APPn, COM, anything else with a length: skipped
        }
    }
}

// The descriptor of a scan from its header: dht, ri: the tables and the restart interval in force; end: of its region.
PCR_HD int resolve_scan(const RegionWalk& w, uint32_t end, const uint32_t dht[8], uint32_t ri, const ImgDesc* img, ScanDesc* sd) {
    const uint32_t s = uni(w.sos), se = uni(w.sos_end), nc = uni((uint32_t)img->nc), progressive = uni((uint32_t)img->progressive);
    const uint64_t h0 = uni(w.sos_head[0]), h1 = uni(w.sos_head[1]);
    uint32_t cid[kMaxComp];
    for (int q = 0; q < kMaxComp; q++) cid[q] = uni((uint32_t)img->cid[q]);
    const uint32_t ns = byte_of(h0, 0);
    if (ns < 1 || ns > nc || se - s < 1 + 2 * ns + 3) return kEFormat;
    sd->ns = (uint8_t)ns;
    uint32_t dc_def[kMaxComp] = {0, 0, 0}, ac_def[kMaxComp] = {0, 0, 0};           // the tables the components name
    uint32_t comp0 = 0;
    for (uint32_t j = 0; j < (uint32_t)kMaxComp; j++) {
        if (j >= ns) continue;
        int c = -1;
        for (int q = 0; q < kMaxComp; q++) if (q < (int)nc && cid[q] == byte_of(h0, 1 + 2 * j)) c = q;
        if (c < 0) return kEFormat;
        const uint32_t td = byte_of(h0, 2 + 2 * j) >> 4, ta = byte_of(h0, 2 + 2 * j) & 15;
        sd->comp[j] = (uint8_t)c;
        if (j == 0) comp0 = (uint32_t)c;
        if (td > 3 || ta > 3) return kEFormat;
#if defined(__HIP_DEVICE_COMPILE__)
        for (uint32_t t = 0; t < 4; t++) { dc_def[j] = t == td ? dht[t] : dc_def[j]; ac_def[j] = t == ta ? dht[4 + t] : ac_def[j]; }   // (indexed, they would go to scratch memory)
#else
        dc_def[j] = dht[td]; ac_def[j] = dht[4 + ta];
#endif
    }
    const uint64_t band = ns == 1 ? h0 >> 24 : ns == 2 ? h0 >> 40 : (h0 >> 56) | (h1 << 8);      // behind the components: Ss, Se, Ah and Al
    const uint32_t Ss = byte_of(band, 0), Se = byte_of(band, 1), Ah = byte_of(band, 2) >> 4, Al = byte_of(band, 2) & 15;
    sd->Ss = (uint8_t)Ss; sd->Se = (uint8_t)Se; sd->Ah = (uint8_t)Ah; sd->Al = (uint8_t)Al;
    for (int j = 0; j < kMaxComp; j++) sd->ac_offc[j] = 0;
    if (!progressive) {
        // Sequential (baseline) file, the format a record of non-progressive images holds (one scan group, or
        // one per component): the scan header must say "all 64 coefficients, full precision".
        if (Ss != 0 || Se != 63 || Ah != 0 || Al != 0) return kEFormat;
        for (uint32_t j = 0; j < (uint32_t)kMaxComp; j++) {
            if (j >= ns) continue;
            if (!dc_def[j] || !ac_def[j]) return kEFormat;
            sd->dc_off[j] = dc_def[j]; sd->ac_offc[j] = ac_def[j];
        }
        sd->ac_off = ac_def[0];
    } else {
        if (Ss > Se || Se > 63 || (Ss == 0 && Se != 0) || (Ss > 0 && ns != 1) || Al > 13) return kEFormat;
        if (Ah != 0 && Ah != Al + 1) return kEFormat;
        for (uint32_t j = 0; j < (uint32_t)kMaxComp; j++) {
            if (j >= ns) continue;
            sd->dc_off[j] = 0;
            if (Ss == 0 && Ah == 0) { if (!dc_def[j]) return kEFormat; sd->dc_off[j] = dc_def[j]; }
        }
        sd->ac_off = 0;
        if (Ss > 0) { if (!ac_def[0]) return kEFormat; sd->ac_off = ac_def[0]; }
    }
    sd->ri = (uint16_t)ri;
    if (ns > 1) { sd->mcu_w = img->mcux; sd->mcus = (uint32_t)img->mcux * img->mcuy; }
    else { sd->mcu_w = img->cw[comp0]; sd->mcus = (uint32_t)img->cw[comp0] * img->ch[comp0]; }
    sd->data_off = se; sd->data_len = end - se;
    return kOk;
}

// A refinement scan works on the positions of its band that are already non-zero.  Those made non-zero by AC first
// scans are read back from the coefficients; those added by earlier refinement scans of the component (not applied to
// the coefficients yet) come from the masks those scans leave, so they are listed here.
PCR_HD int scan_history(ScanDesc* scans, uint32_t g) {
    ScanDesc* sd = &scans[g];
    sd->nhist = 0;
    if (sd->Ss > 0 && sd->Ah > 0) {                // (first scans need no history)
        bool has_first = false;
        for (uint32_t q = 0; q < g; q++) {
            const ScanDesc* e = &scans[q];
            if (e->Ss > 0 && e->comp[0] == sd->comp[0] && e->Ss <= sd->Se && sd->Ss <= e->Se) {
                if (e->Ah == 0) { has_first = true; continue; }
                if (sd->nhist >= kMaxHist) return kEUnsupported;
                sd->hist[sd->nhist++] = (uint8_t)q;
            }
        }
        if (!has_first) return kEFormat;
    }
    sd->valid = 1;
    return kOk;
}

// What is left once all regions are parsed (img->nscans of them): the status of an image whose scans are all valid.
PCR_HD int check_image(const ImgDesc* img, const ScanDesc* scans) {
    if (img->nscans == 0) return kEFormat;
    // the refinement scans of a component are replayed from a list of fixed length when its coefficients are loaded
    for (int c = 0; c < img->nc; c++) {
        int nref = 0;
        for (uint32_t g = 0; g < img->nscans; g++) {
            if (scans[g].Ah == 0) continue;
            for (int j = 0; j < scans[g].ns; j++) if (scans[g].comp[j] == c) nref++;
        }
        if (nref > kApplyMaxScans) return kEUnsupported;
    }
    for (int c = 0; c < img->nc; c++) if (!img->qoff[img->tq[c]]) return kEFormat;
    return kOk;
}

// Parse image i: regions 0..kmax-1.  scans points at this image's G descriptors.
PCR_HD void parse_image(const uint8_t* rec, const uint32_t* off, const uint32_t* len, uint32_t n, uint32_t i,
                        uint32_t nscans_i, uint32_t kmax, ImgDesc* img, ScanDesc* scans) {
    uint32_t dht[8] = {0, 0, 0, 0, 0, 0, 0, 0}, ri = 0;
    for (int t = 0; t < 4; t++) { img->qoff[t] = 0; img->qprec[t] = 0; }
    img->status = kOk; img->nscans = 0; img->nc = 0; img->W = 0; img->H = 0;
    for (int c = 0; c < kMaxComp; c++) img->zmax[c] = 0;
    img->pad = 0;
    uint32_t upto = nscans_i < kmax ? nscans_i : kmax;
    for (uint32_t g = 0; g < upto; g++) {
        scans[g].valid = 0;
        uint32_t p = off[(size_t)g * n + i], L = len[(size_t)g * n + i];
        RegionWalk w;
        int rc = walk_region(rec, p, p + L, g, &w, img);
        if (rc == kOk) {
            for (int t = 0; t < 8; t++) if (w.dht[t]) dht[t] = w.dht[t];
            for (int t = 0; t < 4; t++) if (w.qoff[t]) { img->qoff[t] = w.qoff[t]; img->qprec[t] = w.qprec[t]; }
            if (w.ri >= 0) ri = (uint32_t)w.ri;
            rc = resolve_scan(w, p + L, dht, ri, img, &scans[g]);
        }
        if (rc == kOk) rc = scan_history(scans, g);
        if (rc != kOk) { img->status = rc; return; }
        img->nscans = g + 1;
        for (int j = 0; j < scans[g].ns; j++) {
            const int c = scans[g].comp[j];
            if (scans[g].Se + 1 > img->zmax[c]) img->zmax[c] = (uint8_t)(scans[g].Se + 1);
        }
    }
    img->status = check_image(img, scans);
}

}  // namespace pcr
