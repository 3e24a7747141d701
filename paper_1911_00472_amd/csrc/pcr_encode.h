// Host side of record creation (paper Section 5, "Encoding"): find where each scan of a JPEG file ends,
// group the scans of many files into one record with its index in front, and re-code the quantised
// coefficients of a file as a progressive file (the lossless transcode the paper does with a stock tool
// before it groups scans: same coefficients, ten scans for colour, six for gray).
//
// What is here runs on the CPU: it is done once per dataset, not per batch.  The coefficients a transcode
// starts from come from the device decoder (pcr_decode_coefficients), which reads baseline and progressive
// sources alike; a whole batch is coded there as well (pcr_coder.h), and put together here.
#pragma once
#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <new>
#include <thread>
#include <vector>
#if defined(__SSE2__) && !defined(__HIP_DEVICE_COMPILE__)
#include <emmintrin.h>
#endif

#include "pcr_format.h"
#include "pcr_entropy.h"
#include "pcr_hist.h"
#include "pcr_coder.h"

namespace pcr {
namespace enc {

// work() on `count` threads, this one among them; on as many as the system gives where it gives fewer.  work takes what
// there is to do piece by piece.  Returns whether there was memory for all of it.
template <class F> bool on_threads(uint32_t count, const F& work) {
    std::atomic<bool> enough(true);
    auto run = [&]() { try { work(); } catch (const std::bad_alloc&) { enough = false; } };
    std::vector<std::thread> pool;
    try {
        pool.reserve(count);
        for (uint32_t t = 1; t < count; t++) pool.emplace_back(run);
    } catch (const std::exception&) {}                         // (no more threads, or no memory for their table)
    run();
    for (auto& t : pool) t.join();
    return enough;
}

// ---- scan splitter --------------------------------------------------------------------------------------
// Region s of a file ends where the entropy-coded data of its scan s ends: at the first 0xFF that is not
// followed by 0x00 (a stuffed byte), by a restart marker or by more 0xFF fill leading up to one of those.
// The last region runs to the end of the file.  Returns the number of scans (0: not a well-formed file, or
// more than max_ends scans).
inline int scan_ends(const uint8_t* d, size_t n, uint64_t* ends, int max_ends) {
    if (n < 4 || d[0] != 0xFF || d[1] != 0xD8) return 0;
    int count = 0;
    size_t p = 2;
    auto is_data_follow = [](uint8_t x) { return x == 0x00 || (x >= 0xD0 && x <= 0xD7); };
    while (p + 4 <= n) {
        if (d[p] != 0xFF) return 0;
        const uint8_t m = d[p + 1];
        if (m == 0xFF) { p++; continue; }                      // fill before a marker
        if (m == 0xD9) break;
        const size_t len = ((size_t)d[p + 2] << 8) | d[p + 3];
        if (len < 2 || p + 2 + len > n) return 0;
        p += 2 + len;
        if (m != 0xDA) continue;
        // entropy-coded data: hop from 0xFF to 0xFF
        for (;;) {
            const void* hit = p < n ? memchr(d + p, 0xFF, n - p) : nullptr;
            if (!hit) return 0;                                // data runs off the file: no EOI
            p = (size_t)((const uint8_t*)hit - d);
            size_t q = p + 1;
            while (q < n && d[q] == 0xFF) q++;                 // a run of 0xFF counts as one
            if (q >= n) return 0;
            if (is_data_follow(d[q])) { p = q + 1; continue; }
            break;                                             // a real marker: the region ends at the first 0xFF of the run
        }
        if (count >= max_ends) return 0;
        ends[count++] = p;
    }
    if (count == 0) return 0;
    ends[count - 1] = n;
    return count;
}

// ---- record writer --------------------------------------------------------------------------------------
struct RecordPlan {
    uint32_t n = 0, G = 0;
    uint64_t header_bytes = 0, total = 0;
    std::vector<uint32_t> nscans;                              // [n]
    std::vector<uint64_t> ends;                                // [n][64] region ends of every file
};

constexpr int kMaxScansPerFile = 64;

inline int plan_record(const void* const* files, const size_t* sizes, uint32_t n, RecordPlan* P) {
    if (n == 0 || n > (1u << 24)) return kERange;
    P->n = n; P->G = 0; P->nscans.assign(n, 0); P->ends.assign((size_t)n * kMaxScansPerFile, 0);
    uint64_t payload = 0;
    for (uint32_t i = 0; i < n; i++) {
        if (!files[i]) return kEArg;
        const int s = scan_ends((const uint8_t*)files[i], sizes[i], &P->ends[(size_t)i * kMaxScansPerFile], kMaxScansPerFile);
        if (s <= 0) return kEFormat;
        P->nscans[i] = (uint32_t)s;
        if ((uint32_t)s > P->G) P->G = (uint32_t)s;
        payload += sizes[i];
    }
    const uint64_t raw = hdr_len_pos(n, P->G, P->G, 0);
    P->header_bytes = (raw + 63) / 64 * 64;
    P->total = P->header_bytes + payload;
    if (P->total >= (1ull << 32)) return kEUnsupported;        // offsets inside a record are 32 bits
    return kOk;
}

inline void st_le32(uint8_t* p, uint32_t v) { p[0] = (uint8_t)v; p[1] = (uint8_t)(v >> 8); p[2] = (uint8_t)(v >> 16); p[3] = (uint8_t)(v >> 24); }
inline void st_le64(uint8_t* p, uint64_t v) { st_le32(p, (uint32_t)v); st_le32(p + 4, (uint32_t)(v >> 32)); }

inline void write_record(const RecordPlan& P, const void* const* files, const int32_t* labels, uint8_t* out) {
    const uint32_t n = P.n, G = P.G;
    memset(out, 0, P.header_bytes);
    memcpy(out, "PCR1", 4);
    st_le32(out + 4, 1); st_le32(out + 8, n); st_le32(out + 12, G); st_le64(out + 16, P.header_bytes);
    uint64_t pos = P.header_bytes;
    for (uint32_t g = 0; g < G; g++) {
        for (uint32_t i = 0; i < n; i++) {
            uint32_t len = 0;
            if (g < P.nscans[i]) {
                const uint64_t* e = &P.ends[(size_t)i * kMaxScansPerFile];
                const uint64_t from = g ? e[g - 1] : 0;
                len = (uint32_t)(e[g] - from);
                memcpy(out + pos, (const uint8_t*)files[i] + from, len);
                pos += len;
            }
            st_le32(out + hdr_len_pos(n, G, g, i), len);
        }
        st_le64(out + hdr_group_end_pos(g), pos);
    }
    for (uint32_t i = 0; i < n; i++) {
        st_le32(out + hdr_label_pos(G, i), labels ? (uint32_t)labels[i] : 0u);
        st_le32(out + hdr_nscans_pos(n, G, i), P.nscans[i]);
    }
}

// ---- entry points (record version 2) ----------------------------------------------------------------------
// A scan of a stock file is one serial stream.  The record writer walks every scan once and notes, about every
// `interval` MCUs, a place where a decoder may start: a block boundary outside any end-of-band run, the bit
// offset of that place in the scan's data without the stuffed bytes, and the DC predictions there.  The walk
// needs no coefficient values, only which positions of every block are non-zero so far (the refinement scans'
// zero runs skip those).  Scans with restart markers need no entries: every restart interval is a start already.
struct EntryPoint { uint32_t mcu, bit; int16_t pred[3]; uint16_t zero; };
static_assert(sizeof(EntryPoint) == kEntryBytes, "entry layout");

// Bytes the data of a scan are padded with: a walk looks where it stands once a block, and a block is at most 64 symbols of 32 bits
// and as many correction bits.
constexpr size_t kWalkPad = 512;

// The 57 bits and more at a position, at the upper end.
inline uint64_t bits_at(const uint8_t* d, uint64_t pos) {
    uint64_t v;
    memcpy(&v, d + (pos >> 3), 8);
    return __builtin_bswap64(v) << (pos & 7);
}

// What a walk wants to know of the symbol at the head of a window: the bits it takes, how many positions it goes on by and whether
// a coefficient lies there (in a refinement scan: the zeros it passes), or the run it begins.  Codes of up to kWalkBits bits by look-up, by their
// first kWalkBits bits (0: another one, or none).
constexpr int kWalkBits = 11;
struct WalkTable {
    enum : uint32_t { kCoef = 1u << 16, kRun = 1u << 17, kBad = 1u << 18 };       // | positions or log2 of the run << 8 | bits
    uint32_t lut[1u << kWalkBits];
    const AcTab* tab; bool refine;
    uint32_t entry(uint32_t a) const {                         // a: ac_code's answer
        if (!a) return kBad;
        const uint32_t r = (a >> 4) & 15, sz = a & 15, len = a >> 8;
        if (refine) return sz > 1 ? (uint32_t)kBad : (sz ? kCoef | r << 8 | (len + 1) : (r < 15 ? kRun | r << 8 | (len + r) : 15u << 8 | len));
        return sz ? kCoef | (r + 1) << 8 | (len + sz) : (r < 15 ? kRun | r << 8 | (len + r) : 16u << 8 | len);
    }
    void build(const AcTab* t, bool refinement) {
        tab = t; refine = refinement;
        for (uint32_t i = 0; i < 1u << kWalkBits; i++) {
            // (the same code at both ends of the windows that begin so: it is that code in between)
            const uint32_t a = ac_code(t, i << (32 - kWalkBits)), z = ac_code(t, i << (32 - kWalkBits) | ((1u << (32 - kWalkBits)) - 1));
            lut[i] = a && a == z && (a >> 8) <= (uint32_t)kWalkBits ? entry(a) : 0;
        }
    }
    uint32_t at(uint64_t window) const {
        const uint32_t e = lut[window >> (64 - kWalkBits)];
        return e ? e : entry(ac_code(tab, (uint32_t)(window >> 32)));
    }
};

// Bits set, and the lowest set bit behind the first n set ones (0: there are fewer); BMI2: where the machine has those instructions.
template <bool BMI2> inline uint32_t walk_popcount(uint64_t x) {
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
    if (BMI2) { uint64_t n; asm("popcnt %1, %0" : "=r"(n) : "r"(x) : "cc"); return (uint32_t)n; }
#endif
    return (uint32_t)__builtin_popcountll(x);
}
template <bool BMI2> inline uint64_t walk_nth(uint64_t x, uint32_t n) {
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
    if (BMI2) { uint64_t one; asm("pdep %1, %2, %0" : "=r"(one) : "r"(x), "r"(1ull << n)); return one; }
#endif
    for (; n && x; n--) x &= x - 1;
    return x & (0 - x);
}
inline bool walk_bmi2() {
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
    static const bool has = __builtin_cpu_supports("bmi2") && __builtin_cpu_supports("popcnt");
    return has;
#else
    return false;
#endif
}

// One block of an AC scan outside a run: from bit *pos on, h its non-zero positions so far.  Returns the blocks of the run it ends in,
// itself included (0: none), or -1: no stream that can be followed.
inline int walk_first_block(const uint8_t* d, const WalkTable& T, uint64_t* pos, uint64_t* h, uint32_t Ss, uint32_t Se) {
    uint64_t at = *pos, known = *h;
    uint32_t k = Ss;
    int run = 0;
    while (k <= Se) {
        uint64_t w = bits_at(d, at);
        uint32_t used = 0;
        do {                                                   // (57 bits at least: two symbols of 25 or one of 32)
            const uint32_t e = T.at(w << used);
            if (e & WalkTable::kBad) return -1;
            used += e & 255u;
            if (e & WalkTable::kRun) {
                const uint32_t r = (e >> 8) & 15u;
                run = (int)(1u << r);
                if (r) run += (int)(bits_at(d, at + used - r) >> (64 - r));
                k = 64;
                break;
            }
            k += (e >> 8) & 255u;
            if (e & WalkTable::kCoef) {
                if (k > Se + 1) return -1;
                known |= 1ull << (k - 1);
            }
        } while (k <= Se && used <= 25);
        at += used;
    }
    *pos = at; *h = known;
    return run;
}
template <bool BMI2> inline int walk_refine_block(const uint8_t* d, const WalkTable& T, uint64_t* pos, uint64_t* h, uint64_t band) {
    uint64_t at = *pos, known = *h & band, fresh = 0;         // (a position this scan has made non-zero holds no correction bit, and is no zero behind it)
    uint64_t from = band;                                      // the positions not passed yet
    int run = 0;
    while (from) {
        const uint32_t e = T.at(bits_at(d, at));
        if (e & WalkTable::kBad) return -1;
        at += e & 255u;
        const uint32_t r = (e >> 8) & 15u;
        if (e & WalkTable::kRun) {
            run = (int)(1u << r);
            if (r) run += (int)(bits_at(d, at - r) >> (64 - r));
            break;
        }
        const uint64_t one = walk_nth<BMI2>(~known & from, r);        // over r zeros; a correction bit at every non-zero on the way
        if (!one && (e & WalkTable::kCoef)) return -1;
        const uint64_t passed = one ? one - 1 : ~0ull;
        at += walk_popcount<BMI2>(known & from & passed);
        from &= one ? ~(one | passed) : 0;
        if (e & WalkTable::kCoef) fresh |= one;
    }
    if (run) at += walk_popcount<BMI2>(known & from);          // the rest of the block: corrections only
    *pos = at; *h |= fresh;
    return run;
}

// Entropy-coded data of a scan without stuffed zeros, fill bytes and restart markers; starts[j] = first byte of
// restart interval j.  Stops at the first other marker.
inline void unstuff_scan(const uint8_t* src, uint32_t L, std::vector<uint8_t>* out, std::vector<uint32_t>* starts) {
    out->clear(); starts->assign(1, 0);
    for (uint32_t q = 0; q < L; q++) {
        const void* ff = memchr(src + q, 0xFF, L - q);
        const uint32_t plain = ff ? (uint32_t)((const uint8_t*)ff - (src + q)) : L - q;
        out->insert(out->end(), src + q, src + q + plain);
        q += plain;
        if (q + 1 >= L) break;
        const uint8_t nx = src[q + 1];
        if (nx == 0x00) { out->push_back(0xFF); q++; }
        else if (nx >= 0xD0 && nx <= 0xD7) { starts->push_back((uint32_t)out->size()); q++; }
        else if (nx == 0xFF) continue;
        else break;
    }
}

// ent[g]: entry points of scan g of the file (empty where there are none, also for every scan from the first one
// this walk cannot follow).  ends: the file's region ends (scan_ends).  Returns kOk, or why the frame was refused.
inline int find_entry_points(const uint8_t* file, const uint64_t* ends, uint32_t nscans, uint32_t interval, std::vector<EntryPoint>* ent) {
    for (uint32_t g = 0; g < nscans; g++) ent[g].clear();
    if (interval == 0 || nscans > (uint32_t)kMaxScansPerFile) return kOk;
    uint32_t off[kMaxScansPerFile], len[kMaxScansPerFile];
    for (uint32_t g = 0; g < nscans; g++) { off[g] = g ? (uint32_t)ends[g - 1] : 0u; len[g] = (uint32_t)ends[g] - off[g]; }
    ImgDesc img; std::vector<ScanDesc> sc(nscans);
    memset(&img, 0, sizeof img); memset(sc.data(), 0, sizeof(ScanDesc) * nscans);
    parse_image(file, off, len, 1, 0, nscans, nscans, &img, sc.data());
    if (img.status != kOk) return img.status;
    std::vector<uint64_t> nz[kMaxComp];
    for (int c = 0; c < img.nc; c++) nz[c].assign((size_t)img.bw[c] * img.bh[c], 0);
    std::vector<uint8_t> clean; std::vector<uint32_t> starts;
    std::vector<DcTab> dt(kMaxComp); std::vector<AcTab> at(kMaxComp);
    WalkTable walk;
    const bool bmi2 = walk_bmi2();
    for (uint32_t g = 0; g < nscans; g++) {
        const ScanDesc& sd = sc[g];
        const bool seq = !img.progressive;
        if (!seq && sd.Ss == 0 && sd.Ah > 0) continue;               // DC refinement: one bit per block, nothing to walk
        unstuff_scan(file + sd.data_off, sd.data_len, &clean, &starts);
        const uint32_t nint = sd.ri ? (sd.mcus + sd.ri - 1) / sd.ri : 1;
        if (starts.size() != nint) return kOk;                        // damaged: the decoder will say so
        starts.push_back((uint32_t)clean.size());
        clean.resize(clean.size() + kWalkPad, 0xFF);
        const uint8_t* d = clean.data();
        if (seq || sd.Ss == 0) for (int j = 0; j < sd.ns; j++) dctab_build(&dt[j], file + sd.dc_off[j]);
        if (seq) for (int j = 0; j < sd.ns; j++) actab_build(&at[j], file + sd.ac_offc[j]);
        else if (sd.Ss > 0) { actab_build(&at[0], file + sd.ac_off); walk.build(&at[0], sd.Ah > 0); }
        const int c0 = sd.comp[0];
        const uint64_t band = (sd.Se >= 63 ? ~0ull : ((1ull << (sd.Se + 1)) - 1)) & ~((1ull << sd.Ss) - 1);
        std::vector<EntryPoint>& E = ent[g];
        bool bad = false;
        for (uint32_t iv = 0; iv < nint && !bad; iv++) {
            uint64_t pos = (uint64_t)starts[iv] * 8;
            const uint64_t nbits = (uint64_t)starts[iv + 1] * 8;
            int pred[kMaxComp] = {0, 0, 0};
            uint32_t eobrun = 0;
            const uint32_t m0 = sd.ri ? iv * sd.ri : 0, m1 = sd.ri ? std::min(m0 + sd.ri, sd.mcus) : sd.mcus;
            // AC refinement scans get an entry every interval / 2: a symbol of theirs takes a decoder more than twice as
            // long as one of an AC first scan (zero runs are counted against the block's history, correction bits follow),
            // and a launch of the lane-per-unit decoders takes as long as its longest unit.  So do DC first scans: an MCU
            // of theirs is several symbols (six with 4:2:0 sampling), each found by comparing with the table's codes.
            const bool halved = !seq && interval >= 2 && ((sd.Ss > 0 && sd.Ah > 0) || sd.Ss == 0);
            const uint32_t step = halved ? interval / 2 : interval;
            uint32_t next_entry = step;
            auto entry = [&](uint32_t m) {
                EntryPoint e; e.mcu = m; e.bit = (uint32_t)pos; e.zero = (!seq && sd.Ss > 0) ? 1 : 0;   // (in memory: 1 = written in the short form)
                for (int j = 0; j < kMaxComp; j++) e.pred[j] = (int16_t)pred[j];
                E.push_back(e);
                next_entry = (m / step + 1) * step;
            };
            if (seq || sd.Ss == 0) {                                 // blocks of every scan component of the MCU
                for (uint32_t m = m0; m < m1 && !bad; m++) {
                    if (sd.ri == 0 && m >= next_entry && E.size() < kMaxEntriesPerScan) entry(m);
                    for (int j = 0; j < sd.ns && !bad; j++) {
                        const int c = sd.comp[j];
                        const uint32_t nb = sd.ns > 1 ? (uint32_t)img.hs[c] * img.vs[c] : 1u;
                        for (uint32_t q = 0; q < nb && !bad; q++) {
                            uint64_t w = bits_at(d, pos);
                            const uint32_t e = dc_code(&dt[j], (uint32_t)(w >> 32));
                            if (!e) { bad = true; break; }
                            const uint32_t len = e >> 4, sz = e & 15;
                            pred[j] += extend(sz ? (uint32_t)(w << len >> (64 - sz)) : 0u, (int)sz);
                            pos += len + sz;
                            for (int k = 1; seq && k < 64;) {
                                const uint32_t a = ac_code(&at[j], (uint32_t)(bits_at(d, pos) >> 32));
                                if (!a) { bad = true; break; }
                                const uint32_t r = (a >> 4) & 15, s = a & 15;
                                pos += a >> 8;
                                if (s) { k += (int)r + 1; pos += s; }
                                else if (r == 15) k += 16;
                                else break;
                            }
                            bad = bad || pos > nbits;
                        }
                    }
                }
                continue;
            }
            uint64_t* h = nz[c0].data();
            uint32_t col = m0 % sd.mcu_w;
            h += (size_t)(m0 / sd.mcu_w) * img.bw[c0];
            for (uint32_t m = m0; m < m1 && !bad; m++) {
                if (sd.ri == 0 && m >= next_entry && eobrun == 0 && E.size() < kMaxEntriesPerScan) entry(m);
                int run;
                if (eobrun) {
                    if (sd.Ah > 0) pos += bmi2 ? walk_popcount<true>(h[col] & band) : walk_popcount<false>(h[col] & band);
                    run = (int)eobrun;
                } else if (sd.Ah == 0) run = walk_first_block(d, walk, &pos, &h[col], sd.Ss, sd.Se);
                else run = bmi2 ? walk_refine_block<true>(d, walk, &pos, &h[col], band) : walk_refine_block<false>(d, walk, &pos, &h[col], band);
                bad = run < 0 || pos > nbits;
                eobrun = run > 0 ? (uint32_t)run - 1u : 0u;
                if (++col == sd.mcu_w) { col = 0; h += img.bw[c0]; }
            }
        }
        if (bad) { E.clear(); return kOk; }                         // no entries from here on: later scans build on this one
    }
    return kOk;
}

struct IndexedPlan {
    RecordPlan P;
    uint32_t interval = 0;
    std::vector<std::vector<EntryPoint>> ent;                    // [n * kMaxScansPerFile]
};

inline int plan_record_indexed(const void* const* files, const size_t* sizes, uint32_t n, uint32_t interval, IndexedPlan* Q) {
    int rc = plan_record(files, sizes, n, &Q->P);
    if (rc) return rc;
    Q->interval = interval;
    Q->ent.assign((size_t)n * kMaxScansPerFile, std::vector<EntryPoint>());
    std::atomic<uint32_t> next(0);
    auto work = [&]() {
        for (;;) {
            const uint32_t i = next.fetch_add(1);
            if (i >= n) break;
            (void)find_entry_points((const uint8_t*)files[i], &Q->P.ends[(size_t)i * kMaxScansPerFile], Q->P.nscans[i], interval,
                                    &Q->ent[(size_t)i * kMaxScansPerFile]);   // (a file the walk refuses simply has no entries)
        }
    };
    if (!on_threads(std::max(1u, std::min({16u, std::thread::hardware_concurrency(), n})), work)) return kENoMem;
    uint64_t entry_bytes_total = 0;
    for (const auto& e : Q->ent) entry_bytes_total += e.size() * (uint64_t)((!e.empty() && e[0].zero) ? kEntryBytesShort : kEntryBytes);
    const uint64_t raw = hdr_ecount_pos(n, Q->P.G, Q->P.G, 0);
    Q->P.header_bytes = (raw + 63) / 64 * 64;
    uint64_t payload = 0;
    for (uint32_t i = 0; i < n; i++) payload += sizes[i];
    Q->P.total = Q->P.header_bytes + payload + entry_bytes_total;
    if (Q->P.total >= (1ull << 32)) return kEUnsupported;
    return kOk;
}

inline void write_record_indexed(const IndexedPlan& Q, const void* const* files, const int32_t* labels, uint8_t* out) {
    const RecordPlan& P = Q.P;
    const uint32_t n = P.n, G = P.G;
    memset(out, 0, P.header_bytes);
    memcpy(out, "PCR1", 4);
    st_le32(out + 4, 2); st_le32(out + 8, n); st_le32(out + 12, G); st_le64(out + 16, P.header_bytes);
    st_le32(out + hdr_entry_interval_pos(n, G), Q.interval);
    uint64_t pos = P.header_bytes;
    for (uint32_t g = 0; g < G; g++) {
        for (uint32_t i = 0; i < n; i++) {
            uint32_t len = 0;
            if (g < P.nscans[i]) {
                const uint64_t* e = &P.ends[(size_t)i * kMaxScansPerFile];
                const uint64_t from = g ? e[g - 1] : 0;
                len = (uint32_t)(e[g] - from);
                memcpy(out + pos, (const uint8_t*)files[i] + from, len);
                pos += len;
            }
            st_le32(out + hdr_len_pos(n, G, g, i), len);
        }
        for (uint32_t i = 0; i < n; i++) {                          // the group's entries behind its regions
            const std::vector<EntryPoint>& E = Q.ent[(size_t)i * kMaxScansPerFile + g];
            uint8_t* c = out + hdr_ecount_pos(n, G, g, i);
            const bool brief = !E.empty() && E[0].zero;            // an AC scan: no DC predictions to carry
            const uint32_t field = (uint32_t)E.size() | (brief ? kEntryShortFlag : 0u);
            c[0] = (uint8_t)field; c[1] = (uint8_t)(field >> 8);
            for (const EntryPoint& e : E) {
                st_le32(out + pos, e.mcu); st_le32(out + pos + 4, e.bit);
                if (brief) { pos += kEntryBytesShort; continue; }
                for (int j = 0; j < 3; j++) { out[pos + 8 + 2 * j] = (uint8_t)(uint16_t)e.pred[j]; out[pos + 9 + 2 * j] = (uint8_t)((uint16_t)e.pred[j] >> 8); }
                out[pos + 14] = out[pos + 15] = 0;
                pos += kEntryBytes;
            }
        }
        st_le64(out + hdr_group_end_pos(g), pos);
    }
    for (uint32_t i = 0; i < n; i++) {
        st_le32(out + hdr_label_pos(G, i), labels ? (uint32_t)labels[i] : 0u);
        st_le32(out + hdr_nscans_pos(n, G, i), P.nscans[i]);
    }
}

// ---- progressive encoder --------------------------------------------------------------------------------
// A scan is first turned into tokens (Huffman symbol of one of two table slots + appended bits, or appended
// bits alone), the symbol counts give the scan its own optimal tables, then the tokens are written out.
struct Token { uint8_t slot; uint8_t sym; uint8_t nbits; uint16_t bits; };   // slot 0/1: Huffman table of the scan; 2: bits only; 3: restart marker number sym
constexpr uint8_t kRawBits = 2, kRestartMark = 3;

struct HuffSpec { uint8_t counts[17]; uint8_t symbols[256]; int nsym; uint16_t code[256]; uint8_t size[256]; };

// Code lengths from symbol counts, no code longer than 16 bits and none made of 1-bits only (the procedure of
// the JPEG specification's Annex K.2: a reserved extra symbol takes the all-ones code).
inline void build_table(const uint32_t freq_in[256], HuffSpec* H) {
    long freq[257]; int codesize[257], others[257];
    for (int i = 0; i < 256; i++) freq[i] = (long)freq_in[i];
    freq[256] = 1;
    for (int i = 0; i < 257; i++) { codesize[i] = 0; others[i] = -1; }
    // The symbols that occur, in order; one pass finds the two least (ties: the larger index), the second of which then
    // leaves the list.
    int live[257], nlive = 0;
    for (int i = 0; i < 257; i++) if (freq[i] > 0) live[nlive++] = i;
    while (nlive > 1) {
        int a1 = -1, a2 = -1;
        for (int e = 0; e < nlive; e++) {
            if (a1 < 0 || freq[live[e]] <= freq[live[a1]]) { a2 = a1; a1 = e; }
            else if (a2 < 0 || freq[live[e]] <= freq[live[a2]]) a2 = e;
        }
        const int c1 = live[a1], c2 = live[a2];
        freq[c1] += freq[c2];
        for (int e = a2; e + 1 < nlive; e++) live[e] = live[e + 1];
        nlive--;
        for (int v = c1;; v = others[v]) { codesize[v]++; if (others[v] < 0) { others[v] = c2; break; } }
        for (int v = c2; v >= 0; v = others[v]) codesize[v]++;
    }
    int bits[64] = {0};
    for (int i = 0; i < 257; i++) if (codesize[i]) bits[codesize[i] > 63 ? 63 : codesize[i]]++;
    for (int i = 63; i > 16; i--) {
        while (bits[i] > 0) {
            int j = i - 2;
            while (bits[j] == 0) j--;
            bits[i] -= 2; bits[i - 1] += 1; bits[j + 1] += 2; bits[j] -= 1;
        }
    }
    int longest = 16;
    while (longest > 0 && bits[longest] == 0) longest--;
    if (longest > 0) bits[longest]--;                          // the reserved symbol
    H->counts[0] = 0;
    for (int l = 1; l <= 16; l++) H->counts[l] = (uint8_t)bits[l];
    // symbols in order of code length; inside one length in order of value
    H->nsym = 0;
    for (int l = 1; l <= 63; l++)
        for (int s = 0; s < 256; s++) if (codesize[s] == l) H->symbols[H->nsym++] = (uint8_t)s;
    // canonical codes
    for (int s = 0; s < 256; s++) { H->code[s] = 0; H->size[s] = 0; }
    uint32_t code = 0; int k = 0;
    for (int l = 1; l <= 16; l++) {
        for (int c = 0; c < H->counts[l]; c++, k++) { H->code[H->symbols[k]] = (uint16_t)code; H->size[H->symbols[k]] = (uint8_t)l; code++; }
        code <<= 1;
    }
}

// Bits into bytes, four at a time (one by one where a byte of the four is 0xFF and takes a zero behind it).
class BitWriter {
public:
    explicit BitWriter(std::vector<uint8_t>* out) : out_(out), pos_(out->size()) {}
    void put(uint32_t bits, int n) {                           // n <= 32
        acc_ = (acc_ << n) | (bits & (uint32_t)((1ull << n) - 1u)); have_ += n;
        if (have_ < 32) return;
        const uint32_t w = (uint32_t)(acc_ >> (have_ - 32));
        have_ -= 32;
        room(8);
        if (((~w - 0x01010101u) & w & 0x80808080u) == 0) {     // no byte is 0xFF
            uint8_t* p = out_->data() + pos_;
            p[0] = (uint8_t)(w >> 24); p[1] = (uint8_t)(w >> 16); p[2] = (uint8_t)(w >> 8); p[3] = (uint8_t)w;
            pos_ += 4;
        } else for (int s = 24; s >= 0; s -= 8) byte((uint8_t)(w >> s));
    }
    void finish() {                                            // pad with 1-bits
        const int pad = (8 - have_ % 8) % 8;
        acc_ = (acc_ << pad) | ((1u << pad) - 1u); have_ += pad;
        room(16);
        for (; have_ > 0; have_ -= 8) byte((uint8_t)(acc_ >> (have_ - 8)));
        have_ = 0;
        out_->resize(pos_);
    }
    void marker(uint8_t m) { finish(); out_->push_back(0xFF); out_->push_back(m); pos_ = out_->size(); }
private:
    void room(size_t n) { if (out_->size() - pos_ < n) out_->resize(out_->size() + out_->size() / 2 + 4096); }
    void byte(uint8_t b) { (*out_)[pos_++] = b; if (b == 0xFF) (*out_)[pos_++] = 0x00; }
    std::vector<uint8_t>* out_; size_t pos_;                   // (the vector is longer than what is written, until finish())
    uint64_t acc_ = 0; int have_ = 0;
};

// Which positions of a block (bit k: zig-zag position k) are not zero after the point transform by 0, 1 and 2 bits: what
// the coders below walk over instead of 64 coefficients per block and scan.
struct BlockMasks {
    std::vector<uint64_t> nz[3];
    void fill(const int16_t* plane, size_t blocks) {
        // the order of a mask's bits is changed eight of them at a time
        static const std::vector<uint64_t> order = [] {
            std::vector<uint64_t> t(8 * 256, 0);
            const ZigzagTable zz;
            for (int k = 0; k < 64; k++)
                for (int v = 0; v < 256; v++) if (v >> (zz.natural[k] & 7) & 1) t[(size_t)(zz.natural[k] >> 3) * 256 + v] |= 1ull << k;
            return t;
        }();
        for (auto& m : nz) m.resize(blocks);
        for (size_t b = 0; b < blocks; b++) {
            uint64_t flat[3];
            natural_masks(plane + b * 64, flat);
            for (int s = 0; s < 3; s++) {
                uint64_t m = 0;
                for (int r = 0; r < 8; r++) m |= order[(size_t)r * 256 + (flat[s] >> (8 * r) & 255)];
                nz[s][b] = m;
            }
        }
    }
    static void natural_masks(const int16_t* c, uint64_t flat[3]) {
        flat[0] = flat[1] = flat[2] = 0;
#if defined(__SSE2__) && !defined(__HIP_DEVICE_COMPILE__)
        const __m128i zero = _mm_setzero_si128(), one = _mm_set1_epi16(1), three = _mm_set1_epi16(3);
        for (int q = 0; q < 4; q++) {
            __m128i a = _mm_loadu_si128((const __m128i*)(c + 16 * q)), b = _mm_loadu_si128((const __m128i*)(c + 16 * q + 8));
            a = _mm_max_epi16(a, _mm_subs_epi16(zero, a)); b = _mm_max_epi16(b, _mm_subs_epi16(zero, b));
            flat[0] |= (uint64_t)(uint32_t)_mm_movemask_epi8(_mm_packs_epi16(_mm_cmpgt_epi16(a, zero), _mm_cmpgt_epi16(b, zero))) << (16 * q);
            flat[1] |= (uint64_t)(uint32_t)_mm_movemask_epi8(_mm_packs_epi16(_mm_cmpgt_epi16(a, one), _mm_cmpgt_epi16(b, one))) << (16 * q);
            flat[2] |= (uint64_t)(uint32_t)_mm_movemask_epi8(_mm_packs_epi16(_mm_cmpgt_epi16(a, three), _mm_cmpgt_epi16(b, three))) << (16 * q);
        }
#else
        for (int k = 0; k < 64; k++) {
            const int mag = c[k] < 0 ? -(int)c[k] : c[k];
            flat[0] |= (uint64_t)(mag > 0) << k; flat[1] |= (uint64_t)(mag > 1) << k; flat[2] |= (uint64_t)(mag > 3) << k;
        }
#endif
    }
};

struct Frame {
    int W, H, nc, hmax, vmax;
    int hs[kMaxComp], vs[kMaxComp], tq[kMaxComp], cid[kMaxComp];
    int bw[kMaxComp], bh[kMaxComp], cw[kMaxComp], ch[kMaxComp], mcux, mcuy;
    const int16_t* plane[kMaxComp];                            // [bh][bw][64], natural order inside a block
    BlockMasks masks[kMaxComp];
};

struct ScanSpec { int ns, comp[kMaxComp], Ss, Se, Ah, Al; };

inline int bit_length(int v) { return v ? 32 - __builtin_clz((unsigned)v) : 0; }

// Where a scan's symbols go: a list of tokens, or, with the tables known beforehand, straight into the file.
class TokenSink {
public:
    std::vector<Token> tokens;
    void symbol(uint8_t slot, uint8_t sym, int nbits, uint32_t bits) { tokens.push_back(Token{slot, sym, (uint8_t)nbits, (uint16_t)(bits & 0xFFFFu)}); }
    void raw(uint64_t bits, int n) {
        while (n > 0) { const int take = n < 16 ? n : 16; symbol(kRawBits, 0, take, (uint32_t)(bits >> (n - take)) & ((1u << take) - 1u)); n -= take; }
    }
    void restart(uint8_t m) { tokens.push_back(Token{kRestartMark, m, 0, 0}); }
};
class FileSink {
public:
    FileSink(BitWriter* w, const HuffSpec* H) : w_(w), H_(H) {}
    bool unknown = false;                                      // a symbol the tables hold no code for
    void symbol(uint8_t slot, uint8_t sym, int nbits, uint32_t bits) {
        const int size = H_[slot].size[sym];
        unknown = unknown || size == 0;
        w_->put((uint32_t)H_[slot].code[sym] << nbits | (bits & ((1u << nbits) - 1u)), size + nbits);     // (16 + 16 bits at most)
    }
    void raw(uint64_t bits, int n) {
        if (n > 32) { w_->put((uint32_t)(bits >> (n - 32)), 32); n -= 32; }
        w_->put((uint32_t)bits, n);
    }
    void restart(uint8_t m) { w_->marker((uint8_t)(0xD0 + m)); }
private:
    BitWriter* w_; const HuffSpec* H_;
};

template <class Sink> class ScanCoder {
public:
    // restart_mcus: MCUs of this scan per restart interval (0: no restart markers)
    ScanCoder(const Frame& F, const ScanSpec& S, uint32_t restart_mcus, Sink* sink) : F_(F), S_(S), sink_(*sink), ri_(restart_mcus) {}
    void run() { if (S_.Ss == 0) dc_scan(); else ac_scan(); }

private:
    const Frame& F_; const ScanSpec& S_; Sink& sink_;
    uint32_t ri_, mcu_ = 0, marks_ = 0;                        // restart interval, MCUs begun, markers written
    int pred_[kMaxComp] = {0, 0, 0};                           // DC predictions
    // end-of-band run shared by the blocks of an AC scan, and the correction bits that wait behind it
    struct Bits { uint64_t v; int n; };
    uint32_t eobrun_ = 0;
    std::vector<Bits> pending_;
    const ZigzagTable zz_;

    // A restart interval ends: whatever is pending goes out, a marker follows, predictions start again.
    void begin_mcu() {
        if (ri_ && mcu_ && mcu_ % ri_ == 0) {
            flush_eobrun();
            sink_.restart((uint8_t)(marks_++ & 7));
            pred_[0] = pred_[1] = pred_[2] = 0;
        }
        mcu_++;
    }
    // fn(component of the scan, component, number of the block in its plane)
    template <class Fn> void for_each_block(Fn fn) {
        if (S_.ns > 1) {
            for (int my = 0; my < F_.mcuy; my++) for (int mx = 0; mx < F_.mcux; mx++) {
                begin_mcu();
                for (int j = 0; j < S_.ns; j++) {
                    const int c = S_.comp[j];
                    for (int by = 0; by < F_.vs[c]; by++) for (int bx = 0; bx < F_.hs[c]; bx++)
                        fn(j, c, (size_t)(my * F_.vs[c] + by) * F_.bw[c] + (size_t)(mx * F_.hs[c] + bx));
                }
            }
        } else {
            const int c = S_.comp[0];
            for (int row = 0; row < F_.ch[c]; row++) for (int col = 0; col < F_.cw[c]; col++) { begin_mcu(); fn(0, c, (size_t)row * F_.bw[c] + col); }
        }
    }

    void dc_scan() {
        for_each_block([&](int j, int c, size_t block) {
            const int v = (int)F_.plane[c][block * 64] >> S_.Al;      // arithmetic shift: the point transform of DC
            if (S_.Ah == 0) {
                int diff = v - pred_[c]; pred_[c] = v;
                const int nb = bit_length(diff < 0 ? -diff : diff);
                sink_.symbol((uint8_t)(j == 0 ? 0 : 1), (uint8_t)nb, nb, (uint32_t)(diff < 0 ? diff - 1 : diff));
            } else {
                sink_.raw((uint64_t)(v & 1), 1);
            }
        });
    }

    void flush_eobrun() {
        if (eobrun_ > 0) {
            const int n = bit_length((int)eobrun_) - 1;
            sink_.symbol(0, (uint8_t)(n << 4), n, eobrun_ - (1u << n));
            eobrun_ = 0;
        }
        for (const Bits& b : pending_) sink_.raw(b.v, b.n);
        pending_.clear();
    }

    void ac_scan() {
        const uint64_t band = (S_.Se >= 63 ? ~0ull : (1ull << (S_.Se + 1)) - 1) & ~((1ull << S_.Ss) - 1);
        for_each_block([&](int, int c, size_t block) {
            const int16_t* b = F_.plane[c] + block * 64;
            const uint64_t here = F_.masks[c].nz[S_.Al][block] & band;
            if (S_.Ah == 0) ac_first_block(b, here); else ac_refine_block(b, here, F_.masks[c].nz[S_.Al + 1][block]);
        });
        flush_eobrun();
    }

    void ac_first_block(const int16_t* b, uint64_t m) {
        int prev = S_.Ss - 1;
        if (m) flush_eobrun();
        for (; m; m &= m - 1) {
            const int k = __builtin_ctzll(m), c = b[zz_.natural[k]];
            const int mag = (c < 0 ? -c : c) >> S_.Al;         // magnitudes are shifted, not the signed value
            int run = k - prev - 1;
            prev = k;
            while (run > 15) { sink_.symbol(0, 0xF0, 0, 0); run -= 16; }
            const int nb = bit_length(mag);
            sink_.symbol(0, (uint8_t)((run << 4) | nb), nb, (uint32_t)(c < 0 ? ~mag : mag));
        }
        if (prev < S_.Se) { if (++eobrun_ == 0x7FFF) flush_eobrun(); }
    }

    // m: positions of the band that are not zero; known: those that were not zero before this scan
    void ac_refine_block(const int16_t* b, uint64_t m, uint64_t known) {
        const uint64_t fresh = m & ~known;
        const int last_new = fresh ? 63 - __builtin_clzll(fresh) : -1;   // last position that becomes non-zero in this scan
        int run = 0, prev = S_.Ss - 1;
        Bits corr{0, 0};                                       // correction bits met since the last symbol
        for (; m; m &= m - 1) {
            const int k = __builtin_ctzll(m), c = b[zz_.natural[k]];
            run += k - prev - 1;
            prev = k;
            while (run > 15 && k <= last_new) {                // sixteen zeros, only where a new coefficient still follows
                flush_eobrun();
                sink_.symbol(0, 0xF0, 0, 0);
                run -= 16;
                sink_.raw(corr.v, corr.n); corr = Bits{0, 0};
            }
            if (known >> k & 1) {                              // one more bit of it
                corr.v = corr.v << 1 | (uint64_t)(((c < 0 ? -c : c) >> S_.Al) & 1);
                corr.n++;
                continue;
            }
            flush_eobrun();
            sink_.symbol(0, (uint8_t)((run << 4) | 1), 1, c < 0 ? 0u : 1u);
            sink_.raw(corr.v, corr.n); corr = Bits{0, 0};
            run = 0;
        }
        if (run + (S_.Se - prev) > 0 || corr.n) {
            eobrun_++;
            if (corr.n) {
                if (!pending_.empty() && pending_.back().n + corr.n <= 64) pending_.back() = Bits{pending_.back().v << corr.n | corr.v, pending_.back().n + corr.n};
                else pending_.push_back(corr);
            }
            if (eobrun_ == 0x7FFF) flush_eobrun();
        }
    }
};

inline void put_be16(std::vector<uint8_t>* o, uint32_t v) { o->push_back((uint8_t)(v >> 8)); o->push_back((uint8_t)v); }

inline void write_dht(std::vector<uint8_t>* o, int cls, int id, const HuffSpec& H) {
    o->push_back(0xFF); o->push_back(0xC4);
    put_be16(o, (uint32_t)(2 + 1 + 16 + H.nsym));
    o->push_back((uint8_t)((cls << 4) | id));
    for (int l = 1; l <= 16; l++) o->push_back(H.counts[l]);
    for (int k = 0; k < H.nsym; k++) o->push_back(H.symbols[k]);
}

// The script of the files written here (pcr_hist.h: the device counts the symbols of the same scans).
inline std::vector<ScanSpec> default_script(int nc) {
    std::vector<ScanSpec> s;
    for (int i = 0; i < script_scans(nc); i++) {
        const ScriptScan t = script_scan(nc, i);
        s.push_back(ScanSpec{t.ns, {t.comp[0], t.comp[1], t.comp[2]}, t.Ss, t.Se, t.Ah, t.Al});
    }
    return s;
}

// The frame of a file (its header and quantisation tables) whose coefficients, coef_count of them from `coef` on (null: elsewhere), are
// to be coded.
inline int read_frame(const uint8_t* src, size_t src_bytes, const int16_t* coef, size_t coef_count, ImgDesc* img_out, Frame* frame) {
    if (src_bytes >= (1ull << 32)) return kEUnsupported;
    ImgDesc& img = *img_out; memset(&img, 0, sizeof img);
    ScanDesc first; memset(&first, 0, sizeof first);
    RegionWalk w;
    int rc = walk_region(src, 0, (uint32_t)src_bytes, 0, &w, &img);                   // up to the first scan header
    if (rc == kOk) rc = resolve_scan(w, (uint32_t)src_bytes, w.dht, w.ri >= 0 ? (uint32_t)w.ri : 0u, &img, &first);
    if (rc == kOk) rc = scan_history(&first, 0);
    for (int t = 0; t < 4; t++) { img.qoff[t] = w.qoff[t]; img.qprec[t] = w.qprec[t]; }
    if (rc != kOk) return rc;
    Frame& F = *frame;
    F.W = img.W; F.H = img.H; F.nc = img.nc; F.hmax = img.hmax; F.vmax = img.vmax; F.mcux = img.mcux; F.mcuy = img.mcuy;
    size_t need = 0;
    for (int c = 0; c < img.nc; c++) {
        F.hs[c] = img.hs[c]; F.vs[c] = img.vs[c]; F.tq[c] = img.tq[c]; F.cid[c] = img.cid[c];
        F.bw[c] = img.bw[c]; F.bh[c] = img.bh[c]; F.cw[c] = img.cw[c]; F.ch[c] = img.ch[c];
        if (!img.qoff[img.tq[c]]) return kEFormat;
        F.plane[c] = coef ? coef + need : nullptr;
        need += (size_t)img.bw[c] * img.bh[c] * 64;
    }
    if (need != coef_count) return kERange;
    return kOk;
}

// What stands in a progressive file before its scans.
inline void write_file_head(const uint8_t* src, const ImgDesc& img, const Frame& F, uint32_t restart_interval, std::vector<uint8_t>* out) {
    std::vector<uint8_t>& o = *out;
    o.push_back(0xFF); o.push_back(0xD8);
    bool done[4] = {false, false, false, false};
    for (int c = 0; c < img.nc; c++) {
        const int t = img.tq[c];
        if (done[t]) continue;
        done[t] = true;
        const int bytes = 64 * (img.qprec[t] + 1);
        o.push_back(0xFF); o.push_back(0xDB);
        put_be16(&o, (uint32_t)(2 + 1 + bytes));
        o.push_back((uint8_t)((img.qprec[t] << 4) | t));
        o.insert(o.end(), src + img.qoff[t], src + img.qoff[t] + bytes);
    }
    o.push_back(0xFF); o.push_back(0xC2);
    put_be16(&o, (uint32_t)(8 + 3 * img.nc));
    o.push_back(8); put_be16(&o, img.H); put_be16(&o, img.W); o.push_back((uint8_t)img.nc);
    for (int c = 0; c < img.nc; c++) { o.push_back((uint8_t)F.cid[c]); o.push_back((uint8_t)((img.nc == 1 ? 1 : F.hs[c]) << 4 | (img.nc == 1 ? 1 : F.vs[c]))); o.push_back((uint8_t)F.tq[c]); }
    if (restart_interval) {
        o.push_back(0xFF); o.push_back(0xDD);
        put_be16(&o, 4); put_be16(&o, restart_interval);
    }
}

// What stands in front of a scan's data behind its tables.
inline void write_scan_head(const Frame& F, const ScanSpec& S, std::vector<uint8_t>* out) {
    std::vector<uint8_t>& o = *out;
    o.push_back(0xFF); o.push_back(0xDA);
    put_be16(&o, (uint32_t)(6 + 2 * S.ns));
    o.push_back((uint8_t)S.ns);
    for (int j = 0; j < S.ns; j++) {
        o.push_back((uint8_t)F.cid[S.comp[j]]);
        const int slot = (S.Ss == 0 && j > 0) ? 1 : 0;
        o.push_back((uint8_t)(S.Ss == 0 ? (slot << 4) : slot));
    }
    o.push_back((uint8_t)S.Ss); o.push_back((uint8_t)S.Se); o.push_back((uint8_t)((S.Ah << 4) | S.Al));
}

// How many of n bytes are 0xFF.
inline size_t count_ff(const uint8_t* d, size_t n) {
    size_t all = 0;
    while (n > 0) {                                            // (sums of bytes, which a compiler adds up sixteen at a time)
        const size_t m = std::min<size_t>(n, 240);
        uint8_t some = 0;
        for (size_t i = 0; i < m; i++) some = (uint8_t)(some + (d[i] == 0xFF ? 1 : 0));
        all += some; d += m; n -= m;
    }
    return all;
}

// The progressive file of a frame from what the device made of its coefficients (pcr_coder.h): specs, the tables of its scans (two each);
// bits, how many every scan has (kScriptScansMax); words, the scan's first words, number word_off[scan] of them on.  Returns how
// many bytes it has, and writes them to dst if there is room for them, or else nothing.  (Straight to where they go: by way of a vector,
// with the pages that takes, 64 photographs took longer with sixteen threads than with one.)
inline size_t assemble_progressive(const uint8_t* src, const ImgDesc& img, const Frame& F, const CodeSpec* specs, const uint64_t* bits,
                                   const uint32_t* words, const uint64_t* word_off, uint8_t* dst, size_t room) {
    const std::vector<ScanSpec> script = default_script(img.nc);
    std::vector<uint8_t> head;                                 // what stands ahead of the data of the scans, one behind the other
    std::vector<size_t> ends(script.size());
    write_file_head(src, img, F, 0, &head);
    size_t size = 2;
    auto data_of = [&](size_t at) { return reinterpret_cast<const uint8_t*>(words + word_off[at]); };
    auto bytes_of = [&](size_t at) { return (size_t)((bits[at] + 7) / 8); };
    for (size_t at = 0; at < script.size(); at++) {
        const ScanSpec& S = script[at];
        for (int s = 0; s < 2; s++) {
            const CodeSpec& C = specs[2 * at + s];
            if (C.nsym == 0) continue;
            HuffSpec H;
            H.nsym = (int)C.nsym;
            memcpy(H.counts + 1, C.counts, 16);
            memcpy(H.symbols, C.symbols, C.nsym);
            write_dht(&head, S.Ss == 0 ? 0 : 1, s, H);
        }
        write_scan_head(F, S, &head);
        ends[at] = head.size();
        size += bytes_of(at) + count_ff(data_of(at), bytes_of(at));
    }
    size += head.size();
    if (size > room) return size;
    auto put = [&](const uint8_t* p, size_t n) { memcpy(dst, p, n); dst += n; };
    for (size_t at = 0; at < script.size(); at++) {
        const size_t from = at ? ends[at - 1] : 0;
        put(head.data() + from, ends[at] - from);
        const uint8_t* d = data_of(at);
        for (size_t left = bytes_of(at); left > 0;) {          // a zero behind every byte 0xFF
            const void* ff = memchr(d, 0xFF, left);
            const size_t n = ff ? (size_t)((const uint8_t*)ff - d) + 1 : left;
            put(d, n);
            if (ff) *dst++ = 0;
            d += n; left -= n;
        }
    }
    *dst++ = 0xFF; *dst++ = 0xD9;
    return size;
}

// src: a JPEG file (baseline or progressive) whose frame header and quantisation tables are kept; coef: its
// quantised coefficients, component planes one after the other, each [bh][bw][64] in natural order over the
// MCU-padded block grid.  Appends the progressive file to *out.
// restart_interval: MCUs of each scan between restart markers (0: none; a scan of one component counts its blocks).
// counts (optional): the symbol counts of the scans, [scan][table slot][symbol] (kHistPerImage entries, as k_symbol_hist
// writes them), used for the Huffman tables instead of counting the tokens here.  counts_out (optional): receives the
// counts of the tokens; with it and out == nullptr nothing is written.
inline int transcode_progressive(const uint8_t* src, size_t src_bytes, const int16_t* coef, size_t coef_count, uint32_t restart_interval,
                                 std::vector<uint8_t>* out, const uint32_t* counts = nullptr, uint32_t* counts_out = nullptr) {
    std::vector<uint8_t> scratch;
    if (!out) out = &scratch;
    if (counts_out) memset(counts_out, 0, sizeof(uint32_t) * kHistPerImage);
    if (src_bytes >= (1ull << 32)) return kEUnsupported;
    if (restart_interval > 65535) return kERange;
    ImgDesc img; Frame F;
    const int rc = read_frame(src, src_bytes, coef, coef_count, &img, &F);
    if (rc != kOk) return rc;
    for (int c = 0; c < img.nc; c++) F.masks[c].fill(F.plane[c], (size_t)img.bw[c] * img.bh[c]);
    std::vector<uint8_t>& o = *out;
    write_file_head(src, img, F, restart_interval, out);
    int scan_index = -1;
    for (const ScanSpec& S : default_script(img.nc)) {
        scan_index++;
        TokenSink list;                                            // (only where the symbols are counted here)
        if (!counts) ScanCoder<TokenSink>(F, S, restart_interval, &list).run();
        uint32_t freq[2][256];
        memset(freq, 0, sizeof freq);
        bool used[2] = {false, false};
        if (counts) {
            memcpy(freq, counts + (size_t)scan_index * kHistPerScan, sizeof freq);
            for (int s2 = 0; s2 < 2; s2++) for (int y = 0; y < 256; y++) if (freq[s2][y]) used[s2] = true;
        } else {
            for (const Token& t : list.tokens) if (t.slot < kRawBits) { freq[t.slot][t.sym]++; used[t.slot] = true; }
        }
        if (counts_out) memcpy(counts_out + (size_t)scan_index * kHistPerScan, freq, sizeof freq);
        HuffSpec H[2];
        const int cls = S.Ss == 0 ? 0 : 1;
        for (int s = 0; s < 2; s++) {
            if (used[s]) { build_table(freq[s], &H[s]); write_dht(&o, cls, s, H[s]); }
            else memset(H[s].size, 0, sizeof H[s].size);
        }
        write_scan_head(F, S, &o);
        BitWriter bw(&o);
        FileSink file(&bw, H);
        if (counts) {
            ScanCoder<FileSink>(F, S, restart_interval, &file).run();
            if (file.unknown) return kEFormat;                     // the counts do not fit the coefficients
        } else {
            for (const Token& t : list.tokens) {
                if (t.slot == kRestartMark) file.restart(t.sym);
                else if (t.slot == kRawBits) file.raw(t.bits, t.nbits);
                else file.symbol(t.slot, t.sym, t.nbits, t.bits);
            }
        }
        bw.finish();
    }
    o.push_back(0xFF); o.push_back(0xD9);
    return kOk;
}

}  // namespace enc
}  // namespace pcr
