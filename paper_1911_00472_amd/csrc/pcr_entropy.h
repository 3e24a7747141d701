// Progressive-JPEG entropy decoding for one independently decodable unit (a restart interval
// of one scan of one image), written so that the same code runs in a gfx950 lane and on the
// host.  Decoding follows the JPEG progressive mode (spectral selection + successive
// approximation) that the paper's records are made of (Section 2, "Progressive Image
// Compression"; Section 3: scan k of an image is usable once scans 1..k have been read).
//
// Input is the *unstuffed* entropy-coded data of the unit (FF 00 -> FF, restart markers
// removed); consuming a bit past the unit's end is a data error, never a guess.
//
// Shape of the decoders: ONE WAVEFRONT DECODES ONE UNIT.  Every value below is then the same in
// all 64 lanes, so the compiler keeps it in scalar registers and the loops run on the scalar
// ALU (native 64-bit shifts, population count, find-first-set), paying only for the branch
// actually taken.  All per-scan parameters are passed in registers (LaneScan); the Huffman
// table lives in LDS.
//
// AC refinement is decoded against a 64-bit "already non-zero" mask per block (zig-zag bit
// order) instead of against the coefficients: the serial decoder only finds where new
// coefficients go, their signs, and the string of correction bits (exactly one per already
// non-zero coefficient of the band, in zig-zag order); the arithmetic on the coefficients is
// data-parallel (refine_apply).  DC refinement needs no serial decoder at all: it is one
// bit per block at a position known in advance (dc_refine_bit).
#pragma once
#include "pcr_common.h"

namespace pcr {

// ---------------------------------------------------------------------------------------
// Huffman tables.  Codes of <= 8 bits resolve through `lut`, indexed by the next 8 bits.  In a
// canonical code the longer code words are the numerically largest ones, so all of them lie in
// [limit8, 65536) when left-aligned in 16 bits; `lut2`, indexed by the distance from limit8
// scaled to 128 entries, resolves every long code that owns at least one whole entry, and the
// canonical limits resolve the rest (of a photograph's tables under one symbol in 10 000).  The two look-ups lie one
// behind the other, so that a lane picks its index into either and reads once.  An entry (code_entry) is what a decoder
// needs of the symbol, taken apart; 0 means "not here".
// ---------------------------------------------------------------------------------------
struct AcTab {
    uint16_t lut[256];
    uint16_t lut2[128];         // (right behind lut)
    uint32_t limit[9];          // limit[L-8]: first 16-bit-left-aligned code value NOT of length <= L (L = 8..16)
    uint16_t valptr[8];         // valptr[L-9]: index in huffval of the first code of length L
    uint32_t sh2;               // lut2 index = (code16 - limit[0]) >> sh2
    uint8_t huffval[256];
    uint32_t pad[2];            // (what comes before lutp is copied in 16-byte pieces)
    // both look-ups again, pre-packed for the lanes of a window reader (see packed_entry): everything
    // of a symbol's packed word that does not depend on the bits after the code
    uint32_t lutp[256 + 128];
};
static_assert(sizeof(AcTab) == 1088 + 1536 && sizeof(AcTab) % 16 == 0 && offsetof(AcTab, lut2) == 512, "AcTab layout");

// An AC symbol with a code of `len` bits: bits 0..3 how many bits follow the code (the value of a coefficient, the length
// of an end-of-band run), bits 4..7 the zeros ahead of the position it lands on (0 for an end of band), bits 8..12 len,
// bit 13 end of band, bit 14 coefficient.
constexpr uint32_t kCodeEob = 0x2000u, kCodeCoef = 0x4000u;
PCR_HD uint32_t code_entry(uint32_t len, uint32_t sym) {
    const uint32_t r = sym >> 4, s = sym & 15u;
    if (s) return kCodeCoef | (len << 8) | sym;
    return r == 15u ? (len << 8) | 0xF0u : kCodeEob | (len << 8) | r;
}
// ... and back: (length << 8) | symbol
PCR_HD uint32_t entry_code(uint32_t e) { return (e & 0x1F00u) | ((e & kCodeEob) ? (e & 15u) << 4 : e & 255u); }

// A canonical code's lengths, for building look-ups entry by entry: lim[L] = first left-aligned 16-bit value that is not
// a code of length <= L (so codes of length L occupy lim[L-1] .. lim[L]), first[L] = index of the first code of length L.
struct CanonCode { uint32_t lim[17]; uint32_t first[17]; uint8_t vals[256]; };

// (length << 8) | index of the code at the head of the left-aligned 16-bit value c16; 0 if none of the lengths kLo .. kHi.
// (The limits are counted, not searched: eight reads of LDS that wait for nothing, then two for the length found.)
template <int kLo, int kHi>
PCR_HD uint32_t canon_find(const CanonCode* c, uint32_t c16) {
    uint32_t L = kLo;
#pragma unroll
    for (int q = kLo; q < kHi; q++) L += c16 >= c->lim[q] ? 1u : 0u;
    const uint32_t below = c->lim[L - 1], idx = c->first[L] + ((c16 - below) >> (16 - L));
    return (c16 < c->lim[kHi] && c16 >= below && idx < 256u) ? (L << 8) | idx : 0u;
}

struct DcTab {                  // DC symbols are categories 0..15
    uint8_t lut[256];           // (length << 4) | symbol for codes of <= 8 bits, 0xFF otherwise
    uint32_t limit[9];
    uint16_t valptr[8];
    uint8_t huffval[16];
};
static_assert(sizeof(DcTab) == 324, "DcTab layout");

// Build from a DHT payload: 16 counts followed by the symbols in code order.  Codes of each
// length are consecutive integers in symbol order; moving to the next length doubles the code.
PCR_HD void dctab_build(DcTab* t, const uint8_t* bits_vals) {
    for (int i = 0; i < 256; i++) t->lut[i] = 0xFF;
    uint32_t code = 0; int k = 0;
    for (int L = 1; L <= 16; L++) {
        int cnt = bits_vals[L - 1];
        if (L >= 9) t->valptr[L - 9] = (uint16_t)k;
        for (int j = 0; j < cnt; j++) {
            if (k < 16) {
                uint8_t sym = bits_vals[16 + k];
                t->huffval[k] = sym;
                if (L <= 8) {
                    uint32_t first = code << (8 - L), span = 1u << (8 - L);
                    for (uint32_t e = 0; e < span && first + e < 256; e++) t->lut[first + e] = (uint8_t)((L << 4) | (sym & 15));
                }
            }
            code++; k++;
        }
        if (L >= 8) { uint64_t lim = (uint64_t)code << (16 - L); t->limit[L - 8] = lim > 65536 ? 65536u : (uint32_t)lim; }
        code <<= 1;
    }
}

PCR_HD void actab_build(AcTab* t, const uint8_t* bits_vals) {
    for (int i = 0; i < 256; i++) t->lut[i] = 0;
    for (int i = 0; i < 128; i++) t->lut2[i] = 0;
    // pass 1: short codes, limits
    uint32_t code = 0; int k = 0;
    for (int L = 1; L <= 16; L++) {
        int cnt = bits_vals[L - 1];
        if (L >= 9) t->valptr[L - 9] = (uint16_t)k;
        for (int j = 0; j < cnt; j++) {
            if (k < 256) {
                uint8_t sym = bits_vals[16 + k];
                t->huffval[k] = sym;
                if (L <= 8) {
                    uint32_t first = code << (8 - L), span = 1u << (8 - L);
                    for (uint32_t e = 0; e < span && first + e < 256; e++) t->lut[first + e] = (uint16_t)code_entry((uint32_t)L, sym);
                }
            }
            code++; k++;
        }
        if (L >= 8) { uint64_t lim = (uint64_t)code << (16 - L); t->limit[L - 8] = lim > 65536 ? 65536u : (uint32_t)lim; }
        code <<= 1;
    }
    // pass 2: long codes into lut2
    const uint32_t lim8 = t->limit[0];
    const uint32_t D = 65536u - lim8;
    uint32_t sh2 = 0;
    while (D && ((D - 1) >> sh2) >= 128) sh2++;
    t->sh2 = sh2;
    code = 0; k = 0;
    for (int L = 1; L <= 16; L++) {
        int cnt = bits_vals[L - 1];
        for (int j = 0; j < cnt; j++) {
            if (L >= 9 && k < 256 && (uint32_t)(16 - L) >= sh2) {
                uint64_t c = (uint64_t)code << (16 - L);
                if (c >= lim8 && c < 65536) {
                    uint32_t first = ((uint32_t)c - lim8) >> sh2, span = 1u << (16 - L - sh2);
                    for (uint32_t e = 0; e < span && first + e < 128; e++) t->lut2[first + e] = (uint16_t)code_entry((uint32_t)L, bits_vals[16 + k]);
                }
            }
            code++; k++;
        }
        code <<= 1;
    }
}

// The unstuffed data of a unit is stored as big-endian 32-bit words (the unstuff step swaps the bytes of
// every aligned 4-byte group), so a word is usable as loaded.  The buffer stays readable for some bytes
// past any position a decoder can reach before it checks for an overrun.

// bits [len, len+n) of a 32-bit window (n may be 0)
PCR_HD uint32_t field(uint32_t win, int len, int n) { return n ? (win << len) >> (32 - n) : 0; }

// Hides where a value came from, so that the compiler keeps it in the register it is in instead of
// re-deriving it from other values it would then have to keep alive through a hot loop.
PCR_HD uint32_t opaque(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+s"(v));
#endif
    return v;
}

// The same with the value taken as new each time it is looked at: a test of it stays a scalar compare where it stands
// (hoisted out of a loop it becomes a lane mask, and the branch on that costs three times as much).
PCR_HD uint32_t opaque_here(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(v));
#endif
    return v;
}

// Resolve a code of more than 8 bits.  Returns (length << 8) | symbol, or 0 if it is no code.
PCR_HD uint32_t ac_long_code(const AcTab* t, uint32_t win) {
    const uint32_t c16 = win >> 16;
    const uint32_t lim8 = t->limit[0];
    if (c16 < lim8) return 0;
    const uint32_t i2 = (c16 - lim8) >> t->sh2;
    uint32_t e = i2 < 128 ? t->lut2[i2] : 0;
    if (e) return entry_code(e);
    for (int L = 9; L <= 16; L++) {
        if (c16 < t->limit[L - 8]) {
            uint32_t idx = t->valptr[L - 9] + ((c16 - t->limit[L - 9]) >> (16 - L));
            return idx < 256 ? ((uint32_t)L << 8) | t->huffval[idx] : 0;
        }
    }
    return 0;
}
PCR_HD uint32_t ac_code(const AcTab* t, uint32_t win) {
    uint32_t e = t->lut[win >> 24];
    return e ? entry_code(e) : ac_long_code(t, win);
}
// DC: returns (length << 4) | category, or 0 if it is no code (a valid entry is never 0: length >= 1)
PCR_HD uint32_t dc_code(const DcTab* t, uint32_t win) {
    uint32_t e = t->lut[win >> 24];
    if (e != 0xFF) return e;
    const uint32_t c16 = win >> 16;
    if (c16 < t->limit[0]) return 0;
    for (int L = 9; L <= 16; L++) {
        if (c16 < t->limit[L - 8]) {
            uint32_t idx = t->valptr[L - 9] + ((c16 - t->limit[L - 9]) >> (16 - L));
            return idx < 16 ? ((uint32_t)L << 4) | t->huffval[idx] : 0;
        }
    }
    return 0;
}

PCR_HD int extend(uint32_t v, int s) { return (s && v < (1u << (s - 1))) ? (int)v - (1 << s) + 1 : (int)v; }

// ---------------------------------------------------------------------------------------
// Window reader for the AC scans: the 64 lanes of the wavefront look up, in parallel, the
// Huffman code that WOULD start at each of the next 64 bit offsets of the stream (which code
// starts where does not depend on the decoder's state), and pack what follows from it --
// symbol, total length with its appended bits, the appended value -- into one word per lane.
// The serial part of the decoder then only follows the chain of offsets, fetching the word of
// the offset it stands on with one cross-lane read (readlane), instead of doing a table look-up,
// field extraction, sign extension and bit-buffer refill per symbol on the scalar ALU.
// Codes that neither look-up resolves are left to the serial part (kSymMiss) and decoded on the spot if the chain
// really lands on them.  The window is 96 bits of stream (w0,w1,w2): offsets 0..63 each with
// 32 bits of look-ahead; two more words are always already loaded.
//
// packed word: value (16 bits, signed) << 16 | kSymCoef | kSymEob | total bits (6) << 8 | kSymSpecial | advance (7 bits)
// (see pack_symbol).  Offsets whose code the lanes cannot resolve carry kSymMiss, a word that makes the serial
// part leave its straight line exactly as an end of band does, so that the common path tests nothing extra.
// ---------------------------------------------------------------------------------------
PCR_HD uint32_t bits_at(uint32_t w0, uint32_t w1, uint32_t w2, int j) {      // 32 bits from offset j (0..63)
    const uint32_t hi = j < 32 ? w0 : w1, lo = j < 32 ? w1 : w2;
    return (uint32_t)((((((uint64_t)hi) << 32) | lo) << (j & 31)) >> 32);
}

// e: table entry (length << 8 | symbol), non-zero.  first: AC first scan (size s = s value bits,
// sign-extended here); otherwise refinement (size 1 = one sign bit).  An end-of-band symbol
// (size 0, run r < 15) is followed by r bits of run length in both.
//
// The low 7 bits are how far the symbol moves the decoder on, counted to the position AFTER the one it
// lands on: run + 1 for a coefficient and for sixteen zeros, 65 + run ("past everything") for an end of
// band.  AC first scans add it to the position in the band, refinement scans to the index into the
// block's zero table.  kSymSpecial marks the words the straight line of a decoder cannot finish by itself:
//   kSymMiss   no code the look-ups resolve starts here (a longer one, or no code at all): length 0, advance 127;
//   in a refinement scan, sixteen zeros: it lands on a zero WITHOUT taking it, so it is given the advance
//   of an end of band (80) and redone by hand;
//   kSymInvalid  no code at all (or one that cannot occur in the scan): flags the stream as damaged.
constexpr uint32_t kSymCoef = 0x8000u, kSymEob = 0x4000u, kSymSpecial = 0x80u;
constexpr uint32_t kSymMiss = kSymSpecial | 127u;
constexpr uint32_t kSymInvalid = kSymEob | kSymSpecial | 65u;   // what the AC decoders see where no code matches: an "end of band" of
                                                             // length 0, marked special so that only the by-hand paths need to know it
constexpr uint32_t kZrlAdvance = 16;

PCR_HD uint32_t pack_symbol(uint32_t e, uint32_t win, bool first) {
    const int len = (int)(e >> 8), r = (int)((e >> 4) & 15), s = (int)(e & 15);
    const int nx = s ? (first ? s : 1) : (r != 15 ? r : 0);
    const uint32_t extra = field(win, len, nx);
    const int value = (first && s) ? extend(extra, s) : (int)extra;
    // bit 15: the symbol carries a coefficient; bit 14: it is an end-of-band symbol
    const uint32_t flags = (s ? kSymCoef : 0u) | ((s == 0 && r != 15) ? kSymEob : 0u);
    if (!first && s > 1) return kSymInvalid;                 // sizes above 1 do not exist in a refinement scan
    uint32_t adv = (uint32_t)r + 1u;
    if (flags & kSymEob) adv += 64u;
    else if (!first && s == 0) adv = kSymSpecial | (64u + kZrlAdvance);
    return ((uint32_t)(value & 0xFFFF) << 16) | flags | ((uint32_t)(len + nx) << 8) | adv;
}

// Pre-packed table entry for a symbol whose code has `len` bits: the low 16 bits are those of the packed
// word (advance, total bits, flags), bits 16..20 the code length and bits 21..24 the number of appended
// bits, which finish_packed() replaces by the appended value.  "Not in this table" is kSymMiss.
PCR_HD uint32_t packed_entry(uint32_t e, bool first) {
    if (e == 0) return kSymMiss;
    const uint32_t low = pack_symbol(e, 0, first) & 0xFFFFu;
    if (low == kSymInvalid) return kSymInvalid;               // (no appended bits: finish_packed leaves it alone)
    const uint32_t len = e >> 8, r = (e >> 4) & 15, s = e & 15;
    const uint32_t nx = s ? (first ? s : 1u) : (r != 15 ? r : 0u);
    return low | (len << 16) | (nx << 21);
}
// (No condition: a value is negative where its first bit is 0 and the symbol carries a coefficient, a mask of two sign bits.)
PCR_HD uint32_t finish_packed(uint32_t p, uint32_t win, bool first) {
    const uint32_t len = (p >> 16) & 31, nx = (p >> 21) & 15;
    const uint32_t rest = win << len;
    uint32_t x = (rest >> 1) >> (31 - nx);                    // the nx bits after the code (nx = 0: none)
    if (first) x += (uint32_t)((int32_t)(~rest & (p << 16)) >> 31) & ((~0u << nx) + 1u);
    return (p & 0xFFFFu) | (x << 16);
}
// Entry of lutp for the code at the head of `win`: the 8-bit look-up, or from limit[0] on the one of the longer codes.
PCR_HD uint32_t packed_index(uint32_t win, uint32_t lim8, uint32_t sh2) {
    const uint32_t c16 = win >> 16;
    return c16 < lim8 ? c16 >> 8 : 256u + ((c16 - lim8) >> sh2);
}
// What a symbol moves the decoder on by, as one addend of the packed position the symbol loops keep.
// AC first scan: position in the band << 16 | window offset.
PCR_HD uint32_t first_step(uint32_t word) { return ((word & 127u) << 16) | ((word >> 8) & 63u); }
// AC refinement: window offset << 16 | index into the block's zero table.  Everything that is no new coefficient moves the
// index on by exactly 64, past the table: bit 6 then says so, and the low six bits still name the entry landed on before.
PCR_HD uint32_t refine_step(uint32_t word) {
    const uint32_t adv = word & 127u;
    return (((word >> 8) & 63u) << 16) | (adv < 64u ? adv : 64u);
}
// fills lutp from lut and lut2: entry i by lane (i mod nlanes); call with every lane of the workgroup, after those are complete
PCR_HD void actab_pack(AcTab* t, bool first, uint32_t lane, uint32_t nlanes) {
    for (uint32_t i = lane; i < 256 + 128; i += nlanes) t->lutp[i] = packed_entry(entry_code(i < 256 ? t->lut[i] : t->lut2[i - 256]), first);
}

// packed DC word: difference (16 bits, signed) << 16 | total bits (6) << 8 | category (4)
PCR_HD uint32_t pack_dc(uint32_t e, uint32_t win) {          // e = (length << 4) | category, non-zero
    const int len = (int)(e >> 4), t = (int)(e & 15);
    const int diff = extend(field(win, len, t), t);
    return ((uint32_t)(diff & 0xFFFF) << 16) | ((uint32_t)(len + t) << 8) | (uint32_t)t;
}

// v[lane] = value, lane and value the same in every lane (the lane select travels in m0: a vector instruction of
// this chip reads at most one scalar register besides it)
#if defined(__HIP_DEVICE_COMPILE__)
__device__ inline void write_lane(uint32_t& v, uint32_t value, uint32_t lane) {
    asm volatile("s_mov_b32 m0, %2\n\tv_writelane_b32 %0, %1, m0" : "+v"(v) : "s"(value), "s"(lane) : "m0");
}
#endif

// On the device the stream comes through LDS: kStageWords of it at a time, the next ones under way in registers meanwhile, and
// every lane reads the two words its 32 bits lie in a window ahead.  A window then costs one read and one shift of a lane where
// three scalar words were handed on, two more fetched -- a scalar load comes back with the wait for the look-up -- and the lanes'
// bits picked from them: a gray scan of 92 000 coefficients 4.00 -> 3.62 ms, its refinements 4.60 -> 4.43 and 3.99 -> 3.83 ms,
// plain photographs at scan group 10 5.66 -> 5.42 ms.  (The same feed from a vector register, words picked by scalar reads across
// lanes, was slower than the scalar loads.)
constexpr uint32_t kStageWords = 128, kStageWindows = (kStageWords - 2) / 2;
#if defined(__HIP_DEVICE_COMPILE__)
typedef __attribute__((address_space(3))) uint32_t* StageWords;
#else
typedef uint32_t* StageWords;
#endif
// A lane's part of it.  The words a lane reads are other lanes' writes: put() belongs between two wave_sync (the words read
// before it have been, those read behind it are the new ones), see WindowReader::restage.  (Tests drive sixty-four of these
// over one array.)
struct StagedStream {
    StageWords stage;           // kStageWords words
    const uint32_t* g;          // the stream
    uint32_t lane;
    uint32_t at, last;          // word of the stream the staged ones begin at; last word that is read
    uint32_t left;              // windows of the stage whose words have not been read yet
    uint32_t p0, p1;            // the two words of the window read
    StageWords from;            // where those of the one after it lie in the stage
    uint32_t va, vb;            // the next words of the stream, on their way
    PCR_HD void init(StageWords lds, const uint32_t* words, uint32_t bits, uint32_t lane_id) {
        stage = lds; g = words; lane = lane_id;
        last = (bits >> 5) + 4;
        at = 0u - 2 * kStageWindows;
        fetch();
    }
    PCR_HD void fetch() {                                     // the words behind the stage's windows
        const uint32_t a = at + 2 * kStageWindows + lane, b = a + 64;
        va = g[a < last ? a : last]; vb = g[b < last ? b : last];
    }
    PCR_HD void put() {
        at += 2 * kStageWindows;
        stage[lane] = va; stage[64 + lane] = vb;
        // (a lane whose bits are one whole word reads it as the second of the two: the shift of window() goes from 0 to 31.  Lane 0
        // then reads the word ahead of the stage, which is the end of the table, and uses nothing of it.)
        from = stage + (int)((lane >> 5) - ((lane & 31) == 0 ? 1 : 0));
        left = kStageWindows;
        fetch();
    }
    PCR_HD void read() {
        p0 = from[0]; p1 = from[1];
        from += 2;
        left = opaque(left - 1);
    }
    PCR_HD uint32_t pass(uint32_t n) {                        // over n windows, or to the end of the stage; returns how many are missing
        const uint32_t m = n < left ? n : left;
        from += 2 * m; left -= m;
        return n - m;
    }
    PCR_HD uint32_t window() const {                          // this lane's 32 bits
#if defined(__HIP_DEVICE_COMPILE__)
        return __builtin_amdgcn_alignbit(p0, p1, 32 - lane);
#else
        return (uint32_t)((((uint64_t)p0 << 32) | p1) >> ((32 - lane) & 31));
#endif
    }
};
struct WindowReader {
    const AcTab* tab;
    uint32_t lim8, sh2;         // of tab (see packed_index)
    uint32_t o;                 // offset of the next unread bit inside the window (may run past 63 until normalised)
    uint32_t wbase;             // bits of the stream before the window
    uint32_t mis_bits, total_bits;
    uint32_t lane;              // this lane's offset (device); unused on the host
    uint32_t vinfo;             // this lane's packed word (device)
    uint32_t vstep;             // ... and what it moves the decoder on by, as the symbol loops add it up (see first_step, refine_step)
    bool first;
#if defined(__HIP_DEVICE_COMPILE__)
    StagedStream feed;          // a window ahead
    uint32_t vwin;              // this lane's 32 bits
#else
    StreamPtr p;                // words after n1
    uint32_t w0, w1, w2, n0, n1;
#endif

    // The unit starts sub_bits (0..7) bits into byte byte_off of the segment and holds nbits bits counted from that
    // byte's first bit; pos0: what position() reports for the byte's first bit (0: positions relative to the unit's
    // first byte, as for restart intervals; byte_off * 8: positions in the scan, as for units that start at entry points).
    PCR_HD void init(const uint32_t* words, uint32_t byte_off, uint32_t sub_bits, uint32_t nbits, uint32_t pos0, const AcTab* t, bool first_scan,
                     uint32_t lane_id, uint32_t* lds) {
        first = first_scan; lane = lane_id;
        take_table(t);
        mis_bits = (byte_off & 3) * 8;
        o = mis_bits + sub_bits; wbase = pos0; total_bits = pos0 + nbits + mis_bits;
#if defined(__HIP_DEVICE_COMPILE__)
        feed.init((StageWords)lds, words + (byte_off >> 2), nbits + mis_bits, lane_id);
        restage();
        ahead(); take(); ahead();
#else
        (void)lds;
        p = stream_ptr(words + (byte_off >> 2));
        w0 = p[0]; w1 = p[1]; w2 = p[2]; n0 = p[3]; n1 = p[4]; p += 5;
#endif
        fill();
    }
#if defined(__HIP_DEVICE_COMPILE__)
    __device__ void restage() { wave_sync(); feed.put(); wave_sync(); }
    __device__ void ahead() {
        feed.read();
        if (__builtin_expect(feed.left == 0, 0)) restage();
    }
    __device__ void take() { vwin = feed.window(); }
    __device__ void skip(uint32_t n) {                        // n windows nobody asks for
        while (n) {
            n = feed.pass(n);
            if (feed.left == 0) restage();
        }
    }
#endif
    PCR_HD uint32_t win_at(uint32_t off) const {              // the 32 bits at an offset of the window
#if defined(__HIP_DEVICE_COMPILE__)
        return (uint32_t)__builtin_amdgcn_readlane((int)vwin, (int)off);
#else
        return bits_at(w0, w1, w2, (int)off);
#endif
    }
    PCR_HD void take_table(const AcTab* t) { tab = t; lim8 = uni(t->limit[0]); sh2 = uni(t->sh2); }
    PCR_HD uint32_t word_of(uint32_t win) const { return finish_packed(tab->lutp[packed_index(win, lim8, sh2)], win, first); }
    PCR_HD void fill() {
#if defined(__HIP_DEVICE_COMPILE__)
        vinfo = word_of(vwin);
        vstep = first ? first_step(vinfo) : refine_step(vinfo);
#endif
    }
    // packed word of the offset `off` of the window (0..63); kSymMiss where neither look-up has a code
    PCR_HD uint32_t lookup(uint32_t off) const {
#if defined(__HIP_DEVICE_COMPILE__)
        return (uint32_t)__builtin_amdgcn_readlane((int)vinfo, (int)off);
#else
        return word_of(win_at(off));
#endif
    }
    // the same for an offset that lookup() answered with kSymMiss: a code neither look-up resolves, or garbage
    PCR_HD uint32_t resolve(uint32_t off) const {
        const uint32_t win = win_at(off);
        const uint32_t e = ac_long_code(tab, win);
        return uni(e ? pack_symbol(e, win, first) : kSymInvalid);
    }
    PCR_HD bool exhausted() const { return o >= 64; }         // the next symbol starts beyond the window
    PCR_HD void refill() {
#if defined(__HIP_DEVICE_COMPILE__)
        if (!first && __builtin_expect(o >= 128, 0)) {      // (a first scan moves on by 31 bits at a time)
            const uint32_t n = (o >> 6) - 1;
            o -= 64 * n; wbase += 64 * n;
            skip(n - 1); ahead();
        }
        o -= 64; wbase += 64;
        take();
        fill();
        ahead();
#else
        do { w0 = w2; w1 = n0; w2 = n1; n0 = p[0]; n1 = p[1]; p += 2; o -= 64; wbase += 64; } while (o >= 64);
        fill();
#endif
    }
    // Sequential scans switch tables between blocks: the words of the current window are looked up again.
    PCR_HD void use_table(const AcTab* t) { take_table(t); fill(); }
    // Sequential scans: packed DC word (pack_dc) of the symbol at the current position, decoded on the spot;
    // 0 where the bits are no code of the table.
    PCR_HD uint32_t dc_word(const DcTab* t) const {
        const uint32_t win = win_at(o);
        const uint32_t e = dc_code(t, win);
        return uni(e ? pack_dc(e, win) : 0u);                 // (table reads come back in vector registers)
    }
    // refill() that returns the lanes' words of the window being left (device; 0 on the host)
    PCR_HD uint32_t refill_keep() {
        const uint32_t old = vinfo;
        refill();
        return old;
    }
    // replaces the word of offset `off` (a symbol the serial part resolved by hand)
    PCR_HD void set_word(uint32_t off, uint32_t word) {
#if defined(__HIP_DEVICE_COMPILE__)
        write_lane(vinfo, word, off);
#else
        (void)off; (void)word;
#endif
    }
    PCR_HD void consume(uint32_t n) { o += n; }
    PCR_HD uint32_t position() const { return wbase + o - mis_bits; }       // bits consumed since the unit's first bit
    PCR_HD bool overrun() const { return wbase + o > total_bits; }
    PCR_HD uint32_t overrun_bit() const { return (total_bits - (wbase + o)) >> 31; }   // the same as 0 / 1, without a compare (streams are < 2^31 bits)
};

// Per-lane parameters of the unit being decoded (all in registers).
struct LaneScan {
    uint32_t mcu0, mcu1;        // MCU range [mcu0, mcu1) of the scan handled by this unit
    uint32_t mcu_w;             // MCUs per row of the scan
    int Ss, Se, Al;
    // interleaved DC scans: per scan component j
    int ns;
    uint32_t hs[kMaxComp], vs[kMaxComp], bw[kMaxComp];
    uint32_t poff[kMaxComp];   // element offset of each scan component's plane inside the image's coefficient buffer
    int pred[kMaxComp];        // DC predictions at the unit's first MCU (0 after a restart marker; an entry point brings its own)
};

// ---------------------------------------------------------------------------------------
// How a decoder keeps in step with decoders of other scans of the same blocks that run at the same time (see ChainGate in
// pcr_kernels.h): need(m) before anything of block m of the scan is read that an earlier scan wrote, publish(m) once
// everything the decoder has stored lies in blocks before m or may be seen later, due(bits): whether now is a time to.
// FreeRun: alone, everything it reads was there when it started.
// ---------------------------------------------------------------------------------------
struct FreeRun {
    PCR_HD void need(uint32_t) {}
    PCR_HD bool due(uint32_t) const { return false; }
    PCR_HD void publish(uint32_t) {}
};

// ---------------------------------------------------------------------------------------
// CoefSink: keeps memory off the serial path.  Every symbol the serial part passes goes, as (element
// index, packed word with the value in its top 16 bits), into two vector registers, in the lane whose
// number is the window offset the symbol STARTS at: symbols that start inside one window start at
// different offsets, so no counter is needed.  Each time the bit window slides the lanes whose word
// carries kSymCoef store their value, and all words are cleared.  Words without kSymCoef (an end of
// band, sixteen zeros, an unresolved code) are written too and simply never stored.  The element
// index is checked against the plane's size by the lanes, so the serial part need not clamp what a
// damaged stream makes of it.
// ---------------------------------------------------------------------------------------
struct CoefSink {
    int16_t* plane;                                           // may be null if `dense` is given: then only that copy is written
    int16_t* dense;                                           // optional second copy, one value per block: dense[element index / 64]
    uint32_t limit;                                           // elements of `plane`
    int Al;                                                   // values are stored shifted left by this
    uint32_t vidx; int vval;                                  // device: this lane's pending pair
    PCR_HD void init(int16_t* p, uint32_t elems, int al, int16_t* per_block = nullptr) { plane = p; dense = per_block; limit = elems; Al = al; vidx = 0; vval = 0; }
    // slot: window offset the symbol starts at (0..63); word: packed symbol word
    PCR_HD void emit(uint32_t slot, uint32_t elem, int word) {
#if defined(__HIP_DEVICE_COMPILE__)
        // (the lane select travels in m0: a vector instruction of this chip reads at most one scalar
        // register besides it)
        asm volatile("s_mov_b32 m0, %4\n\tv_writelane_b32 %0, %2, m0\n\tv_writelane_b32 %1, %3, m0"
                     : "+v"(vidx), "+v"(vval) : "s"(elem), "s"(word), "s"(slot) : "m0");
#else
        (void)slot;
        if (((uint32_t)word & kSymCoef) && elem < limit) { const int16_t val = (int16_t)((word >> 16) * (1 << Al)); if (plane) plane[elem] = val; if (dense) dense[elem >> 6] = val; }
#endif
    }
    PCR_HD void flush() {
#if defined(__HIP_DEVICE_COMPILE__)
        if (((uint32_t)vval & kSymCoef) && vidx < limit) {
            const int16_t val = (int16_t)((vval >> 16) * (1 << Al));
            if (plane) plane[vidx] = val;
            if (dense) dense[vidx >> 6] = val;
        }
        vval = 0;
#endif
    }
};

// IndexSink: the same for the AC first scan, with less to write per symbol.  The lane of a window offset already holds the
// packed word of the symbol that starts there (the reader's look-up), so all the serial part leaves in that lane is the
// packed position it has at hand anyway; the lane adds the symbol's own advance and its block's element index, which
// block_from() hands to the lanes from an offset on.  A lane stores if it was given a position and its word carries a
// coefficient.  A symbol the serial part resolved by hand is written back into the reader's words.
struct IndexSink {
    int16_t* plane;
    int16_t* dense;                                           // sequential scans: the compact copy of the DC coefficients, dense[element index / 64]
    uint32_t limit;
    int Al;
    uint32_t vpos;                                            // device: this lane's position in the band << 16 | offset, before its symbol; 0 = none
    uint32_t vbase;                                           // device: element index of position 0 of this lane's block
    PCR_HD void init(int16_t* p, uint32_t elems, int al, int16_t* per_block = nullptr) { plane = p; dense = per_block; limit = elems; Al = al; vpos = 0; vbase = 0; }
    // symbols that start at offset `from` of the window or later belong to the block at `base`
    PCR_HD void block_from(uint32_t from, uint32_t base, uint32_t lane) {
#if defined(__HIP_DEVICE_COMPILE__)
        vbase = lane >= from ? base : vbase;
#else
        (void)from; (void)base; (void)lane;
#endif
    }
    PCR_HD uint32_t elem(uint32_t words) const { return vbase + (vpos >> 16) + (words & 127u); }
    // host build: store at once (there are no lanes to hold anything back)
    PCR_HD void store_now(uint32_t elem, uint32_t word) {
        if ((word & kSymCoef) && elem < limit) {
            plane[elem] = (int16_t)(((int32_t)word >> 16) * (1 << Al));
            if (dense && (elem & 63) == 0) dense[elem >> 6] = plane[elem];
        }
    }
    // words: the lanes' packed words of the window the indices belong to
    PCR_HD void flush(uint32_t words) {
#if defined(__HIP_DEVICE_COMPILE__)
        const uint32_t e = elem(words);
        if ((words & kSymCoef) && vpos && e < limit) plane[e] = (int16_t)(((int32_t)words >> 16) * (1 << Al));
        vpos = 0;
#else
        (void)words;
#endif
    }
    // the same for scans that also carry DC coefficients (element 0 of a block goes to the compact copy as well)
    PCR_HD void flush_with_dc(uint32_t words) {
#if defined(__HIP_DEVICE_COMPILE__)
        const uint32_t e = elem(words);
        if ((words & kSymCoef) && vpos && e < limit) {
            const int16_t val = (int16_t)(((int32_t)words >> 16) * (1 << Al));
            plane[e] = val;
            if ((e & 63) == 0) dense[e >> 6] = val;
        }
        vpos = 0;
#else
        (void)words;
#endif
    }
};

// ---------------------------------------------------------------------------------------
// Window reader for DC first scans: as WindowReader, but an interleaved scan switches between the
// DC tables of its components, so every lane looks its offset up in the table of each scan
// component (once per distinct table) and the serial part picks the word of the component whose
// block it is decoding.  Everything is indexed by scan component with constants: a run-time index
// into the reader would pin it to memory.
// packed word: difference (16 bits, signed) << 16 | total bits (6) << 8 | category (4)
// ---------------------------------------------------------------------------------------

struct DcWindowReader {
    StreamPtr p;
    const DcTab* tab[kMaxComp];     // table of scan component j
    uint32_t w0, w1, w2, n0, n1;
    uint32_t o, wbase, mis_bits, total_bits, lane;
    uint32_t vinfo[kMaxComp];       // this lane's packed word under the table of scan component j
    uint32_t nocode;                // set when the bits at the current position are no code of the table
    int ncomp;
    const uint32_t* g;              // p again, for the vector memory path (as in WindowReader)
    uint32_t vnext;

    PCR_HD void init(const uint32_t* words, uint32_t byte_off, uint32_t sub_bits, uint32_t nbits, const DcTab* t0, const DcTab* t1, const DcTab* t2,
                     int ncomponents, uint32_t lane_id) {                  // (byte_off, sub_bits, nbits: as WindowReader::init)
        tab[0] = t0; tab[1] = t1; tab[2] = t2; ncomp = ncomponents; lane = lane_id;
        mis_bits = (byte_off & 3) * 8;
        p = stream_ptr(words + (byte_off >> 2));
        w0 = p[0]; w1 = p[1]; w2 = p[2]; n0 = p[3]; n1 = p[4]; p += 5;
        g = words + (byte_off >> 2) + 5;
        o = mis_bits + sub_bits; wbase = 0; total_bits = nbits + mis_bits; nocode = 0;
        vinfo[0] = vinfo[1] = vinfo[2] = 0;
        fetch_next();
        fill();
    }
    PCR_HD void fetch_next() {
#if defined(__HIP_DEVICE_COMPILE__)
        vnext = g[lane & 1];
#endif
    }
    PCR_HD void slide() {                                     // on by 64 bits
        w0 = w2; w1 = n0; w2 = n1;
#if defined(__HIP_DEVICE_COMPILE__)
        n0 = (uint32_t)__builtin_amdgcn_readlane((int)vnext, 0); n1 = (uint32_t)__builtin_amdgcn_readlane((int)vnext, 1);
#else
        n0 = p[0]; n1 = p[1];
#endif
        p += 2; g += 2; o -= 64; wbase += 64;
        fetch_next();
    }
    PCR_HD uint32_t word_of(const DcTab* t, uint32_t win) const { const uint32_t e = t->lut[win >> 24]; return e != 0xFF ? pack_dc(e, win) : 0; }
    PCR_HD void fill() {
#if defined(__HIP_DEVICE_COMPILE__)
        const uint32_t win = bits_at(w0, w1, w2, (int)lane);
        vinfo[0] = word_of(tab[0], win);
        if (ncomp > 1) vinfo[1] = tab[1] == tab[0] ? vinfo[0] : word_of(tab[1], win);
        if (ncomp > 2) vinfo[2] = tab[2] == tab[1] ? vinfo[1] : (tab[2] == tab[0] ? vinfo[0] : word_of(tab[2], win));
#endif
    }
    PCR_HD bool exhausted() const { return o >= 64; }
    PCR_HD void refill() {
        do slide(); while (o >= 64);
        fill();
    }
    // packed word of the symbol at the current position (inside the window) for scan component J; where the bits
    // are no code at all it returns 0 (length 0, difference 0) and raises `nocode`
    template <int J> PCR_HD uint32_t peek() {
        uint32_t info;
#if defined(__HIP_DEVICE_COMPILE__)
        info = (uint32_t)__builtin_amdgcn_readlane((int)vinfo[J], (int)o);
#else
        info = word_of(tab[J], bits_at(w0, w1, w2, (int)o));
#endif
        if (__builtin_expect(info == 0, 0)) {                // a code longer than 8 bits, or garbage
            const uint32_t win = bits_at(w0, w1, w2, (int)o);
            const uint32_t e = dc_code(tab[J], win);
            info = uni(e ? pack_dc(e, win) : 0u);            // (table reads come back in vector registers)
            nocode |= uni(e ? 0u : 1u);
        }
        return info;
    }
    PCR_HD void consume(uint32_t n) { o += n; }
    PCR_HD uint32_t overrun_bit() const { return (total_bits - (wbase + o)) >> 31; }
};

// ---------------------------------------------------------------------------------------
// DC first scan.  Non-interleaved scans visit the blocks covering the component's own
// samples, interleaved scans the MCU-padded grid, component by component inside each MCU.
// The sink's plane is the image's coefficient buffer; ls.poff[j] locates the plane of scan component j
// in it ([bh][bw][64] blocks, DC at element 0 of each block).  tj0/1/2: which of the reader's tables each
// scan component uses.
// ---------------------------------------------------------------------------------------
// One DC symbol of scan component J for the block at element e.
template <int J>
PCR_HD void dc_first_block(DcWindowReader* wr, CoefSink* sink, int* pred, uint32_t e, uint32_t* bad) {
    if (wr->exhausted()) {
        *bad |= wr->overrun_bit();                           // never walk far beyond the unit's data
        wr->refill();                                        // (before the flush: the wait for the words fetched a window ago must not include these stores)
        sink->flush();
    }
    const uint32_t info = wr->peek<J>();
    *pred += (int32_t)info >> 16;
    sink->emit(wr->o, e, (int)(((uint32_t)*pred << 16) | kSymCoef));
    wr->consume((info >> 8) & 63);
}

// The common shapes with everything about the MCU known at compile time: NS components, the first one
// HS0 x VS0 blocks per MCU, the others one block (a non-interleaved scan is NS = 1, one block per "MCU" and
// only the blocks that cover the component's samples).  Element indices run along instead of being
// recomputed per MCU.
template <int NS, int HS0, int VS0>
PCR_HD int decode_dc_first_shape(DcWindowReader* wr, const LaneScan& ls, CoefSink* sink) {
    int pred0 = ls.pred[0], pred1 = ls.pred[1], pred2 = ls.pred[2];
    const uint32_t mcu_w = ls.mcu_w;
    const uint32_t my0 = ls.mcu0 / mcu_w;
    uint32_t mx = ls.mcu0 % mcu_w;
    const uint32_t bw0 = ls.bw[0];
    uint32_t e0 = ls.poff[0] + ((my0 * VS0) * bw0 + mx * HS0) * 64;
    uint32_t e1 = NS > 1 ? ls.poff[1] + (my0 * ls.bw[1] + mx) * 64 : 0;
    uint32_t e2 = NS > 2 ? ls.poff[2] + (my0 * ls.bw[2] + mx) * 64 : 0;
    // at the end of a row of MCUs: on to the first block of the next row of MCUs
    const uint32_t wrap0 = (VS0 * bw0 - mcu_w * HS0) * 64;
    const uint32_t wrap1 = NS > 1 ? (ls.bw[1] - mcu_w) * 64 : 0, wrap2 = NS > 2 ? (ls.bw[2] - mcu_w) * 64 : 0;
    uint32_t bad = 0;
    uint32_t left = ls.mcu1 - ls.mcu0;
    while (left != 0) {
#pragma unroll
        for (int by = 0; by < VS0; by++) {
#pragma unroll
            for (int bx = 0; bx < HS0; bx++) dc_first_block<0>(wr, sink, &pred0, e0 + (by * bw0 + bx) * 64, &bad);
        }
        if (NS > 1) dc_first_block<1>(wr, sink, &pred1, e1, &bad);
        if (NS > 2) dc_first_block<2>(wr, sink, &pred2, e2, &bad);
        bad |= wr->nocode;
        e0 += HS0 * 64; e1 += 64; e2 += 64;
        if (++mx == mcu_w) { mx = 0; e0 += wrap0; e1 += wrap1; e2 += wrap2; }
        left = bad ? 0 : left - 1;
    }
    sink->flush();
    bad |= wr->overrun_bit();
    return bad ? kEFormat : kOk;
}

// Any other shape.
template <int J>
PCR_HD void dc_first_component(DcWindowReader* wr, const LaneScan& ls, CoefSink* sink, uint32_t mx, uint32_t my, int* pred, uint32_t* bad) {
    const uint32_t hs = ls.ns > 1 ? ls.hs[J] : 1, vs = ls.ns > 1 ? ls.vs[J] : 1, bw = ls.bw[J];
    uint32_t rowe = ls.poff[J] + ((my * vs) * bw + mx * hs) * 64;       // first block of this MCU in the plane
    for (uint32_t by = 0; by < vs; by++) {
        uint32_t e = rowe;
        for (uint32_t bx = 0; bx < hs; bx++) { dc_first_block<J>(wr, sink, pred, e, bad); e += 64; }
        rowe += bw * 64;
    }
}
PCR_HD int decode_dc_first_any(DcWindowReader* wr, const LaneScan& ls, CoefSink* sink) {
    int pred0 = ls.pred[0], pred1 = ls.pred[1], pred2 = ls.pred[2];
    uint32_t my = ls.mcu0 / ls.mcu_w, mx = ls.mcu0 % ls.mcu_w;
    uint32_t bad = 0;
    uint32_t m = ls.mcu0;
    while (m < ls.mcu1) {
        dc_first_component<0>(wr, ls, sink, mx, my, &pred0, &bad);
        if (ls.ns > 1) dc_first_component<1>(wr, ls, sink, mx, my, &pred1, &bad);
        if (ls.ns > 2) dc_first_component<2>(wr, ls, sink, mx, my, &pred2, &bad);
        bad |= wr->nocode;
        if (++mx == ls.mcu_w) { mx = 0; my++; }
        m = bad ? ls.mcu1 : m + 1;
    }
    sink->flush();
    bad |= wr->overrun_bit();
    return bad ? kEFormat : kOk;
}

// Which of the decoders above fits a scan: 0 = decode_dc_first_any, else an instance of decode_dc_first_shape
// (kDcShapes of them).  ns: components of the scan; hs, vs: their sampling factors in scan order (passed one by
// one: an array argument would pin the caller's copy of them to memory).
constexpr int kDcShapes = 5;
PCR_HD int dc_shape(int ns, uint32_t hs0, uint32_t vs0, uint32_t hs1, uint32_t vs1, uint32_t hs2, uint32_t vs2) {
    if (ns == 1) return 1;
    if (ns == 3 && hs1 == 1 && vs1 == 1 && hs2 == 1 && vs2 == 1) {
        if (hs0 == 2 && vs0 == 2) return 2;
        if (hs0 == 1 && vs0 == 1) return 3;
        if (hs0 == 2 && vs0 == 1) return 4;
    }
    return 0;
}
template <int SHAPE>
PCR_HD int decode_dc_first_as(DcWindowReader* wr, const LaneScan& ls, CoefSink* sink) {
    if (SHAPE == 1) return decode_dc_first_shape<1, 1, 1>(wr, ls, sink);
    if (SHAPE == 2) return decode_dc_first_shape<3, 2, 2>(wr, ls, sink);
    if (SHAPE == 3) return decode_dc_first_shape<3, 1, 1>(wr, ls, sink);
    if (SHAPE == 4) return decode_dc_first_shape<3, 2, 1>(wr, ls, sink);
    return decode_dc_first_any(wr, ls, sink);
}
PCR_HD int decode_dc_first(DcWindowReader* wr, const LaneScan& ls, CoefSink* sink) {
    switch (dc_shape(ls.ns, ls.hs[0], ls.vs[0], ls.hs[1], ls.vs[1], ls.hs[2], ls.vs[2])) {
        case 1: return decode_dc_first_as<1>(wr, ls, sink);
        case 2: return decode_dc_first_as<2>(wr, ls, sink);
        case 3: return decode_dc_first_as<3>(wr, ls, sink);
        case 4: return decode_dc_first_as<4>(wr, ls, sink);
        default: return decode_dc_first_as<0>(wr, ls, sink);
    }
}

// ---------------------------------------------------------------------------------------
// AC first scan of one component, band Ss..Se.  Writes coefficient values in ZIG-ZAG order
// inside each 64-element block (element k of a block is zig-zag position k).  Blocks skipped by
// an end-of-band run are not touched: coefficients must be zero-filled beforehand.
//
// The serial part handles one symbol per loop iteration and does no memory access: a decoded
// coefficient goes, as (element index, value), into the next free lane of two vector registers
// (CoefSink), and the lanes store them all at once each time the bit window slides.  A window
// of 64 bits holds at most 32 coefficient symbols (each is at least 2 bits long), so the 64
// lanes always suffice.  Control flow is structured -- flags and loop conditions instead of
// returns and breaks -- because the compiler turns early exits from nested loops into a state
// variable that is tested after every symbol.
// ---------------------------------------------------------------------------------------
// Non-zero mask of the band Ss..Se of one block in internal (zig-zag) order: what an AC first
// scan over that band has made non-zero.
PCR_HD uint64_t nz_mask_of_block(const int16_t* blk, int Ss, int Se) {
    uint64_t m = 0;
    for (int k = Ss; k <= Se; k++) m |= (uint64_t)(blk[k] != 0) << k;
    return m;
}

// Leaves a symbol at offset `slot` of the window and position kb of the band, before its advance, in the sink (device), or
// stores the word's coefficient at element `elem` at once (host).
PCR_HD void sink_symbol(IndexSink* sink, uint32_t slot, uint32_t kb, uint32_t elem, uint32_t word) {
#if defined(__HIP_DEVICE_COMPILE__)
    (void)elem; (void)word;
    write_lane(sink->vpos, (kb << 16) | slot, slot);
#else
    (void)slot; (void)kb;
    sink->store_now(elem, word);
#endif
}

// The symbols that start inside the current window, one straight line each: a coefficient (run r, then the
// value) and sixteen zeros (r = 15) both move on by r + 1; an end of band and an unresolved code move "past
// everything".  What bounds it is the chain from one symbol's offset to the next on a lone wavefront: the read across
// lanes and the addition behind it (24 cycles), the test (about 10) and the branch (24 taken, 12 not).  So position in
// the band and window offset are ONE register, m0, whose low six bits select the lane of the cross-lane read and write;
// the lanes hold the two advances packed alike, one addition moves both on and one test sees either of them past its end
// (bit 6 of the offset; bits 6 and 7 of the position, which an end of band takes to at most 190); the position goes to the
// sink as it is.  Five instructions per symbol instead of ten.  Four copies follow each other, so that most tests
// are branches not taken.  A gray scan of 92 000 coefficients in 63.7 KB: 5.97 -> 5.29 ms, and with the longer codes looked up
// by the lanes too (they took the serial part some 800 cycles each) and finish_packed without a condition 4.00 ms.
// base_b: element index of the block's position 0.  Returns the offset of the last symbol.
#define PCR_FIRST_SYMBOL(branch)                       \
    "v_readlane_b32 %[st], %[vstep], m0\n\t"           \
    "v_writelane_b32 %[vpos], m0, m0\n\t"              \
    "s_add_i32 m0, m0, %[st]\n\t"                      \
    "s_and_b32 %[t], m0, %[mask]\n\t"                  \
    branch "\n\t"
PCR_HD uint32_t ac_first_symbols(WindowReader* wr, IndexSink* sink, uint32_t* kb_io, uint32_t base_b, uint32_t past) {
    uint32_t kb = *kb_io, o = wr->o, last;
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t st, t;
    (void)base_b;
    asm volatile(
        "s_pack_ll_b32_b16 m0, %[o], %[kb]\n"
        "71:\n"                                              // (see first_loop_aligned)
        "1:\n\t"
        PCR_FIRST_SYMBOL("s_cbranch_scc1 2f")
        PCR_FIRST_SYMBOL("s_cbranch_scc1 2f")
        PCR_FIRST_SYMBOL("s_cbranch_scc1 2f")
        PCR_FIRST_SYMBOL("s_cbranch_scc0 1b")
        "2:\n\t"
        "s_sub_i32 %[last], m0, %[st]\n\t"
        "s_lshr_b32 %[kb], m0, 16\n\t"
        "s_and_b32 %[o], m0, 0x7f"
        : [st] "=&s"(st), [t] "=&s"(t), [last] "=&s"(last), [kb] "+s"(kb), [vpos] "+v"(sink->vpos), [o] "+s"(o)
        : [vstep] "v"(wr->vstep), [mask] "s"(past)
        : "m0", "scc");
    last &= 63u;
#else
    uint32_t at = (kb << 16) | o, st;
    do {
        const uint32_t info = wr->lookup(at & 63u);
        st = first_step(info);
        sink->store_now(base_b + (at >> 16) + (info & 127u), info);
        at += st;
    } while ((at & past) == 0);
    last = (at - st) & 63u; kb = at >> 16; o = at & 0x7Fu;
#endif
    wr->o = o; *kb_io = kb;
    return last;
}
#undef PCR_FIRST_SYMBOL
constexpr uint32_t kFirstPast = 0x00C00040u;                  // position 64 .. 255, or offset 64 .. 127

// Where this stands, once per unit, the code is padded so that the symbol loop behind it begins 16 bytes past a multiple of 32:
// how a loop of 28 bytes a turn lies on the lines it is fetched by is 3 to 5 % of its time, and otherwise left to what stands
// ahead of it.  1024 pictures of 128 x 128 without entry points at scan group 5, us a call with the loop 0, 8, 16, 24 bytes past:
// 288, 292, 278, 280; four records of 256 x 256 2370, 2400, 2290, 2305.  (The padding depends on the distance from here, which is
// the same wherever this ends up.)
PCR_HD void first_loop_aligned() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile(".p2alignl 5, 0xBF800000\n\t.fill ((16 - (71f - 70f)) & 31) / 4, 4, 0xBF800000\n70:");      // (s_nop 0)
#endif
}

template <class Gate>
PCR_HD int decode_ac_first(WindowReader* wr, const LaneScan& ls, IndexSink* sink, Gate& gate) {
    first_loop_aligned();
    const uint32_t Ss = (uint32_t)ls.Ss, Se = (uint32_t)ls.Se;
    const uint32_t bw = ls.bw[0], mcu_w = ls.mcu_w;
    // Positions are kept biased: kb = (zig-zag position of the next candidate) + bias with bias = 63 - Se,
    // so that "the band is complete" reads kb >= 64 whatever Se is, the same bit that says "the window
    // is used up" in the window offset.  After a symbol's advance (run + 1) kb is one past the position
    // it landed on; base_b = element index of the block - bias - 1 makes base_b + kb that element.
    const uint32_t bias = 63 - Se;
    uint32_t left = ls.mcu1 - ls.mcu0;                       // blocks of the unit not finished yet (the current one included)
    uint32_t col = ls.mcu0 % mcu_w;
    uint32_t base_b = ((ls.mcu0 / mcu_w) * bw + col) * 64 - bias - 1;
    const uint32_t row_skip = (bw - mcu_w) * 64;             // elements of the padded grid between two rows of the scan
    uint32_t kb = Ss + bias;
    uint32_t bad = 0;
    const uint32_t past = opaque(kFirstPast);
    sink->block_from(0, base_b, wr->lane);
    uint32_t stored = 0;                                     // the coefficients of blocks before this one have been stored a window ago
    while (left != 0) {
        if (wr->exhausted()) {
            bad |= wr->overrun_bit();                        // never walk far beyond the unit's data
            if (gate.due(wr->wbase)) gate.publish(stored);   // (ahead of this window's stores: those of the last one have had time to get there)
            const uint32_t words = wr->refill_keep();        // (before the flush: the wait for the words fetched a window ago must not include these stores)
            sink->flush(words);
            sink->block_from(0, base_b, wr->lane);
            stored = ls.mcu1 - left;
        }
        const uint32_t last = ac_first_symbols(wr, sink, &kb, base_b, past);
        if (kb >= 64) {                                      // the block is finished, or the lanes left the code to us
            uint32_t info = opaque(wr->lookup(last));        // (a scalar: tested on the scalar unit)
            if (info & kSymSpecial) {                        // a code in neither look-up (or none): the same step by hand
                kb -= kSymMiss & 127;
                info = wr->resolve(wr->o);
                if (info == kSymInvalid) bad |= 1u;          // no code at all
                kb += info & 127;
                wr->set_word(wr->o, info);
                sink_symbol(sink, wr->o, kb - (info & 127), base_b + kb, info);
                wr->consume((info >> 8) & 63);
            }
            if (kb >= 64) {                                  // band complete, or end of band
                uint32_t adv = 1;                            // blocks to move on by
                if (info & kSymEob) {                        // run of 2^r + extra blocks
                    adv = (1u << ((info & 127) - 65)) + (info >> 16);
                } else {
                    bad |= ((64u - kb) >> 31) & (info >> 15);   // a coefficient beyond the band (kb > 64)
                }
                adv = adv < left ? adv : left;
                left = bad ? 0 : left - adv;                 // stop at the first damaged block
                col += adv; base_b += adv * 64; kb = Ss + bias;
                while (col >= mcu_w) { col -= mcu_w; base_b += row_skip; }
                sink->block_from(wr->o, base_b, wr->lane);
            }
        }
    }
    sink->flush(wr->vinfo);
    bad |= wr->overrun_bit();
    return bad ? kEFormat : kOk;
}
PCR_HD int decode_ac_first(WindowReader* wr, const LaneScan& ls, IndexSink* sink) { FreeRun g; return decode_ac_first(wr, ls, sink, g); }

// ---------------------------------------------------------------------------------------
// Sequential (baseline) scan: every block is a DC difference followed by AC run/size pairs up to an end of
// block, the blocks of the components interleaved MCU by MCU (or one component alone).  It is read with the
// AC first scan's reader and symbol loop over the band 1..63: the lanes hold the packed AC word of every
// window offset under ONE table, that of the component being decoded; when the next block belongs to a
// component with another AC table the words of the current window are looked up again (twice per MCU of a
// colour image).  The DC symbol, one per block, is decoded by hand at its position and its word (the running
// DC value) put into the lane of its offset like any other coefficient.
// ---------------------------------------------------------------------------------------
// Tables of the scan's components (pointers into LDS on the device).
struct SeqTables { const DcTab* dc[kMaxComp]; const AcTab* ac[kMaxComp]; };

// One block at element e (its DC), coefficients in zig-zag order behind it.
PCR_HD void sequential_block(WindowReader* wr, IndexSink* sink, const DcTab* dt, const AcTab* at, int* pred, uint32_t e, uint32_t* bad,
                             uint32_t past) {
    if (wr->exhausted()) {
        *bad |= wr->overrun_bit();
        const uint32_t words = wr->refill_keep();
        sink->flush_with_dc(words);
    }
    if (at != wr->tab) {                                     // (what the lanes still hold goes out before their words change)
        sink->flush_with_dc(wr->vinfo);
        wr->use_table(at);
    }
    uint32_t info = wr->dc_word(dt);
    if (info == 0) *bad |= 1u;                               // no code at all
    *pred += (int32_t)info >> 16;
    const uint32_t dcw = ((uint32_t)*pred << 16) | kSymCoef;
    // kb: one past the zig-zag position the last symbol landed on (the band 1..63 needs no bias)
    uint32_t kb = 1;
    const uint32_t base_b = e - 1;
    wr->set_word(wr->o, dcw);
    sink->block_from(wr->o, base_b, wr->lane);
    sink_symbol(sink, wr->o, kb, e, dcw);                    // (its word advances by nothing: element base_b + 1)
    wr->consume((info >> 8) & 63);
    while (kb < 64) {
        if (wr->exhausted()) {
            *bad |= wr->overrun_bit();
            const uint32_t words = wr->refill_keep();
            sink->flush_with_dc(words);
            sink->block_from(0, base_b, wr->lane);
        }
        const uint32_t last = ac_first_symbols(wr, sink, &kb, base_b, past);
        if (kb >= 64) {
            info = opaque(wr->lookup(last));
            if (info & kSymSpecial) {                        // a code in neither look-up (or none): the same step by hand
                kb -= kSymMiss & 127;
                info = wr->resolve(wr->o);
                if (info == kSymInvalid) *bad |= 1u;
                kb += info & 127u;
                wr->set_word(wr->o, info);
                sink_symbol(sink, wr->o, kb - (info & 127u), base_b + kb, info);
                wr->consume((info >> 8) & 63);
            }
            if (kb >= 64) {
                if (info & kSymEob) *bad |= ((info & 127u) != 65u) ? 1u : 0u;     // only the plain end of block exists here
                else *bad |= ((64u - kb) >> 31) & (info >> 15);                   // a coefficient beyond position 63
            }
        }
    }
}

template <int J>
PCR_HD void sequential_component(WindowReader* wr, const LaneScan& ls, const SeqTables& tb, IndexSink* sink, uint32_t mx, uint32_t my, int* pred,
                                 uint32_t* bad, uint32_t past) {
    const uint32_t hs = ls.ns > 1 ? ls.hs[J] : 1, vs = ls.ns > 1 ? ls.vs[J] : 1, bw = ls.bw[J];
    uint32_t rowe = ls.poff[J] + ((my * vs) * bw + mx * hs) * 64;
    for (uint32_t by = 0; by < vs; by++) {
        uint32_t e = rowe;
        for (uint32_t bx = 0; bx < hs; bx++) {
            if (!*bad) sequential_block(wr, sink, tb.dc[J], tb.ac[J], pred, e, bad, past);      // (stop at the first damaged block)
            e += 64;
        }
        rowe += bw * 64;
    }
}

// The sink's plane is the image's coefficient buffer; ls.poff[j] locates the plane of scan component j in it.
// The reader must have been initialised with tb.ac[0] as a first-scan reader.
PCR_HD int decode_sequential(WindowReader* wr, const LaneScan& ls, const SeqTables& tb, IndexSink* sink) {
    int pred0 = ls.pred[0], pred1 = ls.pred[1], pred2 = ls.pred[2];
    uint32_t my = ls.mcu0 / ls.mcu_w, mx = ls.mcu0 % ls.mcu_w;
    uint32_t bad = 0;
    uint32_t m = ls.mcu0;
    const uint32_t past = opaque(kFirstPast);
    while (m < ls.mcu1) {
        sequential_component<0>(wr, ls, tb, sink, mx, my, &pred0, &bad, past);
        if (ls.ns > 1) sequential_component<1>(wr, ls, tb, sink, mx, my, &pred1, &bad, past);
        if (ls.ns > 2) sequential_component<2>(wr, ls, tb, sink, mx, my, &pred2, &bad, past);
        if (++mx == ls.mcu_w) { mx = 0; my++; }
        m = bad ? ls.mcu1 : m + 1;
    }
    sink->flush_with_dc(wr->vinfo);
    bad |= wr->overrun_bit();
    return bad ? kEFormat : kOk;
}

// ---------------------------------------------------------------------------------------
// AC refinement scan.  hist0..: masks written by the earlier AC scans of the
// component (nhist of them).  Per block this writes
//   nzout  positions that become non-zero in this scan,
//   sign   for those positions, 1 = positive,
//   cbits  the correction bits in reading order (first bit read = bit 0).
// ---------------------------------------------------------------------------------------
PCR_HD uint64_t band_mask(int Ss, int Se) { return ((Se >= 63) ? ~0ull : ((1ull << (Se + 1)) - 1)) & ~((1ull << Ss) - 1); }

// What an AC refinement scan leaves per block: one record of kRefWords 64-bit words (zig-zag bit order),
//   [kRefNz]    positions that become non-zero in this scan (later scans need them as history)   } written by phase 1
//   [kRefSign]  signs of the kRefNz positions, 1 = positive                                       } written by
//   [kRefPlus]  positions whose correction bit is 1 (their magnitude grows by 2^Al)              } phase 2
//   [kRefStart] bit offset of the block inside its unit | end-of-band run pending at its start << 32  } written by
//   [kRefHist]  positions of the band already non-zero when the scan starts                      } phase 1
// A scan keeps one array per word, each with one entry per block of the component's plane (word w of block b lies
// at w * blocks + b): every kernel that writes a word for consecutive blocks then writes whole lines (records of five
// words per block, of which a kernel writes two or three, were measured to cost 1.7 - 2.4 times the bytes in partial
// sectors); what the consumers of a finished scan need (the replay of the refinement on the coefficients) is the first
// three words.  On the device the first two arrays are one of pairs, kRefNz and kRefSign of a block side by side: the
// lane decoder, which knows both at the end of a block, writes them with one 16-byte store, and the replay reads them with
// one load.
constexpr int kRefNz = 0, kRefSign = 1, kRefPlus = 2, kRefStart = 3, kRefHist = 4, kRefWords = 5;
PCR_HD size_t ref_word(int w, size_t blk, size_t nblk) {
#if defined(__HIP_DEVICE_COMPILE__)
    if (w <= kRefSign) return 2 * blk + (size_t)w;
#endif
    return (size_t)w * nblk + blk;
}
// u64 words of the records of a scan over a plane of nblk blocks (pairs are 16-byte aligned)
PCR_HD uint64_t ref_words(uint64_t nblk) { return (nblk * kRefWords + 1) & ~1ull; }

// History of a refinement scan: the positions of its band that are non-zero when it starts.  What the
// AC first scans made non-zero is read back from the coefficient plane (one coefficient per lane, a ballot
// of "!= 0"); what earlier refinement scans added is in the records they wrote (p[0..n): their record arrays).
// Device: p[0] is readable also where n is 0 (what is read there is masked off by `some`, 0 or ~0).
struct HistPlanes { const int16_t* coef; const uint64_t* p[kMaxHist]; int n; uint64_t some; };

struct HistWords {                                            // one block's history, combined only when used
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t half;                                            // even lanes: low half, odd lanes: high half of what earlier refinement scans added
    int16_t mine;                                             // this lane's coefficient of the block
#else
    uint64_t a, first;
#endif
};
// On the device the record word is fetched by the vector unit (every lane one half of it) although it is the
// same for all lanes: scalar loads return out of order, so a wait for any LDS result -- there is one ahead of
// every symbol loop -- would also wait for a scalar load issued just before it for two blocks later, and expose
// a trip to memory per block.  Vector loads return in order and have a counter of their own.
PCR_HD HistWords hist_fetch(const HistPlanes& hp, uint32_t blk, uint32_t lane) {
    HistWords w;
    static_assert(kRefNz == 0, "the words that become history are a scan's first array");
    const uint32_t off = (uint32_t)ref_word(kRefNz, blk, 0) * 8;   // (32-bit offsets: a plane has fewer than 2^26 blocks)
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t sel = off + (lane & 1) * 4;
    w.half = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(hp.p[0]) + sel);
    if (__builtin_expect(opaque_here((uint32_t)hp.n) > 1, 0)) {   // scripts with more than two refinement passes over a band
        for (int q = 1; q < kMaxHist; q++) if (q < hp.n) w.half |= *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(hp.p[q]) + sel);
    }
    w.mine = hp.coef[(size_t)blk * 64 + lane];
#else
    (void)lane;
    w.a = 0;
    for (int q = 0; q < kMaxHist; q++) if (q < hp.n) w.a |= *reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(hp.p[q]) + off);
    w.first = nz_mask_of_block(hp.coef + (size_t)blk * 64, 0, 63);
#endif
    return w;
}
PCR_HD uint64_t hist_combine(const HistPlanes& hp, const HistWords& w) {
#if defined(__HIP_DEVICE_COMPILE__)
    const uint64_t a = (uint32_t)__builtin_amdgcn_readlane((int)w.half, 0) | ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)w.half, 1) << 32);
    return (a & hp.some) | __ballot(w.mine != 0);
#else
    (void)hp;
    return w.a | w.first;
#endif
}

// Zero table of one block: entry n (n = 1, 2, ...) belongs to the n-th position of the band that is
// still zero when the scan reaches the block (zig-zag order) and holds the number of non-zero-history
// positions below it -- the correction bits a decoder has stepped over when it lands there -- plus
// kZtLast if nothing is left in the block after it (the band's last position, if it is a zero), both in the top 16 bits.
// Entries beyond the number of zeros are sentinels, "no such zero": all non-zero-history positions of the
// band, plus kZtLast.  Entry 0, where a decoder stands before it has landed anywhere, is 0: no corrections passed.
// With the table the serial decoder does no bit arithmetic per symbol: a run of r zeros followed by
// a new coefficient is "index += r + 1, read the entry", and the entry is what to add to the window
// offset.  kZtLast = 64 pushes that offset past the window, so the one test "offset < 64" ends the
// symbol loop for both reasons, a used-up window and a finished block.
// The 64 lanes build the table in a handful of vector instructions (a prefix count of the two masks
// and one permute); lane i also keeps the index of ITS position so that the set of table entries
// that were taken can be turned back into a mask of positions.
constexpr uint32_t kZtLast = 64;

// v = lane's bit of the wave-uniform mask m ? a : b, without materialising the bit: the mask is used as
// the select operand of a conditional move
PCR_HD uint32_t select_by_mask(uint64_t m, uint32_t a, uint32_t b, uint32_t lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t r;
    (void)lane;
    asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(b), "v"(a), "s"(m));
    return r;
#else
    return ((m >> lane) & 1) ? a : b;
#endif
}

struct ZeroTable {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t ventry, vindex;                                  // lane n: entry n; lane i: table index of position i (63 if not a zero, 0 in lane 0)
#else
    uint32_t entry[64], index[64];
#endif
    // top64: kZtLast << 16 in the lane of the band's last position, 0 elsewhere (the same for every block of a scan).
    // Position 0 is in no refinement scan's band: counted as a zero it is entry 0 and moves the others up by one.
    PCR_HD void build(uint64_t h, uint64_t z, uint32_t nzeros, uint32_t ncorr, uint32_t lane, uint32_t top64) {
        const uint64_t z1 = z | 1u;
#if defined(__HIP_DEVICE_COMPILE__)
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(z1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)z1, 0));
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(h >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)h, 0));
        const uint32_t data = select_by_mask(z1, (below << 16) + top64, (ncorr + kZtLast) << 16, lane);
        const uint32_t dest = select_by_mask(z1, rank, (nzeros + 1) + (lane - rank), lane);      // a permutation of the 64 lanes
        ventry = (uint32_t)__builtin_amdgcn_ds_permute((int)(dest * 4), (int)data);
        vindex = select_by_mask(z1, rank, 63u, lane);
#else
        (void)lane; (void)top64;
        uint32_t rank = 0, below = 0, top = 0;
        for (uint32_t i = 0; i < 64; i++) if ((z | h) >> i & 1) top = i;
        for (uint32_t i = 0; i < 64; i++) {
            const bool iz = (z1 >> i) & 1;
            entry[iz ? rank : nzeros + 1 + (i - rank)] = (iz ? below + (i == top ? kZtLast : 0u) : ncorr + kZtLast) << 16;
            index[i] = iz ? rank : 63u;
            rank += iz; below += (h >> i) & 1;
        }
#endif
    }
    PCR_HD uint32_t at(uint32_t n) const {                    // n <= 63
#if defined(__HIP_DEVICE_COMPILE__)
        return (uint32_t)__builtin_amdgcn_readlane((int)ventry, (int)n);
#else
        return entry[n];
#endif
    }
    // taken: bit n set = a symbol landed on entry n.  Returns the positions of those entries; positions that are
    // no zeros all point at entry 63 and must be masked off by the caller.
    PCR_HD uint64_t positions_of(uint64_t taken) const {
#if defined(__HIP_DEVICE_COMPILE__)
        return __ballot(((taken >> vindex) & 1) != 0);
#else
        uint64_t m = 0;
        for (uint32_t i = 0; i < 64; i++) if ((taken >> index[i]) & 1) m |= 1ull << i;
        return m;
#endif
    }
};

// All LDS and scalar-memory results this wavefront is waiting for have arrived: stated once ahead of a
// hot loop, the wait is not repeated inside it.
PCR_HD void settle_lds() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0xC07F);                      // lgkmcnt(0), the other counters untouched
#endif
}
// The same value in every lane of a vector register, and from there on a value per lane to the compiler.
PCR_HD uint32_t per_lane(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
    return r;
#else
    return v;
#endif
}
// (32-bit byte offsets: a plane has fewer than 2^26 blocks)
PCR_HD void store_word(uint64_t* base, uint32_t bytes, uint64_t v) { *reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(base) + bytes) = v; }
// sets bit n (0..63) of a wave-uniform mask: one scalar instruction
PCR_HD void set_bit(uint64_t* m, uint32_t n) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm("s_bitset1_b64 %0, %1" : "+s"(*m) : "s"(n));
#else
    *m |= 1ull << n;
#endif
}

// The symbols of a refinement scan that start inside the current window.  A new +-1 after r zeros: r zeros are passed, the
// next one is taken, and the decoder is past the corrections on the way.  What bounds it is the chain on a lone wavefront, as in
// ac_first_symbols: two reads across lanes (a symbol's advance at the window offset, the table's entry at the index it
// leads to), each with an addition behind it, the test and the branch.  So index and window offset (less the corrections
// stepped over in this block) are ONE register, *p = offset << 16 | index, whose low six bits select the entry and the bit
// set; an entry added on top is the offset of the next symbol, and one test sees the offset past the window or the
// block (bits 6 and 7 of *q's upper half) and the index past the table (bit 6).  Eight instructions per symbol where index,
// offset and advance apart took eleven; four copies follow each other, so that most branches are not taken.
// Two gray scans of 69 000 and 52 000 new coefficients in 40 and 38 KB: 5.15 -> 4.60 and 4.25 -> 3.99 ms, about half of it from what
// surrounds the loop (one scalar test for "on to the next window", history and records without lane masks and 64-bit adds).
// On return *p is where the last symbol led, *q = *p plus its entry if the index is below 64, *taken holds the entries stood on
// before the last symbol (entry 0, nothing yet, among them).  Returns the step of the last symbol.
constexpr uint32_t kRefinePast = 0x00C00040u;
#define PCR_REFINE_SYMBOL(branch)                      \
    "v_readlane_b32 %[st], %[vstep], m0\n\t"           \
    "s_bitset1_b64 %[tk], %[p]\n\t"                    \
    "s_add_i32 %[p], %[p], %[st]\n\t"                  \
    "v_readlane_b32 %[e], %[vent], %[p]\n\t"           \
    "s_add_i32 %[q], %[p], %[e]\n\t"                   \
    "s_lshr_b32 m0, %[q], 16\n\t"                      \
    "s_and_b32 %[e], %[q], %[mask]\n\t"                \
    branch "\n\t"
#if defined(__HIP_DEVICE_COMPILE__)
// o: window offset of the first symbol; vstep, ventry: the lanes' steps and table entries
__device__ inline uint32_t refine_symbols(uint32_t o, uint32_t vstep, uint32_t ventry, uint32_t* p_io, uint32_t* q_out, uint64_t* taken_io, uint32_t past) {
    uint32_t p = *p_io, q, st, e;
    uint64_t taken = *taken_io;
    asm volatile(
        "s_mov_b32 m0, %[o]\n"
        "1:\n\t"
        PCR_REFINE_SYMBOL("s_cbranch_scc1 2f")
        PCR_REFINE_SYMBOL("s_cbranch_scc1 2f")
        PCR_REFINE_SYMBOL("s_cbranch_scc1 2f")
        PCR_REFINE_SYMBOL("s_cbranch_scc0 1b")
        "2:"
        : [st] "=&s"(st), [e] "=&s"(e), [p] "+s"(p), [q] "=&s"(q), [tk] "+s"(taken)
        : [o] "s"(o), [vstep] "v"(vstep), [vent] "v"(ventry), [mask] "s"(past)
        : "m0", "scc");
    *p_io = p; *q_out = q; *taken_io = taken;
    return st;
}
#endif
PCR_HD uint32_t ac_refine_symbols(const WindowReader* wr, const ZeroTable& zt, uint32_t* p_io, uint32_t* q_out, uint64_t* taken_io, uint32_t past) {
#if defined(__HIP_DEVICE_COMPILE__)
    return refine_symbols(wr->o, wr->vstep, zt.ventry, p_io, q_out, taken_io, past);
#else
    uint32_t p = *p_io, q, st, o = wr->o;
    uint64_t taken = *taken_io;
    do {
        taken |= 1ull << (p & 63u);
        st = refine_step(wr->lookup(o));
        p += st;
        q = p + zt.at(p & 63u);
        o = q >> 16;
    } while ((q & past) == 0);
    *p_io = p; *q_out = q; *taken_io = taken;
    return st;
#endif
}
#undef PCR_REFINE_SYMBOL

// Phase 1 (serial, one wavefront per unit): walk the scan only as far as needed to know where
// every block starts.  For each symbol that means: the code (length, run, size), the zero the run
// ends on and the NUMBER of correction bits stepped over on the way -- both read from the block's
// zero table; the sign and correction bits themselves are not read.  Per block it writes the
// kRefNz, kRefStart and kRefHist words of the block's record.
// The history of the next block is fetched while the current one is decoded.  Conditions are kept
// as integer arithmetic and single compares: a boolean widened to an integer, or two conditions
// and-ed together, cost the compiler a detour through the vector unit or through 64-bit lane masks.
template <class Gate>
PCR_HD int skim_ac_refine(WindowReader* wr, const LaneScan& ls, const HistPlanes& hp, uint64_t* recs, size_t nblk, Gate& gate) {     // nblk: blocks of the component's plane
    const uint32_t bw = ls.bw[0], mcu_w = ls.mcu_w;
    const uint64_t band = band_mask(ls.Ss, ls.Se);
    const uint32_t top64 = wr->lane == (uint32_t)ls.Se ? kZtLast << 16 : 0u;
    const uint32_t past = opaque(kRefinePast);               // (in a register)
    uint32_t left = ls.mcu1 - ls.mcu0;                       // blocks still to do
    const uint32_t row_skip = bw - mcu_w;                    // blocks of the padded grid between two rows of the scan
    const uint32_t last_blk = ((ls.mcu1 - 1) / mcu_w) * bw + (ls.mcu1 - 1) % mcu_w;
    uint64_t* const nz_words = recs + ref_word(kRefNz, 0, nblk);
    uint64_t* const start_words = recs + ref_word(kRefStart, 0, nblk);
    uint64_t* const hist_words = recs + ref_word(kRefHist, 0, nblk);
    uint32_t eobrun = 0;                                     // blocks still covered by an end-of-band run
    uint32_t bad = 0;
    // The history of a block is fetched two blocks ahead (a block of a dozen symbols is shorter than a trip to
    // memory).  One cursor (fblk, fcol) walks the unit's blocks for the fetches, stopping at the last one; b0 / b1
    // remember which block the words under way in h0 / h1 belong to: the block each body works on next.
    uint32_t fcol = ls.mcu0 % mcu_w;
    uint32_t fblk = (ls.mcu0 / mcu_w) * bw + fcol;
    uint32_t b0 = fblk;
    gate.need(ls.mcu0);
    HistWords h0 = hist_fetch(hp, b0, wr->lane);
    fblk++; if (++fcol == mcu_w) { fcol = 0; fblk += row_skip; }
    uint32_t b1 = fblk < last_blk ? fblk : last_blk;
    gate.need(left > 1 ? ls.mcu0 + 1 : ls.mcu0);
    HistWords h1 = hist_fetch(hp, b1, wr->lane);
    ZeroTable zt;
    // One block.  hw, bcur: the block's history and index on entry; on return the fetch for the block two further on
    // is under way in hw and bcur is that block.  (Two copies of this body alternate below, each with its own
    // history registers: handing the words from one variable to the next would mean waiting for the fetch that is
    // still in flight.)
    auto one_block = [&](HistWords& hw, uint32_t& bcur) {
        const uint32_t b = bcur;
        const uint64_t h = hist_combine(hp, hw) & band;           // already non-zero
        const uint64_t z = h ^ band;                         // still zero
        left--;
        fblk++; if (++fcol == mcu_w) { fcol = 0; fblk += row_skip; }
        bcur = fblk < last_blk ? fblk : last_blk;
        const uint32_t m = ls.mcu1 - 1 - left;               // the block's number in the scan
        gate.need(left > 1 ? m + 2 : ls.mcu1 - 1);
        hw = hist_fetch(hp, bcur, wr->lane);
        const uint64_t start = ((uint64_t)eobrun << 32) | wr->position();
        const uint32_t ncorr = (uint32_t)__builtin_popcountll(h);
        uint64_t newm = 0;
        if (eobrun == 0) {                                   // symbols are read only outside an end-of-band run
            const uint32_t nzeros = (uint32_t)__builtin_popcountll(z);   // <= 63: a band never holds position 0
            zt.build(h, z, nzeros, ncorr, wr->lane, top64);
            uint32_t p = wr->o << 16;                        // window offset not counting the correction bits stepped over in this block << 16 | table index stood on (0: none yet)
            uint64_t taken = 0, passed16 = 0;                // table entries stood on, and those of them that sixteen zeros led to
            uint32_t again;
            do {
                uint32_t q, st;
                do {                                         // to the end of the block, window by window
                    if (wr->exhausted()) { const uint32_t before = wr->o; wr->refill(); p -= (before - wr->o) << 16; }
                    settle_lds();
                    st = ac_refine_symbols(wr, zt, &p, &q, &taken, past);
                    wr->o = q >> 16;
                } while (opaque((((q - p) >> 16) | p) & 64u) == 0);
                const uint32_t n = p & 0x7Fu;
                again = 0;
                if (n < 64) {                                // the last zero taken, or a coefficient with no zero left to take (it landed on a sentinel)
                    set_bit(&taken, n);
                    wr->o -= kZtLast;
                    bad |= opaque(nzeros - n) >> 31;
                } else {                                     // past the table: an end of band, a coefficient there is no zero for, or a word to do by hand
                    const uint32_t from = p - st;            // where the symbol stood
                    const uint32_t passed = zt.at(from & 63u) >> 16;   // (no entry that a symbol can follow carries kZtLast)
                    uint32_t info = opaque(wr->lookup(((from >> 16) + passed) & 63u));
                    uint32_t ob = (uint32_t)((int32_t)p >> 16);
                    wr->o = ob + ncorr;                      // the corrections left
                    eobrun = (1u << ((info - 65) & 31)) - 1 + (info >> 16);   // (this block is counted)
                    if (__builtin_expect((info & (kSymEob | kSymSpecial)) != kSymEob, 0)) {
                        eobrun = 0;
                        if ((info & kSymSpecial) == 0) {
                            bad |= 1u;
                        } else {                             // by hand: the symbol again from where it started
                            uint32_t at = from & 63u;
                            if (info == kSymMiss) {          // a code in neither look-up, or none
                                info = wr->resolve(ob + passed);   // (a miss has length 0: ob is still the symbol's)
                                ob += (info >> 8) & 63;
                            }
                            if (info == kSymInvalid) {       // no code at all, or one a refinement scan cannot hold
                                bad |= 1u; wr->o = ob;
                            } else {
                                const uint32_t zrl = info & kSymSpecial;   // sixteen zeros: lands on a zero and leaves it zero
                                at += zrl ? kZrlAdvance : (info & 127);
                                const uint32_t e = at <= nzeros ? zt.at(at) >> 16 : ncorr + kZtLast;   // (nzeros <= 63)
                                wr->o = ob + (e & 63);
                                if (at <= nzeros) set_bit(zrl ? &passed16 : &taken, at);
                                if (e >= kZtLast) {
                                    if (info & kSymEob) eobrun = (1u << ((info - 65) & 31)) - 1 + (info >> 16);
                                    bad |= (info >> 15) & (opaque(nzeros - at) >> 31);
                                } else {
                                    p = (ob << 16) | at;
                                    again = 1;
                                }
                            }
                        }
                    }
                }
            } while (__builtin_expect(again, 0));
            taken &= ~passed16;
            newm = zt.positions_of(taken) & z;                 // (& z: lanes that are no zeros share index 63, which a sentinel can be)
        } else {
            wr->consume(ncorr);
            eobrun--;
        }
        gate.publish(m);                                     // (ahead of this block's record: that of the last block has had time to get there)
        const uint32_t bv = per_lane(b);                     // (byte offsets in a vector register, on constant scalar bases)
        store_word(nz_words, bv * (uint32_t)(ref_word(kRefNz, 1, 0) * 8), newm);
        store_word(start_words, bv * 8, start);
        store_word(hist_words, bv * 8, h);                   // (phase 2 and the refinement replay work on the same history)
        bad |= wr->overrun_bit();
        left = opaque(bad ? 0 : left);                       // stop at the first damaged block
    };
    while (left != 0) {
        one_block(h0, b0);
        if (left == 0) break;
        one_block(h1, b1);
    }
    return bad ? kEFormat : kOk;
}
PCR_HD int skim_ac_refine(WindowReader* wr, const LaneScan& ls, const HistPlanes& hp, uint64_t* recs, size_t nblk) { FreeRun g; return skim_ac_refine(wr, ls, hp, recs, nblk, g); }

// Phase 2 (data-parallel, one lane per block): decode one block completely from its start.
//   words, byte_off  the unit's unstuffed data;  st  the block's kRefStart word;  h  history mask;
//   newm  the positions phase 1 found to become non-zero (kRefNz): the j-th symbol that carries a
//         coefficient lands on the j-th of them, so no zero run has to be counted here
// Returns the sign mask (1 = positive) of the positions that become non-zero and the mask of the positions whose
// correction bit is 1.  The stream holds exactly one correction bit per history-non-zero position of the band, in
// zig-zag order; the bits read between two symbols are dealt out to the history positions passed on the way.
// The lane keeps 64 bits of the stream in a register pair and fetches a word only when 32 of them are used up
// (every lane of a wavefront reads another block: these are plain vector loads), and takes a symbol's correction
// bits out of the 32 bits it looked the symbol up in whenever they fit.

// bits (first bit read = bit 0) dealt out to the set bits of `where`, lowest position first.  The two 32-bit halves of
// `where` are dealt to separately (the low half takes the first popcount(low half) bits): 64-bit shifts and carries
// would double the work of every step.
PCR_HD uint32_t deal_bits32(uint32_t bits, uint32_t where) {
    uint32_t out = 0;
    while (where) {
        const uint32_t low = where & (0u - where);            // the lowest position left
        out |= (bits & 1u) ? low : 0u;
        where ^= low; bits >>= 1;
    }
    return out;
}
PCR_HD uint64_t deal_bits(uint64_t bits, uint64_t where) {
    const uint32_t wlo = (uint32_t)where, whi = (uint32_t)(where >> 32);
    const uint32_t nlo = (uint32_t)__builtin_popcount(wlo);
    const uint32_t lo = deal_bits32((uint32_t)bits, wlo);
    const uint32_t hi = deal_bits32((uint32_t)(nlo < 32 ? bits >> nlo : bits >> 32), whi);   // (at most 63 bits are ever dealt)
    return ((uint64_t)hi << 32) | lo;
}

// position of the n-th (n = 1, 2, ...) set bit of z, or `none` if z has fewer: a binary search on population counts
// (a loop that clears n - 1 bits costs a wavefront its full length whenever one lane needs it)
PCR_HD int nth_set_bit(uint64_t z, uint32_t n, int none) {
    if ((uint32_t)__builtin_popcountll(z) < n) return none;
    uint32_t w = (uint32_t)z, base = 0;
    uint32_t t = (uint32_t)__builtin_popcount(w);
    if (n > t) { n -= t; w = (uint32_t)(z >> 32); base = 32; }
    t = (uint32_t)__builtin_popcount(w & 0xFFFFu); if (n > t) { n -= t; w >>= 16; base += 16; }
    t = (uint32_t)__builtin_popcount(w & 0xFFu);   if (n > t) { n -= t; w >>= 8; base += 8; }
    t = (uint32_t)__builtin_popcount(w & 0xFu);    if (n > t) { n -= t; w >>= 4; base += 4; }
    t = (uint32_t)__builtin_popcount(w & 0x3u);    if (n > t) { n -= t; w >>= 2; base += 2; }
    t = w & 1u;                                     if (n > t) base += 1;
    return (int)base;
}

// (One word is on its way ahead of the buffer: the lanes of a wavefront come to the end of a word at different symbols, and with
// the word fetched when it is needed nearly every symbol waited for memory.  k_refine_blocks, 512 photographs: 222 -> 210 us.)
struct LaneBits {
    const uint32_t* words;
    uint64_t buf;                                             // words[wi] : words[wi + 1]
    uint32_t next;                                            // words[wi + 2]
    uint32_t wi, pos;                                         // next unread bit: bit `pos` (0..31) of buf, counted from its top
    PCR_HD void init(const uint32_t* w, uint32_t bit) { words = w; wi = bit >> 5; pos = bit & 31; buf = ((uint64_t)words[wi] << 32) | words[wi + 1]; next = words[wi + 2]; }
    PCR_HD uint32_t peek() const { return (uint32_t)((buf << pos) >> 32); }          // the next 32 bits
    PCR_HD void skip(uint32_t n) {
        pos += n;
        while (pos >= 32) { wi++; buf = (buf << 32) | next; next = words[wi + 2]; pos -= 32; }
    }
    PCR_HD uint64_t take_reversed(uint32_t n) {               // the next n <= 63 bits, first bit read -> bit 0
        uint64_t out = 0; uint32_t done = 0;
        while (n > 0) {
            const uint32_t t = n > 32 ? 32 : n;
            out |= (uint64_t)(bitrev32(peek()) & (t == 32 ? ~0u : (1u << t) - 1)) << done;
            skip(t); done += t; n -= t;
        }
        return out;
    }
};

PCR_HD void refine_block(const uint32_t* words, uint32_t byte_off, uint64_t st, const AcTab* tab, uint64_t h, uint64_t newm, int Ss, int Se,
                         uint64_t* sign_out, uint64_t* plus_out) {
    const uint64_t band = band_mask(Ss, Se);
    h &= band;
    LaneBits rd;
    rd.init(words, byte_off * 8 + (uint32_t)st);
    const uint32_t ncorr = (uint32_t)__builtin_popcountll(h);
    uint64_t sgn = 0;
    uint64_t corr = 0;                                       // the correction bits in reading order (dealt out to the history positions at the end, once)
    uint32_t taken = 0;                                      // correction bits read so far
    uint32_t n = ncorr;                                      // inside an end-of-band run: all of them, nothing else
    if ((uint32_t)(st >> 32) == 0) {
        uint64_t rem = newm & band;                          // positions still to receive their coefficient
        int k = Ss;                                          // first position not yet passed
        n = 0;
        while (k <= Se) {
            const uint32_t win = rd.peek();
            const uint32_t e = ac_code(tab, win);
            if (!e) break;                                   // phase 1 has already flagged the image
            const uint32_t len = e >> 8, r = (e >> 4) & 15, s = e & 15;
            uint32_t used;                                   // bits of `win` this symbol takes
            int pos;
            if (s) {                                         // code, sign bit, then the corrections passed on the way
                if (!rem) break;
                pos = __builtin_ctzll(rem); rem &= rem - 1;
                sgn |= (uint64_t)((win << len) >> 31) << pos;
                used = len + 1;
            } else if (r == 15) {                            // sixteen zeros: lands on the sixteenth zero from k, which stays zero
                used = len;
                pos = nth_set_bit(~h & band & ~((1ull << k) - 1), 16, Se);
            } else {                                         // end of band: code, run-length bits, then every correction left
                rd.skip(len + r);
                n = ncorr - taken;
                break;
            }
            const uint32_t upto = (uint32_t)__builtin_popcountll(h & ((2ull << pos) - 1));   // corrections at positions <= pos (pos itself is a zero)
            if (upto > taken) {
                const uint32_t m = upto - taken;
                uint64_t bits;
                if (used + m <= 32) {                        // they are in the window already
                    bits = bitrev32(win << used) & ((1u << m) - 1);
                    used += m;
                } else {
                    rd.skip(used); used = 0;
                    bits = rd.take_reversed(m);
                }
                corr |= bits << taken;
                taken = upto;
            }
            rd.skip(used);
            k = pos + 1;
        }
    }
    if (n) corr |= rd.take_reversed(n) << taken;             // (taken + n is at most the number of history positions, 63)
    *sign_out = sgn; *plus_out = deal_bits(corr, h);
}

// ---------------------------------------------------------------------------------------
// Data-parallel part of AC refinement for one coefficient at zig-zag position k of a block.
//   newm, sgn, plus   the block's kRefNz, kRefSign and kRefPlus words of the scan
// ---------------------------------------------------------------------------------------
PCR_HD int16_t refine_apply(int16_t v, int k, uint64_t newm, uint64_t sgn, uint64_t plus, int Al) {
    uint64_t bit = 1ull << k;
    int p = 1 << Al;
    if (plus & bit) v = (int16_t)(v > 0 ? v + p : v - p);
    else if (newm & bit) v = (int16_t)((sgn & bit) ? p : -p);
    return v;
}

// ---------------------------------------------------------------------------------------
// DC refinement: bit number `index` (0 = first bit) of an unstuffed segment.
// ---------------------------------------------------------------------------------------
// words: aligned base of the segment (big-endian words); byte_off: start of the interval in it.
PCR_HD int dc_refine_bit(const uint32_t* words, uint32_t byte_off, uint32_t index) {
    const uint32_t bit = byte_off * 8 + index;
    return (words[bit >> 5] >> (31 - (bit & 31))) & 1;
}

}  // namespace pcr
