// Entropy decoders with ONE LANE PER UNIT: the 64 lanes of a wavefront decode 64 different units (restart intervals or
// entry-point units) of the same kind of scan, each lane with its own bit buffer, Huffman table (the wavefront's copy, in
// LDS, of a table k_headers left in memory) and position in its image's coefficient plane.
//
// When they pay.  A wavefront that decodes one unit on the scalar ALU (pcr_entropy.h) spends about 14 scalar
// instructions per symbol, and the chip issues 256 of those per cycle: a throughput bound that a record with tens of
// thousands of units reaches.  A lane-per-unit wavefront is bound by latency instead: one symbol of every lane per trip
// round a dependent chain (buffer -> table entry -> lengths -> buffer) of one to two thousand cycles, but 64 symbols per
// trip, with a fifth of the instructions all told, and the trips of the wavefronts resident on a SIMD overlap.  With U units the scan takes about
// (symbols of the longest unit) x (chain latency), whatever U is, as long as the U / 64 wavefronts are resident at
// once; the host takes this path for launches with enough units (see lanes_pay in pcr_lib.hip) and the
// one-wavefront-per-unit kernels otherwise (few long units: plain records, small records).
//
// The price of 64 streams in one wavefront is that every branch some lane takes is paid by all: the symbol loop below
// is one straight line per symbol with selects, the rare cases (a code longer than 8 bits, a long end-of-band run that
// crosses rows) sit in short divergent regions.  The decoding procedure is the JPEG progressive mode's (the paper's
// Section 2: spectral selection and successive approximation); results are identical to the scalar decoders'.
#pragma once
#include "pcr_entropy.h"

namespace pcr {

// The decoders below are compiled for the host as well (one "lane", plain arrays for the rings): the CPU tests run them
// against the oracle and, on damaged input, under the sanitizers.
#if !defined(__HIPCC__)
struct uint4 { uint32_t x, y, z, w; };
struct uint2 { uint32_t x, y; };
#endif
// true if `v` holds in any lane of the wavefront that is still in the loop
PCR_HD bool any_lane(bool v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ballot_w64(v) != 0;
#else
    return v;
#endif
}
// the same for what hardly ever holds: the branch behind it is laid out of the way, so that the wavefront runs past it (a
// taken branch costs it the fetch of the instructions it lands on, once per trip of a loop that is little else)
#define PCR_RARELY(v) __builtin_expect(any_lane(v), 0)
// Waits here for every load issued so far (device).  The wait the compiler would otherwise place at a loaded value's
// first use -- or at the first re-use of its register -- can land inside the symbol loop, and a wait for a load is a wait
// for every store issued before it as well: the loop would stand still for the round trip of its own stores in every
// trip.  (s_waitcnt vmcnt(0); the other counters are left at their maxima.)
PCR_HD void loads_arrived() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0x0F70);
#endif
}
// The part of an AcTab (pcr_entropy.h) a lane decoder reads: everything before the pre-packed look-up of the window
// readers.  A wavefront keeps one per scan its lanes decode in LDS, and LDS is what bounds the number of resident
// wavefronts.
struct LaneTab {
    uint16_t lut[256];
    uint16_t lut2[128];
    uint32_t limit[9];
    uint16_t valptr[8];
    uint32_t sh2;
    uint8_t huffval[256];
    uint32_t pad[2];
};
constexpr uint32_t kLaneTabPieces = sizeof(LaneTab) / 16;     // 68
static_assert(sizeof(LaneTab) == 1088 && offsetof(AcTab, lutp) >= sizeof(LaneTab) && offsetof(AcTab, lut2) == offsetof(LaneTab, lut2) &&
              offsetof(AcTab, limit) == offsetof(LaneTab, limit) && offsetof(AcTab, valptr) == offsetof(LaneTab, valptr) &&
              offsetof(AcTab, sh2) == offsetof(LaneTab, sh2) && offsetof(AcTab, huffval) == offsetof(LaneTab, huffval), "a LaneTab is the head of an AcTab");

// What a lane needs to know about its unit (AC scans: one component).
struct LaneUnit {
    const uint32_t* words;        // the scan's unstuffed data as big-endian words
    uint32_t bit0, bit1;          // the unit's bits [bit0, bit1) of that data
    uint32_t mcu0, mcu1, mcu_w;   // blocks [mcu0, mcu1) of the scan, mcu_w per row
    uint32_t bw;                  // blocks per row of the (padded) plane
    uint32_t Ss, Se, Al;
    int16_t* plane; uint32_t plane_elems;
    const LaneTab* tab;
    bool ok;
};

// The loops below are bound by how many instructions stand between one symbol and the next: a lone wavefront issues one
// every eight cycles or so, whatever it is, and a launch takes as long as its longest unit.  Hence the style: conditions
// are kept as sign bits and masks and merged with and / or / bit-field inserts, which are one instruction each, where a
// comparison costs the comparison, a wait for its result and scalar instructions that combine it with others; whatever is
// rare sits behind a branch that is the same for the whole wavefront.

// bits [off, off + width) of v, width 0 included (one instruction on the device; off and width below 32)
PCR_HD uint32_t bit_range(uint32_t v, uint32_t off, uint32_t width) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ubfe(v, off, width);
#else
    return width ? (v >> (off & 31u)) & ((1u << width) - 1u) : 0u;
#endif
}
// all ones if v is negative as a signed number, else zero; the same of one bit of v; a where the mask is ones, b where it
// is zero
PCR_HD uint32_t sign_mask(uint32_t v) { return (uint32_t)((int)v >> 31); }
PCR_HD uint32_t bit_mask(uint32_t v, uint32_t bit) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)__builtin_amdgcn_sbfe((int)v, bit, 1);
#else
    return (uint32_t)((int)(v << (31u - bit)) >> 31);
#endif
}
// v - 1, or 0
PCR_HD uint32_t less_one(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_elementwise_sub_sat(v, 1u);
#else
    return v ? v - 1u : 0u;
#endif
}
PCR_HD uint32_t by_mask(uint32_t mask, uint32_t a, uint32_t b) { return (mask & a) | (~mask & b); }

// A lane's view of its stream: three words of it (w0, w1 and the one after them), and one counter.  With p the position
// of the next unread bit, counted from base16's first bit, and m = p + 63, the counter is kept as n = ~m: then the word
// after w1 has index m >> 5, n (its low five bits) is the amount a funnel shift of w0:w1 takes to put the unread bits at
// the top (w0 ends with the bit before p at the latest, so that the shift is never 32), and the words move on by one where
// bit 5 of n changes.  A symbol's bits are consumed by one subtraction; the word after w1 is read ahead of the trip that
// needs it.
//
// Words come from a ring of kRingWords words per lane in LDS, not from memory: the counter a wavefront waits on for a
// load is shared by its lanes and returns in order, so a loop in which some lane or other fetches a word in every
// trip waits for memory in every trip.  The ring is filled for all lanes at once (refill: 16-byte chunks, as many as
// each lane has room for) whenever some lane is about to run short (short_of), every few dozen symbols; between two
// refills the loop reads no memory at all.  Past the unit's end the chunks repeat, so a lane that follows damaged data
// there reads nothing it should not.
constexpr uint32_t kRingWords = 16;
struct LaneRing { uint32_t w[kRingWords][64]; };             // word i of lane l: row 15 - (i & 15), read without bank conflicts

struct LaneStream {
    const uint4* base16;          // 16-byte aligned address at or before the unit's first word; word indices count from here
    uint32_t* ring;               // this lane's column of the ring (LDS)
    uint32_t n;                   // (see above)
    uint32_t past;                // n when the unit's bits are used up: n below it (as a signed difference) is too far
    uint32_t wr;                  // the ring holds the words before this one (a multiple of 4)
    uint32_t last;                // last chunk of 16 bytes read
    uint32_t w0, w1, w2;
    uint4 v0, v1, v2, v3;         // the chunks behind wr, under way or arrived
    PCR_HD uint32_t next_word() const { return ring[bit_range(n, 5, 4) * 64u]; }
    // Call with every lane that is still decoding.  The chunks written were fetched when the ring was filled the last time,
    // and the next ones set out here: a refill waits for memory only if the ring ran dry sooner than memory answers.
    PCR_HD void refill() {
        const uint32_t room = (kRingWords - (wr - (~n >> 5))) >> 2, c = wr >> 2;   // whole chunks that fit
        static_assert(kRingWords == 16, "the chunks are spelled out (an array indexed in a loop ends up in scratch memory)");
        loads_arrived();
        if (room > 0) put(c, v0);
        if (room > 1) put(c + 1u, v1);
        if (room > 2) put(c + 2u, v2);
        if (room > 3) put(c + 3u, v3);
        wr += room * 4;
        fetch();
    }
    PCR_HD void fetch() {
        const uint32_t c = wr >> 2;
        v0 = chunk(c); v1 = chunk(c + 1u); v2 = chunk(c + 2u); v3 = chunk(c + 3u);
    }
    PCR_HD uint4 chunk(uint32_t c) const { return base16[c < last ? c : last]; }
    PCR_HD void put(uint32_t c, const uint4& v) {
        uint32_t* r = ring + (kRingWords - 4u - (c & 3u) * 4u) * 64u;
        r[192] = v.x; r[128] = v.y; r[64] = v.z; r[0] = v.w;
    }
    // the value of n below which fewer than `words` words lie in the ring behind the one read ahead
    PCR_HD uint32_t low_water(uint32_t words) const { return ~(32u * (wr - 1u - words)); }
    PCR_HD void init(const uint32_t* words, uint32_t bit0, uint32_t bit1, LaneRing* rings, uint32_t lane) {
        const uint32_t* first = words + (bit0 >> 5);
        const uint32_t before = (uint32_t)(reinterpret_cast<uintptr_t>(first) & 15u) >> 2;   // words between the 16-byte boundary and the unit's first
        base16 = reinterpret_cast<const uint4*>(first - before);     // (pointer arithmetic: the address stays a global one)
        ring = &rings->w[0][lane];
        const uint32_t m = before * 32u + (bit0 & 31u) + 63u;
        past = ~(m + (bit1 - bit0));
        last = (m + (bit1 - bit0)) >> 7;                      // (the chunk of the last bit, or the one behind it: slack follows the data)
        n = ~0u; wr = 0;
        fetch();
        refill();                                             // (all four chunks)
        n = ~m;
        const uint32_t i = m >> 5;                            // 1 .. 5
        w0 = ring[(15u - ((i - 2u) & 15u)) * 64u]; w1 = ring[(15u - ((i - 1u) & 15u)) * 64u]; w2 = next_word();   // (i = 1: w0 is not looked at)
    }
    PCR_HD uint32_t window() const {
#if defined(__HIP_DEVICE_COMPILE__)
        return __builtin_amdgcn_alignbit(w0, w1, n);
#else
        return (uint32_t)((((uint64_t)w0 << 32) | w1) >> (n & 31u));
#endif
    }
    PCR_HD void consume(uint32_t bits) {                       // bits in 0..31
        const uint32_t t = n - bits, next = bit_mask(t ^ n, 5);   // (the word index has changed where bit 5 has)
        w0 = by_mask(next, w1, w0); w1 = by_mask(next, w2, w1);
        n = t;
        w2 = next_word();
    }
    PCR_HD uint32_t beyond() const { return n - past; }        // negative once bits past the unit's end have been consumed
};

// A lane's look-up of AC codes: the constants of its table in registers, the table itself in LDS.
constexpr uint32_t kCodeBad = 0x8000u | kCodeEob;           // no code: an end of band without any bits, marked
struct LaneLookup {
    const LaneTab* tab;
    uint32_t lim8, bias, sh2;
    PCR_HD void init(const LaneTab* t) { tab = t; lim8 = t->limit[0]; sh2 = t->sh2; bias = lim8 - (256u << sh2); }
    // The entry (code_entry) of the code at the head of the window, as the table has it (0: in neither look-up).  The index
    // of either look-up is picked first, so one read of LDS serves codes of any length.
    PCR_HD uint32_t entry(uint32_t win) const {
        const uint32_t c16 = win >> 16;
        const uint32_t i = c16 >= lim8 ? (c16 - bias) >> sh2 : win >> 24;
        static_assert(offsetof(LaneTab, lut2) == 512, "lut2 lies right behind lut");
        return reinterpret_cast<const uint16_t*>(tab)[i];
    }
    // ... and what to make of it: kCodeBad if there is no such code.  A decoder reads the entry of the next symbol as soon
    // as it knows where that begins, does the rest of this symbol's work while LDS answers, and looks at it then; an entry of
    // 0 is for by_limits.
    PCR_HD uint32_t resolve(uint32_t e, uint32_t win) const {
        if (PCR_RARELY(e == 0)) {
#if defined(__HIP_DEVICE_COMPILE__)
            asm volatile("");                                 // (keeps the two conditions from being merged into a longer one)
#endif
            if (e == 0) e = by_limits(win >> 16);
        }
        return e;
    }
    // A code neither look-up knows (kCodeBad if there is no such code): limit[L - 8] is the first left-aligned 16-bit value that
    // is not a code of length <= L, so the length is 9 + the number of limits at or below the code.
    PCR_HD uint32_t by_limits(uint32_t c16) const {
        uint32_t L = 9, below = lim8;
#pragma unroll
        for (int q = 1; q <= 7; q++) {
            const uint32_t lim = tab->limit[q];
            const bool over = c16 >= lim;
            L += over ? 1u : 0u; below = over ? lim : below;
        }
        const uint32_t idx = tab->valptr[L - 9] + ((c16 - below) >> (16 - L));
        return (c16 >= lim8 && c16 < tab->limit[8] && idx < 256u) ? code_entry(L, tab->huffval[idx & 255u]) : kCodeBad;
    }
};

// The blocks [mcu0, mcu1) of a unit all lie inside its component's plane.
PCR_HD bool lane_unit_inside(const LaneUnit& U) {
    if (U.mcu0 >= U.mcu1 || U.mcu_w == 0 || U.bw < U.mcu_w) return false;
    const uint32_t row = (U.mcu1 - 1) / U.mcu_w, col = (U.mcu1 - 1) - row * U.mcu_w;
    return (uint64_t)row * U.bw + col < (U.plane_elems >> 6);
}

// AC first scan (one component, band Ss..Se, point transform Al) of one unit.  Every coefficient the unit's symbols
// carry is stored (2 bytes); everything else in the plane was zero-filled before.  One symbol per trip, the three kinds
// of symbol (coefficient after a run, sixteen zeros, end of band) told apart by masks.  Damaged data sets the sign of
// `bad` and is followed to the unit's last block (every store is inside the unit's blocks whatever the data say).
PCR_HD int lane_decode_ac_first(const LaneUnit& U, LaneRing* rings, uint32_t lane) {
    if (!lane_unit_inside(U)) return kEFormat;
    LaneStream st;
    st.init(U.words, U.bit0, U.bit1, rings, lane);
    LaneLookup code;
    code.init(U.tab);
    const uint32_t Ss = U.Ss, Se = U.Se, mcu_w = U.mcu_w, Al = U.Al;
    int16_t* const plane = U.plane;
    uint32_t left = U.mcu1 - U.mcu0;                          // blocks of the unit not finished yet (the current one included)
    const uint32_t row0 = U.mcu0 / mcu_w, col0 = U.mcu0 - row0 * mcu_w;
    int in_row = (int)(mcu_w - col0);                         // blocks left in the row of blocks (the current one included)
    uint32_t base = (row0 * U.bw + col0) * 64;                // element index of the current block
    const uint32_t row_skip = (U.bw - mcu_w) * 64;           // elements of the padded grid between two rows of the scan
    const float rcp_w = 1.0f / (float)mcu_w;
    uint32_t k = Ss, bad = 0;
    uint32_t low = st.low_water(1);                           // (a trip takes one word at most)
    uint32_t next_win = st.window(), next_e = code.entry(next_win);
    while (left != 0) {
        const uint32_t win = next_win;
        uint32_t e = next_e;
        // What is rare -- a ring about to run dry, a code the look-up does not know, a row of blocks at its end -- is asked in
        // one test: a comparison and the branch on it take a wavefront some 37 cycles, as much as four dependent instructions.
        if (PCR_RARELY((int)((st.n - low) | (e - 1u) | (uint32_t)(in_row - 1)) < 0)) {
            if (any_lane((int)(st.n - low) < 0)) { st.refill(); low = st.low_water(1); }
            if (e == 0) e = code.by_limits(win >> 16);
            if (in_row <= 0) {                                // on to the next row of blocks
                if (in_row <= -(int)mcu_w) {                  // an end-of-band run over more than one row
                    uint32_t q = (uint32_t)((float)(-in_row) * rcp_w);      // rows passed, estimated: off by less than 1 + blocks / 2^22
                    const uint32_t margin = 1u + ((uint32_t)-in_row >> 22);
                    q = q > margin ? q - margin : 0;          // never too high; the loop adds what is missing
                    in_row += (int)(q * mcu_w); base += q * row_skip;
                }
                while (in_row <= 0) { in_row += (int)mcu_w; base += row_skip; }
            }
        }
        const uint32_t nx = e & 15u;
        st.consume(bit_range(e, 8, 5) + nx);
        next_win = st.window(); next_e = code.entry(next_win);
        const uint32_t x = win << ((e >> 8) & 31u), extra = bit_range(x, 32u - nx, nx);   // the appended bits: the value, or the length of an end-of-band run
        const uint32_t at = k + bit_range(e, 4, 4);           // the position the symbol lands on (sixteen zeros: the last of them)
        const uint32_t room = Se - at, coef = e << 17;        // negative: beyond the band; negative: a coefficient
        // no code; a coefficient beyond the band; bits beyond the unit's
        bad |= (e << 16) | (room & coef) | st.beyond();
        if ((int)(room | ~coef) >= 0) {
            const uint32_t neg = ~sign_mask(x) & ((1u << nx) - 1u);     // (a value without its top bit stands for a negative one)
            plane[base + at] = (int16_t)((extra - neg) << Al);
        }
        const uint32_t eob = bit_mask(e, 13), done = eob | sign_mask(room - 1u);
        // blocks to move on by: this one and the rest of an end-of-band run
        uint32_t adv = by_mask(eob, (1u << nx) | extra, 1u);
        adv = (adv < left ? adv : left) & done;
        k = by_mask(done, Ss, at + 1u);
        left -= adv; base += adv * 64; in_row -= (int)adv;
    }
    return (int)bad < 0 ? kEFormat : kOk;
}

// ---------------------------------------------------------------------------------------
// DC first scan of one unit (interleaved: up to three components, their blocks MCU by MCU; or one component, block by
// block over the blocks that cover its samples).  A unit's lanes belong to different images, each with its own two or
// three small tables, so the tables do not go through the job mechanism of the AC kernels: every lane keeps its own in
// registers, in a form that needs no look-up -- the first sixteen codes of the table (more are no DC categories; the
// wavefront decoders drop them the same way) in code order, each as its left-aligned 16-bit value.  Canonical codes in
// that form are increasing, so the code at the head of a 16-bit window w is the last one that is <= w: the lane counts
// them, two to an instruction.  One symbol -- one block -- per trip.
// ---------------------------------------------------------------------------------------
constexpr uint32_t kLaneDcCodes = 16;
struct LaneDcCodes {
    uint32_t lim[kLaneDcCodes / 2];                           // left-aligned code of entry i: half i & 1 of word i >> 1; 0xFFFF where there is none (see lane_dc_codes)
    uint64_t len, cat;                                        // 4 bits per entry: code length - 1, category
    uint32_t end;                                             // first left-aligned value that is no code of the (truncated) table
};
// A definition as it is read: sixteen counts and the first sixteen symbols.
struct LaneDcDef { uint32_t w[8]; uint32_t ahead; };         // (the first `ahead` bytes are not its own)

struct LaneDcUnit {
    const uint32_t* words; uint32_t bit0, bit1;               // as LaneUnit
    uint32_t mcu0, mcu1, mcu_w;
    uint32_t ns;                                              // components of the scan
    // per scan component 0, 1, 2:
    uint32_t hs0, hs1, hs2, vs0, vs1, vs2;                    // blocks per MCU (1 x 1 if ns == 1)
    uint32_t bw0, bw1, bw2;                                   // blocks per row of the component's plane
    uint32_t pblk0, pblk1, pblk2;                             // first block of its plane in the image's coefficient buffer
    int pred0, pred1, pred2;                                  // DC predictions at the unit's first MCU
    uint32_t Al;
    int16_t* dense;                                           // the image's compact copy of the DC coefficients: one value per block of the buffer
    int16_t* planes;                                          // the image's coefficient buffer (element 0 of every block), or null
    uint32_t nblocks;                                         // blocks of that buffer
    const uint8_t *def0, *def1, *def2;                        // each scan component's table definition: 16 counts, then the symbols in code order
    const uint8_t* end;                                       // end of the bytes the definitions lie in
    bool ok;
};

// The definition at d (call per lane, for all tables before any is used: the loads are then under way together).  The 32
// bytes are read whatever the definition's length, at the very end of the record (end) from as much ahead of it as is
// missing behind it; a record has more than 32 bytes.
PCR_HD void lane_dc_def(LaneDcDef* D, const uint8_t* d, const uint8_t* end) {
    const uint64_t behind = (uint64_t)(end - d);
    uint32_t ahead = behind >= 32 ? 0u : 32u - (uint32_t)behind;
    struct __attribute__((packed, aligned(1))) Loose { uint4 a, b; };
    const Loose v = *reinterpret_cast<const Loose*>(d - ahead);
    D->w[0] = v.a.x; D->w[1] = v.a.y; D->w[2] = v.a.z; D->w[3] = v.a.w; D->w[4] = v.b.x; D->w[5] = v.b.y; D->w[6] = v.b.z; D->w[7] = v.b.w;
    D->ahead = ahead;
}

// The table of a definition.  Sixteen entries are pushed in at the top of each member and the definition's bytes taken from
// the bottom of its words, so that no register is indexed.  Entries that are not there count as codes at a window of
// sixteen ones: a code if the table's last one is all ones (no file should hold such a table, but the wavefront decoders
// take it).  It is that one then, and all sixteen entries count, so the last of them has its length and category.
PCR_HD void lane_dc_codes(LaneDcCodes* T, LaneDcDef D) {
    auto down = [](uint32_t* w, int n) {                      // n words, one byte down
        for (int q = 0; q + 1 < n; q++) w[q] = (w[q] >> 8) | (w[q + 1] << 24);
        w[n - 1] >>= 8;
    };
    while (PCR_RARELY(D.ahead != 0)) if (D.ahead != 0) { down(D.w, 8); D.ahead--; }
    uint32_t L = 0, code = 0, rem = 0, end = 0, n = 0;
    uint64_t len = 0, cat = 0;
#pragma unroll
    for (uint32_t q = 0; q < kLaneDcCodes / 2; q++) T->lim[q] = 0;
#pragma unroll 1
    for (uint32_t i = 0; i < kLaneDcCodes; i++) {
#pragma unroll 1
        while (rem == 0 && L < 16) { L++; code <<= 1; rem = D.w[0] & 255u; down(D.w, 4); }
        const uint32_t left = code << (16u - L);
        const bool is = rem != 0 && left < 0xFFFFu;
#pragma unroll
        for (uint32_t q = 0; q + 1 < kLaneDcCodes / 2; q++) T->lim[q] = (T->lim[q] >> 16) | (T->lim[q + 1] << 16);
        T->lim[kLaneDcCodes / 2 - 1] = (T->lim[kLaneDcCodes / 2 - 1] >> 16) | (is ? left << 16 : 0xFFFF0000u);
        n += is ? 1u : 0u;
        len = (len >> 4) | (uint64_t)((L - 1u) & 15u) << 60; cat = (cat >> 4) | (uint64_t)(D.w[4] & 15u) << 60;
        down(D.w + 4, 4);
        end = is ? left + (1u << (16u - L)) : end;
        code += rem != 0 ? 1u : 0u; rem -= rem != 0 ? 1u : 0u;
    }
    const uint32_t sh = 4u * (n - 1u) & 63u;                  // the last code's
    T->len = (len & ~0ull >> 4) | (len >> sh) << 60; T->cat = (cat & ~0ull >> 4) | (cat >> sh) << 60; T->end = end;
}

// entries above w (of sixteen)
PCR_HD uint32_t lane_dc_above(const LaneDcCodes& T, uint32_t w) {
#if defined(__HIP_DEVICE_COMPILE__)
    // (written out: the compiler makes sixteen comparisons and selects of it)
    const uint32_t ww = w | (w << 16);
    auto above = [&](uint32_t q) {
        uint32_t r;
        asm("v_pk_sub_u16 %0, %1, %2 clamp\n\tv_pk_min_u16 %0, %0, 1 op_sel_hi:[1,0]" : "=v"(r) : "v"(T.lim[q]), "v"(ww));
        return r;
    };
    const uint32_t a = ((above(0) + above(1)) + (above(2) + above(3))) + ((above(4) + above(5)) + (above(6) + above(7)));    // (halves below 9: no carry)
    return (a & 0xFFFFu) + (a >> 16);
#else
    uint32_t n = 0;
    for (uint32_t q = 0; q < 8; q++) n += ((T.lim[q] & 0xFFFFu) > w ? 1u : 0u) + ((T.lim[q] >> 16) > w ? 1u : 0u);
    return n;
#endif
}

// one symbol: the DC difference at the head of the stream; `bad` gets its sign where there is no code, or no bits
PCR_HD int lane_dc_symbol(LaneStream* st, const LaneDcCodes& T, uint32_t* bad) {
    const uint32_t win = st->window(), w16 = win >> 16;
    const uint32_t sh = 4u * (15u - lane_dc_above(T, w16)) & 63u;
    const uint32_t len = ((uint32_t)(T.len >> sh) & 15u) + 1u, s = (uint32_t)(T.cat >> sh) & 15u;
    st->consume(len + s);
    const uint32_t x = win << len, extra = bit_range(x, 32u - s, s), neg = ~sign_mask(x) & ((1u << s) - 1u);
    *bad |= (T.end - 1u - w16) | st->beyond();
    return (int)(extra - neg);
}

// lanes whose value equals that of the first lane still in the branch
PCR_HD bool as_first(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return v == (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
#else
    (void)v;
    return true;
#endif
}
PCR_HD uint32_t of_first(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
#else
    return v;
#endif
}

// Bound by the latency of one symbol after another: about 330 cycles each, of 46 instructions.  1024 photographs (entry
// points every 64 MCUs) take 55 us; 100 before, when the tables lay in LDS, were read definition byte by byte, and every
// symbol picked its component's members with selects (1250 cycles, 110 instructions).
// The lanes of a wavefront go MCU by MCU, block by block, in step, so which component a block belongs to is the same for
// all of them and costs nothing: lanes whose MCUs look different (another sub-sampling, in another image) go after each
// other.  (Launches are cut so that none are: dc_units_by_shape.)
PCR_HD __attribute__((always_inline)) int lane_decode_dc_first(const LaneDcUnit& U, LaneRing* rings, uint32_t lane) {
    LaneDcDef d0, d1, d2;
    lane_dc_def(&d0, U.def0, U.end); lane_dc_def(&d1, U.def1, U.end); lane_dc_def(&d2, U.def2, U.end);
    LaneStream st;
    st.init(U.words, U.bit0, U.bit1, rings, lane);
    LaneDcCodes t0, t1, t2;
    lane_dc_codes(&t0, d0); lane_dc_codes(&t1, d1); lane_dc_codes(&t2, d2);
    uint32_t left = U.mcu1 - U.mcu0;                          // MCUs not finished yet
    const uint32_t my = U.mcu0 / U.mcu_w;
    uint32_t in_row = U.mcu_w - (U.mcu0 - my * U.mcu_w);      // MCUs left in the row (the current one included)
    // every block lies inside the buffer if those of the last row do
    const uint32_t last_row = (U.mcu1 - 1u) / U.mcu_w;
    auto inside = [&](uint32_t pblk, uint32_t hs, uint32_t vs, uint32_t bw) { return (uint64_t)pblk + ((uint64_t)last_row * vs + vs - 1u) * bw + (uint64_t)U.mcu_w * hs <= U.nblocks; };
    if (U.mcu0 >= U.mcu1 || !inside(U.pblk0, U.hs0, U.vs0, U.bw0) || !inside(U.pblk1, U.hs1, U.vs1, U.bw1) || !inside(U.pblk2, U.hs2, U.vs2, U.bw2)) return kEFormat;
    const uint32_t mx = U.mcu0 - my * U.mcu_w;
    uint32_t b0 = U.pblk0 + my * U.vs0 * U.bw0 + mx * U.hs0, b1 = U.pblk1 + my * U.vs1 * U.bw1 + mx * U.hs1, b2 = U.pblk2 + my * U.vs2 * U.bw2 + mx * U.hs2;   // the MCU's first block of each component
    const uint32_t skip0 = U.vs0 * U.bw0 - U.mcu_w * U.hs0, skip1 = U.vs1 * U.bw1 - U.mcu_w * U.hs1, skip2 = U.vs2 * U.bw2 - U.mcu_w * U.hs2;
    const uint32_t shape = dc_shape(U.ns, U.hs0, U.vs0, U.hs1, U.vs1, U.hs2, U.vs2);
    int pred0 = U.pred0, pred1 = U.pred1, pred2 = U.pred2;
    uint32_t bad = 0;
    bool done = false;
    while (!done) {
        if (!as_first(shape)) continue;                       // (another turn)
        const uint32_t sh = of_first(shape), ns = sh & 15u;
        uint32_t low = st.low_water(1);                       // (a symbol takes one word at most)
        auto blocks = [&](const LaneDcCodes& T, uint32_t hs, uint32_t vs, uint32_t bw, uint32_t b, int* pred) {
            for (uint32_t y = 0; y < vs; y++)
                for (uint32_t x = 0; x < hs; x++) {
                    if (PCR_RARELY((int)(st.n - low) < 0)) { st.refill(); low = st.low_water(1); }
                    *pred += lane_dc_symbol(&st, T, &bad);
                    const int16_t v = (int16_t)((uint32_t)*pred << U.Al);
                    const uint32_t blk = b + y * bw + x;
                    U.dense[blk] = v;
                    if (U.planes) U.planes[(size_t)blk * 64] = v;
                }
        };
        while (left != 0) {
            blocks(t0, (sh >> 4) & 15u, (sh >> 8) & 15u, U.bw0, b0, &pred0);
            if (ns > 1) blocks(t1, (sh >> 12) & 15u, (sh >> 16) & 15u, U.bw1, b1, &pred1);
            if (ns > 2) blocks(t2, (sh >> 20) & 15u, (sh >> 24) & 15u, U.bw2, b2, &pred2);
            left--;
            if ((int)bad < 0) left = 0;                       // stop at the first damaged MCU
            b0 += U.hs0; b1 += U.hs1; b2 += U.hs2; in_row--;
            const uint32_t wrap = sign_mask(in_row - 1u);
            b0 += wrap & skip0; b1 += wrap & skip1; b2 += wrap & skip2; in_row += wrap & U.mcu_w;
        }
        done = true;
    }
    return (int)bad < 0 ? kEFormat : kOk;
}

// ---------------------------------------------------------------------------------------
// AC refinement scan of one unit, complete in one pass: where the new coefficients go, their signs, and the correction
// bits.  The history of a block (which positions of the band are non-zero already) is read from the kRefHist word of
// the block's record, which k_refine_history has written for every block of the scan beforehand; like the stream
// words it comes through a small ring in LDS that all lanes fill at once.  Per block the lane leaves
//   [kRefNz]    positions that become non-zero,   [kRefSign]  their signs (1 = positive),
//   [kRefPlus]  the block's correction bits IN READING ORDER (first bit read = bit 0): k_refine_deal moves them to the
//               history positions they belong to afterwards, one lane per block.
// One trip of the loop is one symbol with the correction bits that follow it, or one block inside an end-of-band run
// (correction bits only).
// ---------------------------------------------------------------------------------------
// position of the n-th (n = 1 .. 16) set bit of z, 64 if there is none
PCR_HD uint32_t nth_zero_position(uint64_t z, uint32_t n) {
    const uint32_t lo = (uint32_t)z, hi = (uint32_t)(z >> 32);
    uint32_t need = 0u - n, t = (uint32_t)__builtin_popcount(lo) + need, off = 0;
    const uint32_t upper = sign_mask(t), w = by_mask(upper, hi, lo);
    need = t > need ? t : need;
    const uint32_t none = sign_mask((uint32_t)__builtin_popcount(w) + need);              // (fewer than n set bits in all)
#pragma unroll
    for (uint32_t width = 16, lg = 4; width > 0; width >>= 1, lg--) {
        t = (uint32_t)__builtin_popcount(bit_range(w, off, width)) + need;
        need = t > need ? t : need;
        off |= (t >> (31u - lg)) & width;
    }
    return off | (upper & 32u) | (none & 64u);
}

constexpr uint32_t kHistRing = 4;
struct LaneHistRing { uint64_t h[kHistRing][64]; };

// What is left of the block is kept relative to the first position k not passed yet: h the history bits from k on (bit 0
// is position k; positions beyond the band are zeros in it), rem the positions of the band from k on.  The zeros are then
// ~h, and a run that ends at relative position p >= rem has run out of the band.
// Damaged data sets the sign of `bad` and is followed to the unit's last block: records are written for the unit's own
// blocks only, whatever the data say.
// RUNS: with a short way through the blocks of end-of-band runs, for units of smooth pictures, where a run covers most of
// the blocks and a unit can be a whole scan (there are no entry points inside a run): 4275 trips for next to no symbols.
// 731 smooth pictures of 600 x 450 at scan group 6: 3.1 ms without, 1.6 with it.  It is a second copy of the loop,
// taken by wavefronts that hold such a unit, because in the loop of all others the mere presence of the other way cost 10 %
// (787 -> 867 us for the refinement launches of 1024 photographs; as a copy 796).
PCR_HD bool lane_mostly_runs(const LaneUnit& U) { return U.bit1 - U.bit0 < U.mcu1 - U.mcu0; }      // (less than a bit per block)

template <bool RUNS>
PCR_HD int lane_decode_ac_refine(const LaneUnit& U, uint64_t* recs, uint32_t nblk, LaneRing* rings, LaneHistRing* hring, uint32_t lane) {
    if (!lane_unit_inside(U) || nblk != U.plane_elems >> 6 || U.Ss == 0) return kEFormat;
    LaneStream st;
    st.init(U.words, U.bit0, U.bit1, rings, lane);
    LaneLookup code;
    code.init(U.tab);
    const uint32_t Ss = U.Ss, band = U.Se - U.Ss + 1u, mcu_w = U.mcu_w, row_skip = U.bw - mcu_w;
    const uint32_t to_place = 63u - U.Se;                     // from the top of a word down to its bottom, once the whole band has passed
    uint32_t left = U.mcu1 - U.mcu0;                          // blocks of the unit not finished yet (the current one included)
    const uint32_t row0 = U.mcu0 / mcu_w, col0 = U.mcu0 - row0 * mcu_w;
    uint32_t blk = row0 * U.bw + col0, in_row = mcu_w - col0; // the current block; blocks left in its row (itself included)
    const uint64_t* hist = recs + ref_word(kRefHist, 0, nblk);
    uint64_t* plus = recs + ref_word(kRefPlus, 0, nblk);
    // The history words of the next blocks: a ring of kHistRing of them in LDS, and the kHistRing after those under way from
    // memory or arrived (h0 .. h3), fetched as the stream's chunks are.  The cursor fblk runs ahead of the decoder's block.
    uint32_t fblk = blk, f_in_row = in_row, fetched = 0, used_up = 0;
    static_assert(kHistRing == 4, "the entries are spelled out (an array indexed in a loop ends up in scratch memory)");
    uint64_t h0, h1, h2, h3;
    auto next_block = [&](uint32_t* b, uint32_t* r) {         // (held at the plane's end: past the unit's last block nothing is looked at)
        *b += 1u; *r -= 1u;
        const bool wrap = *r == 0;
        *b += wrap ? row_skip : 0u; *r = wrap ? mcu_w : *r;
        *b = *b < nblk ? *b : nblk - 1u;
    };
    auto fetch_history = [&]() {
        uint32_t b = fblk, r = f_in_row;
        h0 = hist[b]; next_block(&b, &r);
        h1 = hist[b]; next_block(&b, &r);
        h2 = hist[b]; next_block(&b, &r);
        h3 = hist[b];
    };
    auto more_history = [&]() {                               // every lane: as many blocks' words as its ring has room for
        const uint32_t room = kHistRing - (fetched - used_up);
        loads_arrived();
        if (room > 0) { hring->h[(fetched + 0) & 3u][lane] = h0; next_block(&fblk, &f_in_row); }
        if (room > 1) { hring->h[(fetched + 1) & 3u][lane] = h1; next_block(&fblk, &f_in_row); }
        if (room > 2) { hring->h[(fetched + 2) & 3u][lane] = h2; next_block(&fblk, &f_in_row); }
        if (room > 3) { hring->h[(fetched + 3) & 3u][lane] = h3; next_block(&fblk, &f_in_row); }
        fetched += room;
        fetch_history();
    };
    fetch_history();
    more_history();
    uint64_t h = hring->h[0][lane] >> Ss;                     // (the words hold nothing outside the band)
    uint64_t hn = hring->h[1][lane];                          // the next block's word (as it comes), read a block ahead
    used_up = 2;
    uint64_t newm = 0, sgn = 0, corr = 0;
    uint32_t ncorr = 0, rem = band, eobrun = 0, bad = 0;
    uint32_t low = st.low_water(4);                           // (a trip takes up to four words)
    uint32_t next_win = st.window(), next_e = code.entry(next_win);
    auto block_done = [&]() {                                 // the block's record, and on to the next one
#if defined(__HIP_DEVICE_COMPILE__)
        *reinterpret_cast<ulonglong2*>(recs + ref_word(kRefNz, blk, nblk)) = ulonglong2{newm, sgn};
#else
        recs[ref_word(kRefNz, blk, nblk)] = newm; recs[ref_word(kRefSign, blk, nblk)] = sgn;
#endif
        plus[blk] = corr;
        eobrun = less_one(eobrun);                        // (a run counts the block it starts in)
        left--;
        blk++; in_row--;
        if (PCR_RARELY(in_row == 0)) { blk += in_row == 0 ? row_skip : 0u; in_row = in_row == 0 ? mcu_w : in_row; }
        h = hn >> Ss; hn = hring->h[used_up & 3u][lane]; used_up++;
        newm = 0; sgn = 0; corr = 0; ncorr = 0; rem = band;
    };
    while (left != 0) {
        if (PCR_RARELY((int)(st.n - low) < 0)) { st.refill(); low = st.low_water(4); }
        if (PCR_RARELY(fetched == used_up)) more_history();
        // all lanes inside end-of-band runs: nothing but the corrections of one more block each, mostly none
        if (RUNS && !any_lane(eobrun == 0)) {
            uint32_t todo = (uint32_t)__builtin_popcountll(h), at = 0;
            while (any_lane(todo != 0)) {                     // (31 bits of the window at a time)
                const uint32_t q = todo < 31u ? todo : 31u;
                corr |= (uint64_t)bit_range(bitrev32(st.window()), 0, q) << at;
                st.consume(q);
                at += q; todo -= q;
            }
            bad |= st.beyond();
            block_done();
            next_win = st.window(); next_e = code.entry(next_win);
            continue;
        }
        const uint32_t win = next_win;
        // what the search below needs of the block (while LDS still answers)
        const uint32_t z = ~(uint32_t)h, z16 = (uint32_t)__builtin_popcount(z & 0xFFFFu), z32 = (uint32_t)__builtin_popcount(z);
        const uint32_t hc = (uint32_t)__builtin_popcountll(h);
        const uint32_t in_run = sign_mask(0u - eobrun);       // inside an end-of-band run: no symbol, every correction of the block
        const uint32_t e = by_mask(in_run, kCodeEob, code.resolve(next_e, win));
        const uint32_t nx = e & 15u, r = bit_range(e, 4, 4);
        // A coefficient takes the (r + 1)-th zero from k on, sixteen zeros land on the sixteenth (and leave it zero): a binary
        // search on population counts.  The count still to go is kept negative, as the addend of the next count t: t < 0 says
        // that the zero lies beyond the part counted, and the larger of the two as unsigned numbers is what is still to go
        // either way.  The next 32 positions nearly always hold it.
        uint32_t need = ~r, t = z16 + need;
        uint32_t p = (t >> 27) & 16u;
        need = t > need ? t : need;
#pragma unroll
        for (uint32_t width = 8, lg = 3; width > 0; width >>= 1, lg--) {
            t = (uint32_t)__builtin_popcount(bit_range(z, p, width)) + need;
            need = t > need ? t : need;
            p |= (t >> (31u - lg)) & width;
        }
        if (PCR_RARELY((int)(z32 + ~r) < 0)) p = (int)(z32 + ~r) < 0 ? nth_zero_position(~h, r + 1u) : p;
        const uint32_t eob = bit_mask(e, 13), coef = bit_mask(e, 14);
        const uint32_t past = sign_mask(rem - 1u - p), all = eob | past;   // past: no zero of the band left to land on
        const uint32_t last = by_mask(all, rem - 1u, p);      // what is passed: the positions up to this one
        // the correction bits of the history positions passed follow (of the p positions ahead of the zero all but r): mostly
        // a few, inside the window still
        const uint32_t nc = by_mask(all, hc, p - r);
        const uint32_t used = bit_range(e, 8, 5) + nx;        // bits of the window the symbol takes (30 at most)
        uint32_t fit = 31u - used;
        fit = nc < fit ? nc : fit;
        uint64_t cbits = bit_range(bitrev32(win), used, fit);
        st.consume(used + fit);
        if (PCR_RARELY(fit < nc)) {
            while (fit < nc) {
                const uint32_t q = nc - fit < 31u ? nc - fit : 31u;
                cbits |= (uint64_t)bit_range(bitrev32(st.window()), 0, q) << fit;
                fit += q;
                st.consume(q);
            }
        }
        next_win = st.window(); next_e = code.entry(next_win);
        corr |= cbits << ncorr; ncorr += nc;
        const uint32_t x = win << ((e >> 8) & 31u);
        eobrun = by_mask(eob & ~in_run, (1u << nx) | bit_range(x, 32u - nx, nx), eobrun);
        // no code; no zero to take; sizes above 1 do not exist in a refinement scan; bits beyond the unit's
        bad |= (e << 16) | (coef & (past | (1u - nx))) | st.beyond();
        // the block's masks move down with it, what the symbol made of its position enters at their top
        const uint32_t on = last + 1u, hit = coef & ~past & 0x80000000u;
        h >>= on;
        newm = (newm >> on) | ((uint64_t)hit << 32); sgn = (sgn >> on) | ((uint64_t)(hit & x) << 32);
        rem -= on;
        if (rem == 0) {                                       // the block is complete
            newm >>= to_place; sgn >>= to_place;
            block_done();
        }
    }
    return (int)bad < 0 ? kEFormat : kOk;
}

}  // namespace pcr
