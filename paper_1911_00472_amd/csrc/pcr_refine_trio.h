// AC refinement of one unit by THREE WAVEFRONTS of a workgroup, for launches that take as long as their longest unit.
//
// A lone wavefront issues an instruction every five to ten cycles whatever it is, so what bounds skim_ac_refine is the number of
// instructions between a symbol and the next: some 75 cycles a symbol, which depend on one another, and 600 a window and a block,
// which do not.  Those go to two wavefronts beside it:
//   trio_feed    what would start at each of the next 64 bit offsets, window after window, up to kTrioWindows ahead;
//   trio_keep    the zero tables of the blocks ahead of the walker, and behind it what it leaves of a block turned into the words of
//                the block's record; it is also the one that follows the scans this one builds on, and that others follow;
//   trio_walk    what is left: from symbol to symbol, window to window and block to block, all of it read from LDS a step ahead.
// They hand words on through rings in LDS, with a counter behind each (LDS takes the operations of a wavefront in order: the words
// are there once the counter says so).  Every wait ends: the feeder waits for the walker to leave windows, the keeper for it to
// leave blocks, the walker for either to be ahead of it, which they are unless they wait for it or (the keeper) for scans earlier in
// the chain; the walker gives everything free when it ends, whatever the data were.
//
// What is left: 74 cycles a symbol, 300 a block, 112 a window (one wavefront alone 75, 600 and 600).  512 photographs without entry points,
// all scans side by side at scan group 10: 5.37 -> 3.77 ms, of which the longest walk (90 150 symbols, 3 843 blocks, 5 278 windows) is all but
// some 0.1; 64 gray pictures of 64 x 64 at 6: 106 -> 82 us.  Where the launch is not its longest unit but the instructions of all of them,
// three wavefronts are slower than one (the line: TrioLaunch).
#pragma once

namespace pcr {

constexpr uint32_t kTrioWindows = 16, kTrioBlocks = 8;
struct TrioRings {
    uint32_t words[kTrioWindows][64];                         // windows: what a symbol at each offset does to the walker (TrioWord)
    uint32_t table[kTrioBlocks][64];                          // blocks: the zero table of block b in b % kTrioBlocks (TrioEntry)
    uint32_t out[kTrioBlocks][64];                            // ... what the walker made of it in (b + 1) % kTrioBlocks: entries taken, start word
    // what the walker may go up to: position in the unit of the last window that can be entered, blocks that can be begun (in either case with the one
    // behind it read ahead); what it is done with: blocks, and the position of its window; whether it has ended
    uint32_t win_ready, blk_ready, blk_done, win_used, over, pad[3];
};
static_assert(sizeof(TrioRings) % 16 == 0, "TrioRings layout");
typedef __attribute__((address_space(3))) TrioRings* TrioLds;
typedef volatile __attribute__((address_space(3))) uint32_t* TrioCount;

// TrioWord: what a symbol does to the walker's position, which is table index | window offset (less the corrections stepped over in
// this block) << 8, in one addition.  Bits 0..6 advance of the index (64 for all that is no new coefficient), 8..13 bits of the symbol, 16..30 for an
// end of band the blocks of its run (else 1: the walker's bits from 16 on mean nothing), bit 7 for a symbol that has to be done by
// hand, for the reason in bits 14..15.
// TrioEntry: corrections below the zero the entry belongs to << 8 (ZeroTable), bit 31 if nothing is left in the block behind it.
constexpr uint32_t kTrioByHand = 0x80u, kTrioMiss = 1, kTrioZeros = 2, kTrioInvalid = 3, kTrioLast = 0x80000000u;
// ... in the feeder's look-up of codes: the word's low half, the code's length << 16, 31 - (bits of an end-of-band run's length) << 21
PCR_D uint32_t trio_code(uint32_t e) {
    const uint32_t len = (e >> 8) & 31u, lo = e & 15u, r = (e >> 4) & 15u;
    if (e == 0) return 64u | kTrioByHand | (kTrioMiss << 14) | (31u << 21);
    if (e & kCodeCoef) return (lo == 1u ? (r + 1u) | ((len + 1u) << 8) : 64u | kTrioByHand | (kTrioInvalid << 14)) | (31u << 21);
    if (e & kCodeEob) return 64u | ((len + lo) << 8) | (len << 16) | ((31u - lo) << 21);
    return 64u | kTrioByHand | (len << 8) | (kTrioZeros << 14) | (31u << 21);
}

#if defined(__HIP_DEVICE_COMPILE__)
PCR_D uint32_t trio_read(TrioCount c) {
    const uint32_t v = uni(*c);
    asm volatile("" ::: "memory");
    return v;
}
PCR_D void trio_write(TrioCount c, uint32_t v) {
    asm volatile("" ::: "memory");
    *c = v;
}

// tab: the scan's table in LDS, stage: kStageWords words behind it; words, bits: the stream from the word the unit begins in; wb0: position
// of that word's first bit in the unit
PCR_D void trio_feed(TrioLds T, AcTab* tab, uint32_t* stage, const uint32_t* words, uint32_t bits, uint32_t wb0, uint32_t lane) {
    uint32_t* const code = tab->lutp;
    for (uint32_t i = lane; i < 256 + 128; i += 64) code[i] = trio_code(i < 256 ? tab->lut[i] : tab->lut2[i - 256]);
    wave_sync();
    const uint32_t lim8 = uni(tab->limit[0]), sh2 = uni(tab->sh2);
    StagedStream feed;
    feed.init((StageWords)stage, words, bits, lane);
    auto restage = [&]() { wave_sync(); feed.put(); wave_sync(); };
    auto ahead = [&]() {
        feed.read();
        if (__builtin_expect(feed.left == 0, 0)) restage();
    };
    restage();
    ahead();
    uint32_t w = 0, used = 0, at = 0, win = feed.window(), e = code[packed_index(win, lim8, sh2)];
    ahead();
    do {
        // (the next window's codes are looked up while this one's words are made)
        const uint32_t win_next = feed.window(), e_next = code[packed_index(win_next, lim8, sh2)];
        ahead();
        // the run of an end of band: a one and the bits behind the code
        const uint32_t run = __builtin_amdgcn_alignbit(1u, win << ((e >> 16) & 31u), 1u) >> ((e >> 21) & 31u);
        T->words[w % kTrioWindows][lane] = __builtin_amdgcn_perm(run, e, 0x05040100u);
        w++;
        trio_write(&T->win_ready, wb0 + 64 * (w - 2));
        if (w - used >= kTrioWindows) {
            at = trio_read(&T->win_used); used = (at - wb0) >> 6;
            while (at != ~0u && w - used >= kTrioWindows) {
                __builtin_amdgcn_s_sleep(1);
                at = trio_read(&T->win_used); used = (at - wb0) >> 6;
            }
        }
        win = win_next; e = e_next;
    } while (at != ~0u);
}

// The walker's loop.  A lone wavefront is all there is to it, so it is written out: what bounds it is the chain from one symbol to the
// next (78 cycles: two reads across lanes with an addition behind each, 27 and 31, the shift, the test, and 11 for a branch that is not taken),
// and around it the count of instructions (5 each), the branches taken (25) and the waits for LDS.  Eight copies of a symbol follow
// each other; a block's table and a window's words are read while the ones before them are in use.
//   x      on entry where to go on, on return why it stopped
//   o      window offset of the next symbol;  wb: position of the window in the unit
//   wins   windows that may still be entered, tabs: blocks that may still be begun (what is read ahead for them is there)
//   end    position of the unit's last bit (asked at the end of every ring of windows, so that a walk never goes far beyond it);  ring: the counters
constexpr uint32_t kWalkBlock = 0, kWalkWindow = 1, kWalkOn = 2, kWalkAfterZeros = 3, kWalkDone = 4;       // on entry: begin a block, enter a window, go on in a block, the same behind sixteen zeros, a block is done
constexpr uint32_t kWalkNoTable = 0, kWalkNoWindow = 1, kWalkByHand = 2;                                   // on return
struct TrioWalk {
    uint32_t p, q, st, o, wb, run, m, woff, toff, wins, tabs;
    uint64_t taken;                                           // table entries stood on in the block
    uint32_t vstep, vnext, vent, vahead, vout;                // per lane: this window's words and the next one's, this block's table and the next one's
};
// (set: marks the entry stood on; not done where sixteen zeros led to it, which leave it zero)
#define PCR_TRIO_SYMBOL(set, branch)                   \
    "v_readlane_b32 %[st], %[vstep], m0\n\t"           \
    set                                                \
    "s_add_i32 %[p], %[p], %[st]\n\t"                  \
    "v_readlane_b32 %[t], %[vent], %[p]\n\t"           \
    "s_add_i32 %[q], %[p], %[t]\n\t"                   \
    "s_lshr_b32 m0, %[q], 8\n\t"                       \
    "s_and_b32 %[t], %[q], %[past]\n\t"                \
    branch "\n\t"
#define PCR_TRIO_MARK "s_bitset1_b64 s[40:41], %[p]\n\t"
PCR_D uint32_t trio_walk_on(TrioWalk& W, uint32_t x, uint32_t end, uint32_t ring, uint32_t lane_at) {
    uint32_t t, ncorr, va, vb, vt;
    const uint32_t past = opaque(kTrioLast | 0xC040u), block = opaque(kTrioLast | 0x40u);
    asm volatile(
        "s_mov_b32 m0, %[o]\n\t"
        "v_add_u32_e32 %[vt], %[toff], %[lane_at]\n\t"
        "v_readlane_b32 %[ncorr], %[vent], 63\n\t"
        "s_cmp_eq_u32 %[x], 1\n\ts_cbranch_scc1 13f\n\t"
        "s_cmp_eq_u32 %[x], 2\n\ts_cbranch_scc1 11f\n\t"
        "s_cmp_eq_u32 %[x], 3\n\ts_cbranch_scc1 19f\n\t"
        "s_cmp_eq_u32 %[x], 4\n\ts_cbranch_scc1 16f\n\t"
        // a block begins; its table is here, the next one's sets out
        "10:\n\t"
        "s_sub_u32 %[tabs], %[tabs], 1\n\ts_cbranch_scc1 22f\n\t"
        "s_add_i32 %[toff], %[toff], 0x100\n\t"
        "s_and_b32 %[toff], %[toff], %[tmask]\n\t"
        "v_add_u32_e32 %[vt], %[toff], %[lane_at]\n\t"
        "ds_read_b32 %[vahead], %[vt] offset:%c[table]\n\t"
        "v_readlane_b32 %[ncorr], %[vent], 63\n\t"
        "s_add_i32 %[t], %[wb], m0\n\t"
        "v_writelane_b32 %[vout], %[t], 2\n\t"
        "v_writelane_b32 %[vout], %[run], 3\n\t"
        "s_mov_b64 s[40:41], 0\n\t"
        "s_lshl_b32 %[p], m0, 8\n\t"
        "s_cmp_lg_u32 %[run], 0\n\ts_cbranch_scc1 18f\n\t"
        "11:\n\t"
        "s_cmp_gt_u32 m0, 63\n\ts_cbranch_scc1 13f\n\t"
        "12:\n\t"
        PCR_TRIO_SYMBOL(PCR_TRIO_MARK, "s_cbranch_scc1 14f")
        PCR_TRIO_SYMBOL(PCR_TRIO_MARK, "s_cbranch_scc1 14f")
        PCR_TRIO_SYMBOL(PCR_TRIO_MARK, "s_cbranch_scc1 14f")
        PCR_TRIO_SYMBOL(PCR_TRIO_MARK, "s_cbranch_scc1 14f")
        PCR_TRIO_SYMBOL(PCR_TRIO_MARK, "s_cbranch_scc1 14f")
        PCR_TRIO_SYMBOL(PCR_TRIO_MARK, "s_cbranch_scc1 14f")
        PCR_TRIO_SYMBOL(PCR_TRIO_MARK, "s_cbranch_scc1 14f")
        PCR_TRIO_SYMBOL(PCR_TRIO_MARK, "s_cbranch_scc0 12b")
        "14:\n\t"
        "s_and_b32 %[t], %[q], %[block]\n\ts_cbranch_scc1 15f\n\t"
        "s_bfe_u32 m0, %[q], 0x80008\n\t"
        // on to the next window; its words are here, those of the one after it set out
        "13:\n\t"
        "s_sub_u32 %[wins], %[wins], 1\n\ts_cbranch_scc1 21f\n\t"
        "s_add_i32 %[woff], %[woff], 0x100\n\t"
        "s_and_b32 %[woff], %[woff], %[wmask]\n\t"
        "v_add_u32_e32 %[va], %[woff], %[lane_at]\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_mov_b32_e32 %[vstep], %[vnext]\n\t"
        "ds_read_b32 %[vnext], %[va]\n\t"
        "s_sub_i32 %[p], %[p], 0x4000\n\t"
        "s_add_i32 %[wb], %[wb], 64\n\t"
        "s_sub_i32 m0, m0, 64\n\t"
        "s_cmp_gt_u32 m0, 63\n\ts_cbranch_scc0 12b\n\t"
        "s_branch 13b\n\t"
        "19:\n\t"
        PCR_TRIO_SYMBOL("", "s_cbranch_scc1 14b")
        "s_branch 12b\n\t"
        // inside an end-of-band run: the corrections of the block, nothing else
        "18:\n\t"
        "s_sub_i32 %[run], %[run], 1\n\t"
        "s_bfe_u32 %[t], %[ncorr], 0x60008\n\t"
        "s_add_i32 m0, m0, %[t]\n\t"
        "s_branch 16f\n\t"
        // the last zero taken, or a sentinel landed on
        "17:\n\t"
        "s_bitset1_b64 s[40:41], %[p]\n\t"
        "s_bfe_u32 m0, %[q], 0x80008\n\t"
        "s_branch 16f\n\t"
        // the block ends: by its last zero, by an end of band (the corrections left follow it), or by something else
        "15:\n\t"
        "s_bitcmp1_b32 %[p], 6\n\ts_cbranch_scc0 17b\n\t"
        "s_and_b32 %[t], %[st], 0xC0\n\t"
        "s_cmp_lg_u32 %[t], 0x40\n\ts_cbranch_scc1 23f\n\t"
        "s_sub_i32 %[p], %[p], %[st]\n\t"
        "s_bfe_i32 %[p], %[p], 0x80008\n\t"
        "s_lshr_b32 %[run], %[st], 16\n\t"
        "s_bfe_u32 %[st], %[st], 0x60008\n\t"
        "s_add_i32 %[p], %[p], %[st]\n\t"
        "s_sub_i32 %[run], %[run], 1\n\t"
        "s_bfe_u32 %[t], %[ncorr], 0x60008\n\t"
        "s_add_i32 m0, %[p], %[t]\n\t"
        // the block is done: what there is to know of it to the keeper
        "16:\n\t"
        "v_writelane_b32 %[vout], s40, 0\n\t"
        "v_writelane_b32 %[vout], s41, 1\n\t"
        "s_add_i32 %[m], %[m], 1\n\t"
        "v_mov_b32_e32 %[va], %[m]\n\t"
        "v_mov_b32_e32 %[vb], %[wb]\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_mov_b32_e32 %[vent], %[vahead]\n\t"
        "ds_write_b32 %[vt], %[vout] offset:%c[out]\n\t"
        "ds_write2_b32 %[ring], %[va], %[vb] offset0:2 offset1:3\n\t"
        "s_branch 10b\n"
        // no more windows, or blocks, that are known to be there: asked anew
        "21:\n\t"
        "ds_read_b32 %[va], %[ring] offset:%c[wready]\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_readfirstlane_b32 %[t], %[va]\n\t"
        "s_sub_i32 %[t], %[t], %[wb]\n\t"
        "s_ashr_i32 %[wins], %[t], 6\n\t"
        "s_cmp_gt_u32 %[wb], %[end]\n\ts_cbranch_scc1 24f\n\t"
        "s_cmp_gt_i32 %[wins], 0\n\ts_cbranch_scc1 13b\n"
        "24:\n\ts_mov_b32 %[wins], 0\n\ts_mov_b32 %[x], 1\n\ts_branch 25f\n"
        "22:\n\t"
        "ds_read_b32 %[va], %[ring] offset:%c[bready]\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_readfirstlane_b32 %[t], %[va]\n\t"
        "s_sub_i32 %[tabs], %[t], %[m]\n\t"
        "s_cmp_gt_i32 %[tabs], 0\n\ts_cbranch_scc1 10b\n\t"
        "s_mov_b32 %[tabs], 0\n\ts_mov_b32 %[x], 0\n\ts_branch 25f\n"
        "23:\n\ts_mov_b32 %[x], 2\n"
        "25:\n\t"
        "s_mov_b32 %[o], m0\n\t"
        "s_waitcnt lgkmcnt(0)"
        : [x] "+&s"(x), [p] "+&s"(W.p), [q] "+&s"(W.q), [st] "+&s"(W.st), [t] "=&s"(t), [ncorr] "=&s"(ncorr), [o] "+&s"(W.o), [wb] "+&s"(W.wb), [run] "+&s"(W.run), [m] "+&s"(W.m),
          [woff] "+&s"(W.woff), [toff] "+&s"(W.toff), [wins] "+&s"(W.wins), [tabs] "+&s"(W.tabs), "+&{s[40:41]}"(W.taken),
          [vstep] "+&v"(W.vstep), [vnext] "+&v"(W.vnext), [vent] "+&v"(W.vent), [vahead] "+&v"(W.vahead), [vout] "+&v"(W.vout), [va] "=&v"(va), [vb] "=&v"(vb), [vt] "=&v"(vt)
        : [past] "s"(past), [block] "s"(block), [end] "s"(end), [wready] "n"(0), [bready] "n"(4), [lane_at] "v"(lane_at), [ring] "v"(ring),
          [tmask] "n"((kTrioBlocks - 1) * 256), [wmask] "n"((kTrioWindows - 1) * 256), [table] "n"(offsetof(TrioRings, table)), [out] "n"(offsetof(TrioRings, out))
        : "m0", "scc", "memory");
    return x;
}
#undef PCR_TRIO_SYMBOL
#undef PCR_TRIO_MARK

// tab: the scan's table in LDS (the feeder brings it); words, bits, wb0: as trio_feed; o0: offset of the unit's first bit.  Returns
// whether the walk met anything damaged; a coefficient with no zero left to take is for the keeper to see.
PCR_D uint32_t trio_walk(TrioLds T, const AcTab* tab, const uint32_t* words, uint32_t bits, uint32_t wb0, uint32_t o0, uint32_t blocks, uint32_t lane) {
    TrioWalk W;
    W.p = W.q = W.st = 0; W.o = o0; W.wb = wb0; W.run = 0; W.m = 0; W.woff = 0x100; W.toff = 0; W.tabs = 0;
    W.taken = 0; W.vahead = 0; W.vout = 0;
    const uint32_t end = wb0 + bits;
    uint32_t bad = 0, x = kWalkBlock;
    auto windows = [&]() {                                    // waits until the window behind this one can be entered
        trio_write(&T->win_used, W.wb);
        while ((int32_t)(W.wins = (uint32_t)((int32_t)(trio_read(&T->win_ready) - W.wb) >> 6)) <= 0) {}
    };
    auto next_window = [&]() {                                // (as the loop does it)
        const uint32_t w = (W.wb - wb0) >> 6;
        windows();
        W.wins--;
        W.vstep = W.vnext;
        W.woff = ((w + 2) % kTrioWindows) * 256;
        W.vnext = T->words[(w + 2) % kTrioWindows][lane];
        W.p -= 0x4000; W.o -= 64; W.wb += 64;
    };
    windows();
    W.vstep = T->words[0][lane]; W.vnext = T->words[1][lane];
    while (trio_read(&T->blk_ready) == 0) {}
    W.vent = T->table[0][lane];
    const uint32_t ring = (uint32_t)(size_t)&T->win_ready, lane_at = (uint32_t)(size_t)&T->words[0][lane];
    bool on = true;
    while (on) {
        x = trio_walk_on(W, x, end, ring, lane_at);
        bad |= (end - (W.wb + W.o)) >> 31 & (x == kWalkByHand ? 0u : 1u);      // (never far beyond the unit's data: the loop comes here at the end of every ring of windows at the latest)
        if (x == kWalkNoWindow) {
            windows();
        } else if (x == kWalkNoTable) {
            on = W.m < blocks;
            while (on && (int32_t)(W.tabs = trio_read(&T->blk_ready) - W.m) <= 0) {}
        } else {                                              // by hand: the symbol again from where it started
            auto entry = [&](uint32_t n) { return (uint32_t)__builtin_amdgcn_readlane((int)W.vent, (int)n); };      // n <= 63
            const uint32_t from = W.p - W.st, ncorr = (entry(63) >> 8) & 63u;
            uint32_t at = from & 63u, kind = (W.st >> 14) & 3u, ob = (uint32_t)((int32_t)(from << 16) >> 24) + ((W.st >> 8) & 63u), adv = kZrlAdvance;
            W.o = ob + ncorr;
            x = kWalkDone;
            if ((W.st & kTrioByHand) == 0) {
                bad |= 1u;                                    // a coefficient past the table
            } else {
                uint32_t info = 0;
                if (kind == kTrioMiss) {                      // a code in neither look-up, or none
                    const uint32_t b = W.wb - wb0 + ob + ((entry(at) >> 8) & 63u);      // (a miss has length 0; with the corrections passed it is inside the window)
                    const uint32_t last = (bits >> 5) + 4, i0 = b >> 5 < last ? b >> 5 : last, i1 = i0 + 1 < last ? i0 + 1 : last;
                    const uint32_t win = (uint32_t)((((uint64_t)uni(words[i0]) << 32 | uni(words[i1])) << (b & 31)) >> 32);
                    const uint32_t e = ac_long_code(tab, win);
                    info = uni(e ? pack_symbol(e, win, false) : kSymInvalid);
                    ob += (info >> 8) & 63;
                    kind = info == kSymInvalid ? kTrioInvalid : ((info & kSymSpecial) ? kTrioZeros : 0u);
                    if (kind == 0) adv = info & 127u;
                }
                if (kind == kTrioInvalid) {                   // no code at all, or one a refinement scan cannot hold
                    bad |= 1u;
                } else {
                    at += adv;                                // (sixteen zeros: lands on a zero and leaves it zero)
                    const uint32_t e = at < 64 ? entry(at & 63u) : (ncorr << 8) | kTrioLast;
                    W.o = ob + ((e >> 8) & 63u);
                    if (kind == 0 && at < 64) set_bit(&W.taken, at);
                    if (e & kTrioLast) {
                        if (info & kSymEob) W.run = (1u << ((info - 65) & 31)) - 1 + (info >> 16);
                        bad |= (info >> 15) & (opaque(63u - at) >> 31);
                    } else {
                        W.p = (ob << 8) | at;
                        x = kWalkOn;
                        if (kind == kTrioZeros) {
                            while (W.o >= 64) next_window();
                            x = kWalkAfterZeros;
                        }
                    }
                }
            }
        }
        on = on && bad == 0;                                  // (ends at the first damaged block)
    }
    trio_write(&T->over, 1u);
    trio_write(&T->win_used, ~0u);
    return bad;
}

template <class Gate>
PCR_D uint32_t trio_keep(TrioLds T, const LaneScan& ls, const HistPlanes& hp, uint64_t* recs, size_t nblk, uint32_t lane, Gate& gate) {
    const uint32_t bw = ls.bw[0], mcu_w = ls.mcu_w, blocks = ls.mcu1 - ls.mcu0;
    const uint64_t band = band_mask(ls.Ss, ls.Se);
    const uint32_t top = lane == (uint32_t)ls.Se ? kTrioLast : 0u;
    const uint32_t row_skip = bw - mcu_w;
    const uint32_t first_col = ls.mcu0 % mcu_w, first_blk = (ls.mcu0 / mcu_w) * bw + first_col;
    const uint32_t last_blk = ((ls.mcu1 - 1) / mcu_w) * bw + (ls.mcu1 - 1) % mcu_w;
    uint64_t* const nz_words = recs + ref_word(kRefNz, 0, nblk);
    uint64_t* const start_words = recs + ref_word(kRefStart, 0, nblk);
    uint64_t* const hist_words = recs + ref_word(kRefHist, 0, nblk);
    uint32_t fblk = first_blk, fcol = first_col;              // the block fetched next
    uint32_t sblk = first_blk, scol = first_col;              // the block stored next
    uint32_t hlo = 0, hhi = 0, done = 0, bad = 0;             // hlo, hhi: lane b % kTrioBlocks holds the history of block b
    auto fetch = [&](uint32_t m) {                            // (history words two blocks ahead, as in skim_ac_refine)
        gate.need(ls.mcu0 + (m < blocks ? m : blocks - 1));
        const HistWords w = hist_fetch(hp, fblk < last_blk ? fblk : last_blk, lane);
        fblk++; if (++fcol == mcu_w) { fcol = 0; fblk += row_skip; }
        return w;
    };
    HistWords h0 = fetch(0), h1 = fetch(1);
    auto step = [&](uint32_t i, HistWords& hw) -> bool {
        if (i < blocks) {
            const uint64_t h = hist_combine(hp, hw) & band, z = h ^ band, z1 = z | 1u;
            hw = fetch(i + 2);
            const uint32_t nzeros = (uint32_t)__builtin_popcountll(z), ncorr = (uint32_t)__builtin_popcountll(h);
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(z1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)z1, 0));
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(h >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)h, 0));
            const uint32_t data = select_by_mask(z1, (below << 8) | top, (ncorr << 8) | kTrioLast, lane);
            const uint32_t dest = select_by_mask(z1, rank, (nzeros + 1) + (lane - rank), lane);      // a permutation of the 64 lanes
            T->table[i % kTrioBlocks][dest & 63u] = data;
            trio_write(&T->blk_ready, i + 1 < blocks ? i : blocks);
            write_lane(hlo, (uint32_t)h, i % kTrioBlocks); write_lane(hhi, (uint32_t)(h >> 32), i % kTrioBlocks);
        }
        if (i >= kTrioBlocks - 1) {
            const uint32_t b = i - (kTrioBlocks - 1), slot = b % kTrioBlocks;
            while (done <= b) {
                const uint32_t over = trio_read(&T->over);    // (read ahead of the count: what the walker left before it ended is counted)
                done = trio_read(&T->blk_done);
                if (done <= b) {
                    if (over) return false;
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            const uint32_t v = T->out[(b + 1) % kTrioBlocks][lane];
            const uint64_t h = (uint32_t)__builtin_amdgcn_readlane((int)hlo, (int)slot) | ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hhi, (int)slot) << 32);
            const uint64_t z = h ^ band, z1 = z | 1u;
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(z1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)z1, 0));
            const uint64_t taken = (uint32_t)__builtin_amdgcn_readlane((int)v, 0) | ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)v, 1) << 32);
            const uint64_t start = (uint32_t)__builtin_amdgcn_readlane((int)v, 2) | ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)v, 3) << 32);
            const uint64_t newm = __ballot(((taken >> rank) & 1) != 0) & z;      // (positions that are no zeros are masked off)
            const uint64_t beyond = (taken >> (uint32_t)__builtin_popcountll(z)) >> 1;      // entries past the last zero: a coefficient that had none to take
            bad |= (uint32_t)beyond | (uint32_t)(beyond >> 32);
            gate.publish(ls.mcu0 + b);                        // (ahead of this block's record, as in skim_ac_refine)
            const uint32_t bv = per_lane(sblk);
            store_word(nz_words, bv * (uint32_t)(ref_word(kRefNz, 1, 0) * 8), newm);
            store_word(start_words, bv * 8, start);
            store_word(hist_words, bv * 8, h);
            sblk++; if (++scol == mcu_w) { scol = 0; sblk += row_skip; }
        }
        return true;
    };
    for (uint32_t i = 0; i < blocks + kTrioBlocks - 1; i += 2) {
        if (!step(i, h0)) break;
        if (i + 1 < blocks + kTrioBlocks - 1 && !step(i + 1, h1)) break;
    }
    return bad ? 1u : 0u;
}
#endif

}  // namespace pcr
