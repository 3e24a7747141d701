// Long sequential (baseline) scans with many lanes per scan.
//
// A baseline file without restart markers is one serial stream, and a decoder that follows it from its first bit takes as
// long as it is: 16.5 ms for the 90 KB of a photograph, on a chip that is otherwise idle.  But Huffman streams fall into
// step: a decoder set down anywhere soon reads the same symbols as one that came from the start.  Its state is small -- the
// position, the block of the MCU, the place in the block -- so the stream is cut into pieces, a lane each (kSplitLanes, a
// workgroup per scan):
//   1. every lane decodes its piece as if a first block began there, and leaves the state it ends in;
//   2. every piece that turns out to begin in another state than was assumed is decoded again, until nothing changes.  Piece
//      0 is right from the start, and one that follows a right one is right a round later, so what is left at the end is
//      what one decoder would have seen;
//   3. prefix sums over the blocks and the DC differences of the pieces tell every lane which block it begins in and what
//      its DC predictions are;
//   4. every lane decodes its piece once more and stores the coefficients.
// Falling into step in the block of the MCU is what takes long: a lane that reads luma blocks one place off goes on
// doing so until a chroma block comes, is thrown out of step there, and has one chance in six with every new try: some
// 2500 bits of a 4:2:0 photograph in the median, 23 000 for the worst piece of a file (20 to 40 rounds, most of them with
// few pieces).  Streams that do not fall into step in kSplitRounds rounds are left to k_sequential, as are short ones:
// `done` says which.  64 photographs of 90 KB: 16.5 -> 2.5 ms.
//
// The rounds of a stream that ends with k_sequential are lost: an eighth to a fifth of its time if all of them run.  Such are
// long stretches of identical tiny blocks, for which every phase is as good as any other (one piece comes right per
// round), and high qualities whose blocks take a whole piece each (a 240 x 240 picture at quality 97 has 833 of 943 pieces
// left after 8 rounds, 319 after 32).  The pieces left fall about geometrically, so at rounds 8, 16 and 32 the fall since
// half that round is continued to the last one, and where more than kSplitLeft would be left the kernel gives up at
// once.  Of 33 kinds of files (qualities 75 to 100, 120 to 1600 pixels, flat and noisy) those that would have come right
// in the last rounds are at 20 or below at all three, those given up at round 8 at 76 or above.  (Sixteen pictures of one
// colour, 2048 x 2048 in 4:2:0: 44.1 ms by k_sequential alone, 53.9 after all rounds, 45.8 now; in 4:4:4 102.6, 117.4, 106.7.)
//
// Decoding pieces speculatively until they fall into step is the subject of Klein and Wiseman, "Parallel Huffman Decoding
// with Applications to JPEG Files" (The Computer Journal 46, 2003), and, on GPUs, of Weissenberger and Schmidt, "Accelerating
// JPEG Decompression on GPUs" (HiPC 2021); what is here was written from the idea.
#pragma once
#include "pcr_lanes.h"
#if defined(__HIPCC__)
#include "pcr_kernels.h"
#endif

namespace pcr {

constexpr uint32_t kSplitLanes = 1024, kSplitWaves = kSplitLanes / 64;
constexpr uint32_t kSplitRounds = 64, kSplitLeft = 64;
constexpr uint32_t kSplitLeastBits = 65536;                  // falling into step takes a lane some 20 000 bits, at twice the time per symbol of k_sequential
constexpr uint32_t kSplitPiece = 512;                         // bits per lane at least
constexpr uint32_t kSplitBits = 12, kSplitTabs = 2 * kMaxComp;

struct SplitTables {
    uint16_t lut[kSplitTabs][1u << kSplitBits];               // code_entry of the code at the head of the index, 0: a longer one, or none
    CanonCode code[kSplitTabs];                               // for those
};
// What the lanes of a scan share: scan component j's DC table in bits 4 j .. 4 j + 3 of dc_tabs, its AC table in ac_tabs; block
// b of an MCU: its scan component in bits 2 b .. 2 b + 1 of comps, its column and row in the component's part of the MCU.
struct SplitScan {
    const uint32_t* words; uint32_t bit1;
    uint32_t dc_tabs, ac_tabs, comps, cols, rows, per_mcu;
    // where blocks lie
    uint32_t mcu0, mcu_w, hs0, hs1, hs2, vs0, vs1, vs2, bw0, bw1, bw2, at0, at1, at2;
};
// Where a decoder stands: next bit, block of the MCU, place in the block (0: its DC code comes next).
struct SplitState {
    uint32_t pos, bk;                                         // bk = b * 64 + k
    PCR_D bool operator!=(const SplitState& o) const { return pos != o.pos || bk != o.bk; }
};
struct SplitSums { uint32_t blocks; int dc0, dc1, dc2; };     // block starts passed, sums of the DC differences by component

// The entry of a code the look-up does not resolve.
PCR_D uint32_t split_long_code(const CanonCode* c, uint32_t c16, bool dc) {
    const uint32_t f = canon_find<1, 16>(c, c16);
    if (f == 0 || (dc && (f & 255u) >= 16u)) return kCodeBad;            // (DC: the first sixteen codes are categories)
    const uint32_t v = c->vals[f & 255u];
    return code_entry(f >> 8, dc ? v & 15u : v);
}

PCR_D uint32_t pick(uint32_t c, uint32_t v0, uint32_t v1, uint32_t v2) { return c == 0 ? v0 : (c == 1 ? v1 : v2); }

// The bits a walk moves on by: one at least, whatever the data and the tables hold, so that every walk ends.
PCR_HD uint32_t split_step(uint32_t bits) { return bits < 1u ? 1u : bits; }

// From `from` to the first symbol at or behind bit `end`.  WRITE: stores what it passes, as far as block `total` (block numbers
// count from the unit's first); returns false where the data are no valid stream.  Not WRITE: whatever the data are, the result
// depends on nothing but the state it starts in.
template <bool WRITE>
PCR_D __attribute__((always_inline)) bool split_walk(const SplitScan& S, const SplitTables& T, const SplitState& from, uint32_t end, LaneRing* ring, uint32_t lane, SplitState* to, SplitSums* sums,
                      int16_t* base, int16_t* dense, uint32_t elems, uint32_t block, uint32_t total) {
    uint32_t pos = from.pos, b = from.bk >> 6, k = from.bk & 63u;
    uint32_t blocks = 0;
    int dc0 = 0, dc1 = 0, dc2 = 0;
    uint32_t mx = 0, my = 0, e0 = 0;
    bool good = true;
    auto element_of = [&](uint32_t c, uint32_t b) {           // first element of block b of MCU (mx, my), which is one of component c
        const uint32_t hs = pick(c, S.hs0, S.hs1, S.hs2), vs = pick(c, S.vs0, S.vs1, S.vs2), bw = pick(c, S.bw0, S.bw1, S.bw2), at = pick(c, S.at0, S.at1, S.at2);
        return at + ((my * vs + ((S.rows >> b) & 1u)) * bw + mx * hs + ((S.cols >> b) & 1u)) * 64u;
    };
    if (WRITE) {
        dc0 = sums->dc0; dc1 = sums->dc1; dc2 = sums->dc2;
        const uint32_t at = k ? block - 1u : block;           // inside a block: the one begun by an earlier lane
        const uint32_t m = S.mcu0 + at / S.per_mcu;
        my = m / S.mcu_w; mx = m - my * S.mcu_w;
        if (k) e0 = element_of((S.comps >> (2 * b)) & 3u, b);
    }
    if (pos < end && (!WRITE || block < total || (k && block == total))) {
        LaneStream st;
        st.init(S.words, pos, S.bit1, ring, lane);
        const uint32_t ends = S.bit1 - end;                   // st.beyond() is how many bits are left
        uint32_t low = st.low_water(1);
        const uint32_t per_mcu = S.per_mcu;
        uint32_t b2 = 2u * b;
        // (on a 64-byte line: where the code ahead of it happened to put it made a difference of 3 % of the kernel)
        [[clang::code_align(64)]] while ((int)(st.beyond() - ends) > 0) {
            if (PCR_RARELY((int)(st.n - low) < 0)) { st.refill(); low = st.low_water(1); }
            const uint32_t win = st.window();
            const uint32_t dc = sign_mask(k - 1u);            // (k is 0 .. 63)
            const uint32_t c4 = bit_range(S.comps, b2, 2) * 4u, t = bit_range(by_mask(dc, S.dc_tabs, S.ac_tabs), c4, 4);
            uint32_t e = T.lut[t][win >> (32 - kSplitBits)];
            if (PCR_RARELY(e == 0)) { if (e == 0) e = split_long_code(&T.code[t], win >> 16, dc != 0); }
            const uint32_t len = bit_range(e, 8, 5), nx = e & 15u;
            const uint32_t x = win << len, extra = bit_range(x, 32u - nx, nx);
            const int value = (int)(extra - (~sign_mask(x) & ((1u << nx) - 1u)));   // (a value without its top bit stands for a negative one)
            const uint32_t at = k + bit_range(e, 4, 4);       // the position the symbol lands on (sixteen zeros: the last of them)
            const uint32_t eob = bit_mask(e, 13) & ~dc, none = bit_mask(e, 15);
            // no code; an end-of-band run; a coefficient beyond position 63
            uint32_t bad = none | (eob & sign_mask(0u - nx)) | (bit_mask(e, 14) & sign_mask(63u - at));
            st.consume(split_step(len + nx));
            if (WRITE) {
                const uint32_t c = c4 >> 2;
                if (dc) {
                    if (block >= total) break;                // what follows the last block is padding
                    dc0 += c == 0 ? value : 0; dc1 += c == 1 ? value : 0; dc2 += c == 2 ? value : 0;
                    block++;
                    e0 = element_of(c, b2 >> 1);
                    const int16_t v = (int16_t)(c == 0 ? dc0 : (c == 1 ? dc1 : dc2));
                    if (e0 < elems) { base[e0] = v; dense[e0 >> 6] = v; }
                } else if ((e & kCodeCoef) && at <= 63u && e0 + at < elems) base[e0 + at] = (int16_t)value;
                if ((int)(bad | st.beyond()) < 0) { good = false; break; }      // (or bits past the unit's end)
            } else {
                const uint32_t d = dc & ~none & (uint32_t)value;
                dc0 += (int)(d & sign_mask(c4 - 1u)); dc1 += (int)(d & bit_mask(c4, 2)); dc2 += (int)(d & bit_mask(c4, 3));
                blocks -= dc;                                 // (one more)
            }
            const uint32_t over = eob | bad | sign_mask(62u - at);      // the block ends here (a DC code cannot land there)
            k = ~over & (at + 1u);
            b2 += over & 2u;
            const uint32_t wrap = sign_mask(2u * per_mcu - 1u - b2);
            b2 &= ~wrap;
            if (WRITE && wrap && ++mx == S.mcu_w) { mx = 0; my++; }
        }
        b = b2 >> 1;
        pos = S.bit1 - st.beyond();
    }
    *to = SplitState{pos, b * 64 + k};
    if (!WRITE) *sums = SplitSums{blocks, dc0, dc1, dc2};
    return good;
}

// Whether round `round`, with `count` pieces left, is not worth starting.  half_left: the pieces that were left at half the
// round the fall is looked at next.
PCR_D bool split_stops(uint32_t round, uint32_t count, uint32_t* half_left) {
    if (round < 4 || (round & (round - 1)) != 0) return false;
    if (round == kSplitRounds) return true;
    float left = (float)count;
    const float fall = left / (float)*half_left;
    for (uint32_t n = round < 8 ? 0 : 2 * kSplitRounds / round - 2; n > 0; n--) left *= fall;
    *half_left = count;
    return round >= 8 && left > (float)kSplitLeft;
}

#if defined(__HIPCC__)

// done[u] = 1: unit u needs nothing more.
__global__ void __launch_bounds__(kSplitLanes) k_sequential_split(DevRecord R, const Unit* __restrict__ units, uint32_t* __restrict__ done, const uint32_t* __restrict__ clean32) {
    __shared__ SplitTables T;
    __shared__ LaneRing rings[kSplitWaves];
    // per piece: the state its decoder was last set down in, the one it ended in, what it passed; and the pieces of a round
    __shared__ SplitState s_start[kSplitLanes], s_end[kSplitLanes];
    __shared__ SplitSums s_sums[kSplitLanes], s_part[kSplitWaves];
    __shared__ uint16_t s_list[kSplitLanes];
    __shared__ uint32_t s_count[2];
    __shared__ int s_bad;
    const Unit un = units[blockIdx.x];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    UnitSetup L;
    const int status = group_status(R, un.img);
    unit_setup(R, un, clean32, &L, [status]() { return status == kOk; });
    const ScanDesc* sd = &R.scan[(size_t)un.img * R.G + un.scan];
    const uint32_t bit0 = L.byte_off * 8 + L.sub_bits, bit1 = L.byte_off * 8 + L.nbits;
    const bool mine = L.ok && is_sequential_scan(*sd) && L.ls.ns >= 1 && L.ls.ns <= kMaxComp && bit1 > bit0 && bit1 - bit0 >= kSplitLeastBits;
    if (!mine) { if (tid == 0) done[blockIdx.x] = 0; return; }         // (the same for the whole workgroup: it has the status from one lane)
    // ---- the tables, each once ----
    const uint32_t ns = (uint32_t)L.ls.ns;
    SplitScan S{L.words, bit1, 0, 0, 0, 0, 0, 0, L.ls.mcu0, L.ls.mcu_w, 1, 1, 1, 1, 1, 1, L.ls.bw[0], L.ls.bw[1], L.ls.bw[2], L.ls.poff[0], L.ls.poff[1], L.ls.poff[2]};
    if (ns > 1) { S.hs0 = L.ls.hs[0]; S.hs1 = L.ls.hs[1]; S.hs2 = L.ls.hs[2]; S.vs0 = L.ls.vs[0]; S.vs1 = L.ls.vs[1]; S.vs2 = L.ls.vs[2]; }
    const uint32_t d0 = uni(sd->dc_off[0]), d1 = ns > 1 ? uni(sd->dc_off[1]) : d0, d2 = ns > 2 ? uni(sd->dc_off[2]) : d0;
    const uint32_t a0 = uni(sd->ac_offc[0]), a1 = ns > 1 ? uni(sd->ac_offc[1]) : a0, a2 = ns > 2 ? uni(sd->ac_offc[2]) : a0;
    const uint32_t dj1 = d1 == d0 ? 0u : 1u, dj2 = d2 == d0 ? 0u : (d2 == d1 ? 1u : 2u), aj1 = a1 == a0 ? 3u : 4u, aj2 = a2 == a0 ? 3u : (a2 == a1 ? 4u : 5u);
    S.dc_tabs = dj1 << 4 | dj2 << 8; S.ac_tabs = 3u | aj1 << 4 | aj2 << 8;
    const uint32_t used = 1u | 1u << dj1 | 1u << dj2 | 8u | 1u << aj1 | 1u << aj2;
#pragma unroll
    for (uint32_t j = 0; j < (uint32_t)kMaxComp; j++) {
        const uint32_t hs = pick(j, S.hs0, S.hs1, S.hs2), vs = pick(j, S.vs0, S.vs1, S.vs2);
        if (j < ns)
            for (uint32_t y = 0; y < vs; y++)
                for (uint32_t x = 0; x < hs; x++, S.per_mcu++) { S.comps |= j << (2 * S.per_mcu); S.cols |= x << S.per_mcu; S.rows |= y << S.per_mcu; }
    }
    if (tid == 0) s_bad = 0;
    if (wave < kSplitTabs && ((used >> wave) & 1u)) {
        const uint32_t o = wave == 0 ? d0 : (wave == 1 ? d1 : (wave == 2 ? d2 : (wave == 3 ? a0 : (wave == 4 ? a1 : a2))));
        canon_build(&T.code[wave], HeaderBytes{(GlobalBytes)R.rec, (LdsBytes) nullptr, 0, 0}, o, lane);
    }
    __syncthreads();
    for (uint32_t t = 0; t < kSplitTabs; t++) {
        if (!((used >> t) & 1u)) continue;
        const bool dc = t < (uint32_t)kMaxComp;
        for (uint32_t e = tid; e < (1u << kSplitBits); e += kSplitLanes) {
            const uint32_t f = canon_find<1, kSplitBits>(&T.code[t], e << (16 - kSplitBits));
            const uint32_t v = f ? T.code[t].vals[f & 255u] : 0u;
            T.lut[t][e] = (uint16_t)(f == 0 || (dc && (f & 255u) >= 16u) ? 0u : code_entry(f >> 8, dc ? v & 15u : v));
        }
    }
    __syncthreads();
    // ---- the pieces ----
    const uint32_t bits = bit1 - bit0;
    uint32_t piece = (bits + kSplitLanes - 1) / kSplitLanes;
    if (piece < kSplitPiece) piece = kSplitPiece;
    const uint32_t last = (bits - 1) / piece;                 // the last lane with a piece
    auto end_of = [&](uint32_t p) { return p < last ? bit0 + (p + 1) * piece : bit1; };
    if (tid <= last) { s_start[tid] = SplitState{bit0 + tid * piece, 0}; s_list[tid] = (uint16_t)tid; }
    if (tid == 0) { s_count[0] = last + 1; s_count[1] = 0; }
    __syncthreads();
    // (The pieces of a round are packed into as few wavefronts as hold them: a wavefront with one lane at work takes as long
    // as a full one, and gets in the way of others.)
    uint32_t half_left = 1;                                   // pieces left at half the round the fall is looked at next
    for (uint32_t round = 0;; round++) {
        const uint32_t count = s_count[round & 1];
        if (count == 0) break;
        if (split_stops(round, count, &half_left)) { if (tid == 0) done[blockIdx.x] = 0; return; }       // (the same for everyone)
        if (tid < count) {
            const uint32_t p = s_list[tid];
            SplitState to;
            SplitSums sums;
            split_walk<false>(S, T, s_start[p], end_of(p), &rings[wave], lane, &to, &sums, nullptr, nullptr, 0, 0, 0);
            s_end[p] = to; s_sums[p] = sums;
        }
        __syncthreads();
        bool again = false;
        if (tid > 0 && tid <= last) {
            const SplitState before = s_end[tid - 1];
            again = before != s_start[tid];
            if (again) s_start[tid] = before;
        }
        const uint64_t m = __ballot(again);
        uint32_t at = 0;
        if (lane == 0 && m) at = atomicAdd(&s_count[(round + 1) & 1], (uint32_t)__builtin_popcountll(m));
        at = uni(at);
        if (again) s_list[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] = (uint16_t)tid;
        if (tid == 0) s_count[round & 1] = 0;
        __syncthreads();
    }
    const SplitSums sums = tid <= last ? s_sums[tid] : SplitSums{0, 0, 0, 0};
    // ---- sums of the lanes before ----
    SplitSums incl{lanes_prefix_sum(sums.blocks), (int)lanes_prefix_sum((uint32_t)sums.dc0), (int)lanes_prefix_sum((uint32_t)sums.dc1), (int)lanes_prefix_sum((uint32_t)sums.dc2)};
    if (lane == 63) s_part[wave] = incl;
    __syncthreads();
    SplitSums at{incl.blocks - sums.blocks, incl.dc0 - sums.dc0 + L.ls.pred[0], incl.dc1 - sums.dc1 + L.ls.pred[1], incl.dc2 - sums.dc2 + L.ls.pred[2]};
    uint32_t all = 0;
    for (uint32_t w = 0; w < kSplitWaves; w++) {
        const SplitSums p = s_part[w];
        if (w < wave) { at.blocks += p.blocks; at.dc0 += p.dc0; at.dc1 += p.dc1; at.dc2 += p.dc2; }
        all += p.blocks;
    }
    const uint32_t total = (L.ls.mcu1 - L.ls.mcu0) * S.per_mcu;
    // ---- once more, storing ----
    bool good = true;
    if (tid <= last) {
        SplitState to;
        good = split_walk<true>(S, T, s_start[tid], end_of(tid), &rings[wave], lane, &to, &at, L.base, R.dc + (uni((uint64_t)R.coef_off[un.img]) >> 6), L.base_elems, at.blocks, total);
        if (tid == last && (all < total || (all == total && (to.bk & 63u) != 0))) good = false;      // the data end before the last block does
    }
    if (!good) s_bad = 1;
    __syncthreads();
    if (tid == 0) {
        if (s_bad) R.status[un.img] = kEFormat;
        done[blockIdx.x] = 1;
    }
}

#endif  // __HIPCC__

}  // namespace pcr
