// Long sequential (baseline) scans with many lanes per scan.
//
// A baseline file without restart markers is one serial stream, and a decoder that follows it from its first bit takes as
// long as it is: 16.5 ms for the 90 KB of a photograph, on a chip that is otherwise idle.  But Huffman streams fall into
// step: a decoder set down anywhere soon reads the same symbols as one that came from the start.  Its state is small -- the
// position, the block of the MCU, the place in the block -- so the stream is cut into pieces, a lane each.  What takes long is falling
// into step in the block of the MCU: a lane that reads luma blocks one place off goes on doing so until a chroma block comes, is thrown
// out of step there, and has one chance in six with every new try: some 2500 bits of a 4:2:0 photograph in the median, 23 000 for the
// worst piece of a file.
//
// By tries (k_split_tries, k_split_settle, k_split_store), for launches of few scans:
//   1. the end of every piece is decoded once for each block of the MCU it could begin with (a try): one of them nearly always ends
//      where the one decoder would have;
//   2. every piece is decoded from where each try of the piece before it ended, which says where that leaves the next piece: in one of
//      its own tries (a link), or elsewhere (2 to 15 in a hundred; those are decoded on, a piece a round, until they fall in);
//   3. following the links from the first piece gives every piece's start; prefix sums over the blocks and DC differences of the pieces
//      on that path which block it begins in and what its DC predictions are;
//   4. every piece is decoded once more and its coefficients stored.
// Up to thirteen times the work of one decoder, but only three or four pieces behind each other.  Bound by the issue of vector instructions
// with several scans, by the latency of a symbol (some 75 instructions and two reads of LDS that wait for each other) with one.  64
// photographs of 90 KB, us: 2570 by steps, 990 now (tries 390, settle 350, store 250); one of 99 KB at quality 97, which no step settled, 6200 -> 1500
// the whole call.  The end that is tried is eight blocks long: with six the 64 photographs take 1340 (more to decode on), with ten 1140.
// Blocks of very many bits have more to be decoded on than there is room for (split_dense in pcr_lib.hip); what is left goes in steps.
//
// By steps (k_sequential_split; many scans, scans whose MCUs are one block, and what the tries leave), a workgroup per scan: every lane decodes its piece as if a first
// block began there; every piece that turns out to begin in another state than was assumed is decoded again, until nothing changes (20 to 40
// rounds, most of them with few pieces); then steps 3 and 4.  Streams that do not fall into step are left to k_sequential, as are short
// ones: `done` says which.
//
// The rounds of a stream that ends with k_sequential are lost: an eighth to a fifth of its time if all of them run.  (By steps, that is: long
// stretches of identical tiny blocks, for which every phase is as good as any other, and high qualities whose blocks take a whole piece each.)
// The pieces left fall about geometrically, so at rounds 8, 16 and 32 the fall since half that round is continued to the last one, and
// where more than kSplitLeft would be left the kernel gives up at once.  Of 33 kinds of files (qualities 75 to 100, 120 to 1600 pixels, flat
// and noisy) those that would have come right in the last rounds are at 20 or below at all three, those given up at round 8 at 76 or above.
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
constexpr uint32_t kSplitRounds = 48;                         // of k_split_settle
constexpr uint32_t kSplitLeastBits = 65536;                  // falling into step takes a lane some 20 000 bits, at twice the time per symbol of k_sequential
// Bits of the end of a piece that the tries are made on, and of a piece: eight blocks of the scan's mean, at least and at most (pieces of at least that).
constexpr uint32_t kSplitRunInBlocks = 8, kSplitRunInLeast = 1024, kSplitRunInMost = 4096, kSplitPieceMost = 4096;
constexpr uint32_t kSplitLanePiece = 512;                     // bits of a piece of k_sequential_split at least
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
    uint32_t mx = 0, e0 = 0, m0 = 0, m1 = 0, m2 = 0;          // column of the MCU, first element of the block, of each component's part of the MCU
    bool good = true;
    auto element_of = [&](uint32_t c, uint32_t b) {           // first element of block b of the MCU, which is one of component c
        return pick(c, m0, m1, m2) + (((S.cols >> b) & 1u) * 64u) + (bit_mask(S.rows, b) & pick(c, S.bw0 * 64u, S.bw1 * 64u, S.bw2 * 64u));
    };
    if (WRITE) {
        dc0 = sums->dc0; dc1 = sums->dc1; dc2 = sums->dc2;
        const uint32_t at = k ? block - 1u : block;           // inside a block: the one begun by an earlier lane
        const uint32_t m = S.mcu0 + at / S.per_mcu, my = m / S.mcu_w;
        mx = m - my * S.mcu_w;
        m0 = S.at0 + (my * S.vs0 * S.bw0 + mx * S.hs0) * 64u; m1 = S.at1 + (my * S.vs1 * S.bw1 + mx * S.hs1) * 64u; m2 = S.at2 + (my * S.vs2 * S.bw2 + mx * S.hs2) * 64u;
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
            if (WRITE) {                                      // on to the next MCU, and from the last of a row to the first of the next
                mx -= wrap;
                const uint32_t row = sign_mask(S.mcu_w - 1u - mx);
                m0 += (wrap & (S.hs0 * 64u)) + (row & ((S.vs0 * S.bw0 - S.mcu_w * S.hs0) * 64u));
                m1 += (wrap & (S.hs1 * 64u)) + (row & ((S.vs1 * S.bw1 - S.mcu_w * S.hs1) * 64u));
                m2 += (wrap & (S.hs2 * 64u)) + (row & ((S.vs2 * S.bw2 - S.mcu_w * S.hs2) * 64u));
                mx &= ~row;
            }
        }
        b = b2 >> 1;
        pos = S.bit1 - st.beyond();
    }
    *to = SplitState{pos, b * 64 + k};
    if (!WRITE) *sums = SplitSums{blocks, dc0, dc1, dc2};
    return good;
}

// Whether round `round` of steps, with `count` pieces left, is not worth starting.  half_left: the pieces that were left at half the
// round the fall is looked at next.
constexpr uint32_t kSplitStepRounds = 64, kSplitLeft = 64, kSplitInSteps = 1u << 16;
PCR_D bool split_stops(uint32_t round, uint32_t count, uint32_t* half_left) {
    if (round < 4 || (round & (round - 1)) != 0) return false;
    if (round == kSplitStepRounds) return true;
    float left = (float)count;
    const float fall = left / (float)*half_left;
    for (uint32_t n = round < 8 ? 0 : 2 * kSplitStepRounds / round - 2; n > 0; n--) left *= fall;
    *half_left = count;
    return round >= 8 && left > (float)kSplitLeft;
}

#if defined(__HIPCC__)

// What a unit is given to work in: pieces it is cut into at most, tries of each (the blocks of an MCU), nodes there is room for, where
// its nodes and pieces begin, bits of a piece at least and bits of its end the tries are made on.  The host lays it out from the scan's mean bytes; units that turn out longer have longer pieces.
// No tries: a unit that is not for them.
struct SplitRoom { uint64_t node0; uint32_t piece0, pieces, tries, nodes, least, run_in; };
// A start state of a piece, where its decoder ended and what it passed.  Node p * tries + h: piece p from where try h of the piece
// before ended; behind those, in no order, the starts that no try had.
struct SplitNode { SplitState start, end; SplitSums sums; };
// next[node]: the node of the next piece that starts where this one ended, or
constexpr uint32_t kSplitOpen = 0xFFFD, kSplitLast = 0xFFFE, kSplitNone = 0xFFFF;         // none so far; the last piece; not a node
constexpr uint32_t kSplitNodes = 16384, kSplitFirstNodes = kSplitNodes / 2, kSplitPieces = 2048, kSplitStoreLanes = 256;
// A piece as it is once the one path through the nodes is known: its start, the blocks and DC sums ahead of it.
struct SplitPiece { SplitState start; SplitSums at; };

// The pieces of a unit.
struct SplitCut {
    uint32_t bit0, bit1, piece, last;                         // last: the last piece
    PCR_D uint32_t end_of(uint32_t p) const { return p < last ? bit0 + (p + 1) * piece : bit1; }
};

// Unit, scan and pieces, `most` of them of `least` bits and more (the same for all lanes); false: not a unit for the lanes.
PCR_D bool split_unit(const DevRecord& R, const Unit& un, const uint32_t* __restrict__ clean32, uint32_t most, uint32_t least, UnitSetup* L, SplitScan* S, SplitCut* C) {
    const int status = group_status(R, un.img);
    unit_setup(R, un, clean32, L, [status]() { return status == kOk; });
    const ScanDesc* sd = &R.scan[(size_t)un.img * R.G + un.scan];
    C->bit0 = L->byte_off * 8 + L->sub_bits; C->bit1 = L->byte_off * 8 + L->nbits;
    if (!(L->ok && is_sequential_scan(*sd) && L->ls.ns >= 1 && L->ls.ns <= kMaxComp && C->bit1 > C->bit0 && C->bit1 - C->bit0 >= kSplitLeastBits)) return false;
    const uint32_t ns = (uint32_t)L->ls.ns;
    *S = SplitScan{L->words, C->bit1, 0, 0, 0, 0, 0, 0, L->ls.mcu0, L->ls.mcu_w, 1, 1, 1, 1, 1, 1, L->ls.bw[0], L->ls.bw[1], L->ls.bw[2], L->ls.poff[0], L->ls.poff[1], L->ls.poff[2]};
    if (ns > 1) { S->hs0 = L->ls.hs[0]; S->hs1 = L->ls.hs[1]; S->hs2 = L->ls.hs[2]; S->vs0 = L->ls.vs[0]; S->vs1 = L->ls.vs[1]; S->vs2 = L->ls.vs[2]; }
#pragma unroll
    for (uint32_t j = 0; j < (uint32_t)kMaxComp; j++) {
        const uint32_t hs = pick(j, S->hs0, S->hs1, S->hs2), vs = pick(j, S->vs0, S->vs1, S->vs2);
        if (j < ns)
            for (uint32_t y = 0; y < vs; y++)
                for (uint32_t x = 0; x < hs; x++, S->per_mcu++) { S->comps |= j << (2 * S->per_mcu); S->cols |= x << S->per_mcu; S->rows |= y << S->per_mcu; }
    }
    const uint32_t bits = C->bit1 - C->bit0, even = (bits + most - 1) / most;
    C->piece = even > least ? even : least;
    C->last = (bits - 1) / C->piece;
    return true;
}
// The same for the kernels that go by tries.
PCR_D bool split_unit(const DevRecord& R, const Unit& un, const uint32_t* __restrict__ clean32, const SplitRoom& room, UnitSetup* L, SplitScan* S, SplitCut* C) {
    return split_unit(R, un, clean32, room.pieces, room.least, L, S, C) && S->per_mcu == room.tries && (C->last + 1) * room.tries <= room.nodes;
}

// The tables of a scan, each once, by a workgroup of LANES.
template <uint32_t LANES>
PCR_D void split_tables(const DevRecord& R, const Unit& un, const UnitSetup& L, SplitScan* S, SplitTables* T) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, ns = (uint32_t)L.ls.ns;
    const ScanDesc* sd = &R.scan[(size_t)un.img * R.G + un.scan];
    const uint32_t d0 = uni(sd->dc_off[0]), d1 = ns > 1 ? uni(sd->dc_off[1]) : d0, d2 = ns > 2 ? uni(sd->dc_off[2]) : d0;
    const uint32_t a0 = uni(sd->ac_offc[0]), a1 = ns > 1 ? uni(sd->ac_offc[1]) : a0, a2 = ns > 2 ? uni(sd->ac_offc[2]) : a0;
    const uint32_t dj1 = d1 == d0 ? 0u : 1u, dj2 = d2 == d0 ? 0u : (d2 == d1 ? 1u : 2u), aj1 = a1 == a0 ? 3u : 4u, aj2 = a2 == a0 ? 3u : (a2 == a1 ? 4u : 5u);
    S->dc_tabs = dj1 << 4 | dj2 << 8; S->ac_tabs = 3u | aj1 << 4 | aj2 << 8;
    const uint32_t used = 1u | 1u << dj1 | 1u << dj2 | 8u | 1u << aj1 | 1u << aj2;
    for (uint32_t t = uni(tid >> 6); t < kSplitTabs; t += LANES / 64) {
        if (!((used >> t) & 1u)) continue;
        const uint32_t o = t == 0 ? d0 : (t == 1 ? d1 : (t == 2 ? d2 : (t == 3 ? a0 : (t == 4 ? a1 : a2))));
        canon_build(&T->code[t], HeaderBytes{(GlobalBytes)R.rec, (LdsBytes) nullptr, 0, 0}, o, lane);
    }
    __syncthreads();
    for (uint32_t t = 0; t < kSplitTabs; t++) {
        if (!((used >> t) & 1u)) continue;
        const bool dc = t < (uint32_t)kMaxComp;
        for (uint32_t e = tid; e < (1u << kSplitBits); e += LANES) {
            const uint32_t f = canon_find<1, kSplitBits>(&T->code[t], e << (16 - kSplitBits));
            const uint32_t v = f ? T->code[t].vals[f & 255u] : 0u;
            T->lut[t][e] = (uint16_t)(f == 0 || (dc && (f & 255u) >= 16u) ? 0u : code_entry(f >> 8, dc ? v & 15u : v));
        }
    }
    __syncthreads();
}

// Workgroup (u, c): pieces c (per - 1) + 1 .. (c + 1) (per - 1) of unit u (and piece 0), per = lanes / tries.  First every try of those and of
// the piece before, then every piece from where the tries of the one before ended.
__global__ void __launch_bounds__(kSplitLanes) k_split_tries(DevRecord R, const Unit* __restrict__ units, const SplitRoom* __restrict__ rooms, SplitNode* __restrict__ nodes,
        uint32_t* __restrict__ next, const uint32_t* __restrict__ clean32) {
    __shared__ SplitTables T;
    __shared__ LaneRing rings[kSplitWaves];
    __shared__ SplitState s_end[kSplitLanes];
    __shared__ uint16_t s_list[kSplitLanes];
    __shared__ uint32_t s_count;
    const Unit un = units[blockIdx.x];
    const SplitRoom room = rooms[blockIdx.x];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    UnitSetup L;
    SplitScan S;
    SplitCut C;
    if (!split_unit(R, un, clean32, room, &L, &S, &C)) return;
    const uint32_t H = S.per_mcu, per = kSplitLanes / H, from = blockIdx.y * (per - 1);
    if (from > 0 && from >= C.last) return;
    split_tables<kSplitLanes>(R, un, L, &S, &T);
    const uint32_t a = tid / H, h = tid - a * H, p = from + a;
    const bool mine = a < per && p <= C.last;
    SplitState to{~0u, 0};
    SplitSums sums;
    if (mine && p < C.last) {
        const uint32_t begin = C.bit0 + p * C.piece, end = C.end_of(p);
        split_walk<false>(S, T, SplitState{end - begin > room.run_in ? end - room.run_in : begin, h * 64}, end, &rings[wave], lane, &to, &sums, nullptr, nullptr, 0, 0, 0);
    }
    s_end[tid] = to;
    if (tid == 0) s_count = 0;
    __syncthreads();
    // The starts of this workgroup's pieces, those that are alike once, dealt out to as few wavefronts as hold them.
    const bool ours = mine && (a > 0 || from == 0);
    bool wanted = ours;
    SplitState start{~0u, 0};
    if (p > 0 && ours) {
        start = s_end[tid - H];
        for (uint32_t e = 1; e <= h; e++) wanted = wanted && start != s_end[tid - H - e];
    } else if (p == 0 && h == 0) start.pos = C.bit0;          // (of piece 0 the start is known)
    else wanted = false;
    const uint64_t m = __ballot(wanted);
    uint32_t list = 0;
    if (lane == 0 && m) list = atomicAdd(&s_count, (uint32_t)__builtin_popcountll(m));
    list = uni(list);
    if (wanted) s_list[list + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] = (uint16_t)tid;
    if (ours && !wanted) {
        const uint64_t at = room.node0 + p * H + h;
        nodes[at].start = start; next[at] = kSplitNone;
    }
    __syncthreads();
    if (tid >= s_count) return;                               // (no barrier behind this)
    const uint32_t t = s_list[tid], ta = t / H, tp = from + ta;
    SplitNode node{tp > 0 ? s_end[t - H] : SplitState{C.bit0, 0}, SplitState{0, 0}, SplitSums{0, 0, 0, 0}};
    split_walk<false>(S, T, node.start, C.end_of(tp), &rings[wave], lane, &node.end, &node.sums, nullptr, nullptr, 0, 0, 0);
    uint32_t n = tp == C.last ? kSplitLast : kSplitOpen;
    for (uint32_t e = 0; e < H && n == kSplitOpen; e++) if (!(node.end != s_end[ta * H + e])) n = (tp + 1) * H + e;
    const uint64_t at = room.node0 + tp * H + (t - ta * H);
    nodes[at] = node; next[at] = n;
}

// The node of every piece on the path from the first, if it is known to the end, to path (by all lanes of a workgroup; true for all of them or
// none).  Following it node by node is a read of LDS behind another for every piece, 50 us of them: so the lanes follow every try at the head
// of each kSplitStretch pieces through those first, one lane goes from stretch to stretch, and a lane a stretch writes down what it holds.
constexpr uint32_t kSplitStretch = 32, kSplitStretches = kSplitPieces / kSplitStretch;
struct SplitPath { uint16_t leaves[kSplitStretches][4 * kMaxComp], enters[kSplitStretches]; uint32_t whole; };
PCR_D bool split_follow(const uint16_t* next, uint32_t planned, uint32_t H, uint32_t last, SplitPath* P, uint16_t* path) {
    const uint32_t tid = threadIdx.x, count = last / kSplitStretch + 1;
    auto through = [&](uint32_t i, uint32_t stretch, uint16_t* passed) {     // the node behind the stretch (kSplitLast: it ends with the last piece)
        const uint32_t p1 = (stretch + 1) * kSplitStretch <= last ? (stretch + 1) * kSplitStretch : last + 1;
        for (uint32_t p = stretch * kSplitStretch; p < p1 && i < kSplitOpen; p++) {
            if (passed) passed[p] = (uint16_t)i;
            i = next[i];
        }
        return i;
    };
    if (tid < count * H) {
        const uint32_t stretch = tid / H, h = tid - stretch * H;
        P->leaves[stretch][h] = (uint16_t)through(stretch * kSplitStretch * H + h, stretch, nullptr);
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t i = 0;
        for (uint32_t e = 0; e < count && i < kSplitOpen; e++) {
            P->enters[e] = (uint16_t)i;
            i = i < planned ? P->leaves[e][i - e * kSplitStretch * H] : through(i, e, nullptr);
        }
        P->whole = i == kSplitLast ? 1u : 0u;
    }
    __syncthreads();
    if (!P->whole) return false;
    if (tid < count) through(P->enters[tid], tid, path);
    __syncthreads();
    return true;
}

// One workgroup a unit: what ends in a state that the next piece was not started in is decoded on, a piece a round, until it falls in
// with a node; then the path and the sums along it.  done[u], where it is not 0: unit u has its pieces, and needs nothing but k_split_store; one more
// than the rounds it took.
__global__ void __launch_bounds__(kSplitLanes) k_split_settle(DevRecord R, const Unit* __restrict__ units, const SplitRoom* __restrict__ rooms, SplitNode* __restrict__ all_nodes,
        const uint32_t* __restrict__ all_next, SplitPiece* __restrict__ all_pieces, uint32_t* __restrict__ done, const uint32_t* __restrict__ clean32) {
    __shared__ SplitTables T;
    __shared__ LaneRing rings[kSplitWaves];
    __shared__ uint16_t s_next[kSplitNodes];
    __shared__ SplitSums s_part[kSplitWaves];
    __shared__ SplitPath s_path;
    __shared__ uint32_t s_count;
    const Unit un = units[blockIdx.x];
    const SplitRoom room = rooms[blockIdx.x];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    uint16_t* const path = reinterpret_cast<uint16_t*>(rings);
    static_assert(kSplitStretches * 4 * kMaxComp <= kSplitLanes, "a lane for every try at the head of a stretch");
    static_assert(sizeof rings >= kSplitPieces * sizeof(uint16_t), "the path is kept where the streams were");
    UnitSetup L;
    SplitScan S;
    SplitCut C;
    if (!split_unit(R, un, clean32, room, &L, &S, &C)) { if (tid == 0) done[blockIdx.x] = 0; return; }       // (the same for the whole workgroup)
    SplitNode* const nodes = all_nodes + room.node0;
    const uint32_t H = S.per_mcu, planned = (C.last + 1) * H;
    if (tid == 0) s_count = planned;
    __syncthreads();
    // (a new node begins where the one it follows ended; its piece waits in end.pos until it is decoded)
    auto follow_on = [&](uint32_t node, uint32_t p, const SplitState& start) {
        const uint32_t at = atomicAdd(&s_count, 1u);
        if (at >= room.nodes) return;
        nodes[at].start = start; nodes[at].end = SplitState{p, 0};
        s_next[at] = (uint16_t)kSplitOpen; s_next[node] = (uint16_t)at;
    };
    for (uint32_t i = tid; i < planned; i += kSplitLanes) {
        const uint32_t n = all_next[room.node0 + i];
        s_next[i] = (uint16_t)n;
        if (n == kSplitOpen) follow_on(i, i / H + 1, nodes[i].end);
    }
    __syncthreads();
    bool tables = false;
    uint32_t from = planned, round = 0;
    for (;; round++) {
        const uint32_t upto = s_count;
        if (split_follow(s_next, planned, H, C.last, &s_path, path)) break;   // (what is left does not lie on the path)
        if (upto > room.nodes || upto == from || round == kSplitRounds) { if (tid == 0) done[blockIdx.x] = 0; return; }       // (the same for everyone)
        if (!tables) { split_tables<kSplitLanes>(R, un, L, &S, &T); tables = true; }
        for (uint32_t i = from + tid; i < upto; i += kSplitLanes) {
            const uint32_t p = nodes[i].end.pos;
            SplitState to;
            SplitSums sums;
            split_walk<false>(S, T, nodes[i].start, C.end_of(p), &rings[wave], lane, &to, &sums, nullptr, nullptr, 0, 0, 0);
            nodes[i].sums = sums;
            uint32_t n = p == C.last ? kSplitLast : kSplitOpen;
            for (uint32_t e = 0; e < H && n == kSplitOpen; e++) if (!(to != nodes[(p + 1) * H + e].start)) n = (p + 1) * H + e;
            if (n == kSplitOpen) follow_on(i, p + 1, to);
            else s_next[i] = (uint16_t)n;
        }
        from = upto;
        __syncthreads();
    }
    // ---- sums of the pieces before, two pieces a lane ----
    static_assert(kSplitPieces == 2 * kSplitLanes, "two pieces a lane");
    const uint32_t p0 = 2 * tid;
    SplitSums one{0, 0, 0, 0}, two{0, 0, 0, 0};
    SplitState start0{0, 0}, start1{0, 0};
    if (p0 <= C.last) { const SplitNode& q = nodes[path[p0]]; one = q.sums; start0 = q.start; }
    if (p0 + 1 <= C.last) { const SplitNode& q = nodes[path[p0 + 1]]; two = q.sums; start1 = q.start; }
    const SplitSums sums{one.blocks + two.blocks, one.dc0 + two.dc0, one.dc1 + two.dc1, one.dc2 + two.dc2};
    const SplitSums incl{lanes_prefix_sum(sums.blocks), (int)lanes_prefix_sum((uint32_t)sums.dc0), (int)lanes_prefix_sum((uint32_t)sums.dc1), (int)lanes_prefix_sum((uint32_t)sums.dc2)};
    if (lane == 63) s_part[wave] = incl;
    __syncthreads();
    SplitSums at{incl.blocks - sums.blocks, incl.dc0 - sums.dc0 + L.ls.pred[0], incl.dc1 - sums.dc1 + L.ls.pred[1], incl.dc2 - sums.dc2 + L.ls.pred[2]};
    uint32_t all = 0;
    for (uint32_t w = 0; w < kSplitWaves; w++) {
        const SplitSums q = s_part[w];
        if (w < wave) { at.blocks += q.blocks; at.dc0 += q.dc0; at.dc1 += q.dc1; at.dc2 += q.dc2; }
        all += q.blocks;
    }
    SplitPiece* const pieces = all_pieces + room.piece0;
    if (p0 <= C.last) pieces[p0] = SplitPiece{start0, at};
    if (p0 + 1 <= C.last) pieces[p0 + 1] = SplitPiece{start1, SplitSums{at.blocks + one.blocks, at.dc0 + one.dc0, at.dc1 + one.dc1, at.dc2 + one.dc2}};
    if (tid == 0) { pieces[C.last + 1].at.blocks = all; done[blockIdx.x] = 1 + round; }
}

// Every piece once more, storing: workgroup (u, c) pieces c * kSplitStoreLanes and on of unit u.
__global__ void __launch_bounds__(kSplitStoreLanes) k_split_store(DevRecord R, const Unit* __restrict__ units, const SplitRoom* __restrict__ rooms, const SplitPiece* __restrict__ all_pieces,
        const uint32_t* __restrict__ done, const uint32_t* __restrict__ clean32) {
    __shared__ SplitTables T;
    __shared__ LaneRing rings[kSplitStoreLanes / 64];
    if (!done[blockIdx.x]) return;
    const Unit un = units[blockIdx.x];
    const SplitRoom room = rooms[blockIdx.x];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), p = blockIdx.y * kSplitStoreLanes + tid;
    UnitSetup L;
    SplitScan S;
    SplitCut C;
    if (!split_unit(R, un, clean32, room, &L, &S, &C)) return;
    if (blockIdx.y * kSplitStoreLanes > C.last) return;
    split_tables<kSplitStoreLanes>(R, un, L, &S, &T);
    if (p > C.last) return;
    const SplitPiece* const pieces = all_pieces + room.piece0;
    const uint32_t total = (L.ls.mcu1 - L.ls.mcu0) * S.per_mcu;
    const SplitPiece me = pieces[p];
    SplitSums at = me.at;
    SplitState to;
    bool good = split_walk<true>(S, T, me.start, C.end_of(p), &rings[wave], lane, &to, &at, L.base, R.dc + (uni((uint64_t)R.coef_off[un.img]) >> 6), L.base_elems, at.blocks, total);
    if (p == C.last) {                                        // the data may end before the last block does
        const uint32_t all = pieces[C.last + 1].at.blocks;
        if (all < total || (all == total && (to.bk & 63u) != 0)) good = false;
    }
    if (!good) R.status[un.img] = kEFormat;
}

// By steps; done[u], where it is not 0: unit u needs nothing more; one more than the rounds it took, and kSplitInSteps.
// left: only the units that are left (done[u] is 0), behind the tries.
__global__ void __launch_bounds__(kSplitLanes) k_sequential_split(DevRecord R, const Unit* __restrict__ units, uint32_t* __restrict__ done, uint32_t left, const uint32_t* __restrict__ clean32) {
    if (left && done[blockIdx.x]) return;
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
    SplitScan S;
    SplitCut C;
    if (!split_unit(R, un, clean32, kSplitLanes, kSplitLanePiece, &L, &S, &C)) { if (tid == 0) done[blockIdx.x] = 0; return; }       // (the same for the whole workgroup)
    if (tid == 0) s_bad = 0;
    split_tables<kSplitLanes>(R, un, L, &S, &T);
    const uint32_t last = C.last;                             // the last lane with a piece
    if (tid <= last) { s_start[tid] = SplitState{C.bit0 + tid * C.piece, 0}; s_list[tid] = (uint16_t)tid; }
    if (tid == 0) { s_count[0] = last + 1; s_count[1] = 0; }
    __syncthreads();
    // (The pieces of a round are packed into as few wavefronts as hold them: a wavefront with one lane at work takes as long
    // as a full one, and gets in the way of others.)
    uint32_t half_left = 1, round = 0;                        // half_left: pieces left at half the round the fall is looked at next
    for (;; round++) {
        const uint32_t count = s_count[round & 1];
        if (count == 0) break;
        if (split_stops(round, count, &half_left)) { if (tid == 0) done[blockIdx.x] = 0; return; }       // (the same for everyone)
        if (tid < count) {
            const uint32_t p = s_list[tid];
            SplitState to;
            SplitSums sums;
            split_walk<false>(S, T, s_start[p], C.end_of(p), &rings[wave], lane, &to, &sums, nullptr, nullptr, 0, 0, 0);
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
        good = split_walk<true>(S, T, s_start[tid], C.end_of(tid), &rings[wave], lane, &to, &at, L.base, R.dc + (uni((uint64_t)R.coef_off[un.img]) >> 6), L.base_elems, at.blocks, total);
        if (tid == last && (all < total || (all == total && (to.bk & 63u) != 0))) good = false;      // the data end before the last block does
    }
    if (!good) s_bad = 1;
    __syncthreads();
    if (tid == 0) {
        if (s_bad) R.status[un.img] = kEFormat;
        done[blockIdx.x] = kSplitInSteps + 1 + round;
    }
}

#endif  // __HIPCC__

}  // namespace pcr
