// Long first scans (AC first and DC first) without entry points, with many lanes per scan.
//
// A scan that is one unit is one serial stream, and the wavefront that follows it takes as long as it is: 40 ns a symbol of an AC
// first scan, 80 of an interleaved DC first scan, however idle the chip.  Like baseline scans (pcr_sequential.h, where the idea and
// its sources are) first scans fall into step: pieces are decoded from assumed states, those that turn out to begin in another
// state once more, until nothing changes; prefix sums over the blocks (and DC differences) passed then tell every lane where it
// stands, and all pieces are decoded a last time, storing.  The state is the position and the place in the band (AC: an end of band
// puts any two decoders at the same bit into step) or the block of the MCU (DC).  A piece here is short, a few dozen symbols: falling
// into step takes about as many, and what counts is the longest chain of pieces decoded one after the other.
// Bound by the latency of that chain, some 0.4 us a symbol of a lane; us a call of one plain picture, by wavefronts and by lanes: 500 x 500 at
// scan group 1 541 / 201, at 5 2163 / 230; 1000 x 1000 1925 / 218, 8264 / 401 (the rule and more figures: FirstSplitLaunch).
// Refinement scans cannot be had that way: how many bits a symbol takes depends on which block it is in.
#pragma once
#include "pcr_chains.h"
#include "pcr_sequential.h"

namespace pcr {

constexpr uint32_t kFirstPiece = 128;                       // bits per lane at least
constexpr uint32_t kFirstMostBlocks = 1u << 21;             // of a unit (the sums of a thousand pieces stay below 2^32, whatever the data say)

struct FirstTables {
    uint4 piece[kLaneTabPieces];                            // a LaneTab, or the DcTabs of the scan's components
    static_assert(sizeof(DcTab) * kMaxComp <= sizeof(uint4) * kLaneTabPieces && sizeof(DcTab) % 4 == 0, "they share the room");
};

// From `from` (bk: the place in the band) to the first symbol at or behind bit `end` of an AC first scan.  WRITE: stores what it passes, from
// block `block` of the scan to block `stop`; returns false where the data are no valid stream.  Not WRITE: the result depends on
// nothing but the state it starts in; *blocks: blocks ended.
template <bool WRITE>
PCR_D __attribute__((always_inline)) bool first_ac_walk(const LaneLookup& code, const SplitScan& S, uint32_t Ss, uint32_t Se, uint32_t Al, const SplitState& from, uint32_t end, LaneRing* ring, uint32_t lane,
                      SplitState* to, uint32_t* blocks, int16_t* plane, uint32_t elems, uint32_t block, uint32_t stop) {
    uint32_t k = from.bk, passed = 0, left = WRITE ? (block < stop ? stop - block : 0u) : 1u;
    bool good = true;
    if (from.pos < end && left != 0) {
        LaneStream st;
        st.init(S.words, from.pos, S.bit1, ring, lane);
        const uint32_t ends = S.bit1 - end;                   // st.beyond() is how many bits are left
        uint32_t low = st.low_water(1);
        uint32_t row = 0, col = 0, e0 = 0;
        if (WRITE) { row = block / S.mcu_w; col = block - row * S.mcu_w; e0 = (row * S.bw0 + col) * 64u; }
        while ((int)(st.beyond() - ends) > 0) {
            if (WRITE && left == 0) break;                    // what follows the last block is padding
            if (PCR_RARELY((int)(st.n - low) < 0)) { st.refill(); low = st.low_water(1); }
            const uint32_t win = st.window(), e = code.resolve(code.entry(win), win);
            const uint32_t len = bit_range(e, 8, 5), nx = e & 15u;
            const uint32_t x = win << len, extra = bit_range(x, 32u - nx, nx);
            st.consume(split_step(len + nx));
            const uint32_t at = k + bit_range(e, 4, 4), room = Se - at, coef = e << 17;
            if (WRITE) {
                // no code; a coefficient beyond the band; bits beyond the unit's
                if ((int)((e << 16) | (room & coef) | st.beyond()) < 0) { good = false; break; }
                if ((int)(room | ~coef) >= 0 && e0 + at < elems) plane[e0 + at] = (int16_t)((extra - (~sign_mask(x) & ((1u << nx) - 1u))) << Al);
            }
            const uint32_t eob = bit_mask(e, 13), over = eob | sign_mask(room - 1u);
            const uint32_t adv = by_mask(eob, (1u << nx) | extra, 1u) & over;
            k = by_mask(over, Ss, at + 1u);
            if (WRITE) {
                const uint32_t n = adv < left ? adv : left;
                left -= n; col += n;
                if (col >= S.mcu_w) { const uint32_t q = col / S.mcu_w; row += q; col -= q * S.mcu_w; }
                e0 = (row * S.bw0 + col) * 64u;
            } else passed += adv;
        }
        *to = SplitState{S.bit1 - st.beyond(), k};
    } else *to = from;
    *blocks = passed;
    return good;
}

// The same of a DC first scan (from.bk: the block of the MCU).  sums: WRITE: where the lane stands, in; else what it passed, out.
template <bool WRITE>
PCR_D __attribute__((always_inline)) bool first_dc_walk(const DcTab* tabs, const SplitScan& S, uint32_t Al, const SplitState& from, uint32_t end, LaneRing* ring, uint32_t lane, SplitState* to, SplitSums* sums,
                      int16_t* planes, int16_t* dense, uint32_t elems, uint32_t total) {
    uint32_t b = from.bk, block = WRITE ? sums->blocks : 0u;
    int dc0 = WRITE ? sums->dc0 : 0, dc1 = WRITE ? sums->dc1 : 0, dc2 = WRITE ? sums->dc2 : 0;
    bool good = true;
    if (from.pos < end && (!WRITE || block < total)) {
        LaneStream st;
        st.init(S.words, from.pos, S.bit1, ring, lane);
        const uint32_t ends = S.bit1 - end;
        uint32_t low = st.low_water(1), mx = 0, my = 0;
        if (WRITE) { const uint32_t m = S.mcu0 + block / S.per_mcu; my = m / S.mcu_w; mx = m - my * S.mcu_w; }
        while ((int)(st.beyond() - ends) > 0) {
            if (WRITE && block >= total) break;
            if (PCR_RARELY((int)(st.n - low) < 0)) { st.refill(); low = st.low_water(1); }
            const uint32_t win = st.window(), c = (S.comps >> (2 * b)) & 3u;
            const DcTab* t = tabs + c;
            uint32_t v = t->lut[win >> 24], len = v >> 4, nx = v & 15u, none = 0;
            if (PCR_RARELY(v == 0xFFu)) {
                if (v == 0xFFu) {                             // a code of more than eight bits, or none (the first sixteen codes are categories)
                    const uint32_t c16 = win >> 16;
                    uint32_t below = t->limit[0];
                    len = 9;
#pragma unroll
                    for (int q = 1; q <= 7; q++) { const uint32_t lim = t->limit[q]; if (c16 >= lim) { len++; below = lim; } }
                    const uint32_t idx = len <= 16 ? t->valptr[len - 9] + ((c16 - below) >> (16u - len)) : 16u;
                    none = (c16 >= t->limit[0] && c16 < t->limit[8] && idx < 16u) ? 0u : 1u;
                    nx = none ? 0u : t->huffval[idx & 15u] & 15u;
                    len = none ? 0u : len;
                }
            }
            const uint32_t x = win << len;
            const int value = (int)(bit_range(x, 32u - nx, nx) - (~sign_mask(x) & ((1u << nx) - 1u)));
            st.consume(split_step(len + nx));
            dc0 += c == 0 ? value : 0; dc1 += c == 1 ? value : 0; dc2 += c == 2 ? value : 0;
            if (WRITE) {
                if (none || (int)st.beyond() < 0) { good = false; break; }
                const uint32_t hs = pick(c, S.hs0, S.hs1, S.hs2), vs = pick(c, S.vs0, S.vs1, S.vs2);
                const uint32_t e0 = pick(c, S.at0, S.at1, S.at2) + ((my * vs + ((S.rows >> b) & 1u)) * pick(c, S.bw0, S.bw1, S.bw2) + mx * hs + ((S.cols >> b) & 1u)) * 64u;
                const int16_t p = (int16_t)((uint32_t)(c == 0 ? dc0 : (c == 1 ? dc1 : dc2)) << Al);
                if (e0 < elems) { dense[e0 >> 6] = p; if (planes) planes[e0] = p; }
            }
            block++;
            if (++b == S.per_mcu) { b = 0; if (WRITE && ++mx == S.mcu_w) { mx = 0; my++; } }
        }
        *to = SplitState{S.bit1 - st.beyond(), b};
    } else *to = from;
    if (!WRITE) *sums = SplitSums{block, dc0, dc1, dc2};
    return good;
}

#if defined(__HIPCC__)

// done[u] = 1: unit u needs nothing more.  A workgroup per unit.
template <uint32_t LANES>
__global__ void __launch_bounds__(LANES) k_first_split(DevRecord R, const Unit* __restrict__ units, uint32_t* __restrict__ done, const uint32_t* __restrict__ clean32, uint32_t to_planes) {
    constexpr uint32_t kWaves = LANES / 64;
    __shared__ __attribute__((aligned(16))) FirstTables T;
    __shared__ LaneRing rings[kWaves];
    __shared__ SplitState s_start[LANES], s_end[LANES];
    __shared__ SplitSums s_sums[LANES], s_part[kWaves];
    __shared__ uint16_t s_list[LANES];
    __shared__ uint32_t s_count[2];
    __shared__ int s_bad, s_status;
    const Unit un = units[blockIdx.x];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    UnitSetup L;
    // What becomes of the unit the wavefronts decide together: what they look at here nothing writes while this runs, but for the image's status
    // (workgroups that decode its other units write that word), which one lane reads for all, to be asked behind the first barrier.
    if (tid == 0) s_status = R.status[un.img];
    unit_setup(R, un, clean32, &L, []() { return true; });
    const size_t ig = (size_t)un.img * R.G + un.scan;
    const ScanDesc* sd = &R.scan[ig];
    const uint32_t bit0 = L.byte_off * 8 + L.sub_bits, bit1 = L.byte_off * 8 + L.nbits;
    const bool ac = uni((int)sd->Ss) > 0;
    const uint32_t ns = L.ok ? (uint32_t)L.ls.ns : 0u;
    const bool mine = L.ok && R.img[un.img].progressive && uni((int)sd->Ah) == 0 && !is_sequential_scan(*sd) && ns >= 1 && ns <= (uint32_t)kMaxComp && (!ac || ns == 1) && bit1 > bit0;
    SplitScan S{L.words, bit1, 0, 0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0, 0, 0};
    uint32_t total = 0;
    if (mine) {
        S.mcu0 = L.ls.mcu0; S.mcu_w = L.ls.mcu_w; S.bw0 = L.ls.bw[0]; S.bw1 = L.ls.bw[1]; S.bw2 = L.ls.bw[2]; S.at0 = L.ls.poff[0]; S.at1 = L.ls.poff[1]; S.at2 = L.ls.poff[2];
        if (ns > 1) { S.hs0 = L.ls.hs[0]; S.hs1 = L.ls.hs[1]; S.hs2 = L.ls.hs[2]; S.vs0 = L.ls.vs[0]; S.vs1 = L.ls.vs[1]; S.vs2 = L.ls.vs[2]; }
#pragma unroll
        for (uint32_t j = 0; j < (uint32_t)kMaxComp; j++) {
            const uint32_t hs = pick(j, S.hs0, S.hs1, S.hs2), vs = pick(j, S.vs0, S.vs1, S.vs2);
            if (j < ns)
                for (uint32_t y = 0; y < vs; y++)
                    for (uint32_t x = 0; x < hs; x++, S.per_mcu++) { S.comps |= j << (2 * S.per_mcu); S.cols |= x << S.per_mcu; S.rows |= y << S.per_mcu; }
        }
        const uint64_t all = (uint64_t)(L.ls.mcu1 - L.ls.mcu0) * S.per_mcu;
        total = all <= kFirstMostBlocks ? (uint32_t)all : 0u;
    }
    if (!mine || total == 0) { if (tid == 0) done[blockIdx.x] = 0; return; }
    // ---- the tables (k_headers has built them) ----
    if (ac) {
        const uint4* src = reinterpret_cast<const uint4*>(&R.tabs[R.tab_idx[ig]]);
        for (uint32_t e = tid; e < kLaneTabPieces; e += LANES) T.piece[e] = src[e];
    } else {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(&R.dctabs[R.dctab_idx[ig]]);
        for (uint32_t e = tid; e < ns * (uint32_t)(sizeof(DcTab) / 4); e += LANES) reinterpret_cast<uint32_t*>(T.piece)[e] = src[e];
    }
    // ---- the pieces ----
    const uint32_t bits = bit1 - bit0;
    uint32_t piece = (bits + LANES - 1) / LANES;
    if (piece < kFirstPiece) piece = kFirstPiece;
    const uint32_t last = (bits - 1) / piece;                 // the last lane with a piece
    auto end_of = [&](uint32_t p) { return p < last ? bit0 + (p + 1) * piece : bit1; };
    const uint32_t Ss = (uint32_t)L.ls.Ss, Se = (uint32_t)L.ls.Se, Al = (uint32_t)L.ls.Al, first_bk = ac ? Ss : 0u;
    if (tid <= last) { s_start[tid] = SplitState{bit0 + tid * piece, first_bk}; s_list[tid] = (uint16_t)tid; }
    if (tid == 0) { s_count[0] = last + 1; s_count[1] = 0; s_bad = 0; }
    __syncthreads();
    if (uni(s_status) != kOk) { if (tid == 0) done[blockIdx.x] = 0; return; }
    LaneLookup code;
    code.init(reinterpret_cast<const LaneTab*>(T.piece));     // (of a DC scan: looked at by nobody)
    const DcTab* const dct = reinterpret_cast<const DcTab*>(T.piece);
    uint32_t half_left = 1;
    for (uint32_t round = 0;; round++) {
        const uint32_t count = s_count[round & 1];
        if (count == 0) break;
        if (split_stops(round, count, &half_left)) { if (tid == 0) done[blockIdx.x] = 0; return; }       // (the same for everyone)
        if (tid < count) {
            const uint32_t p = s_list[tid];
            SplitState to;
            SplitSums sums{0, 0, 0, 0};
            if (ac) {
                first_ac_walk<false>(code, S, Ss, Se, Al, s_start[p], end_of(p), &rings[wave], lane, &to, &sums.blocks, nullptr, 0, 0, 0);
                sums.blocks = sums.blocks < total ? sums.blocks : total;      // (an end-of-band run may say anything)
            } else first_dc_walk<false>(dct, S, Al, s_start[p], end_of(p), &rings[wave], lane, &to, &sums, nullptr, nullptr, 0, 0);
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
    // ---- sums of the lanes before ----
    const SplitSums sums = tid <= last ? s_sums[tid] : SplitSums{0, 0, 0, 0};
    const SplitSums incl{lanes_prefix_sum(sums.blocks), (int)lanes_prefix_sum((uint32_t)sums.dc0), (int)lanes_prefix_sum((uint32_t)sums.dc1), (int)lanes_prefix_sum((uint32_t)sums.dc2)};
    if (lane == 63) s_part[wave] = incl;
    __syncthreads();
    SplitSums at{incl.blocks - sums.blocks, incl.dc0 - sums.dc0 + L.ls.pred[0], incl.dc1 - sums.dc1 + L.ls.pred[1], incl.dc2 - sums.dc2 + L.ls.pred[2]};
    uint32_t all = 0;
    for (uint32_t w = 0; w < kWaves; w++) {
        const SplitSums p = s_part[w];
        if (w < wave) { at.blocks += p.blocks; at.dc0 += p.dc0; at.dc1 += p.dc1; at.dc2 += p.dc2; }
        all += p.blocks;
    }
    // ---- once more, storing ----
    bool good = true;
    if (tid <= last) {
        SplitState to;
        uint32_t none;
        if (ac) good = first_ac_walk<true>(code, S, Ss, Se, Al, s_start[tid], end_of(tid), &rings[wave], lane, &to, &none, L.plane[0], L.plane_elems[0], L.ls.mcu0 + at.blocks, L.ls.mcu1);
        else good = first_dc_walk<true>(dct, S, Al, s_start[tid], end_of(tid), &rings[wave], lane, &to, &at, to_planes ? L.base : nullptr, R.dc + (uni((uint64_t)R.coef_off[un.img]) >> 6), L.base_elems, total);
        if (tid == last && all < total) good = false;         // the data end before the last block does
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
