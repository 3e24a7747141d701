// Symbol statistics for the transcode to progressive files (paper Section 5, "Encoding": every image is re-coded as
// a progressive file before its scans are grouped into a record).  An optimised Huffman table needs to know how often
// each symbol occurs in a scan; k_symbol_hist counts that on the device, from the coefficient planes a decode left
// there, for every scan of the script the transcoder writes.  One workgroup per (image, scan): a lane per block, 512 blocks at a
// time in scan order, counting its own symbols into a histogram in LDS; what spans blocks -- end-of-band runs -- is
// settled from two lane masks per wavefront (block puts out the pending run; block ends inside a run).
// The symbol stream is the one pcr_encode.h's ScanCoder writes (the JPEG progressive coding procedures): the two are
// compared count by count in the tests.
#pragma once
#include "pcr_common.h"

namespace pcr {

// The scan scripts stock encoders use by default: DC with one bit held back, the low luma band, chroma, the rest of
// luma, then the held-back bits plane by plane.  nc = 3: 10 scans; nc = 1: 6 scans.
struct ScriptScan { uint8_t ns, comp[kMaxComp], Ss, Se, Ah, Al; };
constexpr int kScriptScansMax = 10;
PCR_HD int script_scans(int nc) { return nc == 3 ? 10 : 6; }
PCR_HD ScriptScan script_scan(int nc, int idx) {
    if (nc == 3) {
        switch (idx) {
            case 0: return ScriptScan{3, {0, 1, 2}, 0, 0, 0, 1};
            case 1: return ScriptScan{1, {0, 0, 0}, 1, 5, 0, 2};
            case 2: return ScriptScan{1, {2, 0, 0}, 1, 63, 0, 1};
            case 3: return ScriptScan{1, {1, 0, 0}, 1, 63, 0, 1};
            case 4: return ScriptScan{1, {0, 0, 0}, 6, 63, 0, 2};
            case 5: return ScriptScan{1, {0, 0, 0}, 1, 63, 2, 1};
            case 6: return ScriptScan{3, {0, 1, 2}, 0, 0, 1, 0};
            case 7: return ScriptScan{1, {2, 0, 0}, 1, 63, 1, 0};
            case 8: return ScriptScan{1, {1, 0, 0}, 1, 63, 1, 0};
            default: return ScriptScan{1, {0, 0, 0}, 1, 63, 1, 0};
        }
    }
    switch (idx) {
        case 0: return ScriptScan{1, {0, 0, 0}, 0, 0, 0, 1};
        case 1: return ScriptScan{1, {0, 0, 0}, 1, 5, 0, 2};
        case 2: return ScriptScan{1, {0, 0, 0}, 6, 63, 0, 2};
        case 3: return ScriptScan{1, {0, 0, 0}, 1, 63, 2, 1};
        case 4: return ScriptScan{1, {0, 0, 0}, 0, 0, 1, 0};
        default: return ScriptScan{1, {0, 0, 0}, 1, 63, 1, 0};
    }
}

// counts of one image: [scan of the script][table slot][symbol]; slot 0: the scan's first (or only) table, slot 1: the
// table of the second and third component of an interleaved DC scan
constexpr uint32_t kHistPerScan = 2 * 256, kHistPerImage = kScriptScansMax * kHistPerScan;

#if defined(__HIPCC__)

PCR_D uint32_t bit_length_u32(uint32_t v) { return v ? 32u - (uint32_t)__builtin_clz(v) : 0u; }

// 64 consecutive blocks of an AC scan: which of them put out the pending end-of-band run, which end inside one.
struct ScanMarks { uint64_t flush, inside; };
// Where those of a scan of an image begin: an image takes the same number for each of its scans, one per 64 of all its blocks.
PCR_HD uint64_t scan_marks_of_image(uint64_t coef_off, uint32_t img) { return (coef_off / 4096 + img) * (uint64_t)kScriptScansMax; }
PCR_D uint64_t scan_marks(const uint64_t* coef_off, uint32_t img, uint32_t sidx) {
    return scan_marks_of_image(coef_off[img], img) + ((coef_off[img + 1] - coef_off[img]) / 4096 + 1) * sidx;
}

// The blocks of a DC scan in scan order.  (Scalars picked by compares: an array indexed with the block's component would lie in scratch
// memory.)
struct DcBlock { uint32_t j; int v, diff; };               // component of the scan, value after the point transform, against the block before
struct DcScanOrder {
    uint32_t several, Al, bpm, first1, first2, mcu_w, total, at1, at2, hs0, hs1, hs2, vs0, vs1, vs2, bw0, bw1, bw2;
    PCR_D DcScanOrder(const ImgDesc* D, const ScriptScan& S) {
        several = S.ns > 1 ? 1u : 0u; Al = S.Al;           // (the scans of the scripts hold all the components, in order)
        const uint32_t blocks0 = (uint32_t)D->bw[0] * D->bh[0], blocks1 = (uint32_t)D->bw[1] * D->bh[1];
        hs0 = several ? D->hs[0] : 1u; hs1 = D->hs[1]; hs2 = D->hs[2]; vs0 = several ? D->vs[0] : 1u; vs1 = D->vs[1]; vs2 = D->vs[2];
        bw0 = D->bw[0]; bw1 = D->bw[1]; bw2 = D->bw[2];
        at1 = blocks0; at2 = blocks0 + blocks1;
        // (each product by itself: of a sum of products of bytes the compiler makes a dot product of four bytes, one of which is not theirs)
        first1 = hs0 * vs0; first2 = first1 + uni(several ? hs1 * vs1 : 0u); bpm = first2 + uni(several ? hs2 * vs2 : 0u);
        mcu_w = several ? D->mcux : D->cw[0];
        total = (several ? (uint32_t)D->mcux * D->mcuy : (uint32_t)D->cw[0] * D->ch[0]) * bpm;
    }
    // restart: MCUs per restart interval (0: none)
    PCR_D DcBlock block(const int16_t* base, uint32_t t, uint32_t restart) const {
        const uint32_t m = t / bpm, within = t - m * bpm;
        const uint32_t j = within < first1 ? 0u : (within < first2 ? 1u : 2u);
        auto of = [&](uint32_t a, uint32_t b, uint32_t c) { return j == 0 ? a : (j == 1 ? b : c); };
        const uint32_t hs = of(hs0, hs1, hs2), vs = of(vs0, vs1, vs2), bw = of(bw0, bw1, bw2);
        const uint32_t w = within - of(0, first1, first2), by = w / hs, bx = w - by * hs;
        const uint32_t my = m / mcu_w, mx = m - my * mcu_w;
        const int16_t* pl = base + (size_t)of(0, at1, at2) * 64;
        const int v = (int)pl[((size_t)(my * vs + by) * bw + mx * hs + bx) * 64] >> Al;
        int pred = 0;
        if (w > 0) {                                        // the block before it inside the MCU
            const uint32_t pby = bx ? by : by - 1, pbx = bx ? bx - 1 : hs - 1;
            pred = (int)pl[((size_t)(my * vs + pby) * bw + mx * hs + pbx) * 64] >> Al;
        } else if (m > 0 && !(restart && m % restart == 0)) {   // the component's last block of the MCU before
            const uint32_t pm = m - 1, pmy = pm / mcu_w, pmx = pm - pmy * mcu_w;
            pred = (int)pl[((size_t)(pmy * vs + vs - 1) * bw + pmx * hs + hs - 1) * 64] >> Al;
        }
        return DcBlock{j, v, v - pred};
    }
};
// Where the plane of a component begins among an image's, in blocks.
PCR_D uint32_t blocks_ahead(const ImgDesc* D, uint32_t c) {
    return (c > 0 ? (uint32_t)D->bw[0] * D->bh[0] : 0u) + (c > 1 ? (uint32_t)D->bw[1] * D->bh[1] : 0u);
}

// planes: the coefficient planes with every scan applied (element k of a block = zig-zag position k); coef_off: [n + 1]
// element offsets of the images.  restart: MCUs per restart interval of the file to be written (0: none; a scan of
// one component counts its blocks).  hist: n * kHistPerImage counters, written (not added to).
// grid: (n, kScriptScansMax), a workgroup each.
// marks, raw_bits (both or neither; restart 0): what k_code_scans wants to know besides -- per 64 blocks of an AC scan which of
// them put out the pending end-of-band run and which end inside one (scan_marks), per scan the bits that belong to no symbol.
// What bounds it is latency: a scan's blocks are one after the other only in their end-of-band runs.  So a workgroup counts 512
// blocks at once, each lane reads its block sixteen bytes ahead of the eight coefficients it looks at (consecutive
// coefficients by themselves were a trip to memory each), and the runs cost a lane a few bit operations.
// 64 baseline photographs: 1.61 ms with a wavefront per scan; now 0.145.
constexpr uint32_t kHistWaves = 8, kHistLanes = 64 * kHistWaves;
__global__ void __launch_bounds__(kHistLanes) k_symbol_hist(const ImgDesc* __restrict__ imgs, const int16_t* __restrict__ planes, const uint64_t* __restrict__ coef_off,
                                                            uint32_t restart, uint32_t* __restrict__ hist, ScanMarks* __restrict__ marks, uint32_t* __restrict__ raw_bits) {
    __shared__ uint32_t h[kHistPerScan], s_raw;
    __shared__ uint64_t s_flush[2][kHistWaves], s_inside[2][kHistWaves];
    const uint32_t img = blockIdx.x, sidx = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    for (uint32_t e = tid; e < kHistPerScan; e += kHistLanes) h[e] = 0;
    if (tid == 0) s_raw = 0;
    __syncthreads();
    const ImgDesc* D = imgs + img;
    const uint32_t nc = D->nc;
    uint32_t* out = hist + (size_t)img * kHistPerImage + (size_t)sidx * kHistPerScan;
    const bool live = (nc == 1 || nc == 3) && (int)sidx < script_scans((int)nc);
    const ScriptScan S = script_scan((int)nc, live ? (int)sidx : 0);
    uint32_t raw = 0;
    if (live) {
        const int16_t* base = planes + coef_off[img];
        if (S.Ss == 0) {
            // ---- DC first: one difference per block against the previous block of the same component in scan order ----
            const DcScanOrder O(D, S);
            for (uint32_t t = tid; t < O.total; t += kHistLanes) {
                if (S.Ah > 0) { raw++; continue; }         // (a DC refinement scan is raw bits: no symbols)
                const DcBlock B = O.block(base, t, restart);
                atomicAdd(&h[(B.j == 0 ? 0u : 256u) + bit_length_u32((uint32_t)(B.diff < 0 ? -B.diff : B.diff))], 1u);
            }
        } else {
            // ---- AC scans (one component): the blocks that cover the component's samples, row by row ----
            const uint32_t c = S.comp[0], cw = D->cw[c], total = cw * (uint32_t)D->ch[c], bw = D->bw[c];
            const int16_t* pl = base + (size_t)blocks_ahead(D, c) * 64;
            uint32_t run = 0;                               // end-of-band run carried along the blocks (the same in all wavefronts)
            auto emit_run = [&](uint32_t r) { atomicAdd(&h[(bit_length_u32(r) - 1u) << 4], 1u); };
            for (uint32_t t0 = 0, round = 0; t0 < total; t0 += kHistLanes, round ^= 1) {
                const uint32_t t = t0 + tid;
                bool emits = false;                         // the block emits a symbol of its own
                int last = -1;                              // the last position that did
                if (t < total) {
                    const uint32_t row = t / cw, col = t - row * cw;
                    const uint4* b = reinterpret_cast<const uint4*>(pl + ((size_t)row * bw + col) * 64);
                    uint32_t zeros = 0;                     // zeros since that position (positions known before this scan are none)
                    uint4 next = b[S.Ss >> 3];
                    for (int j = S.Ss >> 3; j <= S.Se >> 3; j++) {
                        const uint4 v = next;
                        next = b[j < S.Se >> 3 ? j + 1 : j];
                        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int e = 0; e < 8; e++) {
                            const int k = 8 * j + e;
                            if (k < S.Ss || k > S.Se) continue;
                            const int x = (int16_t)(w[e >> 1] >> (16 * (e & 1)));
                            const uint32_t mag = (uint32_t)(x < 0 ? -x : x) >> S.Al;
                            if (mag == 0) { zeros++; continue; }
                            if (S.Ah && mag > 1) { raw++; continue; }       // known already: a correction bit, no symbol
                            // (sixteen zeros go out wherever among them the coder stands when it has passed them)
                            if (zeros > 15) atomicAdd(&h[0xF0], zeros >> 4);
                            atomicAdd(&h[((zeros & 15u) << 4) | (S.Ah ? 1u : bit_length_u32(mag))], 1u);
                            zeros = 0; emits = true; last = k;
                        }
                    }
                }
                // What spans the blocks.  In scan order: a restart boundary and a block that emits a symbol both put out the
                // pending run first; a block with anything behind its last symbol makes it one longer, and 32767 is the
                // longest run there is.
                const uint64_t flush = __ballot(emits || (restart && t < total && t > 0 && t % restart == 0));
                const uint64_t inside = __ballot(t < total && last != S.Se);
                if (lane == 0) {
                    s_flush[round][wave] = flush; s_inside[round][wave] = inside;
                    if (marks && t0 + 64 * wave < total) marks[scan_marks(coef_off, img, sidx) + t0 / 64 + wave] = ScanMarks{flush, inside};
                }
                __syncthreads();                            // (the other pair of lists is free: every wavefront has been through the last round's)
                for (uint32_t q = 0; q < kHistWaves; q++) {
                    const uint64_t X = uni(s_flush[round][q]), N = uni(s_inside[round][q]);
                    const uint32_t first = X ? (uint32_t)__builtin_ctzll(X) : 64u;
                    run += (uint32_t)__builtin_popcountll(first < 64 ? N & ((1ull << first) - 1) : N);     // up to the first that puts it out
                    const bool full = run >= 0x7FFFu;
                    if (full) run -= 0x7FFFu;
                    if (q == wave) {
                        if (lane == 0 && full) emit_run(0x7FFFu);
                        const uint64_t before = (1ull << lane) - 1;
                        if ((X >> lane) & 1) {
                            const uint64_t prev = X & before;          // (the first lane of X puts out what was carried in)
                            const uint32_t mine = prev ? (uint32_t)__builtin_popcountll(N & before & (~0ull << (63 - __builtin_clzll(prev)))) : run;
                            if (mine) emit_run(mine);
                        }
                    }
                    if (X) run = (uint32_t)__builtin_popcountll(N & (~0ull << (63 - __builtin_clzll(X))));
                }
            }
            if (run && tid == 0) emit_run(run);
        }
    }
    if (raw_bits && raw) atomicAdd(&s_raw, raw);
    __syncthreads();
    for (uint32_t e = tid; e < kHistPerScan; e += kHistLanes) out[e] = h[e];
    if (raw_bits && tid == 0) raw_bits[(size_t)img * kScriptScansMax + sidx] = s_raw;
}

#endif  // __HIPCC__

}  // namespace pcr
