// The progressive files of a transcode, coded on the device (paper Section 5, "Encoding": every image is re-coded as a
// progressive file before its scans are grouped into a record).  From the coefficient planes a decode left there and the
// symbol counts of k_symbol_hist:
//   k_code_tables   the optimised Huffman tables of every scan, and how many bits the scan takes with them
//   k_code_scans    the entropy-coded bits of every scan, without stuffed bytes
// The host puts the files together (pcr_encode.h): headers, tables, and the bits with the stuffed bytes in.  Symbols, tables and
// bits are those of pcr_encode.h's coder, byte for byte (tests/test_gpu_transcode.py).
#pragma once
#include "pcr_common.h"
#include "pcr_hist.h"

namespace pcr {

// A table as a file holds it.
struct CodeSpec { uint8_t counts[16]; uint32_t nsym; uint8_t symbols[256]; };      // counts[l]: codes of l + 1 bits

#if defined(__HIPCC__)

// The least of a 64-bit key over the wavefront, in all lanes.
PCR_D uint64_t lanes_min(uint64_t v) {
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint64_t o = __shfl_xor(v, (int)d, 64);
        v = o < v ? o : v;
    }
    return uni(v);
}

// Code lengths, symbols and codes of the tables: a wavefront per table, the two of a scan in a workgroup.  The procedure is
// that of Annex K.2 of the JPEG specification: merge the two least counts (ties: the larger symbol first) until one is left,
// with a reserved 257th symbol that takes the all-ones code, then shorten what is longer than 16 bits.  A lane holds five
// symbols; a symbol knows the group it has been merged into and how often that was merged.
// codes: [n][scan][slot][256], code << 8 | bits.  bits: [n][scan].  raw_bits: see k_symbol_hist.
// What bounds it is latency: a merge is two reductions over the wavefront, one after the other, and the 60 to 150 merges of a
// table follow each other.  64 photographs: 53 us.
__global__ void __launch_bounds__(128) k_code_tables(const ImgDesc* __restrict__ imgs, const uint32_t* __restrict__ hist, const uint32_t* __restrict__ raw_bits,
                                                     CodeSpec* __restrict__ specs, uint32_t* __restrict__ codes, uint64_t* __restrict__ bits) {
    __shared__ uint32_t s_len[2][64], s_base[2][18], s_first[2][18];
    __shared__ uint64_t s_bits[2];
    const uint32_t lane = threadIdx.x & 63, slot = uni(threadIdx.x >> 6);
    const size_t scan = (size_t)blockIdx.x * kScriptScansMax + blockIdx.y;
    const uint32_t* h = hist + scan * kHistPerScan + slot * 256;
    CodeSpec* spec = specs + scan * 2 + slot;
    uint32_t* code = codes + (scan * 2 + slot) * 256;
    uint32_t count[4], group[5], depth[5];
    uint64_t freq[5];
    for (uint32_t j = 0; j < 4; j++) { count[j] = h[lane + 64 * j]; freq[j] = count[j]; }
    freq[4] = lane == 0 ? 1 : 0;                               // the reserved symbol, number 256
    uint32_t live = 0;
    for (uint32_t j = 0; j < 5; j++) { group[j] = lane + 64 * j; depth[j] = 0; live += (uint32_t)__builtin_popcountll(__ballot(freq[j] != 0)); }
    const uint32_t nsym = live - 1;
    for (; live > 1; live--) {
        // a group goes by the number of one of its symbols, which holds its count (the others: 0)
        constexpr uint64_t kNone = ~0ull;
        uint64_t key[5], a = kNone, b = kNone;
        for (uint32_t j = 0; j < 5; j++) { key[j] = freq[j] ? freq[j] << 16 | (511u - (lane + 64 * j)) : kNone; a = key[j] < a ? key[j] : a; }
        a = lanes_min(a);
        for (uint32_t j = 0; j < 5; j++) b = key[j] < b && key[j] != a ? key[j] : b;
        b = lanes_min(b);
        const uint32_t ga = 511u - (uint32_t)(a & 0xFFFFu), gb = 511u - (uint32_t)(b & 0xFFFFu);
        for (uint32_t j = 0; j < 5; j++) {
            if (lane + 64 * j == ga) freq[j] += b >> 16;
            if (lane + 64 * j == gb) freq[j] = 0;
            if (group[j] == ga || group[j] == gb) { group[j] = ga; depth[j]++; }
        }
    }
    // ---- how many symbols have each length, and the symbols in order of length and number (the reserved one counts, but is not listed) ----
    uint32_t mine = 0, ranked = 0, rank[4] = {0, 0, 0, 0};
    for (uint32_t l = 1; l < 64 && ranked < nsym; l++) {       // (counts of 32 bits: no length comes near 64)
        uint32_t all = 0;
        for (uint32_t j = 0; j < 4; j++) {
            const bool here = depth[j] == l && count[j] != 0;
            const uint64_t m = __ballot(here);
            if (here) rank[j] = ranked + all + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1));
            all += (uint32_t)__builtin_popcountll(m);
        }
        ranked += all;
        if (lane == l) mine = all;
    }
    if (nsym && lane == uni(depth[4])) mine++;                 // (lane 0 holds the reserved symbol)
    uint32_t* len = s_len[slot];
    uint32_t* base = s_base[slot];
    len[lane] = mine;
    wave_sync();
    if (lane == 0) {
        for (int i = 63; i > 16; i--)
            while (len[i] > 0) {
                int j = i - 2;
                while (len[j] == 0) j--;
                len[i] -= 2; len[i - 1] += 1; len[j + 1] += 2; len[j] -= 1;
            }
        int longest = 16;
        while (longest > 0 && len[longest] == 0) longest--;
        if (longest > 0) len[longest]--;                       // the reserved symbol
        uint32_t first = 0, before = 0;
        for (int l = 1; l <= 16; l++) { s_first[slot][l] = first; base[l] = before; first = (first + len[l]) << 1; before += len[l]; }
        base[17] = before;
    }
    wave_sync();
    if (lane < 16) spec->counts[lane] = (uint8_t)len[lane + 1];
    if (lane == 0) spec->nsym = base[17];
    // ---- the codes, and the bits the scan takes ----
    const ScriptScan S = script_scan((int)imgs[blockIdx.x].nc, (int)blockIdx.y);
    uint64_t total = 0;
    for (uint32_t j = 0; j < 4; j++) {
        const uint32_t s = lane + 64 * j;
        uint32_t c = 0;
        if (count[j] != 0) {
            uint32_t l = 1;
            while (l < 16 && rank[j] >= base[l + 1]) l++;
            c = (s_first[slot][l] + rank[j] - base[l]) << 8 | l;
            spec->symbols[rank[j]] = (uint8_t)s;
            // behind the code: the bits of a DC difference, of a new coefficient (its sign, in a refinement scan), of a run's length
            const uint32_t size = s & 15u, run = s >> 4;
            const uint32_t extra = S.Ss == 0 ? s : (size ? (S.Ah ? 1u : size) : (run < 15 ? run : 0u));
            total += (uint64_t)count[j] * (l + extra);
        }
        code[s] = c;
    }
    for (uint32_t d = 1; d < 64; d <<= 1) total += __shfl_xor(total, (int)d, 64);
    if (lane == 0) s_bits[slot] = total;
    __syncthreads();
    if (threadIdx.x == 0) bits[scan] = s_bits[0] + s_bits[1] + raw_bits[scan];
}

// Blocks of the longest end-of-band run there is.
constexpr uint32_t kLongestRun = 0x7FFF;

// Length of the end-of-band run that begins at block t: the blocks that end inside one, up to the next that puts it out.
PCR_D uint32_t run_from(const ScanMarks* marks, uint32_t words, uint32_t t) {
    uint32_t w = t >> 6;
    const uint64_t from = ~0ull << (t & 63);
    uint64_t flush = marks[w].flush & (from << 1), inside = marks[w].inside & from;     // (block t's own symbols are ahead of the run)
    uint32_t run = 0;
    for (;;) {
        if (flush) { run += (uint32_t)__builtin_popcountll(inside & ((flush & (0 - flush)) - 1)); break; }
        run += (uint32_t)__builtin_popcountll(inside);
        if (++w >= words || run >= kLongestRun) break;
        flush = marks[w].flush; inside = marks[w].inside;
    }
    return run < kLongestRun ? run : kLongestRun;
}

// A block of an AC first scan: put(symbol, bits behind the code, how many).
template <class Put> PCR_D void code_first_block(const uint4* b, const ScriptScan& S, Put put) {
    uint32_t zeros = 0;
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
            const uint32_t mag = (uint32_t)(x < 0 ? -x : x) >> S.Al;           // magnitudes are shifted, not the signed value
            if (mag == 0) { zeros++; continue; }
            for (; zeros > 15; zeros -= 16) put(0xF0u, 0u, 0u);
            const uint32_t nb = bit_length_u32(mag);
            put(zeros << 4 | nb, x < 0 ? mag ^ ((1u << nb) - 1u) : mag, nb);
            zeros = 0;
        }
    }
}

// What a refinement scan has to say of a block, as masks of the positions of its band: known: not zero before this scan; fresh: not
// zero from this scan on; low: the bit this scan adds; minus: negative.
struct RefineBlock { uint64_t known, fresh, low, minus; };
PCR_D RefineBlock refine_block(const uint4* b, const ScriptScan& S) {
    RefineBlock M{0, 0, 0, 0};
    uint4 next = b[S.Ss >> 3];
    for (int j = S.Ss >> 3; j <= S.Se >> 3; j++) {
        const uint4 v = next;
        next = b[j < S.Se >> 3 ? j + 1 : j];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        uint32_t known = 0, fresh = 0, low = 0, minus = 0;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int x = (int16_t)(w[e >> 1] >> (16 * (e & 1)));
            const uint32_t mag = (uint32_t)(x < 0 ? -x : x) >> S.Al;
            known |= (mag > 1 ? 1u : 0u) << e; fresh |= (mag == 1 ? 1u : 0u) << e; low |= (mag & 1u) << e; minus |= (x < 0 ? 1u : 0u) << e;
        }
        M.known |= (uint64_t)known << (8 * j); M.fresh |= (uint64_t)fresh << (8 * j); M.low |= (uint64_t)low << (8 * j); M.minus |= (uint64_t)minus << (8 * j);
    }
    const uint64_t band = (S.Se >= 63 ? ~0ull : (1ull << (S.Se + 1)) - 1) & ~((1ull << S.Ss) - 1);
    M.known &= band; M.fresh &= band;
    return M;
}
// Its symbols, and the correction bits each has behind it: put as above, raw(bits, how many) for correction bits.  Those behind the last
// symbol come back in *rest, *nrest.
template <class Put, class Raw> PCR_D void code_refine_block(const RefineBlock& M, const ScriptScan& S, Put put, Raw raw, uint64_t* rest, uint32_t* nrest) {
    uint64_t corr = 0;
    uint32_t ncorr = 0;
    int prev = S.Ss - 1;
    if (M.fresh) {
        const int last = 63 - __builtin_clzll(M.fresh);
        uint32_t run = 0;
        for (uint64_t m = (M.known | M.fresh) & (last < 63 ? (2ull << last) - 1 : ~0ull); m; m &= m - 1) {
            const int k = __builtin_ctzll(m);
            run += (uint32_t)(k - prev - 1);
            prev = k;
            for (; run > 15; run -= 16) { put(0xF0u, 0u, 0u); raw(corr, ncorr); corr = 0; ncorr = 0; }
            if (M.known >> k & 1) { corr = corr << 1 | (M.low >> k & 1); ncorr++; continue; }
            put(run << 4 | 1u, (uint32_t)(~M.minus >> k & 1), 1u);
            raw(corr, ncorr); corr = 0; ncorr = 0;
            run = 0;
        }
    }
    for (uint64_t m = M.known & (prev < 0 ? ~0ull : ~1ull << prev); m; m &= m - 1) { corr = corr << 1 | (M.low >> __builtin_ctzll(m) & 1); ncorr++; }
    *rest = corr; *nrest = ncorr;
}

// The bits of the scans of images first .. first + gridDim.x - 1: a workgroup per (image, scan), 512 blocks at a time, a lane per
// block.  A block's bits are counted, a prefix sum says where they go, and they are written into words in LDS, which then go out
// in one piece (kCodeWords of them at a time, where the blocks take more: the lanes go through their blocks again for each).  An
// end-of-band run's code is written by the block that begins it -- in the stream its correction bits follow, block by
// block -- which looks its length up in the marks.
// word_off: [images][scan] + 1, where the words of a scan begin in `words` (big-endian, the last one's rest zeros behind the
// padding of its byte).
// What bounds it is the work of a lane on its block, symbol by symbol with most of the others waiting, in the longest scan.  64
// photographs: 0.38 ms, and 6 MB of bits to the host, where 30 MB of coefficients went before and 16 threads took 8 ms to code them.
constexpr uint32_t kCodeWaves = 8, kCodeLanes = 64 * kCodeWaves, kCodeWords = 4096;
__global__ void __launch_bounds__(kCodeLanes) k_code_scans(const ImgDesc* __restrict__ imgs, const int16_t* __restrict__ planes, const uint64_t* __restrict__ coef_off,
                                                           const ScanMarks* __restrict__ all_marks, const uint32_t* __restrict__ codes, const uint64_t* __restrict__ word_off,
                                                           uint32_t first, uint32_t* __restrict__ words) {
    __shared__ uint32_t s_code[2 * 256], s_words[kCodeWords], s_sum[kCodeWaves], s_carry;
    const uint32_t img = first + blockIdx.x, sidx = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const ImgDesc* D = imgs + img;
    const uint32_t nc = D->nc;
    if ((nc != 1 && nc != 3) || (int)sidx >= script_scans((int)nc)) return;
    const ScriptScan S = script_scan((int)nc, (int)sidx);
    const uint32_t* code = codes + ((size_t)img * kScriptScansMax + sidx) * 2 * 256;
    for (uint32_t e = tid; e < 2 * 256; e += kCodeLanes) s_code[e] = code[e];
    if (tid == 0) s_carry = 0;
    __syncthreads();
    const uint64_t* wo = word_off + (size_t)blockIdx.x * kScriptScansMax + sidx;
    const uint64_t out0 = wo[0], room = wo[1] - wo[0];
    const int16_t* base = planes + coef_off[img];
    const bool dc = S.Ss == 0;
    const DcScanOrder O(D, S);
    const uint32_t c = S.comp[0], cw = D->cw[c], total = dc ? O.total : cw * (uint32_t)D->ch[c], bw = D->bw[c];
    const int16_t* pl = base + (size_t)blocks_ahead(D, c) * 64;
    const ScanMarks* marks = all_marks + scan_marks(coef_off, img, sidx);
    const uint32_t nmarks = (total + 63) / 64;
    uint64_t done = 0;                                         // words written
    uint32_t have = 0;                                         // bits of the next one (in s_carry)
    uint32_t run = 0;                                          // end-of-band run carried along the blocks, below kLongestRun
    for (uint32_t t0 = 0; t0 < total; t0 += kCodeLanes) {
        const uint32_t t = t0 + tid;
        const bool on = t < total;
        const uint4* b = nullptr;
        uint32_t mine = 0;                                     // bits of the block
        uint32_t run_code = 0, run_bits = 0;                   // the code of the run that begins here, its length's bits behind it
        DcBlock B{0, 0, 0};
        RefineBlock M{0, 0, 0, 0};
        uint64_t rest = 0;
        uint32_t nrest = 0;
        auto count = [&](uint32_t sym, uint32_t, uint32_t n) { mine += (s_code[sym] & 255u) + n; };
        if (dc) {
            if (on) {
                B = O.block(base, t, 0);
                if (S.Ah) mine = 1;
                else { const uint32_t nb = bit_length_u32((uint32_t)(B.diff < 0 ? -B.diff : B.diff)); mine = (s_code[(B.j ? 256u : 0u) + nb] & 255u) + nb; }
            }
        } else {
            // what spans blocks: in this lane's 64, and in those of the wavefronts before
            bool begins = false;
            for (uint32_t q = 0; q < kCodeWaves; q++) {
                const uint32_t w = t0 / 64 + q;
                if (w >= nmarks) break;
                const uint64_t X = marks[w].flush, N = marks[w].inside;
                const uint32_t ahead = (uint32_t)__builtin_popcountll(X ? N & ((X & (0 - X)) - 1) : N);      // of those carried in: up to the first that puts the run out
                if (q == wave) {
                    const uint64_t put_out = X & ((2ull << lane) - 1), before = N & ((1ull << lane) - 1);
                    uint32_t r = put_out ? (uint32_t)__builtin_popcountll(before & (~0ull << (63 - __builtin_clzll(put_out)))) : run + (uint32_t)__builtin_popcountll(before);
                    if (r >= kLongestRun) r -= kLongestRun;
                    begins = (N >> lane & 1) && r == 0;
                }
                run += ahead;
                if (run >= kLongestRun) run -= kLongestRun;
                if (X) run = (uint32_t)__builtin_popcountll(N & (~0ull << (63 - __builtin_clzll(X))));
            }
            if (on) {
                const uint32_t row = t / cw, col = t - row * cw;
                b = reinterpret_cast<const uint4*>(pl + ((size_t)row * bw + col) * 64);
                if (begins) {
                    const uint32_t length = run_from(marks, nmarks, t), nb = bit_length_u32(length) - 1u, e = s_code[nb << 4];
                    run_code = (e >> 8) << nb | (length - (1u << nb)); run_bits = (e & 255u) + nb;
                    mine = run_bits;
                }
                if (S.Ah) {
                    M = refine_block(b, S);
                    code_refine_block(M, S, count, [&](uint64_t, uint32_t n) { mine += n; }, &rest, &nrest);
                    mine += nrest;
                } else code_first_block(b, S, count);
            }
        }
        const uint32_t incl = lanes_prefix_sum(mine);
        if (lane == 63) s_sum[wave] = incl;
        __syncthreads();
        uint32_t start = have + incl - mine, all = have;
        for (uint32_t q = 0; q < kCodeWaves; q++) { const uint32_t s = s_sum[q]; start += q < wave ? s : 0u; all += s; }
        __syncthreads();                                       // (blocks inside a run may have no bits at all, and the loop below no turn)
        const uint32_t nwords = (all + 31) / 32;
        for (uint32_t w0 = 0; w0 < nwords; w0 += kCodeWords) {
            const uint32_t here = nwords - w0 < kCodeWords ? nwords - w0 : kCodeWords;
            for (uint32_t e = tid; e < here; e += kCodeLanes) s_words[e] = e + w0 == 0 ? s_carry : 0u;
            __syncthreads();
            uint32_t pos = start;
            auto bits = [&](uint32_t v, uint32_t n) {          // 1 to 32 of them
                const uint32_t at = (pos >> 5) - w0, sh = pos & 31u;
                const uint64_t x = (uint64_t)v << (64u - sh - n);
                if (at < here) atomicOr(&s_words[at], (uint32_t)(x >> 32));
                if (sh + n > 32u && at + 1u < here) atomicOr(&s_words[at + 1u], (uint32_t)x);
                pos += n;
            };
            auto put = [&](uint32_t sym, uint32_t v, uint32_t n) { const uint32_t e = s_code[sym]; bits((e >> 8) << n | v, (e & 255u) + n); };
            auto raw = [&](uint64_t v, uint32_t n) {
                if (n > 32) { bits((uint32_t)(v >> (n - 32u)), 32u); n -= 32u; v &= 0xFFFFFFFFull; }
                if (n) bits((uint32_t)v & (n < 32 ? (1u << n) - 1u : ~0u), n);
            };
            if (on) {
                if (dc) {
                    if (S.Ah) bits((uint32_t)B.v & 1u, 1u);
                    else {
                        const uint32_t nb = bit_length_u32((uint32_t)(B.diff < 0 ? -B.diff : B.diff));
                        put((B.j ? 256u : 0u) + nb, (uint32_t)(B.diff < 0 ? B.diff - 1 : B.diff) & ((1u << nb) - 1u), nb);
                    }
                } else if (S.Ah) {
                    uint64_t v; uint32_t n;
                    code_refine_block(M, S, put, raw, &v, &n);
                    if (run_bits) bits(run_code, run_bits);
                    raw(rest, nrest);
                } else {
                    code_first_block(b, S, put);
                    if (run_bits) bits(run_code, run_bits);
                }
            }
            __syncthreads();
            const bool last = w0 + here == nwords && (all & 31u) != 0;       // (its last word waits for the next blocks' bits)
            for (uint32_t e = tid; e < here - (last ? 1u : 0u); e += kCodeLanes)
                if (done + w0 + e < room) words[out0 + done + w0 + e] = __builtin_bswap32(s_words[e]);
            if (tid == 0) s_carry = last ? s_words[here - 1] : 0u;
            __syncthreads();
        }
        done += all / 32; have = all & 31u;
    }
    if (tid == 0 && have && done < room) {
        const uint32_t pad = (8u - have) & 7u;                 // 1-bits to the end of the byte
        words[out0 + done] = __builtin_bswap32(s_carry | ((1u << pad) - 1u) << (32u - have - pad));
    }
}

#endif  // __HIPCC__

}  // namespace pcr
