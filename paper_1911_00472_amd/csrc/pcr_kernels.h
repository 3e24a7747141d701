// gfx950 kernels of the PCR decode path.  One kernel per step:
//   k_index      scan-group index (prefix sums of region lengths)
//   k_headers    JPEG marker parsing and Huffman tables, one workgroup per image
//   k_unstuff    byte un-stuffing + restart-interval location, one or four wavefronts per (image, scan); zero fills
//   k_decode_waves   progressive Huffman decode, one wavefront per unit: a restart
//                interval of a scan, or the stretch between two entry points of the record (the whole scan
//                where there is neither)
//   k_refine_blocks   second phase of AC refinement, one lane per block
//   k_dc_first_lanes, k_ac_first_lanes, k_ac_refine_lanes   the same scans with one LANE per unit (pcr_lanes.h), for
//                launches with very many units; k_refine_history, k_refine_deal: per-block work before and after
//   k_apply      data-parallel refinement (DC bits, AC corrections and new coefficients)
//   k_pixel      de-quantise + IDCT + chroma replication + YCbCr->RGB + store
//   k_gather     materialise an image's scan prefix (parity hook)
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "pcr_common.h"
#include "pcr_format.h"
#include "pcr_chains.h"
#include "pcr_entropy.h"
#include "pcr_refine_trio.h"
#include "pcr_lanes.h"
#include "pcr_pixel.h"

namespace pcr {

// Everything a kernel needs to find its data; passed by value.
// Wave priority.  A decode call on one record usually shares the GPU with calls on other records (other
// streams).  The AC entropy kernels then keep every SIMD busy with long-running wavefronts that issue
// scalar instructions back to back, and instruction arbitration serves the oldest wavefronts first: a short
// data-parallel kernel of another record (unstuff, fill, phase 2 of refinement, pixels) was measured to run
// 3-8 times longer than alone, holding up its record's dependency chain.  These kernels therefore raise
// their own wavefronts' issue priority (s_setprio; stream priorities are not touched); the DC first kernel,
// few and latency-bound wavefronts, takes a middle value.  The AC entropy kernels stay at the default.
PCR_D void short_kernel_priority() { __builtin_amdgcn_s_setprio(3); }

// Workgroups are handed to the chip's eight dies (XCDs, each with its own L2) round-robin by their index.  Kernels whose
// neighbouring work items write neighbouring memory (the runs of MCUs of one image row, the rows of cells of one image)
// take item xcd_major(blockIdx.x, gridDim.x) instead of item blockIdx.x: every die then works through one contiguous
// eighth of the list, so the cache lines two neighbours share are completed in one L2 instead of being written back
// in parts from two.
constexpr uint32_t kXcds = kDies;
PCR_D uint32_t xcd_major(uint32_t b, uint32_t n) {
    const uint32_t q = n / kXcds, r = n - q * kXcds, x = b % kXcds, i = b / kXcds;
    return x * q + (x < r ? x : r) + i;
}
// A store of T (made of 32-bit words) that asks the caches to make no room for it.  Which stores do is the host's to say (pixels_past, rows_past and fill_past in pcr_lib.hip).
template <class T, int WORDS = sizeof(T) / 4> PCR_D void put_past(void* p, const uint32_t* w) {
    typedef uint32_t V __attribute__((ext_vector_type(WORDS), aligned(alignof(T))));
    V v;
#pragma unroll
    for (int e = 0; e < WORDS; e++) v[e] = w[e];
    __builtin_nontemporal_store(v, reinterpret_cast<V*>(p));
}
// the value of the lane before this one (lane 0: `first`), and the sum over the lanes up to this one
PCR_D uint32_t lane_before(uint32_t v, uint32_t first) { return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138, 0xF, 0xF, false); }   // wave_shr:1
PCR_D uint32_t lanes_prefix_sum(uint32_t v) {
    uint32_t x = v;
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);           // row_shr:1, 2, 4, 8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);           // row_bcast:15 into rows 1 and 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);           // row_bcast:31 into rows 2 and 3
    return x;
}
PCR_D void dc_kernel_priority() { __builtin_amdgcn_s_setprio(2); }

struct DevRecord {
    const uint8_t* rec;        // record bytes
    uint8_t* clean;            // unstuffed entropy data, same offsets as rec
    uint64_t nbytes;           // of rec
    uint32_t n, G;
    uint32_t* off;             // [G][n] absolute region offsets (k_index)
    const uint32_t* len;       // [G][n] region lengths (inside rec's header)
    const uint32_t* nscans;    // [n] (inside rec's header)
    ImgDesc* img;              // [n]
    ScanDesc* scan;            // [n][G]
    const uint64_t* coef_off;  // [n+1] int16 units
    const uint64_t* out_off;   // [n+1] bytes
    const uint64_t* mask_off;  // [n][G] u64 units into masks (AC scans)
    const uint32_t* slot_base; // [n][G] first entry of the scan in ivl_start
    const uint32_t* slot_cnt;  // [n][G] intervals of the scan
    uint32_t* ivl_start;       // per scan: intervals+1 offsets into the clean segment
    int16_t* coef;
    int16_t* dc;               // the DC coefficients, one per block in the order of the blocks of `coef` (written by the DC first scans and
                               // by sequential scans): what the pixel kernels read; element 0 of a block in `coef` holds it only for the
                               // coefficient export
    uint64_t* masks;
    int32_t* status;           // [n]
    int32_t* status_out;       // [n], the caller's (null: not wanted): filled by the pixel kernel of the call (hand_out_status)
    AcTab* tabs;               // Huffman tables of the AC scans, written by k_headers
    const uint32_t* tab_idx;   // [n][G] index into tabs
    DcTab* dctabs;             // the DC tables of the DC first scans, three slots per scan (one per scan component)
    const uint32_t* dctab_idx; // [n][G] first slot of the scan in dctabs
    const uint32_t* ent_off;   // [n][G] record offset of the scan's entry points (0: none; then slot_cnt - 1 of them)
};

// segment of a scan in the clean buffer: 4-byte aligned base (big-endian words)
PCR_HD uint32_t clean_base(uint32_t data_off) { return (data_off + 3u) & ~3u; }

// --------------------------------------------------------------------------------------
// k_index: off[g][i] = start of group g + sum of len[g][j], j < i.  One workgroup per group.
// --------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_index(DevRecord R, uint32_t kmax) {
    __shared__ uint32_t part[256];
    __shared__ uint32_t carry;
    short_kernel_priority();
    uint32_t g = blockIdx.x;
    if (g >= kmax) return;
    uint64_t hb = ld_le64(R.rec + 16);
    uint64_t start = g == 0 ? hb : ld_le64(R.rec + hdr_group_end_pos(g - 1));
    if (threadIdx.x == 0) carry = (uint32_t)start;
    __syncthreads();
    for (uint32_t base = 0; base < R.n; base += 256) {
        uint32_t i = base + threadIdx.x;
        uint32_t v = i < R.n ? R.len[(size_t)g * R.n + i] : 0;
        part[threadIdx.x] = v;
        __syncthreads();
        for (uint32_t d = 1; d < 256; d <<= 1) {           // inclusive Hillis-Steele scan
            uint32_t t = threadIdx.x >= d ? part[threadIdx.x - d] : 0;
            __syncthreads();
            part[threadIdx.x] += t;
            __syncthreads();
        }
        if (i < R.n) R.off[(size_t)g * R.n + i] = carry + part[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == 255) carry += part[255];
        __syncthreads();
    }
}

// --------------------------------------------------------------------------------------
// k_headers: the marker segments of one image per workgroup, and the Huffman tables of its scans.
//   1. where the regions of scan groups 0 .. kmax-1 lie: the offsets k_index left, or (own_index, most records, one
//      launch fewer) the sum of the lengths ahead of the image's, taken here;
//   2. the first bytes of every region into LDS, all of them at once -- a walk over marker segments is a chain of
//      reads that depend on one another, and from memory each of them is a trip of a microsecond;
//   3. one WAVEFRONT PER REGION walks its segments (walk_region), then reads its scan header (resolve_scan) with the tables
//      and the restart interval in force, which ballots over the regions find;
//   4. one wavefront puts together which scans refine which (the scans' headers handed round its lanes) and checks the image;
//   5. one wavefront per TABLE builds it from its definition, every lane its share of the entries.
// What bounds it is code that runs once: a workgroup passes through all of it, from a cold instruction cache, and each
// branch that lanes take differently costs its mask arithmetic.  So the walk is scalar code with one place that reads (24
// bytes at a time); with a lane per region, byte reads and the parse's state in vector registers the walk was 28 000 cycles
// of the 94 000 a workgroup of ten scans took, the search for the scans refined 22 000 and the tables, dealt out by scan, 28 000;
// now 18 000, 6 000 and 12 000.  us for 64 gray pictures of 6 scans 22.8 -> 16.2, small ragged ones of 10 scans 43.0 -> 26.6,
// 1024 of 256 x 256 at scan group 5 38.5 -> 27.2 (with k_index ahead of it, 8 more), 512 photographs of 10 scans 48.9 -> 30.8.
// Workgroups have a wavefront per scan group, kHeaderWaves at most: with eight of them at every scan group, of which seven
// had nothing to do at scan group 1, the kernel stood in the way of the pixel writers of other records (four records
// in flight, ms per step at scan groups 1 and 2: 0.745 and 2.18, now 0.675 and 2.08; alone nothing changes).  Records
// small enough for own_index leave the chip empty anyway and keep the eight, which sum the lengths.
// keep_status: a fidelity upgrade builds on planes decoded earlier; an image those calls found damaged stays so.
// tables from scan k0 on are built (none: k0 = kmax); dc_too = 0: the DC first scans of this call are all decoded by
// k_dc_first_lanes, which builds its own tables.
// --------------------------------------------------------------------------------------
constexpr int kHeaderWaves = 8, kHeaderLanes = 64 * kHeaderWaves;
constexpr uint32_t kMaxGroups = 64;                        // (parse_record_header refuses more)
constexpr uint32_t kHeaderStage = 16384;                   // bytes of LDS for the heads of the regions, shared out evenly
constexpr uint32_t kHeaderWindow = 1024;                   // ... but at most this much per region (a first region with its tables is 600-700 bytes)
constexpr uint32_t kHeaderWideImages = 512;                // kHeaderWaves wavefronts per workgroup whatever the scan group up to this many images
// Beyond this many images the workgroups are more than find room at once with eight wavefronts each: four at most.  us a call, eight / four:
// 2048 pictures of 24 x 34 at scan group 9 262 / 245, of 15 to 40 pixels at 7 215 / 195, two records of 2048 of 70 x 54 at 5 314 / 295,
// four of 2048 of 30 x 30 at 9 715 / 646; but 800 of 64 x 64 at 10 249 / 255, 1000 of 48 x 48 at 10 246 / 253.
constexpr uint32_t kHeaderNarrowImages = 1024;
// own_index up to this many images (a workgroup sums n lengths per scan group), but beyond half of it only up to scan group
// kHeaderWaves.  us a call with k_index / without: 1024 pictures of 256 x 256 at scan group 5 271 / 263, four records of
// 1024 photographs at 1 708 / 695, at 10 6022 / 6042, of 64 x 64 at 10 721 / 717; 2048 pictures of 256 x 256 at 1 209 / 197, at 5 502 / 492,
// at 10 1158 / 1151.
constexpr uint32_t kOwnIndexImages = 2048;

// Record bytes by record offset: from the staged window, or (past it: long comments and profiles) from memory.
// (The address spaces are spelled out: through two generic pointers every read became a flat one.)
typedef const __attribute__((address_space(3))) uint8_t* LdsBytes;
typedef const __attribute__((address_space(1))) uint8_t* GlobalBytes;
struct HeaderBytes {
    GlobalBytes rec; LdsBytes lds; uint32_t base, count, room;   // room: bytes of the window, of which `count` are staged
    PCR_D uint8_t operator[](uint32_t p) const { const uint32_t o = p - base; return o < count ? lds[o] : rec[p]; }
};
// Twenty-four bytes, little endian; what lies at the region's end or behind it says nothing.
struct DeviceHead {
    uint64_t v[3];
    PCR_D uint32_t byte(uint32_t i) const { return byte_of(v[i >> 3], i & 7); }     // (i: a constant, after inlining)
    PCR_D void skip_marker() { v[0] = (v[0] >> 32) | (v[1] << 32); v[1] = (v[1] >> 32) | (v[2] << 32); v[2] >>= 32; }
    PCR_D static uint32_t sum_bytes(uint64_t x) { return __builtin_amdgcn_sad_u8((uint32_t)x, 0u, __builtin_amdgcn_sad_u8((uint32_t)(x >> 32), 0u, 0u)); }
    PCR_D uint32_t counts() const { return sum_bytes(v[0] >> 8) + sum_bytes(v[1]) + byte_of(v[2], 0); }
    PCR_D void first16(uint64_t h[2]) const { h[0] = v[0]; h[1] = v[1]; }
};
// (Called with a wavefront, all lanes the same.  end: of the region the window is the head of.  The window starts on 16 bytes, and four bytes behind it may be read.)
PCR_D DeviceHead head_at(const HeaderBytes& b, uint32_t p, uint32_t end) {
    const uint32_t o = p - b.base;
    uint32_t w[6] = {0, 0, 0, 0, 0, 0};
    if (o + 24 <= b.room) {
        typedef const __attribute__((address_space(3))) uint32_t* LdsWords;
        const LdsWords at = (LdsWords)(b.lds + (o & ~3u));
#pragma unroll
        for (int t = 0; t < 6; t++) w[t] = __builtin_amdgcn_alignbyte(at[t + 1], at[t], o & 3);
    } else {
#pragma unroll 1
        for (uint32_t t = 0; t < 24; t++) {
            const uint32_t x = t < end - p ? b.rec[p + t] : 0u;
#pragma unroll
            for (int q = 0; q < 5; q++) w[q] = __builtin_amdgcn_alignbyte(w[q + 1], w[q], 1);
            w[5] = (w[5] >> 8) | (x << 24);
        }
    }
    DeviceHead h;
#pragma unroll
    for (int t = 0; t < 3; t++) h.v[t] = ((uint64_t)uni(w[2 * t + 1]) << 32) | uni(w[2 * t]);
    return h;
}

// From a DHT payload (16 counts, then the symbols in code order); call with a whole wavefront.
PCR_D void canon_build(CanonCode* c, const HeaderBytes& def, uint32_t at, uint32_t lane) {
    const uint32_t mine = lane < 16 ? def[at + lane] : 0u;
    const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)lanes_prefix_sum(mine), 15);       // symbols in all
    for (uint32_t i = lane; i < 256; i += 64) c->vals[i] = i < k ? def[at + 16 + i] : (uint8_t)0;
    // the codes of a length end, left-aligned, where those of all lengths up to it together do
    const uint32_t ends = lanes_prefix_sum(lane < 16 ? mine << (15 - lane) : 0u), lim = ends > 65536u ? 65536u : ends;
    const uint32_t first = lanes_prefix_sum(mine) - mine;
    if (lane < 16) { c->lim[lane + 1] = lim; c->first[lane + 1] = first; }
    if (lane == 16) c->lim[0] = 0;
}
// What actab_build and actab_pack make of the definition, entry by entry (same contents).
PCR_D void actab_build_wave(AcTab* t, const CanonCode* c, bool first, uint32_t lane) {
    const uint32_t lim8 = c->lim[8], D = 65536u - lim8;
    uint32_t sh2 = 0;
    while (D && ((D - 1) >> sh2) >= 128) sh2++;
    for (uint32_t e = lane; e < 256; e += 64) {
        const uint32_t f = canon_find<1, 8>(c, e << 8);
        const uint32_t v = f ? (f & 0xFF00u) | c->vals[f & 255u] : 0u;
        t->lut[e] = (uint16_t)(f ? code_entry(f >> 8, v & 255u) : 0u);
        t->lutp[e] = packed_entry(v, first);
        t->huffval[e] = c->vals[e];
    }
    for (uint32_t e = lane; e < 128; e += 64) {
        const uint32_t c16 = lim8 + (e << sh2);
        const uint32_t f = c16 < 65536u ? canon_find<9, 16>(c, c16) : 0u;
        const uint32_t v = (f && 16u - (f >> 8) >= sh2) ? (f & 0xFF00u) | c->vals[f & 255u] : 0u;
        t->lut2[e] = (uint16_t)(v ? code_entry(v >> 8, v & 255u) : 0u);
        t->lutp[256 + e] = packed_entry(v, first);
    }
    if (lane < 9) t->limit[lane] = c->lim[8 + lane];
    if (lane < 8) t->valptr[lane] = (uint16_t)c->first[9 + lane];
    if (lane == 0) t->sh2 = sh2;
}
// ... and dctab_build (only the first sixteen codes are DC categories).
PCR_D void dctab_build_wave(DcTab* t, const CanonCode* c, uint32_t lane) {
    for (uint32_t e = lane; e < 256; e += 64) {
        const uint32_t f = canon_find<1, 8>(c, e << 8);
        t->lut[e] = (f && (f & 255u) < 16u) ? (uint8_t)(((f >> 8) << 4) | (c->vals[f & 255u] & 15)) : (uint8_t)0xFF;
    }
    if (lane < 16) t->huffval[lane] = c->vals[lane];
    if (lane < 9) t->limit[lane] = c->lim[8 + lane];
    if (lane < 8) t->valptr[lane] = (uint16_t)c->first[9 + lane];
}

// LDS of a workgroup: the heads of the regions of kmax scan groups, a code per wavefront, what the walks found.  (With room for the most
// of everything, 30 KB, five workgroups fitted a compute unit whatever there was to do.  us a launch for 2048 pictures at scan groups 1 / 3 / 4, then and now: 37.6 / 43.4 / 45.0,
// 25.0 / 34.8 / 35.5.)
PCR_HD uint32_t header_stage(uint32_t kmax) { return kmax * kHeaderWindow < kHeaderStage ? kmax * kHeaderWindow : kHeaderStage; }
PCR_HD uint32_t header_lds(uint32_t kmax, uint32_t waves) {
    static_assert(sizeof(CanonCode) % 4 == 0 && sizeof(RegionWalk) % alignof(ScanDesc) == 0 && sizeof(ScanDesc) % 4 == 0 && alignof(RegionWalk) <= 8 && sizeof(CanonCode) % 8 == 0, "they follow each other");
    return header_stage(kmax) + 16 + waves * (uint32_t)sizeof(CanonCode) + kmax * (uint32_t)(sizeof(RegionWalk) + sizeof(ScanDesc));
}
__global__ void __launch_bounds__(kHeaderLanes, 8) k_headers(DevRecord R, uint32_t kmax, uint32_t keep_status, uint32_t own_index, uint32_t k0, uint32_t dc_too) {
    extern __shared__ __attribute__((aligned(16))) uint8_t stage[];          // (header_lds: as much as the scans of the call take)
    CanonCode* const s_code = reinterpret_cast<CanonCode*>(stage + header_stage(kmax) + 16);
    RegionWalk* const s_walk = reinterpret_cast<RegionWalk*>(s_code + (blockDim.x >> 6));
    ScanDesc* const s_scan = reinterpret_cast<ScanDesc*>(s_walk + kmax);
    __shared__ uint32_t s_off[kMaxGroups], s_len[kMaxGroups];
    __shared__ int s_rc[kMaxGroups];
    __shared__ ImgDesc s_img;
    __shared__ uint16_t s_job[kMaxGroups * kMaxComp];        // tables to build: scan group | component of the scan << 8
    __shared__ uint32_t s_njobs;
    short_kernel_priority();
    const uint32_t i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lanes = blockDim.x, waves = lanes >> 6;
    const uint32_t n = R.n, nsc = R.nscans[i];
    uint32_t upto = nsc < kmax ? nsc : kmax;
    if (upto > kMaxGroups) upto = kMaxGroups;               // (cannot happen: the header check refuses such records)
    // ---- where the regions lie ----
    if (own_index) {
        for (uint32_t g = wave; g < upto; g += waves) {      // (512 of a group's loads at once, eight lengths per lane)
            const uint32_t* len = R.len + (size_t)g * n;
            const uint64_t start = ld_le64(R.rec + (g == 0 ? 16 : hdr_group_end_pos(g - 1)));
            const uint32_t mine = len[i];
            constexpr uint32_t kHalf = 8;
            uint32_t before = 0;
            for (uint32_t first = 0; first < i; first += 64 * kHalf) {
                uint32_t t[kHalf];
#pragma unroll
                for (uint32_t j = 0; j < kHalf; j++) { const uint32_t at = first + 64 * j + lane; t[j] = len[at < i ? at : i]; }
#pragma unroll
                for (uint32_t j = 0; j < kHalf; j++) before += first + 64 * j + lane < i ? t[j] : 0u;
            }
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) before += (uint32_t)__shfl_xor((int)before, d);
            if (lane == 0) { s_off[g] = (uint32_t)start + before; s_len[g] = mine; }
        }
    } else if (tid < upto) { s_off[tid] = R.off[(size_t)tid * n + i]; s_len[tid] = R.len[(size_t)tid * n + i]; }
    for (uint32_t e = tid; e < sizeof(ScanDesc) / 4 * upto; e += lanes) reinterpret_cast<uint32_t*>(s_scan)[e] = 0;
    for (uint32_t e = tid; e < sizeof(ImgDesc) / 4; e += lanes) reinterpret_cast<uint32_t*>(&s_img)[e] = 0;
    __syncthreads();
    // ---- their first bytes ----
    uint32_t window = upto ? (kHeaderStage / upto) & ~15u : 0u;
    if (window > kHeaderWindow) window = kHeaderWindow;
    const uint32_t pieces = window >> 4;                     // 16-byte pieces per region
    for (uint32_t e = tid; e < pieces * upto; e += lanes) {
        const uint32_t g = e / pieces, o = (e - g * pieces) * 16, L = s_len[g];
        if (o >= L) continue;
        const uint8_t* src = R.rec + s_off[g] + o;
        uint8_t* dst = stage + g * window + o;
        if (o + 16 <= L) {
            struct __attribute__((packed, aligned(1))) Sixteen { uint32_t a, b, c, d; };
            const Sixteen t = *reinterpret_cast<const Sixteen*>(src);
            *reinterpret_cast<uint4*>(dst) = uint4{t.a, t.b, t.c, t.d};
        } else for (uint32_t b = 0; b < L - o; b++) dst[b] = src[b];
    }
    __syncthreads();
    auto bytes_of = [&](uint32_t g) {
        const uint32_t len = uni(s_len[g]);
        return HeaderBytes{(GlobalBytes)R.rec, (LdsBytes)(stage + g * window), uni(s_off[g]), len < window ? len : window, window};
    };
    // ---- the walk, a wavefront per region ----
    for (uint32_t g = wave; g < upto; g += waves) {
        const uint32_t at = uni(s_off[g]), end = at + uni(s_len[g]);
        const int rc = walk_region(bytes_of(g), at, end, g, &s_walk[g], &s_img);
        if (lane == 0) s_rc[g] = rc;
    }
    __syncthreads();
    for (uint32_t g = wave; g < upto; g += waves) {
        // what is in force at the scan: the last definition in this region or an earlier one
        const RegionWalk& w = s_walk[lane < upto ? lane : 0];
        uint32_t dht[8], ri;
#pragma unroll
        for (int t = 0; t < 8; t++) {
            const uint32_t def = w.dht[t];
            const uint64_t m = __ballot(lane <= g && def != 0);
            dht[t] = m ? (uint32_t)__builtin_amdgcn_readlane((int)def, 63 - __builtin_clzll(m)) : 0u;
        }
        {
            const int def = w.ri;
            const uint64_t m = __ballot(lane <= g && def >= 0);
            ri = m ? (uint32_t)__builtin_amdgcn_readlane(def, 63 - __builtin_clzll(m)) : 0u;
        }
        const int walked = uni(s_rc[g]);
        if (walked == kOk) {
            const int rc = resolve_scan(s_walk[g], uni(s_off[g]) + uni(s_len[g]), dht, ri, &s_img, &s_scan[g]);
            if (lane == 0) s_rc[g] = rc;
        }
    }
    if (wave == waves - 1) {                                 // quantisation tables: the last definition of all
        const RegionWalk& w = s_walk[lane < upto ? lane : 0];
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const uint32_t off = w.qoff[t], prec = w.qprec[t];
            const uint64_t m = __ballot(lane < upto && off != 0);
            const int last = m ? 63 - __builtin_clzll(m) : 0;
            const uint32_t qo = (uint32_t)__builtin_amdgcn_readlane((int)off, last), qp = (uint32_t)__builtin_amdgcn_readlane((int)prec, last);
            if (lane == 0) { s_img.qoff[t] = m ? qo : 0u; s_img.qprec[t] = (uint8_t)(m ? qp : 0u); }
        }
    }
    __syncthreads();
    if (wave == 0) {
        int rc = lane < upto ? s_rc[lane] : kOk;
        // scan_history, the reach of the components and check_image, every scan's header handed round the lanes
        ScanDesc* sd = &s_scan[lane < upto ? lane : 0];
        const uint32_t ns = sd->ns, Ss = sd->Ss, Se = sd->Se, comp = sd->comp[0];
        uint32_t key = Ss | (Se << 6) | (sd->Ah ? 1u << 12 : 0u) | (comp << 13);
#pragma unroll
        for (uint32_t j = 0; j < (uint32_t)kMaxComp; j++) if (j < ns) key += 1u << (15 + 2 * sd->comp[j]);     // how often the scan names each component
        uint64_t hist = 0;
        uint32_t nhist = 0, has_first = 0, over = 0;
        const bool refines = Ss > 0 && sd->Ah > 0;
        for (uint32_t q = 0; q + 1 < upto; q++) {
            const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)key, (int)q);
            if ((k & 63) == 0) continue;
            const bool of = refines && q < lane && ((k >> 13) & 3) == comp && (k & 63) <= Se && Ss <= ((k >> 6) & 63);
            if ((k & (1u << 12)) == 0) has_first |= of ? 1u : 0u;
            else if (of) {
                if (nhist >= (uint32_t)kMaxHist) over = 1;
                else { hist |= (uint64_t)q << (8 * nhist); nhist++; }
            }
        }
        if (lane < upto && rc == kOk) {
            sd->nhist = (uint8_t)nhist;
#pragma unroll
            for (int t = 0; t < kMaxHist; t++) if ((uint32_t)t < nhist) sd->hist[t] = (uint8_t)(hist >> (8 * t));
            rc = over ? kEUnsupported : (refines && !has_first ? kEFormat : kOk);
            if (rc == kOk) sd->valid = 1;
        }
        const uint64_t bad = __ballot(lane < upto && rc != kOk);
        const uint32_t good = bad ? (uint32_t)__builtin_ctzll(bad) : upto;            // scans ahead of the first damaged region
        const int first_rc = __shfl(rc, bad ? (int)good : 0);
        uint32_t reach[kMaxComp] = {0, 0, 0}, nref[kMaxComp] = {0, 0, 0};             // per component: how far its scans reach, how many refine it
        for (uint32_t q = 0; q < good; q++) {
            const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)key, (int)q), z = ((k >> 6) & 63) + 1;
#pragma unroll
            for (int c = 0; c < kMaxComp; c++) {
                const uint32_t named = (k >> (15 + 2 * c)) & 3;
                if (named && z > reach[c]) reach[c] = z;
                if (k & (1u << 12)) nref[c] += named;
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < kMaxComp; c++) s_img.zmax[c] = (uint8_t)reach[c];
            s_img.nscans = good;
        }
        {
            const uint32_t jobs = lane < k0 || lane >= upto ? 0u : Ss > 0 ? 1u : (dc_too && sd->Ah == 0 && s_img.progressive) ? ns : 0u;
            const uint32_t end = lanes_prefix_sum(jobs);
            for (uint32_t j = 0; j < jobs; j++) s_job[end - jobs + j] = (uint16_t)(lane | (j << 8));
            if (lane == 63) s_njobs = end;
        }
        if (lane >= good && lane < upto) s_scan[lane].valid = 0;
        int st = bad ? first_rc : kOk;
        if (!bad) {                                          // (as check_image)
            if (good == 0) st = kEFormat;
            else {
#pragma unroll
                for (int c = 0; c < kMaxComp; c++) if (st == kOk && c < s_img.nc && nref[c] > (uint32_t)kApplyMaxScans) st = kEUnsupported;
#pragma unroll
                for (int c = 0; c < kMaxComp; c++) if (st == kOk && c < s_img.nc && !s_img.qoff[s_img.tq[c]]) st = kEFormat;
            }
        }
        if (lane == 0) {
            s_img.status = st;
            if (!(keep_status && R.status[i] != kOk)) R.status[i] = st;
        }
    }
    __syncthreads();
    {
        uint32_t* dst = reinterpret_cast<uint32_t*>(&R.scan[(size_t)i * R.G]);
        static_assert(sizeof(ScanDesc) % 4 == 0, "ScanDesc is copied as dwords");
        for (uint32_t e = tid; e < sizeof(ScanDesc) / 4 * upto; e += lanes) dst[e] = reinterpret_cast<const uint32_t*>(s_scan)[e];
        uint32_t* di = reinterpret_cast<uint32_t*>(&R.img[i]);
        for (uint32_t e = tid; e < sizeof(ImgDesc) / 4; e += lanes) di[e] = reinterpret_cast<const uint32_t*>(&s_img)[e];
    }
    if (s_img.status != kOk) return;
    // ---- the tables ----
    CanonCode* code = &s_code[wave];
    const uint32_t njobs = s_njobs;
    for (uint32_t job = wave; job < njobs; job += waves) {
        const uint32_t g = s_job[job] & 255u, j = s_job[job] >> 8;
        const ScanDesc& sd = s_scan[g];
        const size_t ig = (size_t)i * R.G + g;
        // (a table may have been defined ahead of this scan's own region: in memory then, unless it is region 0)
        canon_build(code, bytes_of(g), sd.Ss > 0 ? sd.ac_off : sd.dc_off[j], lane);
        wave_sync();
        if (sd.Ss > 0) actab_build_wave(&R.tabs[R.tab_idx[ig]], code, sd.Ah == 0, lane);
        else dctab_build_wave(&R.dctabs[R.dctab_idx[ig] + j], code, lane);
        wave_sync();
    }
}

// --------------------------------------------------------------------------------------
// k_unstuff: per (image, scan) remove stuffed zeros, fill bytes and restart markers from the entropy-coded segment, stop at
// the first other marker, note where each restart interval begins -- and, in the same launch, clear the memory the
// decoders expect to be zero (fills: a bandwidth-bound job beside a latency-bound one).
//
// 64 lanes x 16 bytes per step and wavefront, the next step's bytes under way meanwhile.  A byte is
// judged by itself and the byte before it, which for a lane's first byte comes from its neighbour by a lane shift: FF says
// nothing yet; after FF, 00 stands for a data byte FF, D0..D7 is a restart marker, FF is fill, anything else the marker
// that ends the segment; every other byte is data.  A lane classifies its sixteen bytes at once (one flag bit per byte in
// two 64-bit words), squeezes out the few it drops and puts the rest at its place in LDS (a prefix sum over the lanes says
// where); whole 16-byte chunks are then stored as the big-endian words the decoders read.
// A step takes a wavefront about 1.5 us whatever the others do, so the scans of a group that are long on average
// (kUnstuffWide bytes) get the four wavefronts of a workgroup (three barriers per step of 4 KB), the others one each.
// (Before: a workgroup per scan, 2 KB per step with four barriers and no loads ahead, 128 us for the 81 MB of 1024
// photographs, and 71 us for the fill after it.)
// --------------------------------------------------------------------------------------
constexpr uint32_t kUnstuffWaves = 4, kUnstuffManyWaves = 16, kUnstuffStep = 1024;
// What binding a handle to a record clears, pieces of 16 bytes, and 64 bytes behind the record (anywhere; null: none), in one launch: five or
// six memory fills were a dispatch of some microseconds each, behind the copy of the bytes and one after the other.  Bound by the launch
// (the largest piece is as long as the record).  us from host memory to training tensors: two
// photographs at scan group 1 368 -> 305, 293 of 139 to 356 pixels at 6 475 -> 430 (of 4 x 512 photographs at 5 the runs differ by more than that).
struct BindFill { uint4* p[5]; uint64_t n16[5]; uint32_t word[5], count; uint8_t* tail; };
__global__ void __launch_bounds__(256) k_bind_fill(BindFill F) {
    const uint64_t at = (uint64_t)blockIdx.x * 256 + threadIdx.x, step = (uint64_t)gridDim.x * 256;
#pragma unroll
    for (uint32_t f = 0; f < 5; f++) {
        if (f >= F.count) break;
        const uint4 v{F.word[f], F.word[f], F.word[f], F.word[f]};
        for (uint64_t i = at; i < F.n16[f]; i += step) F.p[f][i] = v;
    }
    if (F.tail && at < 64) F.tail[at] = 0;
}

constexpr int kMaxFills = 3;
struct FillList { uint4* p[kMaxFills]; size_t n16[kMaxFills]; uint32_t rows, past; };  // 16-byte pieces; rows of workgroups that share the work; past: see put_past

// 0x80 in every byte of the result whose byte in x is zero (exact, no carries between bytes)
PCR_D uint64_t zero_bytes(uint64_t x) {
    const uint64_t m = 0x7F7F7F7F7F7F7F7Full;
    return ~(((x & m) + m) | x | m);
}
// the flags (0x80 per byte) of the bytes below byte n (n >= 8: all; n < 0: none)
PCR_D uint64_t flags_below(int n) { return n >= 8 ? 0x8080808080808080ull : (n <= 0 ? 0ull : ((1ull << (8 * n)) - 1) & 0x8080808080808080ull); }
struct __attribute__((packed, aligned(1))) LooseU64 { uint64_t v; };
struct __attribute__((packed, aligned(1))) LooseU32 { uint32_t v; };
struct __attribute__((packed, aligned(1))) LooseU16 { uint16_t v; };

// What a launch works through: scan groups in order of decreasing length; first[e]: the first unstuffing workgroup of entry
// e (first[count]: their number); bit e of `wide`: one scan per workgroup, else one per wavefront.
// kUnstuffWide, in bytes of a group's mean scan; us of the launch with the line at 1024 / 3072 / 6144 / 12288 / never: 1024
// photographs at scan group 2 89 / 89 / 99 / 99 / 99, 5 109 / 108 / 98 / 98 / 103, 10 143 / 129 / 132 / 132 / 141; 256 pictures
// of 600 x 450 in 4:4:4 at 5 90 / 90 / 90 / 105 / 152; 128 of 1024 x 1024 at 10 114 / 114 / 131 / 131 / 279; 1024 of 256 x 256 at
// 5 43 / 31 / 31 / 31 / 31.
constexpr uint32_t kUnstuffWide = 6144;
// Few long scans leave most of the chip idle while each takes a step after the other: a workgroup has kUnstuffManyWaves wavefronts
// where all scans of a launch find room at once that way and the longest group's are several steps of the narrower ones.
// us of the launch, four wavefronts and sixteen: 38 pictures of 361 to 924 pixels at scan group 8 84 / 66, 24 of 896 x 952 at 6 57 / 47, one of
// 1000 x 700 at 3 37 / 30, the baseline file of a picture of 393 x 609 38.6 / 27.7.
constexpr uint32_t kUnstuffManyScans = 512, kUnstuffManyBytes = 12288;
struct UnstuffPlan { uint64_t wide; uint32_t count; uint32_t first[kMaxGroups + 1]; uint8_t group[kMaxGroups]; };

// One scan by W wavefronts (1, or those of a workgroup); wave: this one's number among them.  buf: W steps and
// 32 bytes; tot: W words.
template <uint32_t W>
PCR_D void unstuff_scan(const DevRecord& R, uint32_t i, uint32_t g, uint8_t* buf, uint32_t* tot, uint32_t wave, uint32_t lane) {
    auto together = [&]() { if (W > 1) __syncthreads(); else wave_sync(); };
    const ImgDesc& img = R.img[i];
    if (img.status != kOk || g >= img.nscans) return;
    const size_t ig = (size_t)i * R.G + g;
    const ScanDesc& sd = R.scan[ig];
    const uint32_t off = uni(sd.data_off), L = uni(sd.data_len), sb = uni(R.slot_base[ig]), sc = uni(R.slot_cnt[ig]);
    const uint8_t* src = R.rec + off;
    uint8_t* dst = R.clean + clean_base(off);
    // sixteen bytes from p on (bytes past the segment are whatever follows it in the record, and are not looked at) and, for
    // lane 0, the byte ahead of them
    auto load = [&](uint32_t p, uint64_t* lo, uint64_t* hi, uint32_t* prev) {
        *lo = *hi = 0; *prev = 0;
        if (p >= L) return;
        if (lane == 0 && p > 0) *prev = src[p - 1];
        if ((uint64_t)off + p + 16 <= R.nbytes) {
            *lo = reinterpret_cast<const LooseU64*>(src + p)->v; *hi = reinterpret_cast<const LooseU64*>(src + p + 8)->v;
        } else for (uint32_t q = 0; q < 16 && p + q < L; q++) {
            if (q < 8) *lo |= (uint64_t)src[p + q] << (8 * q); else *hi |= (uint64_t)src[p + q] << (8 * (q - 8));
        }
    };
    const uint32_t mine = (wave * 64 + lane) * 16, step = W * kUnstuffStep;
    uint32_t out_total = 0, rst_total = 0, have = 0;          // bytes stored; restart markers seen; bytes waiting in buf
    uint64_t nlo, nhi;
    uint32_t nprev;
    load(mine, &nlo, &nhi, &nprev);
    bool stop = false;
    for (uint32_t base = 0; base < L && !stop; base += step) {
        uint64_t lo = nlo, hi = nhi;
        const uint32_t before = lane_before((uint32_t)(hi >> 56), nprev);
        load(base + step + mine, &nlo, &nhi, &nprev);
        const int nvalid = (int)(L - base) - (int)mine;       // (may be more than sixteen, or negative)
        const uint64_t vlo = flags_below(nvalid), vhi = flags_below(nvalid - 8);
        const uint64_t flo = zero_bytes(~lo), fhi = zero_bytes(~hi);
        const uint64_t plo = (flo << 8) | (before == 0xFF ? 0x80ull : 0), phi = (fhi << 8) | (flo >> 63 << 7);      // the byte before is FF
        const uint64_t zlo = zero_bytes(lo), zhi = zero_bytes(hi);
        uint64_t klo = vlo & ((~flo & ~plo) | (plo & zlo)), khi = vhi & ((~fhi & ~phi) | (phi & zhi));
        uint64_t rlo = 0, rhi = 0;
        bool ends = false;                                    // the marker that ends the segment is among this wavefront's bytes
        if (__ballot(((plo & vlo & ~zlo) | (phi & vhi & ~zhi)) != 0)) {   // (rare) FF with something other than a stuffed zero behind it
            const uint64_t d = 0xF8F8F8F8F8F8F8F8ull, e = 0xD0D0D0D0D0D0D0D0ull;
            rlo = vlo & plo & zero_bytes((lo & d) ^ e); rhi = vhi & phi & zero_bytes((hi & d) ^ e);
            const uint64_t slo = vlo & plo & ~zlo & ~rlo & ~flo, shi = vhi & phi & ~zhi & ~rhi & ~fhi;
            const uint64_t who = __ballot((slo | shi) != 0);
            if (who) {                                        // drop what lies at or behind it
                ends = true;
                const uint32_t first = (uint32_t)__builtin_ctzll(who);
                const int upto = lane < first ? 16 : (lane > first ? 0 : (slo ? __builtin_ctzll(slo) >> 3 : 8 + (__builtin_ctzll(shi) >> 3)));
                klo &= flags_below(upto); khi &= flags_below(upto - 8); rlo &= flags_below(upto); rhi &= flags_below(upto - 8);
            }
        }
        // the stuffed zeros kept stand for the FF ahead of them
        const uint64_t tlo = klo & plo, thi = khi & phi;
        lo |= (tlo >> 7) * 0xFF; hi |= (thi >> 7) * 0xFF;
        uint32_t nkeep = (uint32_t)__builtin_popcountll(klo) + (uint32_t)__builtin_popcountll(khi);
        uint32_t nrst = (uint32_t)__builtin_popcountll(rlo) + (uint32_t)__builtin_popcountll(rhi);
        const uint32_t incl = lanes_prefix_sum(nkeep | (nrst << 16));
        uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63), ahead = 0;   // of all wavefronts; of those before this one
        stop = ends;
        if (W > 1) {                                          // (a wavefront's counts are below 2^11 and 2^10)
            if (lane == 0) tot[wave] = all | (ends ? 0x80000000u : 0u);
            __syncthreads();
            uint32_t sum = 0;
            stop = false;
#pragma unroll
            for (uint32_t q = 0; q < W; q++) {
                const uint32_t t = uni(tot[q]);
                if (q == wave) {
                    ahead = sum;
                    if (stop) nkeep = nrst = 0;               // the segment ended ahead of this wavefront's bytes
                }
                sum += stop ? 0u : t & 0x7FFFFFFFu;
                stop = stop || (t >> 31);
            }
            all = sum;
        }
        const uint32_t at = have + (ahead & 0xFFFF) + (incl & 0xFFFF) - nkeep;
        if (nrst) {                                           // (rare) where the next intervals begin: behind the bytes kept ahead of each marker
            uint32_t r = rst_total + (ahead >> 16) + (incl >> 16) - nrst;
            for (uint64_t m = rlo; m; m &= m - 1) { r++; if (r < sc) R.ivl_start[sb + r] = out_total + at + (uint32_t)__builtin_popcountll(klo & ((m & (0 - m)) - 1)); }
            for (uint64_t m = rhi; m; m &= m - 1) { r++; if (r < sc) R.ivl_start[sb + r] = out_total + at + (uint32_t)__builtin_popcountll(klo) + (uint32_t)__builtin_popcountll(khi & ((m & (0 - m)) - 1)); }
        }
        rst_total += all >> 16;
        // squeeze the dropped bytes out, the highest first (few lanes have any, and mostly one)
        uint64_t dlo = 0x8080808080808080ull & ~klo, dhi = 0x8080808080808080ull & ~khi;
        if (nkeep == 0) dlo = dhi = 0;
        while (dlo | dhi) {
            if (dhi) {
                const uint32_t sh = (63u - (uint32_t)__builtin_clzll(dhi)) & 56u;
                dhi &= ~(0x80ull << sh);
                const uint64_t low = (1ull << sh) - 1;
                hi = (hi & low) | ((hi >> 8) & ~low);
            } else {
                const uint32_t sh = (63u - (uint32_t)__builtin_clzll(dlo)) & 56u;
                dlo &= ~(0x80ull << sh);
                const uint64_t low = (1ull << sh) - 1;
                lo = (lo & low) | (((lo >> 8) & ~low) & 0x00FFFFFFFFFFFFFFull) | (hi << 56);
                hi >>= 8;
            }
        }
        uint8_t* p = buf + at;
        if (nkeep == 16) { reinterpret_cast<LooseU64*>(p)->v = lo; reinterpret_cast<LooseU64*>(p + 8)->v = hi; }
        else {
            if (nkeep & 8) { reinterpret_cast<LooseU64*>(p)->v = lo; p += 8; lo = hi; }
            if (nkeep & 4) { reinterpret_cast<LooseU32*>(p)->v = (uint32_t)lo; p += 4; lo >>= 32; }
            if (nkeep & 2) { reinterpret_cast<LooseU16*>(p)->v = (uint16_t)lo; p += 2; lo >>= 16; }
            if (nkeep & 1) *p = (uint8_t)lo;
        }
        together();
        have += all & 0xFFFF;
        const uint32_t full = have >> 4, c = wave * 64 + lane;   // whole chunks: one per lane at most (fewer than sixteen bytes were waiting)
        uint4 left{0, 0, 0, 0};
        if (c < full) {
            const uint4 v = *reinterpret_cast<const uint4*>(buf + c * 16);
            *reinterpret_cast<uint4*>(dst + out_total + c * 16) = uint4{__builtin_bswap32(v.x), __builtin_bswap32(v.y), __builtin_bswap32(v.z), __builtin_bswap32(v.w)};
        }
        if (c == 0) left = *reinterpret_cast<const uint4*>(buf + full * 16);
        together();
        if (c == 0) *reinterpret_cast<uint4*>(buf) = left;    // (the next step writes behind its first have & 15 bytes, some of them into the rest of it)
        together();
        out_total += full * 16; have &= 15u;
    }
    const uint32_t c = wave * 64 + lane;
    // what is left: whole words (their unused bytes lie ahead of the next segment: a marker and its length are four bytes)
    if (c * 4 < have) *reinterpret_cast<uint32_t*>(dst + out_total + c * 4) = __builtin_bswap32(*reinterpret_cast<const uint32_t*>(buf + c * 4));
    out_total += have;
    if (c == 0) {
        R.ivl_start[sb] = 0;
        // intervals whose restart marker never showed up get an empty range; the end goes last
        for (uint32_t r = rst_total + 1; r <= sc; r++) R.ivl_start[sb + r] = out_total;
        R.ivl_start[sb + sc] = out_total;
        if (rst_total + 1 != (sd.ri ? sc : 1u)) R.status[i] = kEFormat;      // (without restart intervals the units of a scan start at entry points)
    }
    if (sd.Ss == 0 && sd.Ah != 0) {
        // DC refinement is read in place later (one bit per block): check every interval is long enough
        __threadfence_block();
        together();
        uint32_t bpm = 0;
        for (int q = 0; q < sd.ns; q++) bpm += sd.ns > 1 ? (uint32_t)img.hs[sd.comp[q]] * img.vs[sd.comp[q]] : 1;
        for (uint32_t r = c; r < sc; r += W * 64) {
            const uint32_t m0 = sd.ri ? r * sd.ri : 0, m1 = sd.ri ? (m0 + sd.ri < sd.mcus ? m0 + sd.ri : sd.mcus) : sd.mcus;
            const uint32_t bits = (R.ivl_start[sb + r + 1] - R.ivl_start[sb + r]) * 8;
            if ((m1 - m0) * bpm > bits) R.status[i] = kEFormat;
        }
    }
}

struct ApplyUnit { uint32_t img; uint32_t comp; };
struct ApplyScan { uint64_t mask_off; uint32_t slot; uint32_t data_base; uint32_t mcu_w; uint16_t ri; uint8_t Ss, Se, Ah, Al, ns, before, bpm, pad[3]; };
struct ApplyList { uint32_t n, nac; ApplyScan sc[kApplyMaxScans]; };       // AC scans first (nac of them), then DC scans; both in file order
// The lists of a call (none: nau = 0), made by the first `groups` workgroups of the unstuffing launch.
struct ApplyJob { const ApplyUnit* au; ApplyList* lists; uint32_t nau, kmax, groups; };

// Gathers, per (image, component), the scans that matter for refinement (AC scans of the component in file order, DC
// refinement scans) into a compact list.
// A wavefront per (image, component), a lane per scan: the loads of all scans are under way together.  (A lane per image
// and component walking its scans took 9.4 us for 1024 images, nearly all of it waiting for one load after another.)
constexpr int kApplyPrepWaves = 4;                          // (in a launch of its own; else as many as a workgroup of that launch has)
PCR_D void apply_prep(const DevRecord& R, const ApplyUnit* __restrict__ au, uint32_t nau, uint32_t kmax, ApplyList* lists, uint32_t group) {
    const uint32_t u = group * (blockDim.x >> 6) + uni(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    if (u >= nau) return;
    const ApplyUnit a = au[u];
    const ImgDesc* img = &R.img[a.img];
    const uint32_t c = a.comp;
    ApplyList* L = &lists[u];
    const uint32_t upto = img->nscans < kmax ? img->nscans : kmax;
    uint32_t n = 0;
    for (uint32_t dc = 0; dc < 2; dc++) {                    // (AC first scans are in the planes already)
        for (uint32_t g0 = 0; g0 < upto; g0 += 64) {
            const uint32_t g = g0 + lane;
            const size_t ig = (size_t)a.img * R.G + (g < upto ? g : 0u);
            const ScanDesc sd = R.scan[ig];
            ApplyScan e;
            e.Ss = sd.Ss; e.Se = sd.Se; e.Ah = sd.Ah; e.Al = sd.Al; e.ns = sd.ns; e.ri = sd.ri; e.mcu_w = sd.mcu_w;
            e.mask_off = R.mask_off[ig]; e.slot = R.slot_base[ig]; e.data_base = clean_base(sd.data_off);
            e.before = 0; e.bpm = 0; e.pad[0] = e.pad[1] = e.pad[2] = 0;
            bool has = false;
            uint32_t before = 0, bpm = 0;
#pragma unroll
            for (uint32_t q = 0; q < (uint32_t)kMaxComp; q++) {
                if (q >= sd.ns) continue;
                const uint32_t cq = sd.comp[q];
                if (cq == c) { has = true; before = bpm; }
                bpm += sd.ns > 1 ? (uint32_t)img->hs[cq] * img->vs[cq] : 1u;
            }
            if (dc) { e.before = (uint8_t)before; e.bpm = (uint8_t)bpm; } else has = sd.comp[0] == c;
            const bool take = g < upto && sd.Ah != 0 && (sd.Ss == 0 ? 1u : 0u) == dc && has;
            const uint64_t all = __builtin_amdgcn_ballot_w64(take);
            const uint32_t at = n + (uint32_t)__builtin_popcountll(all & ((1ull << lane) - 1u));
            if (take && at < (uint32_t)kApplyMaxScans) L->sc[at] = e;
            n += (uint32_t)__builtin_popcountll(all);
        }
        n = n < (uint32_t)kApplyMaxScans ? n : (uint32_t)kApplyMaxScans;
        if (!dc && lane == 0) L->nac = n;
    }
    if (lane == 0) L->n = n;
}
// (a launch of its own while stage timing is on)
__global__ void __launch_bounds__(64 * kApplyPrepWaves) k_apply_prep(DevRecord R, ApplyJob A) { apply_prep(R, A.au, A.nau, A.kmax, A.lists, blockIdx.x); }

// Workgroups [0, A.groups) make the refinement lists: a launch of their own behind the entropy decoders took 5.5 us and the gap to the next
// (64 gray pictures at scan group 6 186 -> 182 us a call, 256 ragged ones 364 -> 359).  A multiple of kDies, so that the others keep their dies.
// The other P.first[P.count] + kDies * F.rows: fill_turn says which of them fill, the others unstuff.  (Every second
// or fourth single workgroup, as before, put the whole fill on four or two of the eight dies: 202 and 214 us for 1024
// photographs at scan groups 9 and 10, of which the 0.5 GB fill is the larger part, against 118 and 131.)
template <uint32_t WAVES>
__global__ void __launch_bounds__(64 * WAVES) k_unstuff(DevRecord R, UnstuffPlan P, FillList F, uint32_t period, ApplyJob A) {
    __shared__ __attribute__((aligned(16))) uint8_t buf[WAVES * (kUnstuffStep + 32)];
    __shared__ uint32_t tot[WAVES];
    short_kernel_priority();
    const uint32_t tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63;
    if (blockIdx.x < A.groups) { apply_prep(R, A.au, A.nau, A.kmax, A.lists, blockIdx.x); return; }
    const FillTurn turn = fill_turn(blockIdx.x - A.groups, F.rows, period);
    if (turn.fills) {
        for (int f = 0; f < kMaxFills; f++) {
            uint4* p = F.p[f];
            const size_t n16 = F.n16[f], stride = (size_t)F.rows * kDies * (64 * WAVES);
            const uint32_t zero[4] = {0, 0, 0, 0};
            if (F.past) { for (size_t e = (size_t)turn.index * (64 * WAVES) + tid; e < n16; e += stride) put_past<uint4>(p + e, zero); }
            else for (size_t e = (size_t)turn.index * (64 * WAVES) + tid; e < n16; e += stride) p[e] = make_uint4(0, 0, 0, 0);
        }
        return;
    }
    const uint32_t u = turn.index;
    uint32_t e = 0;
    while (e + 1 < P.count && u >= P.first[e + 1]) e++;
    if (e >= P.count) return;
    const uint32_t g = P.group[e], at = u - P.first[e];
    if ((P.wide >> e) & 1) {
        if (at < R.n) unstuff_scan<WAVES>(R, at, g, buf, tot, wave, lane);
    } else {
        const uint32_t i = at * WAVES + wave;
        if (i < R.n) unstuff_scan<1>(R, i, g, buf + wave * (kUnstuffStep + 32), tot, 0, lane);
    }
}

// --------------------------------------------------------------------------------------
// Entropy kernels: ONE WAVEFRONT PER UNIT (a restart interval of one scan of one image).
// Everything the decoder touches is a function of the block and the wavefront's number in it, i.e. wave-uniform, so the
// compiler keeps the decoder state in scalar registers and runs it on the scalar ALU with
// native 64-bit shifts, population counts and find-first-set; the Huffman table sits in LDS.
// A serial bit-stream decoder has no use for 64 lanes, but a lone wavefront issues only about
// one instruction per ten cycles whatever its width, and packing 64 different streams into one
// wavefront makes every loop iteration pay for the union of all lanes' branches; one stream
// per wavefront costs only the branch actually taken and lets thousands of streams interleave
// on the SIMDs.  The host orders units by decreasing byte length (longest first).
// (With tens of thousands of units per launch the balance tips: see pcr_lanes.h and the kernels
// k_ac_first_lanes / k_ac_refine_lanes below, which the host takes for such launches.)
// --------------------------------------------------------------------------------------
constexpr int kEntropyLanes = 64;
// clean32 is R.clean again, as a separate restrict-qualified kernel argument: the kernels only read the unstuffed
// data, and knowing that nothing written here aliases it lets the compiler fetch it with scalar loads (straight into
// scalar registers, waited for at the first use) instead of vector loads followed by a read-first-lane.

struct UnitSetup {
    const uint32_t* words;        // segment base, unit start and length for the window readers
    uint32_t byte_off, sub_bits, nbits, pos0;
    LaneScan ls;
    int16_t* plane[kMaxComp];     // planes of the scan's components
    uint32_t plane_elems[kMaxComp];
    int16_t* base;                // the image's coefficient buffer (all planes)
    uint32_t base_elems;
    bool ok;
};

// The status of an image, read once for all wavefronts of the workgroup.  Workgroups that decode other units of the image write that word
// in the same launch: wavefronts that are to meet at a barrier behind it must not each read it for themselves.
PCR_D int group_status(const DevRecord& R, uint32_t img) {
    __shared__ int s_status;
    if (threadIdx.x == 0) s_status = R.status[img];
    __syncthreads();
    return uni(s_status);
}
// good: whether the image's status is kOk.  (A call, so that where a wavefront reads the word for itself it does so behind the image's address: ahead of
// it the decoders of short launches took 0.3 to 0.5 % longer.)
template <class Good>
PCR_D void unit_setup(const DevRecord& R, const Unit& un, const uint32_t* __restrict__ clean32, UnitSetup* L, const Good& good) {
    L->ok = false;
    const ImgDesc* img = &R.img[un.img];
    if (!good() || un.scan >= img->nscans) return;
    const size_t ig = (size_t)un.img * R.G + un.scan;
    const ScanDesc* sd = &R.scan[ig];
    if (!sd->valid) return;
    const uint32_t sb = R.slot_base[ig];
    const uint32_t ri = sd->ri, mcus = sd->mcus;
    LaneScan& ls = L->ls;
    ls.mcu_w = uni(sd->mcu_w);
    ls.pred[0] = ls.pred[1] = ls.pred[2] = 0;
    const uint32_t sc = R.slot_cnt[ig];
    if (ri == 0 && sc > 1) {
        // Units of a scan without restart markers start at the record's entry points: unit j runs from entry j-1
        // (the scan's start for j = 0) to entry j (the scan's end for the last unit).
        const uint32_t stride = uni(entry_stride(ld_le16(R.rec + hdr_ecount_pos(R.n, R.G, un.scan, un.img))));   // 16 bytes, or 8 without DC predictions
        const uint8_t* e = R.rec + uni(R.ent_off[ig]) + (size_t)stride * un.interval;             // entry j; entry j-1 lies one stride before it
        const uint32_t total = uni(R.ivl_start[sb + sc]) * 8;                                    // bits of the scan's unstuffed data
        uint32_t m0 = 0, bit0 = 0, m1 = mcus, bit1 = total;
        if (un.interval > 0) {
            const uint8_t* p = e - stride;
            m0 = uni(ld_le32(p)); bit0 = uni(ld_le32(p + 4));
            if (stride == kEntryBytes) { ls.pred[0] = uni((int)(int16_t)ld_le16(p + 8)); ls.pred[1] = uni((int)(int16_t)ld_le16(p + 10)); ls.pred[2] = uni((int)(int16_t)ld_le16(p + 12)); }
        }
        if (un.interval + 1 < sc) { m1 = uni(ld_le32(e)); bit1 = uni(ld_le32(e + 4)); }
        if (!(m0 < m1 && m1 <= mcus && bit0 <= bit1 && bit1 <= total)) { R.status[un.img] = kEFormat; return; }   // entries out of order or out of range
        ls.mcu0 = m0; ls.mcu1 = m1;
        L->byte_off = bit0 >> 3; L->sub_bits = bit0 & 7; L->nbits = bit1 - (bit0 & ~7u); L->pos0 = bit0 & ~7u;
    } else {
        const uint32_t b0 = R.ivl_start[sb + un.interval], b1 = R.ivl_start[sb + un.interval + 1];
        ls.mcu0 = uni(ri ? un.interval * ri : 0);
        ls.mcu1 = uni(ri ? (ls.mcu0 + ri < mcus ? ls.mcu0 + ri : mcus) : mcus);
        if (ls.mcu0 >= mcus) return;
        L->byte_off = uni(b0); L->sub_bits = 0; L->nbits = uni(b1 > b0 ? b1 - b0 : 0) * 8; L->pos0 = 0;
    }
    ls.Ss = uni((int)sd->Ss); ls.Se = uni((int)sd->Se); ls.Al = uni((int)sd->Al); ls.ns = uni((int)sd->ns);
    int16_t* base = R.coef + uni((uint64_t)R.coef_off[un.img]);
    size_t poff[kMaxComp + 1]; poff[0] = 0;
#pragma unroll
    for (int c = 0; c < kMaxComp; c++) poff[c + 1] = poff[c] + (c < img->nc ? (size_t)uni((uint32_t)img->bw[c]) * uni((uint32_t)img->bh[c]) * 64 : 0);
#pragma unroll
    for (int j = 0; j < kMaxComp; j++) {
        const int c = uni(j < ls.ns ? (int)sd->comp[j] : 0);
        ls.hs[j] = uni((uint32_t)img->hs[c]); ls.vs[j] = uni((uint32_t)img->vs[c]); ls.bw[j] = uni((uint32_t)img->bw[c]);
        const size_t po = c == 0 ? poff[0] : (c == 1 ? poff[1] : poff[2]);
        ls.poff[j] = (uint32_t)po;
        L->plane[j] = base + po;
        L->plane_elems[j] = (uint32_t)((c == 0 ? poff[1] : (c == 1 ? poff[2] : poff[3])) - po);
    }
    L->base = base;
    L->base_elems = (uint32_t)poff[kMaxComp];
    L->words = clean32 + (uni(clean_base(sd->data_off)) >> 2);
    L->ok = true;
}

// The same for a wavefront that is alone with its unit.
PCR_D void unit_setup(const DevRecord& R, const Unit& un, const uint32_t* __restrict__ clean32, UnitSetup* L) {
    unit_setup(R, un, clean32, L, [&]() { return R.status[un.img] == kOk; });
}

// What earlier kernels wrote and this one only reads, at a wave-uniform address: a scalar load, which arrives in scalar
// registers and does not stand in the way of the loads behind it.
template <class T> PCR_D T load_const(const T* p) { return *(const __attribute__((address_space(4))) T*)p; }
// The caller's copy of an image's status, from the workgroup of the pixel kernel that has the image's first tile.  (As a copy of its own
// behind that kernel it was one more command that waits for the one before it.  Pictures of 16 to 43 pixels, two records of 130 at scan
// group 2: 112 us a call with it, 80 without; 120 of 88 x 103 at 6: 135 and 130.)
PCR_D void hand_out_status(const DevRecord& R, uint32_t img, uint32_t tile) {
    if (R.status_out && tile == 0) {
        const int32_t st = load_const(&R.status[img]);
        if (threadIdx.x == 0) R.status_out[img] = st;
    }
}
// Where this stands its arguments have been loaded: loads that depend on nothing but the image's number are then under
// way together.  (The compiler moves each to its first use, behind the branches, and waits for one after the other.)
PCR_D void wanted_now(uint32_t a) { asm volatile("" :: "s"(a)); }
PCR_D void wanted_now(uint64_t a) { asm volatile("" :: "s"(a)); }
// a value per component, picked by a component number (per lane or wave-uniform) out of three wave-uniform ones
PCR_D uint32_t pick3(uint32_t c, uint32_t a0, uint32_t a1, uint32_t a2) { return c == 0 ? a0 : (c == 1 ? a1 : a2); }

// a descriptor through a wave-uniform pointer, as dwords
template <class T> PCR_D void load_desc(const T* ip, T* D) {
    const __attribute__((address_space(4))) uint32_t* src = (const __attribute__((address_space(4))) uint32_t*)ip;
    uint32_t* dst = reinterpret_cast<uint32_t*>(D);
#pragma unroll
    for (uint32_t e = 0; e < sizeof(T) / 4; e++) dst[e] = src[e];
}
template <class T> PCR_D void desc_wanted_now(const T& D) {
    const uint32_t* w = reinterpret_cast<const uint32_t*>(&D);
#pragma unroll
    for (uint32_t e = 0; e < sizeof(T) / 4; e++) wanted_now(w[e]);
}
PCR_D void wanted_now(const ImgDesc& D) { desc_wanted_now(D); }
PCR_D void wanted_now(const ScanDesc& D) { desc_wanted_now(D); }

// The same in vector registers; a descriptor as its words (loaded whole: the loads of single members end up behind the
// branches that use them).
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
PCR_D void arrived(uint32_t a) { asm volatile("" :: "v"(a)); }
PCR_D void arrived(uint64_t a) { asm volatile("" :: "v"(a)); }
template <class T> struct DescWords {
    static constexpr uint32_t kQuads = sizeof(T) / 16, kRest = sizeof(T) / 4 - 4 * kQuads;
    uint4v q[kQuads]; uint32_t r[kRest ? kRest : 1];
    PCR_D void load(const T* p) {
        struct __attribute__((packed, aligned(4))) Quad { uint4v v; };
#pragma unroll
        for (uint32_t e = 0; e < kQuads; e++) q[e] = reinterpret_cast<const Quad*>(p)[e].v;
#pragma unroll
        for (uint32_t e = 0; e < kRest; e++) r[e] = reinterpret_cast<const uint32_t*>(p)[4 * kQuads + e];
    }
    PCR_D void here() const {
#pragma unroll
        for (uint32_t e = 0; e < kQuads; e++) asm volatile("" :: "v"(q[e]));
#pragma unroll
        for (uint32_t e = 0; e < kRest; e++) asm volatile("" :: "v"(r[e]));
    }
    // the member of `bytes` bytes at offset off (constants, after inlining)
    PCR_D uint32_t at(size_t off, uint32_t bytes) const {
        const uint32_t e = (uint32_t)off / 4, w = e < 4 * kQuads ? q[e / 4][e % 4] : r[e - 4 * kQuads];
        return bytes == 4 ? w : (w >> (8 * (off % 4))) & ((1u << (8 * bytes)) - 1u);
    }
};
#define PCR_MEMBER(D, T, m, i) ((D).at(offsetof(T, m) + (i) * sizeof(((T*)0)->m[0]), sizeof(((T*)0)->m[0])))
#define PCR_FIELD(D, T, m) ((D).at(offsetof(T, m), sizeof(((T*)0)->m)))

// What the set-up of a unit reads, in two rounds of loads that depend on nothing but the unit and on the first round: loads
// that are each behind a check of the one before cost a trip to memory each, eight or nine of them ahead of a lane's first
// symbol.  (Every address is inside its buffer whatever the descriptors say; the checks come afterwards.)
struct LaneUnitInfo {
    DescWords<ImgDesc> img; DescWords<ScanDesc> sd;
    bool ok, entries;                                         // the unit can be decoded, as far as these tell; it runs from one entry point to another
    uint32_t ns, Ss, Se, Ah, Al, mcu_w;
    uint64_t coef0;
    uint32_t m0, m1, b0, b1;                                  // its MCUs, its bits in the scan's unstuffed data
    uint64_t preds;                                           // DC predictions of the entry point it starts at, or zeros
    PCR_D uint32_t bw(uint32_t c) const { return pick(c, PCR_MEMBER(img, ImgDesc, bw, 0), PCR_MEMBER(img, ImgDesc, bw, 1), PCR_MEMBER(img, ImgDesc, bw, 2)); }
    PCR_D uint32_t bh(uint32_t c) const { return pick(c, PCR_MEMBER(img, ImgDesc, bh, 0), PCR_MEMBER(img, ImgDesc, bh, 1), PCR_MEMBER(img, ImgDesc, bh, 2)); }
    PCR_D uint32_t hs(uint32_t c) const { return pick(c, PCR_MEMBER(img, ImgDesc, hs, 0), PCR_MEMBER(img, ImgDesc, hs, 1), PCR_MEMBER(img, ImgDesc, hs, 2)); }
    PCR_D uint32_t vs(uint32_t c) const { return pick(c, PCR_MEMBER(img, ImgDesc, vs, 0), PCR_MEMBER(img, ImgDesc, vs, 1), PCR_MEMBER(img, ImgDesc, vs, 2)); }
    PCR_D uint32_t nblk(uint32_t c) const { return c < PCR_FIELD(img, ImgDesc, nc) ? bw(c) * bh(c) : 0u; }
    PCR_D uint32_t before(uint32_t c) const { return (c > 0 ? nblk(0) : 0u) + (c > 1 ? nblk(1) : 0u); }      // blocks of the planes ahead of it
    PCR_D static uint32_t pick(uint32_t c, uint32_t a0, uint32_t a1, uint32_t a2) { return c == 0 ? a0 : (c == 1 ? a1 : a2); }
};
PCR_D uint64_t loose64(const uint8_t* p) { return reinterpret_cast<const LooseU64*>(p)->v; }
PCR_D __attribute__((always_inline)) void lane_unit_info(const DevRecord& R, const Unit& un, LaneUnitInfo* I) {
    const size_t ig = (size_t)un.img * R.G + un.scan;
    auto in_record = [&](uint64_t at, uint32_t bytes) { return R.rec + (at + bytes <= R.nbytes ? at : R.nbytes - bytes); };   // (a record has more than 24 bytes)
    // first round
    I->img.load(&R.img[un.img]); I->sd.load(&R.scan[ig]);
    const uint32_t status = (uint32_t)R.status[un.img], sc = R.slot_cnt[ig], ent = R.ent_off[ig];
    const uint32_t field = reinterpret_cast<const LooseU16*>(in_record(hdr_ecount_pos(R.n, R.G, un.scan, un.img), 2))->v;
    const uint32_t i0 = R.ivl_start[un.slot + un.interval], i1 = R.ivl_start[un.slot + un.interval + 1];
    I->coef0 = R.coef_off[un.img];
    I->img.here(); I->sd.here(); arrived(status); arrived(sc); arrived(ent); arrived(field); arrived(i0); arrived(i1); arrived(I->coef0);
    I->ns = PCR_FIELD(I->sd, ScanDesc, ns); I->Ss = PCR_FIELD(I->sd, ScanDesc, Ss); I->Se = PCR_FIELD(I->sd, ScanDesc, Se);
    I->Ah = PCR_FIELD(I->sd, ScanDesc, Ah); I->Al = PCR_FIELD(I->sd, ScanDesc, Al); I->mcu_w = PCR_FIELD(I->sd, ScanDesc, mcu_w);
    const uint32_t mcus = PCR_FIELD(I->sd, ScanDesc, mcus), ri = PCR_FIELD(I->sd, ScanDesc, ri);
    I->entries = ri == 0 && sc > 1;
    // second round: the scan's end, the entry points ahead of and behind the unit
    const uint32_t stride = entry_stride(field);
    const uint64_t e = (uint64_t)ent + (uint64_t)stride * un.interval;
    const bool first = un.interval == 0, last = un.interval + 1 >= sc;
    const uint64_t ahead = I->entries && !first ? e - stride : 0;
    const uint8_t *pa = in_record(ahead, 8), *pp = in_record(ahead + 8, 8), *pb = in_record(I->entries && !last ? e : 0, 8);
    const uint32_t total = R.ivl_start[un.slot + (I->entries ? sc : 0u)] * 8;
    const uint64_t ea = loose64(pa), eb = loose64(pb), ep = loose64(pp);
    arrived(total); arrived(ea); arrived(eb); arrived(ep);
    const uint32_t r0 = ri ? un.interval * ri : 0u, r1 = ri ? (r0 + ri < mcus ? r0 + ri : mcus) : mcus;
    I->m0 = I->entries ? (first ? 0u : (uint32_t)ea) : r0; I->m1 = I->entries && !last ? (uint32_t)eb : (I->entries ? mcus : r1);
    I->b0 = I->entries ? (first ? 0u : (uint32_t)(ea >> 32)) : i0 * 8; I->b1 = I->entries ? (last ? total : (uint32_t)(eb >> 32)) : (i1 > i0 ? i1 : i0) * 8;
    I->preds = !I->entries || first || stride != kEntryBytes ? 0u : ep;
    I->ok = status == (uint32_t)kOk && un.scan < PCR_FIELD(I->img, ImgDesc, nscans) && PCR_FIELD(I->sd, ScanDesc, valid) != 0 && I->mcu_w != 0 && (I->entries || I->m0 < mcus);
    if (I->ok && I->entries && !(I->m0 < I->m1 && I->m1 <= mcus && I->b0 <= I->b1 && I->b1 <= total)) { R.status[un.img] = kEFormat; I->ok = false; }   // entries out of order or out of range
}

// The same checks and ranges as unit_setup (pcr_kernels.h), without the assumption that the unit is wave-uniform.
PCR_D void lane_unit_setup(const DevRecord& R, const Unit& un, const uint32_t* __restrict__ clean32, LaneUnit* U) {
    LaneUnitInfo I;
    lane_unit_info(R, un, &I);
    U->ok = I.ok && I.ns == 1 && I.Ss != 0;
    const uint32_t c = PCR_MEMBER(I.sd, ScanDesc, comp, 0);
    U->mcu0 = I.m0; U->mcu1 = I.m1; U->bit0 = I.b0; U->bit1 = I.b1; U->mcu_w = I.mcu_w;
    U->Ss = I.Ss; U->Se = I.Se; U->Al = I.Al;
    U->bw = I.bw(c);
    U->plane_elems = U->bw * I.bh(c) * 64;
    U->plane = R.coef + I.coef0 + (size_t)I.before(c) * 64;
    U->words = clean32 + (clean_base(PCR_FIELD(I.sd, ScanDesc, data_off)) >> 2);
    U->tab = nullptr;                                         // (the kernel points it at the job's copy in LDS)
}

// One job of a lane-per-unit kernel: units [first, first + count) of the launch's list, count <= 64, and the scans they
// belong to (image * scans per image + scan), kLaneTabs at most: one Huffman table each.
constexpr int kLaneTabs = 8;
struct LaneJob { uint32_t first, count, ntab; uint32_t key[kLaneTabs]; };

// The AC tables of a job on their way into LDS, straight from memory: bring with every lane of the wavefront, have once
// they are needed (the set-up of the units goes on beside them).  Where the tables lie is read first, for all at once: with
// each table behind its own index and its own branch the eight of a job were eight trips to memory one after the other.
PCR_D void lane_tables_bring(const DevRecord& R, const LaneJob& job, const Unit& un, uint4 (*tabs)[kLaneTabPieces]) {
    const uint32_t t = threadIdx.x;
    static_assert(kLaneTabPieces > kEntropyLanes && kLaneTabPieces <= 2 * kEntropyLanes, "two pieces per lane");
    uint32_t at[kLaneTabs];
#pragma unroll
    for (uint32_t sl = 0; sl < (uint32_t)kLaneTabs; sl++) {
        const uint32_t k = job.key[sl < job.ntab ? sl : 0u];
        at[sl] = load_const(&R.tab_idx[k < R.n * R.G ? k : 0u]);
    }
#pragma unroll
    for (uint32_t sl = 0; sl < (uint32_t)kLaneTabs; sl++) wanted_now(at[sl]);
    arrived(un.img); arrived(un.scan);                        // (the lane's unit, on its way since before: waited for here, not behind the tables)
    auto to_lds = [](const uint4* from, uint4* to) {          // lane l's piece to to[l]
        __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)from, (__attribute__((address_space(3))) void*)to, 16, 0, 0);
    };
#pragma unroll
    for (uint32_t sl = 0; sl < (uint32_t)kLaneTabs; sl++) {
        if (sl >= job.ntab) continue;                         // (the same for all lanes)
        const uint4* src = reinterpret_cast<const uint4*>(&R.tabs[at[sl]]);
        to_lds(src + t, &tabs[sl][0]);
        if (t < kLaneTabPieces - kEntropyLanes) to_lds(src + kEntropyLanes + t, &tabs[sl][kEntropyLanes]);
    }
}
PCR_D void lane_tables_have() {
    __builtin_amdgcn_s_waitcnt(0x0F70);                       // (vmcnt 0)
    __syncthreads();
}
// the slot of the table of scan `key` (>= kLaneTabs: not among the job's -- the host never makes such a job)
PCR_D uint32_t lane_table_slot(const DevRecord& R, const LaneJob& job, uint32_t key) {
    uint32_t slot = ~0u;
#pragma unroll
    for (uint32_t sl = 0; sl < (uint32_t)kLaneTabs; sl++)
        if (sl < job.ntab && job.key[sl] == key && key < R.n * R.G) slot = sl;
    return slot;
}

// The scans of a component that build on each other -- its AC first scans, then one refinement scan after another -- are
// decoded side by side by the wavefronts of one workgroup, each following the one before it through the image: a
// refinement scan needs of a block only what the earlier scans made of that block.  (One launch after the other took the
// SUM of the scans' times, and a scan's time is that of its longest unit: 2.9 + 4.7 + 6.0 ms for photographs without
// entry points; side by side they take about the longest of them.)
//
// done[w]: blocks of the scan that wavefront w has finished and whose results are in memory (a workgroup's wavefronts run
// on one compute unit and share its vector cache: no more than the order of the operations is needed to see them).  A
// wavefront waits only for wavefronts before it in the chain, and every wavefront ends by releasing all of its blocks,
// whatever became of its unit: every wait ends.
// units [first, first + count), a wavefront each; refines: those of them that are of refinement scans; byte w of waits: the earlier wavefronts that wavefront w follows
struct UnitChain { uint32_t first; uint16_t count, refines; uint64_t waits; };

struct ChainGate {
    uint32_t* done;
    uint32_t self, waits;
    bool watched;                                             // some wavefront follows this one
    uint32_t avail;                                           // blocks before this one have been released by all this wavefront follows
    PCR_D void need(uint32_t m) {
        if (m < avail) return;
        for (;;) {
            uint32_t least = ~0u;
            for (uint32_t w = waits; w; w &= w - 1) {
                const uint32_t d = uni(__hip_atomic_load(&done[__builtin_ctz(w)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                least = d < least ? d : least;
            }
            avail = least;
            if (m < avail) break;
            __builtin_amdgcn_s_sleep(4);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
    PCR_D bool due(uint32_t bits) const { return watched && ((bits >> 6) & 3u) == 0; }      // (every fourth window)
    PCR_D void publish(uint32_t m) {
        if (!watched) return;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __hip_atomic_store(&done[self], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

PCR_D ChainGate chain_gate(const UnitChain& ch, uint32_t* done, uint32_t wave) {
    uint64_t all = ch.waits | (ch.waits >> 32);
    all |= all >> 16; all |= all >> 8;
    ChainGate gate{done, wave, (uint32_t)(ch.waits >> (8 * wave)) & 255u, ((all >> wave) & 1u) != 0, 0u};
    if (gate.waits == 0) gate.avail = ~0u;
    return gate;
}

// What a wavefront keeps in LDS: the AC table of its scan and the words of the stream it is at, or the DC tables of its components.
constexpr uint32_t kWaveTabBytes = sizeof(AcTab) + kStageWords * sizeof(uint32_t), kWaveDcTabBytes = kMaxComp * sizeof(DcTab);
static_assert(kWaveDcTabBytes <= kWaveTabBytes, "one area serves both");

PCR_D int wave_dc_first(const DevRecord& R, const Unit& un, const UnitSetup& L, DcTab* tabs, uint32_t lane, bool to_planes) {
    dc_kernel_priority();
    const ScanDesc* sd = &R.scan[(size_t)un.img * R.G + un.scan];
    const uint32_t o0 = sd->dc_off[0], o1 = L.ls.ns > 1 ? sd->dc_off[1] : o0, o2 = L.ls.ns > 2 ? sd->dc_off[2] : o0;
    // distinct tables of the scan's components: slot 0 always, slot 1/2 when a component uses another one
    int tj1 = 0, tj2 = 0, ntab = 1;
    if (o1 != o0) { tj1 = 1; ntab = 2; }
    if (o2 == o1) tj2 = tj1; else if (o2 != o0) { tj2 = ntab; ntab++; }
    {                                                       // built by k_headers: copy the distinct ones
        const uint32_t* src = reinterpret_cast<const uint32_t*>(&R.dctabs[R.dctab_idx[(size_t)un.img * R.G + un.scan]]);
        uint32_t* dst = reinterpret_cast<uint32_t*>(&tabs[0]);
        constexpr uint32_t kWords = sizeof(DcTab) / 4;
        for (uint32_t e = lane; e < kWords; e += kEntropyLanes) {
            dst[e] = src[e];
            if (tj1 == 1) dst[kWords + e] = src[kWords + e];
            if (tj2 != 0 && tj2 != tj1) dst[(uint32_t)tj2 * kWords + e] = src[2 * kWords + e];
        }
    }
    wave_sync();
    DcWindowReader wr;                                      // tables by scan component
    wr.init(L.words, L.byte_off, L.sub_bits, L.nbits, &tabs[0], &tabs[uni(tj1)], &tabs[uni(tj2)], L.ls.ns, lane);
    CoefSink sink;
    // (to_planes = 0: only the compact copy, one value per block -- all a decode without AC scans and refinements reads)
    sink.init(to_planes ? L.base : nullptr, L.base_elems, L.ls.Al, R.dc + (uni((uint64_t)R.coef_off[un.img]) >> 6));
    return decode_dc_first(&wr, L.ls, &sink);
}

PCR_D void bring_ac_table(const DevRecord& R, size_t ig, AcTab* tab, uint32_t lane) {         // (built by k_headers)
    const uint4* src = reinterpret_cast<const uint4*>(&R.tabs[R.tab_idx[ig]]);
    uint4* dst = reinterpret_cast<uint4*>(tab);
    for (uint32_t e = lane; e < sizeof(AcTab) / 16; e += kEntropyLanes) dst[e] = src[e];
    wave_sync();
}
PCR_D HistPlanes hist_planes(const DevRecord& R, const Unit& un, const ScanDesc* sd, const UnitSetup& L) {
    // (the history is read through plain pointers: earlier scans may be writing it in this very launch)
    HistPlanes hp;
    hp.coef = L.plane[0];
    hp.n = sd->nhist;
#pragma unroll
    for (int q = 0; q < kMaxHist; q++) hp.p[q] = R.masks + uni((uint64_t)R.mask_off[(size_t)un.img * R.G + sd->hist[q < hp.n ? q : 0]]);
    hp.n = uni(hp.n);
    hp.some = hp.n > 0 ? ~0ull : 0ull;
    if (hp.n == 0) hp.p[0] = reinterpret_cast<const uint64_t*>(hp.coef);   // (16 bytes a block are read of its 128)
    return hp;
}
template <class Gate>
PCR_D int wave_ac(const DevRecord& R, const Unit& un, const UnitSetup& L, AcTab* tab, uint32_t lane, Gate& gate) {
    const size_t ig = (size_t)un.img * R.G + un.scan;
    const ScanDesc* sd = &R.scan[ig];
    bring_ac_table(R, ig, tab, lane);
    WindowReader wr;
    if (sd->Ah == 0) {
        wr.init(L.words, L.byte_off, L.sub_bits, L.nbits, L.pos0, tab, true, lane, reinterpret_cast<uint32_t*>(tab + 1));
        IndexSink sink;
        sink.init(L.plane[0], L.plane_elems[0], L.ls.Al);
        return decode_ac_first(&wr, L.ls, &sink, gate);
    }
    const HistPlanes hp = hist_planes(R, un, sd, L);
    wr.init(L.words, L.byte_off, L.sub_bits, L.nbits, L.pos0, tab, false, lane, reinterpret_cast<uint32_t*>(tab + 1));
    return skim_ac_refine(&wr, L.ls, hp, R.masks + uni((uint64_t)R.mask_off[ig]), L.plane_elems[0] >> 6, gate);
}

// One of the three wavefronts of a refinement unit (pcr_refine_trio.h).
constexpr uint32_t kTrioWalk = 0, kTrioFeed = 1, kTrioKeep = 2;
template <class Gate>
PCR_D __attribute__((always_inline)) void trio_unit(const DevRecord& R, const Unit& un, const UnitSetup& L, uint4* area, uint32_t part, uint32_t lane, Gate& gate) {
#if defined(__HIP_DEVICE_COMPILE__)
    const size_t ig = (size_t)un.img * R.G + un.scan;
    const ScanDesc* sd = &R.scan[ig];
    AcTab* tab = reinterpret_cast<AcTab*>(area);
    const TrioLds T = (TrioLds)(reinterpret_cast<uint8_t*>(area) + kWaveTabBytes);
    const uint32_t mis = (L.byte_off & 3) * 8, bits = L.nbits + mis, wb0 = L.pos0 - mis;
    const uint32_t* const words = L.words + (L.byte_off >> 2);
    if (part == kTrioFeed) {
        bring_ac_table(R, ig, tab, lane);
        trio_feed(T, tab, reinterpret_cast<uint32_t*>(tab + 1), words, bits, wb0, lane);
        return;
    }
    uint32_t bad;
    if (part == kTrioWalk) {
        bad = trio_walk(T, tab, words, bits, wb0, mis + L.sub_bits, L.ls.mcu1 - L.ls.mcu0, lane);
    } else {
        const HistPlanes hp = hist_planes(R, un, sd, L);
        bad = trio_keep(T, L.ls, hp, R.masks + uni((uint64_t)R.mask_off[ig]), L.plane_elems[0] >> 6, lane, gate);
    }
    if (bad) R.status[un.img] = kEFormat;
#endif
}

// Workgroup b: chain b of `chains`, or (without them) unit b of `units`, with a wavefront per unit.  Dynamic LDS:
// kWaveTabBytes per wavefront.  ROLES: which kinds of scans there may be among them (each kind on its own has
// more of the scalar registers: 26 are spilled for AC scans that follow, 107 with all kinds).  FOLLOW: some scan of the launch follows another one; without it the decoders carry nothing of
// the gate, which costs an AC first scan three per cent of its instructions (plain photographs, four records in flight at
// scan group 5, ms per step: 8.55 with, 7.95 without).
constexpr int kWavesDc = 1, kWavesAc = 2;
template <int ROLES, class Gate>
PCR_D __attribute__((always_inline)) void wave_unit(const DevRecord& R, const Unit& un, const UnitSetup& L, uint4* tabs, uint32_t lane, bool to_planes, Gate& gate) {
    const ScanDesc* sd = &R.scan[(size_t)un.img * R.G + un.scan];
    int rc = kEFormat;                                        // (a unit in the wrong launch: the descriptors disagree with the host's)
    if (uni((int)sd->Ss) > 0) { if (ROLES & kWavesAc) rc = wave_ac(R, un, L, reinterpret_cast<AcTab*>(tabs), lane, gate); }
    else if ((ROLES & kWavesDc) && uni((int)sd->Ah) == 0 && R.img[un.img].progressive) rc = wave_dc_first(R, un, L, reinterpret_cast<DcTab*>(tabs), lane, to_planes);
    if (rc != kOk) R.status[un.img] = rc;
}
template <int ROLES, bool FOLLOW>
__global__ void __launch_bounds__(kEntropyLanes * kChainWaves) k_decode_waves(DevRecord R, const Unit* __restrict__ units, const UnitChain* __restrict__ chains,
        const uint32_t* __restrict__ clean32, uint32_t to_planes, const uint32_t* __restrict__ had) {
    extern __shared__ uint4 wave_tabs[];
    __shared__ uint32_t done[kChainWaves];
    if (!FOLLOW && had && had[blockIdx.x]) return;            // (the many lanes of k_first_split have dealt with it)
    const uint32_t wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
    UnitChain ch{blockIdx.x, 1, 0, 0};
    if (chains) ch = chains[blockIdx.x];
    if (FOLLOW) {
        if (threadIdx.x < kChainWaves) done[threadIdx.x] = 0;
        __syncthreads();
    }
    if (wave >= ch.count) return;
    const Unit un = units[ch.first + wave];
    UnitSetup L;
    unit_setup(R, un, clean32, &L);
    if (FOLLOW) {
        ChainGate gate = chain_gate(ch, done, wave);
        if (L.ok) wave_unit<ROLES>(R, un, L, wave_tabs + wave * (kWaveTabBytes / 16), lane, to_planes != 0, gate);
        gate.publish(~0u);
    } else if (L.ok) { FreeRun gate; wave_unit<ROLES>(R, un, L, wave_tabs, lane, to_planes != 0, gate); }
}

// The same with three wavefronts for every unit of a refinement scan (pcr_refine_trio.h): wavefronts 0 .. count - 1 are those of
// k_decode_waves, behind them come the feeder and the keeper of the first refinement scan of the chain, of the second, and so on.  Without chains
// every unit is of a refinement scan.  Dynamic LDS: kWaveTabBytes per scan and sizeof(TrioRings) per refinement scan.  All wavefronts of a
// workgroup have to agree on whether there is anything to decode, so the image's status is read once.
constexpr uint32_t kTrioChainWaves = 16;
template <int ROLES, bool FOLLOW>
__global__ void __launch_bounds__(kEntropyLanes * kTrioChainWaves) k_decode_trios(DevRecord R, const Unit* __restrict__ units, const UnitChain* __restrict__ chains,
        const uint32_t* __restrict__ clean32, uint32_t to_planes, const uint32_t* __restrict__ had) {
    extern __shared__ uint4 wave_tabs[];
    __shared__ uint32_t done[kChainWaves];
    if (had && had[blockIdx.x]) return;                       // (the many lanes of k_first_split have dealt with it)
    const uint32_t wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
    UnitChain ch{blockIdx.x, 1, 1, 0};
    if (FOLLOW) ch = chains[blockIdx.x];
    const uint32_t count = ch.count, refines = ch.refines, trios = (uint32_t)__builtin_popcount(refines);
    uint32_t which = wave, part = kTrioWalk;                  // the scan, and the part of it if it is a refinement scan
    if (wave >= count) {
        uint32_t rest = refines;
        for (uint32_t j = (wave - count) >> 1; j && rest; j--) rest &= rest - 1;
        which = rest ? (uint32_t)__builtin_ctz(rest) : 0u;
        part = ((wave - count) & 1u) ? kTrioKeep : kTrioFeed;
    }
    auto area_of = [&](uint32_t scan) { return wave_tabs + (scan * kWaveTabBytes + (uint32_t)__builtin_popcount(refines & ((1u << scan) - 1u)) * (uint32_t)sizeof(TrioRings)) / 16; };
    if (FOLLOW && threadIdx.x < kChainWaves) done[threadIdx.x] = 0;
    if (wave < count && ((refines >> wave) & 1u) && lane < 8) {
        const TrioLds T = (TrioLds)(reinterpret_cast<uint8_t*>(area_of(wave)) + kWaveTabBytes);
        (&T->win_ready)[lane] = 0;
    }
    const Unit un = units[ch.first + which];
    const int status = group_status(R, un.img);               // (behind its barrier: the counters are zero)
    if (wave >= count + 2 * trios) return;
    UnitSetup L;
    unit_setup(R, un, clean32, &L, [&]() { return status == kOk; });
    uint4* const area = area_of(which);
    const bool refine = (refines >> which) & 1u;
    if (part == kTrioWalk) __builtin_amdgcn_s_setprio(1);
    if (FOLLOW) {
        ChainGate gate = chain_gate(ch, done, which);
        if (L.ok && refine) trio_unit(R, un, L, area, part, lane, gate);
        else if (L.ok) wave_unit<ROLES>(R, un, L, area, lane, to_planes != 0, gate);
        if (!refine || part == kTrioKeep) gate.publish(~0u);
    } else if (L.ok) { FreeRun gate; trio_unit(R, un, L, area, part, lane, gate); }
}

// The same scan kind with one LANE per unit (pcr_lanes.h).  One wavefront per job: up to 64 consecutive units of the
// launch's list that use at most kLaneTabs different Huffman tables between them (the host cuts the list that way; the
// units of one scan lie together).  The tables (built by k_headers) are copied into LDS first: every lane looks
// its codes up in its own table, and 64 scattered reads of memory per symbol would bound the kernel by the rate at
// which the memory pipeline takes requests.
PCR_D __attribute__((always_inline)) void ac_first_job(const DevRecord& R, const Unit* __restrict__ units, const LaneJob& job, const uint32_t* __restrict__ clean32,
        uint4 (*tabs)[kLaneTabPieces], LaneRing* rings) {
    const uint32_t t = threadIdx.x;
    const bool mine = t < job.count;
    const Unit un = units[job.first + (mine ? t : 0u)];
    const uint32_t key = un.img * R.G + un.scan;
    lane_tables_bring(R, job, un, tabs);
    const uint32_t slot = lane_table_slot(R, job, key);
    LaneUnit U;
    U.ok = false;
    if (mine && slot < (uint32_t)kLaneTabs) lane_unit_setup(R, un, clean32, &U);
    lane_tables_have();
    if (!U.ok) return;
    U.tab = reinterpret_cast<const LaneTab*>(&tabs[slot][0]);
    const int rc = lane_decode_ac_first(U, rings, t);
    if (rc != kOk) R.status[un.img] = rc;
}
__global__ void __launch_bounds__(kEntropyLanes) k_ac_first_lanes(DevRecord R, const Unit* __restrict__ units, const LaneJob* __restrict__ jobs,
        const uint32_t* __restrict__ clean32) {
    __shared__ uint4 tabs[kLaneTabs][kLaneTabPieces];
    __shared__ LaneRing rings;
    ac_first_job(R, units, jobs[blockIdx.x], clean32, tabs, &rings);
}

// AC refinement scans with one lane per unit: as k_ac_first_lanes.  k_refine_history must have run for the scans of the
// launch, k_refine_deal must follow.
__global__ void __launch_bounds__(kEntropyLanes) k_ac_refine_lanes(DevRecord R, const Unit* __restrict__ units, const LaneJob* __restrict__ jobs,
        const uint32_t* __restrict__ clean32) {
    __shared__ uint4 tabs[kLaneTabs][kLaneTabPieces];
    __shared__ LaneRing rings;
    __shared__ LaneHistRing hring;
    const LaneJob job = jobs[blockIdx.x];
    const uint32_t t = threadIdx.x;
    const bool mine = t < job.count;
    Unit un = units[job.first + (mine ? t : 0u)];
    const uint32_t key = un.img * R.G + un.scan;
    lane_tables_bring(R, job, un, tabs);
    const uint32_t slot = lane_table_slot(R, job, key);
    LaneUnit U;
    U.ok = false;
    if (mine && slot < (uint32_t)kLaneTabs) lane_unit_setup(R, un, clean32, &U);
    lane_tables_have();
    if (!U.ok) return;
    U.tab = reinterpret_cast<const LaneTab*>(&tabs[slot][0]);
    uint64_t* recs = R.masks + R.mask_off[key];
    const int rc = any_lane(lane_mostly_runs(U)) ? lane_decode_ac_refine<true>(U, recs, U.plane_elems >> 6, &rings, &hring, t)
                                                 : lane_decode_ac_refine<false>(U, recs, U.plane_elems >> 6, &rings, &hring, t);
    if (rc != kOk) R.status[un.img] = rc;
}

// DC first scans with one lane per unit (pcr_lanes.h: lane_decode_dc_first): 64 consecutive units of the launch's list
// per wavefront, whatever images they belong to -- every lane builds its own small tables.  The checks and ranges are
// those of unit_setup.
PCR_D __attribute__((always_inline)) void lane_dc_unit_setup(const DevRecord& R, const Unit& un, const uint32_t* __restrict__ clean32, uint32_t to_planes, LaneDcUnit* U) {
    LaneUnitInfo I;
    lane_unit_info(R, un, &I);
    U->ok = I.ok && I.Ss == 0 && I.Ah == 0 && PCR_FIELD(I.img, ImgDesc, progressive) != 0 && I.ns >= 1 && I.ns <= (uint32_t)kMaxComp;
    U->pred0 = (int)(int16_t)I.preds; U->pred1 = (int)(int16_t)(I.preds >> 16); U->pred2 = (int)(int16_t)(I.preds >> 32);
    U->mcu0 = I.m0; U->mcu1 = I.m1; U->bit0 = I.b0; U->bit1 = I.b1; U->mcu_w = I.mcu_w;
    U->ns = I.ns; U->Al = I.Al;
    const bool one = I.ns == 1;                                 // a scan of one component goes block by block
    // scan component j is component c of the image (sampling factors are 1 or 2: the parser refuses anything else)
    auto component = [&](uint32_t j, uint32_t comp, uint32_t dc_off, uint32_t* hs, uint32_t* vs, uint32_t* bw, uint32_t* pblk, const uint8_t** def) {
        const uint32_t c = j < I.ns ? comp : 0u;
        *hs = one ? 1u : I.hs(c); *vs = one ? 1u : I.vs(c); *bw = I.bw(c);
        *pblk = I.before(c);
        *def = R.rec + (j < I.ns ? dc_off : PCR_MEMBER(I.sd, ScanDesc, dc_off, 0));
    };
    component(0, PCR_MEMBER(I.sd, ScanDesc, comp, 0), PCR_MEMBER(I.sd, ScanDesc, dc_off, 0), &U->hs0, &U->vs0, &U->bw0, &U->pblk0, &U->def0);
    component(1, PCR_MEMBER(I.sd, ScanDesc, comp, 1), PCR_MEMBER(I.sd, ScanDesc, dc_off, 1), &U->hs1, &U->vs1, &U->bw1, &U->pblk1, &U->def1);
    component(2, PCR_MEMBER(I.sd, ScanDesc, comp, 2), PCR_MEMBER(I.sd, ScanDesc, dc_off, 2), &U->hs2, &U->vs2, &U->bw2, &U->pblk2, &U->def2);
    U->end = R.rec + R.nbytes;
    U->nblocks = I.nblk(0) + I.nblk(1) + I.nblk(2);
    U->dense = R.dc + (I.coef0 >> 6);
    U->planes = to_planes ? R.coef + I.coef0 : nullptr;
    U->words = clean32 + (clean_base(PCR_FIELD(I.sd, ScanDesc, data_off)) >> 2);
}

// Workgroup `block` of the lanes' DC decoders: units [starts[block], starts[block + 1]) of the launch, or sixty-four after
// sixty-four where there are no starts.
PCR_D __attribute__((always_inline)) void dc_first_units(const DevRecord& R, const Unit* __restrict__ units, uint32_t nunits, const uint32_t* __restrict__ starts, uint32_t block,
        const uint32_t* __restrict__ clean32, uint32_t to_planes, LaneRing* rings) {
    short_kernel_priority();
    const uint32_t t = threadIdx.x, u = (starts ? load_const(&starts[block]) : block * kEntropyLanes) + t;
    if (starts) nunits = load_const(&starts[block + 1]);
    const Unit un = units[u < nunits ? u : 0u];
    LaneDcUnit U;
    U.ok = false;
    if (u < nunits) lane_dc_unit_setup(R, un, clean32, to_planes, &U);
    if (!U.ok) return;
    const int rc = lane_decode_dc_first(U, rings, t);
    if (rc != kOk) R.status[un.img] = rc;
}
__global__ void __launch_bounds__(kEntropyLanes, 4) k_dc_first_lanes(DevRecord R, const Unit* __restrict__ units, uint32_t nunits,
        const uint32_t* __restrict__ starts, const uint32_t* __restrict__ clean32, uint32_t to_planes) {
    __shared__ LaneRing rings;
    dc_first_units(R, units, nunits, starts, blockIdx.x, clean32, to_planes, &rings);
}
// DC and AC first scans of one level in one launch: the first dc_blocks workgroups are k_dc_first_lanes', the others
// k_ac_first_lanes'.  Both take as long as their longest unit and leave most of the chip idle meanwhile; one behind the
// other they took the sum: 1024 x 256 x 256 at scan group 5 62 us for the DC scans by wavefronts + 82, 1024 photographs
// at 2 136 + 108.  (Kept on their own where stages are timed, and for calls with only one of the two.)
__global__ void __launch_bounds__(kEntropyLanes, 4) k_first_lanes(DevRecord R, const Unit* __restrict__ dc_units, uint32_t n_dc, const uint32_t* __restrict__ dc_starts, uint32_t dc_blocks,
        const Unit* __restrict__ ac_units, const LaneJob* __restrict__ jobs, const uint32_t* __restrict__ clean32, uint32_t to_planes) {
    __shared__ uint4 tabs[kLaneTabs][kLaneTabPieces];
    __shared__ LaneRing rings;
    if (blockIdx.x < dc_blocks) dc_first_units(R, dc_units, n_dc, dc_starts, blockIdx.x, clean32, to_planes, &rings);
    else ac_first_job(R, ac_units, jobs[blockIdx.x - dc_blocks], clean32, tabs, &rings);
}

// Sequential (baseline) scans: the DC and AC tables of every scan component, once per distinct table.  done: which of the
// first n_done units the lanes have dealt with (k_split_settle).
__global__ void __launch_bounds__(kEntropyLanes) k_sequential(DevRecord R, const Unit* __restrict__ units, const uint32_t* __restrict__ done, uint32_t n_done,
        const uint32_t* __restrict__ clean32) {
    __shared__ uint32_t stage_[1 + kStageWords];            // (a word is read ahead of it)
    uint32_t* stage = stage_ + 1;
    __shared__ DcTab dtabs[kMaxComp];
    __shared__ AcTab atabs[kMaxComp];
    if (blockIdx.x < n_done && done[blockIdx.x]) return;
    const Unit un = units[blockIdx.x];
    UnitSetup L;
    unit_setup(R, un, clean32, &L);
    if (!L.ok) return;
    const ScanDesc* sd = &R.scan[(size_t)un.img * R.G + un.scan];
    if (!is_sequential_scan(*sd)) { R.status[un.img] = kEFormat; return; }      // (a unit in the wrong launch)
    const uint32_t d0 = sd->dc_off[0], d1 = L.ls.ns > 1 ? sd->dc_off[1] : d0, d2 = L.ls.ns > 2 ? sd->dc_off[2] : d0;
    const uint32_t a0 = sd->ac_offc[0], a1 = L.ls.ns > 1 ? sd->ac_offc[1] : a0, a2 = L.ls.ns > 2 ? sd->ac_offc[2] : a0;
    int dj1 = 0, dj2 = 0, nd = 1, aj1 = 0, aj2 = 0, na = 1;
    if (d1 != d0) { dj1 = 1; nd = 2; }
    if (d2 == d1) dj2 = dj1; else if (d2 != d0) { dj2 = nd; nd++; }
    if (a1 != a0) { aj1 = 1; na = 2; }
    if (a2 == a1) aj2 = aj1; else if (a2 != a0) { aj2 = na; na++; }
    if (threadIdx.x == 0) { dctab_build(&dtabs[0], R.rec + d0); actab_build(&atabs[0], R.rec + a0); }
    if (threadIdx.x == 1) {
        if (dj1 == 1) dctab_build(&dtabs[1], R.rec + d1);
        if (aj1 == 1) actab_build(&atabs[1], R.rec + a1);
    }
    if (threadIdx.x == 2) {
        if (dj2 != 0 && dj2 != dj1) dctab_build(&dtabs[dj2], R.rec + d2);
        if (aj2 != 0 && aj2 != aj1) actab_build(&atabs[aj2], R.rec + a2);
    }
    __syncthreads();
    for (int t = 0; t < na; t++) actab_pack(&atabs[t], true, threadIdx.x, kEntropyLanes);
    __syncthreads();
    SeqTables tb;
    tb.dc[0] = &dtabs[0]; tb.dc[1] = &dtabs[uni(dj1)]; tb.dc[2] = &dtabs[uni(dj2)];
    tb.ac[0] = &atabs[0]; tb.ac[1] = &atabs[uni(aj1)]; tb.ac[2] = &atabs[uni(aj2)];
    WindowReader wr;
    wr.init(L.words, L.byte_off, L.sub_bits, L.nbits, L.pos0, tb.ac[0], true, threadIdx.x, stage);
    IndexSink sink;
    sink.init(L.base, L.base_elems, 0, R.dc + (uni((uint64_t)R.coef_off[un.img]) >> 6));
    const int rc = decode_sequential(&wr, L.ls, tb, &sink);
    if (rc != kOk) R.status[un.img] = rc;
}


// Phase 2 of AC refinement: one lane per block of the scan.
struct RefineScan { uint32_t img; uint32_t scan; };
// The per-block helpers of the lane decoders take their work from a list instead: chunk `chunk` (256 blocks) of scan
// `entry` of the launch's RefineScan list -- the planes of a record differ in size by an order of magnitude (luma and
// chroma, small and large images), and a grid sized for the largest would be mostly workgroups that find nothing to do.
struct RefineTile { uint32_t entry; uint32_t chunk; };

// What the lane-per-unit refinement decoder needs before and after it, one lane per block of the scan (the grid of
// k_refine_blocks).  k_refine_history: the kRefHist word of every block -- which positions of the band are non-zero
// when the scan starts: what the AC first scans left in the coefficient plane, and what earlier refinement scans of the
// band added (their kRefNz words).  k_refine_deal: the correction bits the decoder left in reading order go to the
// history positions they belong to (kRefPlus as every consumer reads it).
// Where the work of a tile lies: its entry, then everything that depends on the image and the scan alone in ONE round of scalar
// loads.  (Read where it was used, each member behind the branch before it, a workgroup waited five times in a row before
// its first word of the records.  1024 photographs, four records in flight, and 256 of 600 x 450, us per launch: k_refine_history 177 ->
// 137 and 59 -> 52, k_refine_deal 73 -> 69 and 22 -> 21.)
struct RefinePlace {
    ImgDesc D; ScanDesc S;
    uint32_t img, chunk, status, tab, slot, cw, ncov, bw, plane;
    size_t ig;
    uint64_t mask, coef;
};
PCR_D void refine_place(const DevRecord& R, const RefineScan* rs, const RefineTile* tiles, RefinePlace* P) {
    const uint64_t tile = load_const(reinterpret_cast<const uint64_t*>(tiles) + blockIdx.x);
    const uint64_t a = load_const(reinterpret_cast<const uint64_t*>(rs) + (uint32_t)tile);
    P->chunk = (uint32_t)(tile >> 32);
    P->img = (uint32_t)a;
    P->ig = (size_t)P->img * R.G + (uint32_t)(a >> 32);
    load_desc(R.img + P->img, &P->D);
    load_desc(R.scan + P->ig, &P->S);
    P->status = (uint32_t)load_const(&R.status[P->img]);
    P->tab = load_const(&R.tab_idx[P->ig]);
    P->slot = load_const(&R.slot_base[P->ig]);
    P->mask = load_const(&R.mask_off[P->ig]);
    P->coef = load_const(&R.coef_off[P->img]);
    wanted_now(P->D); wanted_now(P->S); wanted_now(P->status); wanted_now(P->tab); wanted_now(P->slot); wanted_now(P->mask); wanted_now(P->coef);
    const uint32_t c = P->S.comp[0];
    P->cw = pick3(c, P->D.cw[0], P->D.cw[1], P->D.cw[2]);
    P->ncov = P->cw * pick3(c, P->D.ch[0], P->D.ch[1], P->D.ch[2]);
    P->bw = pick3(c, P->D.bw[0], P->D.bw[1], P->D.bw[2]);
    P->plane = P->bw * pick3(c, P->D.bh[0], P->D.bh[1], P->D.bh[2]);
}
static_assert(sizeof(RefineTile) == 8 && offsetof(RefineTile, entry) == 0 && sizeof(RefineScan) == 8 && offsetof(RefineScan, img) == 0, "taken as 64-bit words");
// k_refine_history works through the padded plane (blocks the image does not cover included: they hold zeros), 64
// consecutive blocks -- 8 KB of coefficients -- per wavefront: lane i of step j loads 16-byte chunk 64 j + i of them, so
// that every load instruction reads one contiguous kilobyte, turns its eight coefficients into eight mask bits, and leaves
// the byte in LDS where the lane that owns the block picks up all eight.  grid: one workgroup per tile (chunks of the padded planes).
__global__ void __launch_bounds__(256) k_refine_history(DevRecord R, const RefineScan* __restrict__ rs, const RefineTile* __restrict__ tiles) {
    __shared__ __attribute__((aligned(8))) uint8_t bytes[4][64 * 8];
    short_kernel_priority();
    RefinePlace P;
    refine_place(R, rs, tiles, &P);
    if (P.status != (uint32_t)kOk || P.chunk * 256 >= P.plane) return;
    const uint32_t plane = P.plane, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t blk0 = P.chunk * 256 + wave * 64, blk = blk0 + lane;
    const uint32_t nhist = P.S.nhist < kMaxHist ? P.S.nhist : kMaxHist;
    uint64_t from[kMaxHist];                                  // the records of the scans this one builds on
    uint32_t band0;                                           // first and last position of the first of them
    {
        const size_t i0 = (size_t)P.img * R.G;
#pragma unroll
        for (uint32_t q = 0; q < (uint32_t)kMaxHist; q++) from[q] = load_const(&R.mask_off[i0 + (q < nhist ? P.S.hist[q] : 0u)]);
        static_assert(offsetof(ScanDesc, Ss) % 4 == 2 && offsetof(ScanDesc, Se) == offsetof(ScanDesc, Ss) + 1, "the upper half of a word");
        band0 = load_const(reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(&R.scan[i0 + (nhist ? P.S.hist[0] : 0u)]) + (offsetof(ScanDesc, Ss) & ~3u))) >> 16;
#pragma unroll
        for (uint32_t q = 0; q < (uint32_t)kMaxHist; q++) wanted_now(from[q]);
        wanted_now(band0);
    }
    uint64_t m = 0;
    // An earlier refinement scan of the very same band has this word already: what it started from and what it added
    // are what this scan starts from (16 bytes per block instead of the block's 128 bytes of coefficients).
    const bool from_records = nhist && band0 == (P.S.Ss | ((uint32_t)P.S.Se << 8));
    if (from_records) {
        if (blk < plane) m = R.masks[from[0] + ref_word(kRefHist, blk, plane)];
    } else {
        const uint32_t c = P.S.comp[0], n0 = (uint32_t)P.D.bw[0] * P.D.bh[0], n1 = (uint32_t)P.D.bw[1] * P.D.bh[1];
        const size_t po = (size_t)(c > 0 ? n0 : 0u) * 64 + (size_t)(c > 1 ? n1 : 0u) * 64;
        const uint4* src = reinterpret_cast<const uint4*>(R.coef + P.coef + po) + (size_t)blk0 * 8;
        const uint32_t chunk = lane & 7u;                     // (the same in every step: 64 is a multiple of 8)
        const bool wanted = chunk >= (uint32_t)(P.S.Ss >> 3) && chunk <= (uint32_t)(P.S.Se >> 3);
#pragma unroll
        for (uint32_t j = 0; j < 8; j++) {
            const uint32_t e = j * 64 + lane;                 // chunk e & 7 of block blk0 + (e >> 3)
            uint32_t bits = 0;
            if (wanted && blk0 + (e >> 3) < plane) {
                const uint4 v = src[e];
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (uint32_t q = 0; q < 4; q++) bits |= ((w[q] & 0xFFFFu) ? 1u : 0u) << (2 * q) | ((w[q] >> 16) ? 2u : 0u) << (2 * q);
            }
            bytes[wave][e] = (uint8_t)bits;
        }
    }
    __syncthreads();
    if (blk >= plane) return;
    if (!from_records) m = *reinterpret_cast<const uint64_t*>(&bytes[wave][lane * 8]);
#pragma unroll
    for (uint32_t q = 0; q < (uint32_t)kMaxHist; q++) if (q < nhist) m |= R.masks[from[q] + ref_word(kRefNz, blk, plane)];
    R.masks[P.mask + ref_word(kRefHist, blk, plane)] = m & band_mask(P.S.Ss, P.S.Se);
}
// grid: one workgroup per tile (chunks of the blocks the image covers)
__global__ void __launch_bounds__(256) k_refine_deal(DevRecord R, const RefineScan* __restrict__ rs, const RefineTile* __restrict__ tiles) {
    short_kernel_priority();
    RefinePlace P;
    refine_place(R, rs, tiles, &P);
    const uint32_t b = P.chunk * 256 + threadIdx.x, plane = P.plane;
    if (P.status != (uint32_t)kOk || b >= P.ncov) return;
    const uint32_t blk = (b / P.cw) * P.bw + (b % P.cw);
    uint64_t* rec = R.masks + P.mask;
    rec[ref_word(kRefPlus, blk, plane)] = deal_bits(rec[ref_word(kRefPlus, blk, plane)], rec[ref_word(kRefHist, blk, plane)]);
}

__global__ void __launch_bounds__(256) k_refine_blocks(DevRecord R, const RefineScan* __restrict__ rs, const RefineTile* __restrict__ tiles) {
    __shared__ __attribute__((aligned(16))) AcTab tab;
    short_kernel_priority();
    RefinePlace P;
    refine_place(R, rs, tiles, &P);
    if (P.status != (uint32_t)kOk || P.chunk * 256 >= P.ncov) return;
    const uint32_t b = P.chunk * 256 + threadIdx.x, at = b < P.ncov ? b : P.ncov - 1;
    const size_t blk = (size_t)(at / P.cw) * P.bw + (at % P.cw), plane = P.plane;
    uint64_t* rec = R.masks + P.mask;
    // (the block's words and its unit's start are on their way while the table is)
    const uint64_t h = rec[ref_word(kRefHist, blk, plane)], st = rec[ref_word(kRefStart, blk, plane)], newm = rec[ref_word(kRefNz, blk, plane)];   // (h: the history phase 1 worked on)
    const uint32_t start = R.ivl_start[P.slot + (P.S.ri ? at / P.S.ri : 0)];
    {
        constexpr uint32_t kPieces = offsetof(AcTab, lutp) / 16;                     // (what ac_code reads)
        const uint4* src = reinterpret_cast<const uint4*>(&R.tabs[P.tab]);
        if (threadIdx.x < kPieces) reinterpret_cast<uint4*>(&tab)[threadIdx.x] = src[threadIdx.x];
    }
    arrived(h); arrived(st); arrived(newm); arrived(start);
    __syncthreads();
    if (b >= P.ncov) return;
    const uint32_t* words = reinterpret_cast<const uint32_t*>(R.clean + clean_base(P.S.data_off));
    uint64_t sgn, plus;
    refine_block(words, start, st, &tab, h, newm, P.S.Ss, P.S.Se, &sgn, &plus);
    rec[ref_word(kRefSign, blk, plane)] = sgn; rec[ref_word(kRefPlus, blk, plane)] = plus;
}

// --------------------------------------------------------------------------------------
// Refinement, data-parallel.  One lane per coefficient of every block of a component
// (natural order within the block, so loads and stores are contiguous).
//   k = 0: DC refinement scans -- the block's bit sits at a position fixed by the scan's block
//          order (and restart intervals), so it is simply fetched and OR-ed in;
//   k > 0: replay the AC scans of the component in file order: first scans only extend the
//          non-zero mask, refinement scans add a correction bit or place a new +-2^Al.
// --------------------------------------------------------------------------------------
// apply_prep (in the unstuffing launch) has gathered, per (image, component), the scans that matter for refinement; k_apply then
// runs one lane per coefficient, a workgroup covering kApplyChunk consecutive coefficients.
constexpr uint32_t kApplyChunk = 4096;

// DC refinement of the block at (row, col) of a component with sampling hs x vs: the block's bit sits at
// a position fixed by the scan's block order and restart intervals; returns the bit (0 / 1), 0 for a block
// a non-interleaved scan does not visit.
PCR_D uint32_t dc_refinement_bit(const DevRecord& R, const ApplyScan& S, uint32_t row, uint32_t col, uint32_t hs, uint32_t vs, bool covered) {
    uint32_t m, within;
    if (S.ns > 1) { m = (row >> (vs - 1)) * S.mcu_w + (col >> (hs - 1)); within = S.before + (row & (vs - 1)) * hs + (col & (hs - 1)); }   // (sampling factors are 1 or 2)
    else { if (!covered) return 0; m = row * S.mcu_w + col; within = 0; }
    const uint32_t ivl = S.ri ? m / S.ri : 0;
    const uint32_t bit = (m - ivl * S.ri) * S.bpm + within;
    const uint32_t* words = reinterpret_cast<const uint32_t*>(R.clean + S.data_base);
    return (uint32_t)dc_refine_bit(words, R.ivl_start[S.slot + ivl], bit);
}

__global__ void __launch_bounds__(256) k_apply(DevRecord R, const ApplyUnit* __restrict__ au, const ApplyList* __restrict__ lists) {
    __shared__ ApplyList L;
    const ApplyUnit a = au[blockIdx.y];
    const ImgDesc* img = &R.img[a.img];
    if (R.status[a.img] != kOk) return;
    const int c = a.comp;
    const uint32_t bw = img->bw[c], nblk = bw * img->bh[c];
    const uint32_t first = blockIdx.x * kApplyChunk;
    if (first >= nblk * 64) return;
    {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(&lists[blockIdx.y]);
        uint32_t* dst = reinterpret_cast<uint32_t*>(&L);
        for (uint32_t e = threadIdx.x; e < sizeof(ApplyList) / 4; e += 256) dst[e] = src[e];
    }
    __syncthreads();
    const uint32_t n = L.n;
    const uint32_t cw = img->cw[c], ch = img->ch[c], hs = img->hs[c], vs = img->vs[c];
    const size_t plane = nblk;
    int16_t* pl = R.coef + R.coef_off[a.img];
    for (int q = 0; q < c; q++) pl += (size_t)img->bw[q] * img->bh[q] * 64;
    for (uint32_t idx = first + threadIdx.x; idx < first + kApplyChunk && idx < nblk * 64; idx += 256) {
        const uint32_t b = idx >> 6; const int k = (int)(idx & 63);  // element k of a block = zig-zag position k
        const uint32_t row = b / bw, col = b % bw;
        const bool covered = row < ch && col < cw;
        const int16_t v0 = pl[idx];
        int16_t v = v0;
        for (uint32_t e = 0; e < n; e++) {
            const ApplyScan& S = L.sc[e];
            if (S.Ss == 0) {
                if (k != 0) continue;
                if (dc_refinement_bit(R, S, row, col, hs, vs, covered)) v |= (int16_t)(1 << S.Al);
            } else if (k != 0 && covered && k >= S.Ss && k <= S.Se) {
                const uint64_t* rec = R.masks + S.mask_off;
                v = refine_apply(v, k, rec[ref_word(kRefNz, b, nblk)], rec[ref_word(kRefSign, b, nblk)], rec[ref_word(kRefPlus, b, nblk)], S.Al);
            }
        }
        if (v != v0) pl[idx] = v;
    }
}

// Parity hook: internal planes (zig-zag order inside each block) -> natural order.
__global__ void __launch_bounds__(256) k_export_natural(const int16_t* in, int16_t* out, size_t n) {
    __shared__ uint8_t zz[64];
    if (threadIdx.x < 64) zz[threadIdx.x] = (uint8_t)zigzag_lookup(threadIdx.x);
    __syncthreads();
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * 256;
    for (; i < n; i += stride) out[(i & ~(size_t)63) + zz[i & 63]] = in[i];
}

// --------------------------------------------------------------------------------------
// k_crop_resize: the training tail.  For every image one box of the decoded pixels is resized to
// out_h x out_w with bilinear interpolation on pixel centres (no anti-aliasing; samples beyond the
// box's edge repeat the edge), optionally mirrored left to right, normalised per channel and written
// as half precision, channel-planar: out[((i * C + c) * out_h + oy) * out_w + ox].
// One lane per output sample position (all channels); a workgroup covers 32 columns of 8 rows (the usual
// training sizes are multiples of 32), so a wavefront stores two runs of 64 contiguous bytes per channel.
// grid (ceil(out_w / 32), ceil(out_h / 8), n).  A box that does not lie inside its image is clamped into it.
// dims: width and height per image and out_off: byte offset of every image in `in`, both as laid down when the
// record was opened (the descriptors in device memory are only filled by a decode call).
// --------------------------------------------------------------------------------------
struct CropBox { int32_t x0, y0, w, h, flip; };

// floor(num / den) and the remainder in [0, den), den > 0, |num| < 2^31: the quotient is guessed in single
// precision (off by one at most for the quotients that occur, below 2^17) and put right with the remainder
PCR_D void floor_div(int num, int den, float inv_den, int* q, int* r) {
    int g = (int)floorf((float)num * inv_den);
    int rem = num - g * den;
    if (rem < 0) { g--; rem += den; }
    if (rem >= den) { g++; rem -= den; }
    *q = g; *r = rem;
}

// Where output sample (oy, ox) of a resize looks: the two source rows and columns (absolute, the box's edge samples
// repeated) and the weights of the second (f) and the first (g) of them.
// (f is the remainder times the rounded reciprocal of 2 * out size, g one minus that product, rounded once: their sum can miss one by a
// last place.  Both are made here, so that every kernel that interpolates gives the very same bits however it hands them on.)
struct TailTap { int a, b; float f, g; };
PCR_D TailTap tail_tap(int o, int out, int first, int size) {
    const int d = 2 * out;
    const float inv = 1.0f / (float)d;
    int l, r;
    floor_div((2 * o + 1) * size - out, d, inv, &l, &r);
    TailTap t;
    t.f = __fmul_rn((float)r, inv); t.g = __builtin_fmaf(-(float)r, inv, 1.0f);
    t.a = first + min(max(l, 0), size - 1); t.b = first + min(max(l + 1, 0), size - 1);
    return t;
}
PCR_D TailTap tail_row(const CropBox& b, int oy, int out_h) { return tail_tap(oy, out_h, b.y0, b.h); }
PCR_D TailTap tail_col(const CropBox& b, int ox, int out_w) { return tail_tap(b.flip ? out_w - 1 - ox : ox, out_w, b.x0, b.w); }
// A box as the tail uses it: clamped into its W x H image.
PCR_D CropBox clamp_box(CropBox b, int W, int H) {
    b.x0 = min(max(b.x0, 0), W - 1); b.y0 = min(max(b.y0, 0), H - 1);
    b.w = min(max(b.w, 1), W - b.x0); b.h = min(max(b.h, 1), H - b.y0);
    return b;
}
// One channel of one output sample from its four source values (whole numbers 0..255; y, x: its row's and its column's weights),
// normalised, as half precision.  The operations are spelled out one by one, so that every kernel that interpolates gives the
// very same bits.
PCR_D __half tail_value(float aa, float ab, float ba, float bb, const TailTap& x, const TailTap& y, float mean, float istd) {
    const float top = __fmaf_rn(x.f, ab, __fmul_rn(x.g, aa));
    const float bot = __fmaf_rn(x.f, bb, __fmul_rn(x.g, ba));
    const float v = __fmaf_rn(y.f, bot, __fmul_rn(y.g, top));
    return __float2half_rn(__fmul_rn(__fsub_rn(__fmul_rn(v, 1.0f / 255.0f), mean), istd));
}

__global__ void __launch_bounds__(256) k_crop_resize(const uint32_t* __restrict__ dims, const uint64_t* __restrict__ out_off,
        const uint8_t* __restrict__ in, const CropBox* __restrict__ boxes,
        int out_h, int out_w, int C, float m0, float m1, float m2, float s0, float s1, float s2, __half* __restrict__ out) {
    const uint32_t i = blockIdx.z;
    const int ox = (int)(blockIdx.x * 32 + (threadIdx.x & 31)), oy = (int)(blockIdx.y * 8 + (threadIdx.x >> 5));
    if (ox >= out_w || oy >= out_h) return;
    const int W = (int)dims[2 * i], H = (int)dims[2 * i + 1];
    if (W < 1 || H < 1) return;
    const CropBox b = clamp_box(boxes[i], W, H);
    // source point relative to the box, as an exact fraction: ((2 o + 1) * size - out) / (2 * out) pixels
    const TailTap y = tail_row(b, oy, out_h), x = tail_col(b, ox, out_w);
    const uint8_t* img = in + out_off[i];
    const uint8_t* paa = img + ((size_t)y.a * W + x.a) * C; const uint8_t* pab = img + ((size_t)y.a * W + x.b) * C;
    const uint8_t* pba = img + ((size_t)y.b * W + x.a) * C; const uint8_t* pbb = img + ((size_t)y.b * W + x.b) * C;
    const float mean[3] = {m0, m1, m2}, istd[3] = {s0, s1, s2};
    __half* dst = out + ((size_t)i * C * out_h + oy) * out_w + ox;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        if (c < C) dst[(size_t)c * out_h * out_w] = tail_value((float)paa[c], (float)pab[c], (float)pba[c], (float)pbb[c], x, y, mean[c], istd[c]);
    }
}

// --------------------------------------------------------------------------------------
// k_pixel: one workgroup per run of consecutive MCUs of one image (raster order over its MCU grid, across the
// ends of MCU rows), ONE LANE PER 8x8 BLOCK.
//   phase A  the lane loads its block's 64 coefficients (eight 16-byte loads; chunks that no scan <= k can have
//            touched are not read), replays the component's refinement scans on them, de-quantises, and runs the
//            whole 8x8 inverse DCT in registers: zig-zag order becomes register naming, the row and the column
//            pass need no exchange between lanes, no LDS and no barrier.  The constant factors of the transform
//            (1/2 per pass, cos(pi/4) on terms 0 and 4) are folded into the de-quantisation table.  The clamped
//            samples stay in the lane's registers.
//   phase B  twice, for the upper and for the lower half of the pixel rows of the MCUs: the lanes put the part of
//            their block that lies in the half into LDS, MCU by MCU (per MCU the rows of each component as one small
//            row-major plane; a component that only has its DC writes one sample per block: the block is flat);
//            then chroma replication + colour + one rounding + store: one lane per group of 12 output bytes (4 RGB
//            pixels; 8 gray ones) of two pixel rows of one MCU, lanes ordered along the image rows, the samples
//            read from LDS as 16- and 8-byte vectors, each row written with one (possibly unaligned) store.
// Two pixel rows per lane in phase B (indices, and with 4:2:0 the chroma samples, fetched once for both) took 1024
// photographs from 361 to 288 us (scan group 2) and from 527 to 463 (scan group 10: 0.93 GB of coefficients, masks and
// pixels, 2.0 TB/s; the rest is vector issue).  Folding the half of the rounding into luma and centring the samples
// before the transform saves another 5 %, but moves pixels whose value lies on the edge of rounding (2 in 100 000).
// The kernel is bound by memory latency times occupancy, not by arithmetic.  Occupancy is bounded by LDS, which is
// why the samples go through it in halves (128 bytes per lane at a time: four wavefronts per SIMD instead of two,
// measured a third faster); and the chain of dependent trips to memory is kept short: the image's descriptor is read
// with scalar loads (no copy through LDS, no barrier), and the coefficient loads are issued before the tables of the
// prologue are built.  (A decode without any AC scan goes
// through k_pixel_flat instead.)
// The refinement is applied here, on the way in: the coefficient planes hold what the first scans wrote, and the
// lane replays the component's refinement scans from the records the refinement kernels left (exactly what k_apply
// does for the coefficient export, the only caller that needs the refined values in memory).  lists / list_idx:
// the per-(image, component) scan lists of apply_prep and their index by image * 3 + component (-1: nothing to
// refine); both null if no scan <= k refines.  kRefine = false compiles the replay out.
// boxes (optional): one box per image; runs of MCUs that do not touch their image's box are skipped altogether
// (their pixels are left as they are): for callers that go on to read only the boxes (pcr_decode_crop_batch).
// --------------------------------------------------------------------------------------
constexpr int kPixLanes = 128;             // blocks per workgroup (the samples of half a run take kPixLanes * 128 bytes of LDS)

struct PixelTile { uint32_t img; uint32_t mcu0; };          // first MCU of the run
typedef short short2v __attribute__((ext_vector_type(2)));
typedef short short8 __attribute__((ext_vector_type(8)));

// w / d as (w * recip16(d)) >> 16, exact while w * d < 65536
PCR_HD uint32_t recip16(uint32_t d) { return d ? 65536u / d + 1u : 0u; }

PCR_HD uint32_t blocks_per_mcu(const ImgDesc& d) {
    uint32_t b = 0;
    for (int c = 0; c < d.nc; c++) b += (uint32_t)d.hs[c] * d.vs[c];
    return b;
}
// Samples of an MCU in LDS: 32 per block for half of its pixel rows, and some that stay empty.  A wavefront converts a
// pixel row of several MCUs at a time, each lane sixteen bytes of it; with nothing between the MCUs their rows lie a
// multiple of 256 bytes apart, on the same banks.  groups: lanes per pixel row of an MCU.
PCR_HD uint32_t pixel_mcu_samples(uint32_t bpm, uint32_t groups) { return bpm * 32 + 4 * groups; }
PCR_HD uint32_t pixel_row_groups(uint32_t nc, uint32_t hmax) { return 8 * hmax / (nc == 1 ? 8u : 4u); }
constexpr uint32_t kPixSamples = 4368;     // what a workgroup holds: 21 MCUs of 4:2:0, 42 of 4:4:4, 121 gray ones (eight workgroups to a compute unit)
PCR_HD uint32_t pixel_mcus(uint32_t bpm, uint32_t groups) {
    const uint32_t by_lanes = (uint32_t)kPixLanes / bpm, by_lds = kPixSamples / pixel_mcu_samples(bpm, groups);
    return by_lanes < by_lds ? by_lanes : by_lds;
}
PCR_HD uint32_t pixel_mcus_per_tile(const ImgDesc& d) { return pixel_mcus(blocks_per_mcu(d), pixel_row_groups(d.nc, d.hmax)); }   // >= 10: an MCU has at most 12 blocks

// 8-point inverse transform with the constant factors taken out: in[u] must already carry the 1/2 of the pass and,
// for u = 0 and 4, cos(pi/4).  out[x] = sum_u in'[u] cos((2x+1) u pi / 16).
PCR_D void idct8_scaled(float& x0, float& x1, float& x2, float& x3, float& x4, float& x5, float& x6, float& x7) {
    const float c1 = 0.98078528040323044913f, c2 = 0.92387953251128675613f, c3 = 0.83146961230254523708f,
                c5 = 0.55557023301960222474f, c6 = 0.38268343236508977173f, c7 = 0.19509032201612826785f;
    const float a = x0 + x4, b = x0 - x4;
    const float p = x2 * c2 + x6 * c6, q = x2 * c6 - x6 * c2;
    const float e0 = a + p, e1 = b + q, e2 = b - q, e3 = a - p;
    const float o0 = x1 * c1 + x3 * c3 + x5 * c5 + x7 * c7;
    const float o1 = x1 * c3 - x3 * c7 - x5 * c1 - x7 * c5;
    const float o2 = x1 * c5 - x3 * c1 + x5 * c7 + x7 * c3;
    const float o3 = x1 * c7 - x3 * c5 + x5 * c3 - x7 * c1;
    x0 = e0 + o0; x7 = e0 - o0; x1 = e1 + o1; x6 = e1 - o1;
    x2 = e2 + o2; x5 = e2 - o2; x3 = e3 + o3; x4 = e3 - o3;
}
// The factor folded into the quantiser step of zig-zag position k: 1/2 per pass, cos(pi/4) for row or column 0 and 4.
// Bit k of the words: positions with row and column 0 or 4, and those with one of them.
struct PixFolds {
    uint64_t both, once;
    constexpr PixFolds() : both(0), once(0) {
        for (int k = 0; k < 64; k++) {
            const uint32_t p = (uint32_t)zigzag_natural(k), u = p & 7, v = p >> 3;
            const bool a = (u & 3) == 0, b = (v & 3) == 0;
            if (a && b) both |= 1ull << k; else if (a || b) once |= 1ull << k;
        }
    }
};

// byte `which` of `word` := v rounded half up and clamped to [0, 255] (v is finite); the other bytes are kept.
// (The conversion instruction saturates and is exact on integers, which floor(v + 1/2) is.)
PCR_D uint32_t put_u8(float v, uint32_t which, uint32_t word) {
    return __builtin_amdgcn_cvt_pk_u8_f32(__builtin_floorf(v + 0.5f), which, word);
}

// Four values rounded half up and clamped to [0, 255], as bytes.  The conversion instruction rounds as the mode register
// says; turned to downwards for it (and back to nearest behind it) it saves every byte its floor.
#define PCR_ROUND_DOWN "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 2\n\t"
#define PCR_ROUND_NEAREST "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0"
PCR_D uint32_t four_u8(float a, float b, float c, float d) {
    uint32_t w;
    asm(PCR_ROUND_DOWN
        "v_cvt_pk_u8_f32 %0, %1, 0, 0\n\tv_cvt_pk_u8_f32 %0, %2, 1, %0\n\tv_cvt_pk_u8_f32 %0, %3, 2, %0\n\tv_cvt_pk_u8_f32 %0, %4, 3, %0\n\t"
        PCR_ROUND_NEAREST : "=&v"(w) : "v"(a + 0.5f), "v"(b + 0.5f), "v"(c + 0.5f), "v"(d + 0.5f));
    return w;
}
// The colour conversion of all pixel kernels (the same instructions everywhere, so that the pixels do not depend on which
// kernel wrote them): luma y, chroma u, v around zero.
PCR_D void to_rgb(float y, float u, float v, float* r, float* g, float* b) {
    *r = __builtin_fmaf(1.402f, v, y);
    *g = __builtin_fmaf(-0.714136f, v, __builtin_fmaf(-0.344136f, u, y));
    *b = __builtin_fmaf(1.772f, u, y);
}
// the twelve bytes of four pixels
PCR_D void rgb_words(const float y[4], const float u[4], const float v[4], uint32_t w[3]) {
    float r[4], g[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; i++) { to_rgb(y[i], u[i], v[i], &r[i], &g[i], &b[i]); r[i] += 0.5f; g[i] += 0.5f; b[i] += 0.5f; }
    asm(PCR_ROUND_DOWN
        "v_cvt_pk_u8_f32 %0, %3, 0, 0\n\tv_cvt_pk_u8_f32 %1, %7, 0, 0\n\tv_cvt_pk_u8_f32 %2, %11, 0, 0\n\t"
        "v_cvt_pk_u8_f32 %0, %4, 1, %0\n\tv_cvt_pk_u8_f32 %1, %8, 1, %1\n\tv_cvt_pk_u8_f32 %2, %12, 1, %2\n\t"
        "v_cvt_pk_u8_f32 %0, %5, 2, %0\n\tv_cvt_pk_u8_f32 %1, %9, 2, %1\n\tv_cvt_pk_u8_f32 %2, %13, 2, %2\n\t"
        "v_cvt_pk_u8_f32 %0, %6, 3, %0\n\tv_cvt_pk_u8_f32 %1, %10, 3, %1\n\tv_cvt_pk_u8_f32 %2, %14, 3, %2\n\t"
        PCR_ROUND_NEAREST
        : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2])
        : "v"(r[0]), "v"(g[0]), "v"(b[0]), "v"(r[1]), "v"(g[1]), "v"(b[1]), "v"(r[2]), "v"(g[2]), "v"(b[2]), "v"(r[3]), "v"(g[3]), "v"(b[3]));
}

// What the pixel kernels need to know about an image, all wave-uniform (read through a wave-uniform pointer, so
// with scalar loads): sampling, blocks per MCU, where a component's samples start inside an MCU's part of the
// sample tile (rb) and their row length there (rs), first block of its plane in the image's coefficient buffer.
struct PixGeom {
    uint32_t nc, W, H, hmax, vmax, mcux, mcuy, bpm;
    uint32_t hs[kMaxComp], vs[kMaxComp], nbl[kMaxComp], rb[kMaxComp], rs[kMaxComp], plane0[kMaxComp], npl[kMaxComp], bw[kMaxComp], zmx[kMaxComp], cw[kMaxComp], ch[kMaxComp];
    bool flat[kMaxComp];
};
PCR_D void pix_geom(const ImgDesc& D, PixGeom* g) {
    const ImgDesc* ip = &D;
    g->nc = ip->nc; g->W = ip->W; g->H = ip->H; g->hmax = ip->hmax; g->vmax = ip->vmax; g->mcux = ip->mcux; g->mcuy = ip->mcuy;
    uint32_t bpm = 0, p0 = 0;
#pragma unroll
    for (uint32_t c = 0; c < kMaxComp; c++) {
        const bool on = c < g->nc;
        g->hs[c] = on ? ip->hs[c] : 0; g->vs[c] = on ? ip->vs[c] : 0;
        g->nbl[c] = g->hs[c] * g->vs[c]; g->rb[c] = bpm * 64; g->rs[c] = g->hs[c] * 8; bpm += g->nbl[c];
        g->bw[c] = on ? ip->bw[c] : 0;
        g->npl[c] = on ? g->bw[c] * (uint32_t)ip->bh[c] : 0;         // blocks of the component's plane
        g->plane0[c] = p0; p0 += g->npl[c];
        g->zmx[c] = on ? ip->zmax[c] : 0; g->cw[c] = on ? ip->cw[c] : 0; g->ch[c] = on ? ip->ch[c] : 0;
        g->flat[c] = on && g->zmx[c] <= 1;
    }
    g->bpm = bpm;
}

// The lane's block: component c, block (brow, bcol) of the component's plane.
struct PixBlock { uint32_t c, hs, vs, brow, bcol, b, zm, nblk; const int16_t* coef; const int16_t* dc; bool covered; };   // nblk: blocks of the component's plane;   // dc: the block's entry of the compact DC copy
// j: number of the block inside its MCU (components one after the other, each vs rows of hs blocks); (my, mx): the MCU
PCR_D void pix_block(const DevRecord& R, const PixGeom& G, uint64_t coef0, uint32_t j, uint32_t my, uint32_t mx, PixBlock* B, uint32_t* by_out, uint32_t* bx_out) {
    const uint32_t c = j < G.nbl[0] ? 0u : (j < G.nbl[0] + G.nbl[1] ? 1u : 2u);
    const uint32_t jj = j - pick3(c, 0u, G.nbl[0], G.nbl[0] + G.nbl[1]);
    B->c = c; B->hs = pick3(c, G.hs[0], G.hs[1], G.hs[2]); B->vs = pick3(c, G.vs[0], G.vs[1], G.vs[2]);
    const uint32_t bx = jj & (B->hs - 1), by = jj >> (B->hs - 1);                  // (sampling factors are 1 or 2)
    B->brow = my * B->vs + by; B->bcol = mx * B->hs + bx;
    B->b = B->brow * pick3(c, G.bw[0], G.bw[1], G.bw[2]) + B->bcol;
    B->zm = pick3(c, G.zmx[0], G.zmx[1], G.zmx[2]);
    B->nblk = pick3(c, G.npl[0], G.npl[1], G.npl[2]);
    B->coef = R.coef + coef0 + ((size_t)pick3(c, G.plane0[0], G.plane0[1], G.plane0[2]) + B->b) * 64;
    B->dc = R.dc + (coef0 >> 6) + pick3(c, G.plane0[0], G.plane0[1], G.plane0[2]) + B->b;
    B->covered = B->brow < pick3(c, G.ch[0], G.ch[1], G.ch[2]) && B->bcol < pick3(c, G.cw[0], G.cw[1], G.cw[2]);
    *by_out = by; *bx_out = bx;
}
// The block's coefficients as they lie in memory (zig-zag order, two to a word), chunks beyond zm left zero; returns the
// DC coefficient, which comes from the compact copy (the planes hold it only for the coefficient export) and is put in its
// place when the loads have arrived (pix_samples): here it would have the lane wait for them.
PCR_D int16_t pix_load(const PixBlock& B, uint4 v[8]) {
    const int16_t dc = *B.dc;
#pragma unroll
    for (int ch = 0; ch < 8; ch++) {
        v[ch] = uint4{0, 0, 0, 0};
        if (B.zm > 1 && (uint32_t)ch * 8 < B.zm) v[ch] = *reinterpret_cast<const uint4*>(B.coef + ch * 8);
    }
    return dc;
}
// DC of the block after the component's DC refinement scans
template <bool kRefine>
PCR_D int pix_dc(const DevRecord& R, const PixBlock& B, int dcv, const ApplyList* rlc) {
    const uint32_t nref = kRefine ? rlc->n : 0;
    for (uint32_t e = kRefine ? rlc->nac : 0u; e < nref; e++)
        if (dc_refinement_bit(R, rlc->sc[e], B.brow, B.bcol, B.hs, B.vs, B.covered)) dcv |= 1 << rlc->sc[e].Al;
    return dcv;
}
// One or two refinement passes over the block's coefficients, two coefficients to a word.  A position either grows (it
// was non-zero: + 2^Al with its own sign) or is new (it was zero: +- 2^Al by the sign its pass gave) or stays: one step
// with one sign, taken from the coefficient or from the pass.  lo: the positions that change in the pass at bit Al, hi:
// those of the pass before it at bit Al + 1 (or none): a position new in that pass may grow in this one and does so with
// the same sign, so both passes are one step of 0 .. 3 times 2^Al.  neg: the new positions that are negative, of both.
// Sixteen positions at a time are laid out so that a shift puts an even and an odd one into the two halves of a word:
// six instructions for two coefficients and both passes (ten per coefficient one by one).
PCR_D uint32_t pair_mad(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(short2v, a) * __builtin_bit_cast(short2v, b) + __builtin_bit_cast(short2v, c));
}
PCR_D uint32_t pair_sign(uint32_t a) { return __builtin_bit_cast(uint32_t, __builtin_bit_cast(short2v, a) >> (short)15); }
PCR_D void pix_refine(uint32_t cw[32], uint64_t neg, uint64_t hi, uint64_t lo, uint32_t Al) {
    const uint32_t one = 0x00010001u << Al, above = ((0xFFFEu << Al) & 0xFFFFu) * 0x00010001u;     // 2^Al, and -2^(Al+1), in both halves
#pragma unroll
    for (int g = 0; g < 4; g++) {
        auto spread = [g](uint64_t m) {                       // bit p of the sixteen: at p, and at p + 15
            const uint32_t w = g < 2 ? (uint32_t)m : (uint32_t)(m >> 32), h = (g & 1) ? w >> 16 : w & 0xFFFFu;
            return h | (h << 15);
        };
        const uint32_t n = spread(neg), m = (spread(lo) & 0x55555555u) | ((spread(hi) & 0x55555555u) << 1);
#pragma unroll
        for (int j = 0; j < 8; j++) {
            uint32_t& c = cw[8 * g + j];
            const uint32_t step = (pair_sign((n << (15 - 2 * j)) | c) & above) | one;
            c = pair_mad((m >> (2 * j)) & 0x00030003u, step, c);
        }
    }
}
// Refinement replay, de-quantisation and the 8x8 inverse transform of the lane's block; the clamped samples are left in
// F[8 y + x].  qc: the component's folded quantiser steps (zig-zag order); rlc: its refinement scan list.
template <bool kRefine>
PCR_D void pix_samples(const DevRecord& R, const PixBlock& B, const uint4 v[8], int16_t dc, const float* qc, const ApplyList* rlc, float F[64]) {
    uint32_t cw[32];
#pragma unroll
    for (int ch = 0; ch < 8; ch++) { cw[4 * ch] = v[ch].x; cw[4 * ch + 1] = v[ch].y; cw[4 * ch + 2] = v[ch].z; cw[4 * ch + 3] = v[ch].w; }
    cw[0] = (cw[0] & 0xFFFF0000u) | (uint16_t)dc;
    if (kRefine) {
        const uint32_t nref = rlc->n, nac = B.covered ? rlc->nac : 0u;
        // A pass's part of the block's record: positions that become non-zero and their signs, positions whose magnitude
        // grows (all inside the scan's band).  Those of the first two passes are under way together, the DC bits beside them.
        auto pass = [&](uint32_t e, ulonglong2* ns, uint64_t* pl) {
            const uint64_t* rec = R.masks + rlc->sc[e].mask_off;
            *ns = *reinterpret_cast<const ulonglong2*>(rec + ref_word(kRefNz, B.b, B.nblk));
            *pl = rec[ref_word(kRefPlus, B.b, B.nblk)];
        };
        ulonglong2 ns0{0, 0}, ns1{0, 0};
        uint64_t pl0 = 0, pl1 = 0;
        if (nac > 0) pass(0, &ns0, &pl0);
        if (nac > 1) pass(1, &ns1, &pl1);
        for (uint32_t e = rlc->nac; e < nref; e++)
            if (dc_refinement_bit(R, rlc->sc[e], B.brow, B.bcol, B.hs, B.vs, B.covered)) cw[0] |= (1u << rlc->sc[e].Al) & 0xFFFFu;
        // the passes gathered and not made yet: usual scripts refine bit by bit, and the last two are made together
        uint64_t neg = ns0.x & ~ns0.y, hi = 0, lo = ns0.x | pl0;
        uint32_t al = nac > 0 ? rlc->sc[0].Al : 0u, passes = nac > 0 ? 1u : 0u;
        for (uint32_t e = 1; e < nac; e++) {
            if (e > 1) pass(e, &ns1, &pl1);
            const uint32_t Al = rlc->sc[e].Al;
            const bool joins = passes == 1 && Al + 1u == al;
            if (passes != 0 && !joins) { pix_refine(cw, neg, hi, lo, al); neg = 0; passes = 0; }
            hi = joins ? lo : 0; lo = ns1.x | pl1; neg |= ns1.x & ~ns1.y; al = Al; passes++;
        }
        if (passes != 0) pix_refine(cw, neg, hi, lo, al);
    }
    auto coef = [&](int k) { return (float)(int)(int16_t)(uint16_t)(cw[k >> 1] >> (16 * (k & 1))); };
#pragma unroll
    for (int k4 = 0; k4 < 16; k4++) {                        // natural order: F[8 v + u]
        const float4 qq = *reinterpret_cast<const float4*>(qc + 4 * k4);
        F[zigzag_lookup(4 * k4)] = coef(4 * k4) * qq.x; F[zigzag_lookup(4 * k4 + 1)] = coef(4 * k4 + 1) * qq.y;
        F[zigzag_lookup(4 * k4 + 2)] = coef(4 * k4 + 2) * qq.z; F[zigzag_lookup(4 * k4 + 3)] = coef(4 * k4 + 3) * qq.w;
    }
    // the level shift: the DC term reaches every sample with weight one (its folded factor is exactly 1/8 and the
    // transforms only add it), so 128 is added to that once instead of to the 64 samples
    F[0] += 128.f;
#pragma unroll
    for (int r = 0; r < 8; r++)
        idct8_scaled(F[8 * r], F[8 * r + 1], F[8 * r + 2], F[8 * r + 3], F[8 * r + 4], F[8 * r + 5], F[8 * r + 6], F[8 * r + 7]);
#pragma unroll
    for (int x = 0; x < 8; x++)
        idct8_scaled(F[x], F[8 + x], F[16 + x], F[24 + x], F[32 + x], F[40 + x], F[48 + x], F[56 + x]);
#pragma unroll
    for (int e = 0; e < 64; e++) F[e] = clamp255(F[e]);
}
// rows y0 .. y0 + kRows - 1 of the block's samples to dst[(y - y0) * row_len + x]
template <int y0, int kRows>
PCR_D void pix_put_rows(const float F[64], float* dst, uint32_t row_len) {
#pragma unroll
    for (int y = 0; y < kRows; y++) {
        *reinterpret_cast<float4*>(dst + y * row_len) = float4{F[8 * (y0 + y)], F[8 * (y0 + y) + 1], F[8 * (y0 + y) + 2], F[8 * (y0 + y) + 3]};
        *reinterpret_cast<float4*>(dst + y * row_len + 4) = float4{F[8 * (y0 + y) + 4], F[8 * (y0 + y) + 5], F[8 * (y0 + y) + 6], F[8 * (y0 + y) + 7]};
    }
}
// Half kHalf (0: upper, 1: lower) of the pixel rows of an MCU: the part of the lane's block that lies in it, to the
// component's rows of the half (sampling factors are 1 or 2: a block of a component with two block rows per MCU lies
// in one half whole, any other block has four sample rows in each).  dst: the block's first sample row in the half.
// A flat block (flat: only its DC) is one sample.
template <int kHalf>
PCR_D void pix_put_half(const float F[64], bool flat, uint32_t vs, uint32_t by, float* dst, uint32_t row_len) {
    if (vs == 2) {
        if (by != (uint32_t)kHalf) return;
        if (flat) dst[0] = F[0]; else pix_put_rows<0, 8>(F, dst, row_len);
    } else {
        if (flat) dst[0] = F[0]; else pix_put_rows<4 * kHalf, 4>(F, dst, row_len);
    }
}
// The components' folded quantiser steps into LDS; every lane of the workgroup (of two wavefronts or more) calls it.  The
// loads of all components are under way together, and where they lie is known from the descriptor in registers: a chain of
// loads that each wait for the one before is what a kernel of short workgroups waits for most.
struct PixQuant { uint32_t off[kMaxComp], wide[kMaxComp]; };
PCR_D void pix_quant_where(const ImgDesc& D, PixQuant* Q) {
    const uint32_t prec = (uint32_t)D.qprec[0] | (uint32_t)D.qprec[1] << 8 | (uint32_t)D.qprec[2] << 16 | (uint32_t)D.qprec[3] << 24;
    // (Picked from the descriptor in registers; read from memory once more it was one more trip ahead of the steps.  The compiler is not to
    // see that they are members of one array: indexed, the descriptor goes to scratch memory, and k_pixel takes half as long again.)
    uint32_t q0 = D.qoff[0], q1 = D.qoff[1], q2 = D.qoff[2], q3 = D.qoff[3];
    asm("" : "+s"(q0), "+s"(q1), "+s"(q2), "+s"(q3));
#pragma unroll
    for (uint32_t c = 0; c < kMaxComp; c++) {
        const uint32_t tq = D.tq[c] & 3u;
        Q->off[c] = tq & 2u ? (tq & 1u ? q3 : q2) : (tq & 1u ? q1 : q0);
        Q->wide[c] = (prec >> (8 * tq)) & 255u;
    }
}
struct PixSteps { uint32_t hi[2], lo[2]; };                  // a step's bytes as loaded (an 8-bit one twice): of component `wave`, and of component 2
PCR_D void pix_quant_load(const DevRecord& R, const PixQuant& Q, uint32_t nc, uint32_t tid, PixSteps* S) {
    const uint32_t wave = uni(tid >> 6), k = tid & 63u;
#pragma unroll
    for (uint32_t j = 0; j < 2; j++) {                        // (no branch: the loads would be waited for at its end)
        const uint32_t c = j == 1 ? 2u : wave, d = c < nc ? c : 0u;
        const uint32_t wide = pick3(d, Q.wide[0], Q.wide[1], Q.wide[2]) ? 1u : 0u;
        const uint8_t* q = R.rec + pick3(d, Q.off[0], Q.off[1], Q.off[2]) + (k << wide);
        S->hi[j] = q[0]; S->lo[j] = q[wide];
    }
}
PCR_D void pix_quant_table(const PixQuant& Q, const PixSteps& S, uint32_t nc, float (*qz)[68], uint32_t tid, uint32_t nthreads) {
    const uint32_t wave = uni(tid >> 6), k = tid & 63u;
    // Which positions have the transform's cos(pi/4) folded in twice and once: bit k of the words.
    constexpr PixFolds folds{};
    const uint64_t both = folds.both >> k, once = folds.once >> k;
    const float f = (both & 1u) ? 0.125f : ((once & 1u) ? 0.25f * 0.70710678118654752440f : 0.25f);   // (cos(pi/4) squared is exactly 1/2: a block with only its DC is exactly DC x step / 8)
    auto step = [&](uint32_t c, uint32_t j) { return (float)(pick3(c, Q.wide[0], Q.wide[1], Q.wide[2]) ? S.hi[j] << 8 | S.lo[j] : S.hi[j]) * f; };
    if (wave < nc) qz[wave][k] = step(wave, 0);
    if (nthreads == 128 && wave == 0 && nc > 2) qz[2][k] = step(2, 1);    // (two wavefronts: the first has component 2 as well)
}
// the refinement scan lists of the image's components into LDS (all of them under way together)
PCR_D void pix_lists(const ApplyList* __restrict__ lists, const int32_t* __restrict__ list_idx, uint32_t img, uint32_t nc, ApplyList* rl, uint32_t tid) {
    constexpr uint32_t kWords = sizeof(ApplyList) / 4;
    const int32_t* at = list_idx + img * kMaxComp;
    const int32_t l0 = at[0], l1 = at[1], l2 = at[2];
    uint32_t w[kMaxComp], x[kMaxComp];
    static_assert(kWords > 128 && kWords <= 256, "two words per lane of 128");
    const uint32_t e0 = tid, e1 = tid + 128;
#pragma unroll
    for (uint32_t c = 0; c < kMaxComp; c++) {
        const int32_t li = c == 0 ? l0 : (c == 1 ? l1 : l2);
        const uint32_t* src = reinterpret_cast<const uint32_t*>(&lists[li]);
        w[c] = x[c] = 0;                                     // (n = 0 where there is none)
        if (c < nc && li >= 0) { if (e0 < 128) w[c] = src[e0]; if (e1 < kWords) x[c] = src[e1]; }
    }
#pragma unroll
    for (uint32_t c = 0; c < kMaxComp; c++) {
        uint32_t* dst = reinterpret_cast<uint32_t*>(&rl[c]);
        if (c < nc) { if (e0 < 128) dst[e0] = w[c]; if (e1 < kWords) dst[e1] = x[c]; }
    }
}

// four consecutive samples of a component for the output pixels x0 .. x0+3 of a pixel row (x0 a multiple of 4):
// row: the component's row of the MCU; sh: 1 if the component has half the horizontal resolution
PCR_D void four_samples(const float* row, uint32_t x0, uint32_t sh, float v[4]) {
    if (sh == 0) { const float4 t = *reinterpret_cast<const float4*>(row + x0); v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w; }
    else { const float2 t = *reinterpret_cast<const float2*>(row + (x0 >> 1)); v[0] = v[1] = t.x; v[2] = v[3] = t.y; }
}

// The first n (< 12) bytes of w0 w1 w2 to p with at most three stores (a row's last, narrower group: a loop over
// the bytes would cost every wavefront that holds a row end its full length)
PCR_D void store_head(uint8_t* p, uint32_t w0, uint32_t w1, uint32_t w2, uint32_t n) {
    struct __attribute__((packed, aligned(1))) U32 { uint32_t v; };
    struct __attribute__((packed, aligned(1))) U16 { uint16_t v; };
    const uint32_t words[3] = {w0, w1, w2};
    uint32_t done = 0;
    if (n >= 8) { reinterpret_cast<U32*>(p)->v = w0; reinterpret_cast<U32*>(p + 4)->v = w1; done = 8; }
    else if (n >= 4) { reinterpret_cast<U32*>(p)->v = w0; done = 4; }
    const uint32_t w = done == 8 ? words[2] : (done == 4 ? words[1] : words[0]);       // the word the rest comes from
    if (n - done >= 2) { reinterpret_cast<U16*>(p + done)->v = (uint16_t)w; if (n - done == 3) p[done + 2] = (uint8_t)(w >> 16); }
    else if (n - done == 1) p[done] = (uint8_t)w;
}

// past: pixels stored past the caches (pixels_past).  The choice is made at every store; as a kernel of its own for them it takes the same time (0.3 % less for
// two records of 128 pictures of 1024 x 1024).
//
// 120 registers at most, and not the 128 that four wavefronts per SIMD could have: with four of them a SIMD has 32 left for a wavefront of another launch.  At
// 121 (with the two stores of twelve bytes below the other way round) k_bind_fill of a loader's next slot took 119 us beside this kernel instead of 19, and
// 4 x 1024 photographs at scan group 2 2475 us a pass instead of 2220.  Where a change or another compiler takes it over the line, something is to
// be kept in LDS or worked out again that was kept in registers: the attribute that limits them has no effect below what launch bounds allow.
template <bool kRefine, bool kPlanes>
__global__ void __launch_bounds__(kPixLanes, 4) k_pixel(DevRecord R, const PixelTile* __restrict__ tiles, uint8_t* __restrict__ out,
                                                     const ApplyList* __restrict__ lists, const int32_t* __restrict__ list_idx,
                                                     const CropBox* __restrict__ boxes, uint32_t past) {
    // samples of half the pixel rows of the run: 32 per block
    __shared__ __attribute__((aligned(16))) float tile[kPixSamples];
    // quantiser steps in zig-zag order times the folded transform factors; the rows of the three components start
    // four banks apart, so that lanes of different components read them without bank conflicts
    __shared__ __attribute__((aligned(16))) float qz[kMaxComp][68];
    __shared__ ApplyList rl[kRefine ? kMaxComp : 1];       // refinement scan lists of the components (n = 0: none)
    // per MCU of the run: how many of its pixel columns and rows lie inside the image, less one (four bits each), and its
    // first byte, counted from the first one of the run's first row of MCUs (below 2^23: at most 2 x 16 rows of 65535 pixels
    // of a wide image, or what 121 MCUs hold)
    __shared__ uint32_t place[kPixLanes];
    short_kernel_priority();
    const uint32_t item = xcd_major(blockIdx.x, gridDim.x);
    const uint32_t timg = uni(tiles[item].img), mcu0 = uni(tiles[item].mcu0);
    hand_out_status(R, timg, mcu0);
    const uint32_t tid = threadIdx.x;
    // Everything the run needs to know of its image, asked for at once, and the quantiser steps, the block's coefficients and
    // the lists behind it: three round trips to memory ahead of the transform where there were eight, one after the other,
    // half of a workgroup's time (measured: 53 % of the wavefronts' cycles waiting, now 39).  With the rows of the MCUs apart
    // in LDS (pixel_mcu_samples) and both refinement passes at once (pix_refine), us for a record
    // decoded alone: 1024 x 256 x 256 at scan group 5 137 -> 114, 128 x 1024 x 1024 254 -> 224, 256 x 600 x 450 4:4:4 at scan group 10
    // 356 -> 219, 1024 photographs 460 -> 317.
    ImgDesc D;
    load_desc(R.img + timg, &D);
    const bool dead = load_const(&R.status[timg]) != kOk;
    const uint64_t coef0 = load_const(&R.coef_off[timg]), out0 = load_const(&R.out_off[timg]);
    wanted_now(D); wanted_now((uint32_t)dead); wanted_now(coef0); wanted_now(out0);
    PixGeom G;
    pix_geom(D, &G);
    PixQuant Q;
    pix_quant_where(D, &Q);
    const uint32_t nc = G.nc, W = G.W, H = G.H, mcux = G.mcux, bpm = G.bpm;
    const uint32_t mcu_px_w = 8 * G.hmax, mcu_px_h = 8 * G.vmax;
    if (bpm == 0 || bpm > 12) return;                       // (cannot happen for an image the parser accepted)
    const uint32_t gpm = pixel_row_groups(nc, G.hmax);      // groups per pixel row of an MCU: 1, 2 or 4
    const uint32_t per = pixel_mcus(bpm, gpm);
    const uint32_t total = mcux * G.mcuy;
    if (mcu0 >= total) return;
    const uint32_t nm = total - mcu0 < per ? total - mcu0 : per;      // MCUs of this run
    if (boxes) {                                            // (clamped into the image exactly as k_crop_resize clamps it)
        CropBox b = boxes[timg];
        b.x0 = min(max(b.x0, 0), (int)W - 1); b.y0 = min(max(b.y0, 0), (int)H - 1);
        b.w = min(max(b.w, 1), (int)W - b.x0); b.h = min(max(b.h, 1), (int)H - b.y0);
        const uint32_t r0 = mcu0 / mcux, r1 = (mcu0 + nm - 1) / mcux;          // MCU rows the run touches
        if ((int)(r0 * mcu_px_h) >= b.y0 + b.h || (int)((r1 + 1) * mcu_px_h) <= b.y0) return;
        if (r0 == r1) {
            const uint32_t c0 = mcu0 - r0 * mcux;
            if ((int)(c0 * mcu_px_w) >= b.x0 + b.w || (int)((c0 + nm) * mcu_px_w) <= b.x0) return;
        }
    }
    const uint32_t row0 = mcu0 / mcux;                      // the run's first row of MCUs
    // ---- phase A, first half: the quantiser steps, the lane's block and its loads ----
    PixSteps steps;
    pix_quant_load(R, Q, nc, tid, &steps);
    const uint32_t m = (tid * recip16(bpm)) >> 16, j = tid - m * bpm;
    const bool mine = !dead && m < nm;
    PixBlock B;
    uint32_t by = 0, bx = 0;
    uint4 v[8];
    int16_t dc = 0;
    if (mine) {
        const uint32_t M = mcu0 + m, my = M / mcux, mx = M - my * mcux;
        pix_block(R, G, coef0, j, my, mx, &B, &by, &bx);
        dc = pix_load(B, v);
    }
    // ---- prologue tables (the loads above are under way meanwhile) ----
    if (kRefine) pix_lists(lists, list_idx, timg, nc, rl, tid);
    pix_quant_table(Q, steps, nc, qz, tid, kPixLanes);
    if (tid < nm) {
        const uint32_t M = mcu0 + tid, my = M / mcux, mx = M - my * mcux;
        const uint32_t x = mx * mcu_px_w, y = my * mcu_px_h;
        const uint32_t vw = W - x < mcu_px_w ? W - x : mcu_px_w, vh = H - y < mcu_px_h ? H - y : mcu_px_h;      // (every MCU holds a pixel)
        place[tid] = (vw - 1u) | (vh - 1u) << 4 | ((my - row0) * mcu_px_h * W + x) * nc << 8;
    }
    __syncthreads();
    // ---- phase A, second half: the block's samples, in registers ----
    float S[64];
    const bool flatb = mine && B.zm <= 1;                   // flat: one sample stands for the block
    if (mine) {
        const ApplyList* rlc = &rl[kRefine ? B.c : 0];
        asm volatile("" : "+v"(dc), "+v"(v[0].x));            // (or what is done with them, and the wait for the loads, comes right behind the loads)
        if (flatb) S[0] = clamp255((float)pix_dc<kRefine>(R, B, dc, rlc) * qz[B.c][0] + 128.f);
        else pix_samples<kRefine>(R, B, v, dc, qz[B.c], rlc, S);
    }
    if (kPlanes) {
        // Instead of pixels: the lane's block, rounded, into the component's own plane of bytes (`out`: one byte per
        // coefficient slot, so a component's plane lies where its coefficient plane lies, [rows of samples][bw * 8]),
        // for k_triangle_rgb.  A damaged image's planes are left alone; that kernel writes its pixels as zeros.
        if (mine) {
            const uint32_t pw = pick3(B.c, G.bw[0], G.bw[1], G.bw[2]) * 8;
            uint8_t* pd = out + coef0 + (size_t)pick3(B.c, G.plane0[0], G.plane0[1], G.plane0[2]) * 64 + (size_t)(B.brow * 8) * pw + B.bcol * 8;
#pragma unroll
            for (int y = 0; y < 8; y++) {
                uint2 w;
                if (flatb) {
                    w.x = w.y = four_u8(S[0], S[0], S[0], S[0]);
                } else {
                    w.x = four_u8(S[8 * y], S[8 * y + 1], S[8 * y + 2], S[8 * y + 3]);
                    w.y = four_u8(S[8 * y + 4], S[8 * y + 5], S[8 * y + 6], S[8 * y + 7]);
                }
                *reinterpret_cast<uint2*>(pd + (size_t)y * pw) = w;
            }
        }
        return;
    }
    // ---- phase B: one lane per group of output bytes of two pixel rows of one MCU, the upper half of the pixel rows of
    // the MCUs first, then the lower: the samples of half a run are what the workgroup holds in LDS at a time.  (Two
    // rows at a time: the indices, and with 4:2:0 the chroma terms, serve both.) ----
    const uint32_t shx0 = G.hs[0] == G.hmax ? 0 : 1, shy0 = G.vs[0] == G.vmax ? 0 : 1;       // sampling factors are 1 or 2
    const uint32_t shx1 = nc > 1 && G.hs[1] != G.hmax, shy1 = nc > 1 && G.vs[1] != G.vmax;
    const uint32_t shx2 = nc > 2 && G.hs[2] != G.hmax, shy2 = nc > 2 && G.vs[2] != G.vmax;
    const bool halves = (shx1 & shy1 & shx2 & shy2) && !shx0 && !shy0;                      // 4:2:0
    const uint32_t ppg = nc == 1 ? 8u : 4u;                 // pixels per group and row: 8 gray bytes, or 12 bytes of RGB
    const uint32_t lg = gpm == 4 ? 2u : (gpm == 2 ? 1u : 0u);
    const uint32_t half_h = mcu_px_h >> 1;                  // pixel rows of an MCU per half: 4 or 8
    const uint32_t items = nm * (half_h >> 1) * gpm;
    const uint32_t rcpn = nm > 1 ? 0xFFFFFFFFu / nm + 1u : 0u;       // q / nm as the high word of q * rcpn: exact while q * nm < 2^32
    const uint32_t mstride = pixel_mcu_samples(bpm, gpm);
    uint8_t* const first = out + out0 + (size_t)row0 * mcu_px_h * W * nc;
    const uint32_t line = W * nc;
    // component c's four samples for pixels x0.. of row ly (counted inside the half) of MCU mm: a flat component has one per block
    auto fetch = [&](uint32_t c, uint32_t mm, uint32_t ly, uint32_t x0, uint32_t shx, uint32_t shy, float s[4]) {
        if (G.flat[c]) {
            const float f = tile[mm * mstride + (G.rb[c] >> 1) + ((x0 >> shx) >> 3) * 8];      // (a half holds one block row of the component, or half of one)
            s[0] = s[1] = s[2] = s[3] = f;
        } else four_samples(tile + mm * mstride + (G.rb[c] >> 1) + (ly >> shy) * G.rs[c], x0, shx, s);
    };
#pragma unroll
    for (int half = 0; half < 2; half++) {
        if (half) __syncthreads();                          // (the upper half has been read)
        if (mine) {
            float* const dst = tile + m * mstride + (pick3(B.c, G.rb[0], G.rb[1], G.rb[2]) >> 1) + bx * 8;
            if (half == 0) pix_put_half<0>(S, flatb, B.vs, by, dst, B.hs * 8);
            else pix_put_half<1>(S, flatb, B.vs, by, dst, B.hs * 8);
        }
        __syncthreads();
        for (uint32_t it = tid; it < items; it += kPixLanes) {
            // lanes run along the image rows: group, then MCU, then pair of pixel rows
            const uint32_t g = it & (gpm - 1), q = it >> lg;
            const uint32_t lyp = nm > 1 ? __umulhi(q, rcpn) : q, mm = q - lyp * nm, lyh = 2 * lyp;
            const uint32_t ly = lyh + half * half_h;        // the first of the two pixel rows inside the MCU
            const uint32_t pl = place[mm];
            const uint32_t x0 = g * ppg, vw = (pl & 15u) + 1u, vh = ((pl >> 4) & 15u) + 1u;
            if (ly >= vh || x0 >= vw) continue;
            uint8_t* const wp = first + ((pl >> 8) + ly * line + x0 * nc);
            const uint32_t left = vw - x0;                  // pixels of the group inside the image
            const bool both = ly + 1 < vh;
            if (nc == 1) {
#pragma unroll
                for (uint32_t row = 0; row < 2; row++) {
                    float a[4], bq[4];
                    fetch(0, mm, lyh + row, x0, 0, 0, a); fetch(0, mm, lyh + row, x0 + 4, 0, 0, bq);
                    uint32_t w0 = 0, w1 = 0;
                    if (!dead) { w0 = four_u8(a[0], a[1], a[2], a[3]); w1 = four_u8(bq[0], bq[1], bq[2], bq[3]); }
                    if (row && !both) continue;
                    if (left >= 8) {
                        struct __attribute__((packed, aligned(1))) Eight { uint32_t a, b; };
                        Eight e8; e8.a = w0; e8.b = w1;
                        const uint32_t w[2] = {w0, w1};
                        if (past) put_past<Eight>(wp + row * line, w); else *reinterpret_cast<Eight*>(wp + row * line) = e8;
                    } else {
                        store_head(wp + row * line, w0, w1, 0u, left);
                    }
                }
            } else {
                auto store = [&](uint32_t row, const uint32_t w[3]) {
                    uint8_t* const p = wp + row * line;
                    if (left >= 4) {
                        struct __attribute__((packed, aligned(1))) Twelve { uint32_t a, b, c; };
                        Twelve tw; tw.a = w[0]; tw.b = w[1]; tw.c = w[2];
                        // one (possibly unaligned) 12-byte store
                        if (!past) *reinterpret_cast<Twelve*>(p) = tw; else put_past<Twelve>(p, w);
                    } else {
                        store_head(p, w[0], w[1], w[2], left * 3);
                    }
                };
                if (dead) {
                    const uint32_t w[3] = {0, 0, 0};
                    store(0, w);
                    if (both) store(1, w);
                } else if (halves) {                        // two chroma samples for the eight pixels
                    float cb[4], cr[4];
                    fetch(1, mm, lyh, x0, 1, 1, cb); fetch(2, mm, lyh, x0, 1, 1, cr);
                    const float u0 = cb[0] - 128.f, u1 = cb[2] - 128.f, v0 = cr[0] - 128.f, v1 = cr[2] - 128.f;
                    const float u[4] = {u0, u0, u1, u1}, v[4] = {v0, v0, v1, v1};
#pragma unroll
                    for (uint32_t row = 0; row < 2; row++) {
                        if (row && !both) continue;
                        float ys[4]; uint32_t w[3];
                        fetch(0, mm, lyh + row, x0, 0, 0, ys);
                        rgb_words(ys, u, v, w);
                        store(row, w);
                    }
                } else {
#pragma unroll 1
                    for (uint32_t row = 0; row < (both ? 2u : 1u); row++) {
                        float ys[4], cb[4], cr[4]; uint32_t w[3];
                        fetch(0, mm, lyh + row, x0, shx0, shy0, ys); fetch(1, mm, lyh + row, x0, shx1, shy1, cb); fetch(2, mm, lyh + row, x0, shx2, shy2, cr);
#pragma unroll
                        for (int i = 0; i < 4; i++) { cb[i] -= 128.f; cr[i] -= 128.f; }
                        rgb_words(ys, cb, cr, w);
                        store(row, w);
                    }
                }
            }
        }
    }
}

// --------------------------------------------------------------------------------------
// k_pixel_flat: the pixel stage of a decode that holds DC coefficients only (scan groups ahead of every AC scan):
// every block is flat, so an 8x8 cell of output pixels has ONE colour.  One lane per cell (runs of kFlatLanes cells in
// raster order over the image's grid of cells): it reads the DC of the block of each component that covers its cell
// from the compact DC plane (sampling factors are 1 or 2, so a cell lies inside one block of every component),
// de-quantises, converts the colour once and writes the cell's rows, 24 bytes each (8 gray bytes), with unaligned
// vector stores.  No LDS and no barrier; the work per output byte is a few instructions, which is what bounds a
// kernel whose input is 1/64 of its output.  The arithmetic is k_pixel's, so the pixels are the same.
// --------------------------------------------------------------------------------------
constexpr int kFlatLanes = 256;
PCR_HD uint32_t flat_cells(uint32_t W, uint32_t H) { return ((W + 7) >> 3) * ((H + 7) >> 3); }

// only DCs decoded for every component?  (the host launches the flat kernels only for such decodes)
PCR_D bool flat_image(const ImgDesc& D) {
    bool ok = D.nc == 1 || D.nc == 3;
    for (uint32_t c = 0; c < kMaxComp; c++) if (c < D.nc && D.zmax[c] > 1) ok = false;
    return ok;
}
// The output bytes of cell (cx, cy): four pixels as three words (w0 w1 w2; a cell row of eight pixels is w0 w1 w2 w0 w1 w2),
// for a gray image four equal bytes in each.  dcp: the image's compact DC plane.
PCR_D void flat_cell_words(const DevRecord& R, const ImgDesc& D, const int16_t* dcp, uint32_t cx, uint32_t cy, bool dead, uint32_t* w0, uint32_t* w1, uint32_t* w2) {
    float s[kMaxComp];
    uint32_t plane0 = 0;
#pragma unroll
    for (uint32_t c = 0; c < kMaxComp; c++) {
        s[c] = 128.f;
        if (c < D.nc) {
            const uint32_t bcol = (cx * D.hs[c]) >> (D.hmax - 1), brow = (cy * D.vs[c]) >> (D.vmax - 1);      // (sampling factors are 1 or 2)
            // (picked with compares: an index computed at run time would put the whole descriptor into scratch memory)
            const uint32_t tq = D.tq[c] & 3;
            const uint32_t qoff = tq == 0 ? D.qoff[0] : (tq == 1 ? D.qoff[1] : (tq == 2 ? D.qoff[2] : D.qoff[3]));
            const uint32_t qprec = tq == 0 ? D.qprec[0] : (tq == 1 ? D.qprec[1] : (tq == 2 ? D.qprec[2] : D.qprec[3]));
            const uint8_t* q = R.rec + qoff;
            const float q0 = (qprec ? (float)ld_be16(q) : (float)q[0]) * 0.125f;
            s[c] = clamp255((float)dcp[plane0 + brow * D.bw[c] + bcol] * q0 + 128.f);
            plane0 += (uint32_t)D.bw[c] * D.bh[c];
        }
    }
    if (D.nc == 1) { const uint32_t g = four_u8(s[0], s[0], s[0], s[0]); *w0 = g; *w1 = g; *w2 = g; }
    else {
        float rf, gf, bf;
        to_rgb(s[0], s[1] - 128.f, s[2] - 128.f, &rf, &gf, &bf);
        const uint32_t w = four_u8(rf, gf, bf, rf);
        *w0 = w; *w1 = __builtin_amdgcn_perm(w, w, 0x01000201u); *w2 = __builtin_amdgcn_perm(w, w, 0x02010002u);
    }
    if (dead) { *w0 = 0; *w1 = 0; *w2 = 0; }
}

__global__ void __launch_bounds__(kFlatLanes) k_pixel_flat(DevRecord R, const PixelTile* __restrict__ tiles, uint8_t* __restrict__ out,
                                                           const CropBox* __restrict__ boxes) {
    short_kernel_priority();
    const uint32_t item = xcd_major(blockIdx.x, gridDim.x);
    const uint32_t timg = uni(tiles[item].img), cell0 = uni(tiles[item].mcu0);
    hand_out_status(R, timg, cell0);
    ImgDesc D;
    load_desc(R.img + timg, &D);
    const uint32_t nc = D.nc, W = D.W, H = D.H;
    const uint32_t cells_w = (W + 7) >> 3, total = cells_w * ((H + 7) >> 3);
    const uint32_t cell = cell0 + threadIdx.x;
    if (!flat_image(D)) return;
    if (cell >= total) return;
    // cell / cells_w as the high word of a product: exact while cell * cells_w < 2^32 (and the factor fits: cells_w > 1)
    const uint32_t cy = cells_w == 1 ? cell : ((uint64_t)total * cells_w < (1ull << 32) ? __umulhi(cell, 0xFFFFFFFFu / cells_w + 1u) : cell / cells_w);
    const uint32_t cx = cell - cy * cells_w;
    const uint32_t x = cx * 8, y = cy * 8;
    if (boxes) {                                            // (clamped into the image exactly as k_crop_resize clamps it)
        CropBox b = boxes[timg];
        b.x0 = min(max(b.x0, 0), (int)W - 1); b.y0 = min(max(b.y0, 0), (int)H - 1);
        b.w = min(max(b.w, 1), (int)W - b.x0); b.h = min(max(b.h, 1), (int)H - b.y0);
        if ((int)x >= b.x0 + b.w || (int)x + 8 <= b.x0 || (int)y >= b.y0 + b.h || (int)y + 8 <= b.y0) return;
    }
    const bool dead = uni((uint32_t)(R.status[timg] != kOk)) != 0;
    uint32_t w0, w1, w2;
    flat_cell_words(R, D, R.dc + (R.coef_off[timg] >> 6), cx, cy, dead, &w0, &w1, &w2);
    const uint32_t npx = W - x < 8 ? W - x : 8, nrows = H - y < 8 ? H - y : 8;
    const size_t pitch = (size_t)W * nc;
    uint8_t* wp = out + R.out_off[timg] + (size_t)y * pitch + (size_t)x * nc;
    struct __attribute__((packed, aligned(1))) Words2 { uint32_t a, b; };
    struct __attribute__((packed, aligned(1))) Words4 { uint32_t a, b, c, d; };
    if (npx == 8) {
        if (nc == 1) {
            Words2 e; e.a = w0; e.b = w0;
            for (uint32_t r = 0; r < nrows; r++, wp += pitch) *reinterpret_cast<Words2*>(wp) = e;
        } else {
            Words4 e; e.a = w0; e.b = w1; e.c = w2; e.d = w0;
            Words2 f; f.a = w1; f.b = w2;
            for (uint32_t r = 0; r < nrows; r++, wp += pitch) { *reinterpret_cast<Words4*>(wp) = e; *reinterpret_cast<Words2*>(wp + 16) = f; }
        }
    } else {                                                // the image's last, narrower column of cells
        const uint32_t nb = npx * nc;
        for (uint32_t r = 0; r < nrows; r++, wp += pitch)
            for (uint32_t i = 0; i < nb; i++) wp[i] = (uint8_t)((nc == 1 ? w0 : (i % 12 < 4 ? w0 : (i % 12 < 8 ? w1 : w2))) >> (8 * (i & 3)));
    }
}

// --------------------------------------------------------------------------------------
// k_pixel_flat_rows: the same pixels written as whole aligned 16-byte chunks, for images of at most kFlatRowCells
// cells per row decoded without crop boxes (the usual case; k_pixel_flat serves the rest).  One wavefront per row of
// cells (many short workgroups in flight hide the chain descriptor -> DC -> LDS -> stores better than few wide ones).  The eight pixel rows the cells cover are equal and lie one behind the other in the output, so the band is
// one run of bytes that repeats the pixel row; the lanes first make that row in LDS (one cell each), then write the
// band chunk by chunk -- a chunk is sixteen bytes of the repeated row from the chunk's distance to the band's start
// modulo the row length -- and the few bytes ahead of the first and behind the last whole chunk one by one.
// Measured on this chip, writing a decoded record's pixels this way takes 0.10 ms per 490 MB against 0.14 ms for
// 24-byte pieces at the cells' own addresses.
// --------------------------------------------------------------------------------------
constexpr int kFlatRowCells = 1024, kFlatRowLanes = 64;
PCR_HD bool flat_rows_fit(uint32_t W) { return ((W + 7) >> 3) <= (uint32_t)kFlatRowCells; }
// LDS bytes a launch needs for images of at most `cells` cells per row: 24 bytes per cell, the repeated 32 bytes, slack
PCR_HD uint32_t flat_rows_lds(uint32_t cells) { return cells * 24 + 64; }

__global__ void __launch_bounds__(kFlatRowLanes) k_pixel_flat_rows(DevRecord R, const PixelTile* __restrict__ tiles, uint8_t* __restrict__ out, uint32_t max_cells, uint32_t past) {
    // the pixel row: 24 bytes per cell (8 for a gray image), then its first 32 bytes again so that a chunk may run past its end
    extern __shared__ __attribute__((aligned(16))) uint32_t pat[];
    short_kernel_priority();
    const uint32_t item = xcd_major(blockIdx.x, gridDim.x);
    const uint32_t timg = uni(tiles[item].img), cy = uni(tiles[item].mcu0);      // (mcu0: the row of cells)
    hand_out_status(R, timg, cy);
    ImgDesc D;
    load_desc(R.img + timg, &D);
    const uint32_t nc = D.nc, W = D.W, H = D.H, tid = threadIdx.x;
    const uint32_t cells_w = (W + 7) >> 3;
    if (!flat_image(D) || cells_w > max_cells || cy * 8 >= H) return;      // (wave-uniform: no lane is left behind at a barrier)
    const bool dead = uni((uint32_t)(R.status[timg] != kOk)) != 0;
    const int16_t* dcp = R.dc + (R.coef_off[timg] >> 6);
    for (uint32_t cx = tid; cx < cells_w; cx += kFlatRowLanes) {
        uint32_t w0, w1, w2;
        flat_cell_words(R, D, dcp, cx, cy, dead, &w0, &w1, &w2);
        if (nc == 1) { pat[2 * cx] = w0; pat[2 * cx + 1] = w0; }
        else { uint32_t* d = pat + 6 * cx; d[0] = w0; d[1] = w1; d[2] = w2; d[3] = w0; d[4] = w1; d[5] = w2; }
    }
    __syncthreads();
    const uint32_t pitch = W * nc;                           // bytes of a pixel row (< 2^15 here)
    uint8_t* pb = reinterpret_cast<uint8_t*>(pat);
    uint32_t wrap = 0;
    if (tid < 32) wrap = pb[tid % pitch];
    __syncthreads();                                        // (the last cell may have written past the row's end: read first, then overwrite)
    if (tid < 32) pb[pitch + tid] = (uint8_t)wrap;
    __syncthreads();
    const uint32_t nrows = H - cy * 8 < 8 ? H - cy * 8 : 8;
    const uint32_t len = nrows * pitch;                     // bytes of the band (< 2^18)
    uint8_t* band = out + R.out_off[timg] + (size_t)cy * 8 * pitch;
    const uint32_t head = (uint32_t)((16 - (reinterpret_cast<uintptr_t>(band) & 15)) & 15);   // bytes ahead of the first aligned chunk
    const float inv_pitch = 1.0f / (float)pitch;
    // distance from the band's start -> position in the pixel row (p < 2^24: the quotient in single precision is off by at most one)
    auto in_row = [&](uint32_t p) {
        uint32_t r = (uint32_t)((float)p * inv_pitch);
        int32_t q = (int32_t)(p - r * pitch);
        if (q < 0) q += (int32_t)pitch; else if (q >= (int32_t)pitch) q -= (int32_t)pitch;
        return (uint32_t)q;
    };
    if (head >= len) {                                      // a band shorter than one chunk
        for (uint32_t p = tid; p < len; p += kFlatRowLanes) band[p] = pb[in_row(p)];
        return;
    }
    const uint32_t nchunks = (len - head) >> 4, tail0 = head + (nchunks << 4);
    for (uint32_t j = tid; j < nchunks; j += kFlatRowLanes) {
        const uint32_t p = head + (j << 4), q = in_row(p);
        const uint32_t* s = pat + (q >> 2);
        const uint32_t a = s[0], b = s[1], c = s[2], d = s[3], e = s[4], sh = q & 3;
        uint4 v;
        v.x = __builtin_amdgcn_alignbyte(b, a, sh); v.y = __builtin_amdgcn_alignbyte(c, b, sh);
        v.z = __builtin_amdgcn_alignbyte(d, c, sh); v.w = __builtin_amdgcn_alignbyte(e, d, sh);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        if (past) put_past<uint4>(band + p, w); else *reinterpret_cast<uint4*>(band + p) = v;
    }
    if (tid < head) band[tid] = pb[tid];                    // (head < 16 <= the repeated part)
    if (tid < len - tail0) band[tail0 + tid] = pb[in_row(tail0 + tid)];
}

// --------------------------------------------------------------------------------------
// k_triangle_rgb: pixels from planes of rounded samples (k_pixel<., true>) with the chroma up-sampling stock decoders
// use instead of replication: every output sample of a component at half resolution is 3/4 of the nearer and 1/4 of the
// farther sample of the component's grid, down the columns first, then along the rows; beyond the component's own
// samples (ceil(W hs / hmax) x ceil(H vs / vmax)) the nearest one stands in.  On integer samples these weights are exact
// in single precision.  One lane per four pixels of a row.  grid: (ceil(items of the largest image / 256), images).
// --------------------------------------------------------------------------------------
PCR_D float triangle_sample(const uint8_t* p, uint32_t pw, uint32_t xc, uint32_t yc, uint32_t fx, uint32_t fy, uint32_t x, uint32_t y) {
    if (fx == 1 && fy == 1) return (float)p[(size_t)y * pw + x];
    const uint32_t xi = fx == 2 ? x >> 1 : x;
    uint32_t xj = fx == 2 ? ((x & 1) ? xi + 1 : (xi ? xi - 1 : 0)) : xi;
    if (xj >= xc) xj = xc - 1;
    const uint32_t yi = fy == 2 ? y >> 1 : y;
    uint32_t yj = fy == 2 ? ((y & 1) ? yi + 1 : (yi ? yi - 1 : 0)) : yi;
    if (yj >= yc) yj = yc - 1;
    const float a0 = (float)p[(size_t)yi * pw + xi], a1 = (float)p[(size_t)yj * pw + xi];
    const float c0 = fy == 2 ? 0.75f * a0 + 0.25f * a1 : a0;
    if (fx != 2) return c0;
    const float b0 = (float)p[(size_t)yi * pw + xj], b1 = (float)p[(size_t)yj * pw + xj];
    const float c1 = fy == 2 ? 0.75f * b0 + 0.25f * b1 : b0;
    return 0.75f * c0 + 0.25f * c1;
}

__global__ void __launch_bounds__(256) k_triangle_rgb(DevRecord R, const uint8_t* __restrict__ planes, uint8_t* __restrict__ out) {
    const uint32_t img = blockIdx.y;
    ImgDesc D;
    load_desc(R.img + img, &D);
    const uint32_t W = D.W, H = D.H, nc = D.nc;
    const uint32_t gw = (W + 3) >> 2;                        // groups of four pixels per row
    const uint32_t item = blockIdx.x * 256 + threadIdx.x;
    if (item >= gw * H || (nc != 1 && nc != 3)) return;
    const uint32_t y = item / gw, x0 = (item - y * gw) * 4;
    const uint32_t npx = W - x0 < 4 ? W - x0 : 4;
    const bool dead = R.status[img] != kOk;
    float s[kMaxComp][4];
    uint32_t plane0 = 0;
#pragma unroll
    for (uint32_t c = 0; c < kMaxComp; c++) {
        if (c < nc && !dead) {
            const uint8_t* p = planes + R.coef_off[img] + (size_t)plane0 * 64;
            const uint32_t pw = (uint32_t)D.bw[c] * 8, fx = D.hmax / D.hs[c], fy = D.vmax / D.vs[c];
            const uint32_t xc = (W * D.hs[c] + D.hmax - 1) / D.hmax, yc = (H * D.vs[c] + D.vmax - 1) / D.vmax;
            for (uint32_t i = 0; i < 4; i++) s[c][i] = i < npx ? triangle_sample(p, pw, xc, yc, fx, fy, x0 + i, y) : 0.f;
        } else for (uint32_t i = 0; i < 4; i++) s[c][i] = 0.f;
        plane0 += c < nc ? (uint32_t)D.bw[c] * D.bh[c] : 0;
    }
    uint8_t* wp = out + R.out_off[img] + ((size_t)y * W + x0) * nc;
    if (nc == 1) {
        for (uint32_t i = 0; i < npx; i++) wp[i] = dead ? 0 : (uint8_t)put_u8(s[0][i], 0, 0);
        return;
    }
    uint32_t w0 = 0, w1 = 0, w2 = 0;
    if (!dead) {
        float r[4], g[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float u = s[1][i] - 128.f, w = s[2][i] - 128.f;
            r[i] = s[0][i] + 1.402f * w; g[i] = s[0][i] - 0.344136f * u - 0.714136f * w; b[i] = s[0][i] + 1.772f * u;
        }
        w0 = put_u8(r[0], 0, w0); w0 = put_u8(g[0], 1, w0); w0 = put_u8(b[0], 2, w0); w0 = put_u8(r[1], 3, w0);
        w1 = put_u8(g[1], 0, w1); w1 = put_u8(b[1], 1, w1); w1 = put_u8(r[2], 2, w1); w1 = put_u8(g[2], 3, w1);
        w2 = put_u8(b[2], 0, w2); w2 = put_u8(r[3], 1, w2); w2 = put_u8(g[3], 2, w2); w2 = put_u8(b[3], 3, w2);
    }
    if (npx == 4) {
        struct __attribute__((packed, aligned(1))) Twelve { uint32_t a, b, c; };
        Twelve tw; tw.a = w0; tw.b = w1; tw.c = w2;
        *reinterpret_cast<Twelve*>(wp) = tw;
    } else {
        for (uint32_t i = 0; i < npx * 3; i++) wp[i] = (uint8_t)((i < 4 ? w0 : (i < 8 ? w1 : w2)) >> (8 * (i & 3)));
    }
}

// --------------------------------------------------------------------------------------
// k_smooth: the five lowest AC coefficients of every block of a component of which only the DC first scan has been
// received, predicted from the DC coefficients of the block and its eight neighbours (T.81 K.8: the coefficients of
// the quadratic surface whose means over the nine blocks are the nine DC values; what stock decoders show for the
// first scans of a progressive file).  Integer form: weights 36/256, 9/256 and 5/256 of the de-quantised DC
// differences, rounded to a multiple of the coefficient's own quantiser step, halves away from zero, limited to
// +-1023; a neighbour beyond the component's block grid is the nearest block inside it.
// kClear = false: writes the first 16-byte chunk of each such block of the coefficient planes (zig-zag positions
// 0..7: 1..5 predicted, the others zero; the pixel kernel takes position 0 from the compact DC copy) and raises the
// component's zmax to 6, so that k_pixel reads that chunk and nothing more.  kClear = true, after k_pixel: the chunks
// are zero again and zmax is 1, the state an upgrade to a higher scan group builds on.
// grid: (kSmoothGroups, images); 256 lanes, a block per lane and trip.
// --------------------------------------------------------------------------------------
constexpr uint32_t kSmoothGroups = 8;
PCR_D int smooth_predict(int64_t w, int64_t q0, int64_t delta, int64_t qz) {
    const int64_t num = w * q0 * delta, den = 256 * qz;
    int64_t v = num >= 0 ? (num + den / 2) / den : -((-num + den / 2) / den);
    v = v > 1023 ? 1023 : (v < -1023 ? -1023 : v);
    return (int)v;
}
template <bool kClear>
__global__ void __launch_bounds__(256) k_smooth(DevRecord R) {
    __shared__ uint32_t does[kMaxComp];                      // per component: 1 if it holds its DC first scan and nothing else
    __shared__ uint32_t qs[kMaxComp][6];                     // its quantiser steps of zig-zag positions 0..5
    const uint32_t img = blockIdx.y, tid = threadIdx.x;
    ImgDesc* ip = R.img + img;
    const uint32_t nc = ip->nc;
    if (ip->status != kOk || !ip->progressive || nc > kMaxComp) return;
    if (tid < kMaxComp) {
        uint32_t carried = 0, dc_first = 0, tq = 0;
        if (tid < nc) {
            tq = ip->tq[tid];
            const ScanDesc* sc = R.scan + (size_t)img * R.G;
            const uint32_t ng = ip->nscans < R.G ? ip->nscans : R.G;
            for (uint32_t g = 0; g < ng; g++)
                for (uint32_t j = 0; j < sc[g].ns && j < kMaxComp; j++)
                    if (sc[g].comp[j] == tid) { carried++; dc_first += (sc[g].Ss == 0 && sc[g].Se == 0 && sc[g].Ah == 0) ? 1u : 0u; }
        }
        const bool on = carried == 1 && dc_first == 1 && ip->qoff[tq] != 0;
        does[tid] = on ? 1u : 0u;
        if (on) {
            const uint8_t* q = R.rec + ip->qoff[tq];
            const bool wide = ip->qprec[tq] != 0;
            // (a step of zero, which the standard does not allow, predicts nothing: DC step zero makes every difference zero,
            // and a coefficient with step zero de-quantises to zero whatever it is; the divisor only must not be zero)
            for (uint32_t k = 0; k < 6; k++) { const uint32_t v = wide ? ld_be16(q + 2 * k) : q[k]; qs[tid][k] = (v || k == 0) ? v : 1u; }
        }
    }
    __syncthreads();
    uint32_t plane0 = 0;
    for (uint32_t c = 0; c < nc; c++) {
        const uint32_t bw = ip->bw[c], bh = ip->bh[c], nb = bw * bh;
        if ((uint64_t)(plane0 + nb) * 64 > R.coef_off[img + 1] - R.coef_off[img]) return;   // (cannot happen for an image the parser accepted)
        if (does[c]) {
            if (blockIdx.x == 0 && tid == 0) ip->zmax[c] = kClear ? 1 : 6;
            const int16_t* dc = R.dc + (R.coef_off[img] >> 6) + plane0;
            int16_t* planes = R.coef + R.coef_off[img] + (size_t)plane0 * 64;
            const int64_t q0 = qs[c][0], q1 = qs[c][1], q2 = qs[c][2], q3 = qs[c][3], q4 = qs[c][4], q5 = qs[c][5];
            for (uint32_t b = blockIdx.x * 256 + tid; b < nb; b += kSmoothGroups * 256) {
                short8 o = short8{0, 0, 0, 0, 0, 0, 0, 0};
                if (!kClear) {
                    const uint32_t by = b / bw, bx = b - by * bw;
                    const uint32_t xl = bx ? bx - 1 : 0, xr = bx + 1 < bw ? bx + 1 : bx, ya = by ? by - 1 : 0, yb = by + 1 < bh ? by + 1 : by;
                    const int64_t al = dc[ya * bw + xl], a = dc[ya * bw + bx], ar = dc[ya * bw + xr];
                    const int64_t l = dc[by * bw + xl], m = dc[b], r = dc[by * bw + xr];
                    const int64_t bl = dc[yb * bw + xl], be = dc[yb * bw + bx], br = dc[yb * bw + xr];
                    o[1] = (short)smooth_predict(36, q0, l - r, q1);
                    o[2] = (short)smooth_predict(36, q0, a - be, q2);
                    o[3] = (short)smooth_predict(9, q0, a + be - 2 * m, q3);
                    o[4] = (short)smooth_predict(5, q0, (al - ar) - (bl - br), q4);
                    o[5] = (short)smooth_predict(9, q0, l + r - 2 * m, q5);
                }
                *reinterpret_cast<short8*>(planes + (size_t)b * 64) = o;
            }
        }
        plane0 += nb;
    }
}

// --------------------------------------------------------------------------------------
// k_pixel_smooth_flat: the pixels of a decode that holds DC first scans only, with k_smooth's predictions, without the
// detour through the coefficient planes and the full transform: one lane per 8x8 cell of pixels, as in k_pixel_flat.
// A block with zig-zag coefficients 0..5 only is
//     f(y, x) = F00 / 8 + a (F01 c1(x) + F02 c2(x)) + a (F10 c1(y) + F20 c2(y)) + F11 c1(x) c1(y) / 4,
//     a = 1 / (4 sqrt 2),  c1(t) = cos((2t + 1) pi / 16),  c2(t) = cos((2t + 1) pi / 8),
// a sum of a function of x, a function of y and one product: per component the lane keeps the two functions of x for
// its eight pixel columns and the two of y for its eight pixel rows (a cell of a component at half resolution covers
// four of the block's sample columns or rows, each twice), and a sample costs two operations.  Clamping, colour
// conversion and rounding as everywhere.  The predictions are the same integers k_smooth writes (32-bit arithmetic when
// the quantiser table has 8-bit entries: 36 x 255 x four DC coefficients fits).  Launched by the host only when every scan decoded
// is a DC first scan; a component without its DC scan reads as zero and is not predicted.
// grid: the flat tile list (runs of kFlatLanes cells of one image).
// --------------------------------------------------------------------------------------
PCR_D int smooth_predict32(uint32_t w, uint32_t q0, int delta, uint32_t qz) {
    const uint32_t mag = (uint32_t)(delta < 0 ? -delta : delta);
    const uint32_t num = w * q0 * mag, den = 256u * qz;
    uint32_t v = (num + den / 2) / den;
    v = v > 1023u ? 1023u : v;
    return delta < 0 ? -(int)v : (int)v;
}
__global__ void __launch_bounds__(kFlatLanes) k_pixel_smooth_flat(DevRecord R, const PixelTile* __restrict__ tiles, uint8_t* __restrict__ out) {
    __shared__ uint32_t does[kMaxComp];
    short_kernel_priority();
    const uint32_t item = xcd_major(blockIdx.x, gridDim.x);
    const uint32_t timg = uni(tiles[item].img), cell0 = uni(tiles[item].mcu0);
    hand_out_status(R, timg, cell0);
    ImgDesc D;
    load_desc(R.img + timg, &D);
    const uint32_t nc = D.nc, W = D.W, H = D.H;
    if (!flat_image(D)) return;
    if (threadIdx.x < kMaxComp) {
        uint32_t carried = 0, dc_first = 0;
        if (threadIdx.x < nc && D.progressive) {
            const ScanDesc* sc = R.scan + (size_t)timg * R.G;
            const uint32_t ng = D.nscans < R.G ? D.nscans : R.G;
            for (uint32_t g = 0; g < ng; g++)
                for (uint32_t j = 0; j < sc[g].ns && j < kMaxComp; j++)
                    if (sc[g].comp[j] == threadIdx.x) { carried++; dc_first += (sc[g].Ss == 0 && sc[g].Se == 0 && sc[g].Ah == 0) ? 1u : 0u; }
        }
        does[threadIdx.x] = (carried == 1 && dc_first == 1) ? 1u : 0u;
    }
    __syncthreads();
    const uint32_t cells_w = (W + 7) >> 3, total = cells_w * ((H + 7) >> 3);
    const uint32_t cell = cell0 + threadIdx.x;
    if (cell >= total) return;
    const uint32_t cy = cells_w == 1 ? cell : ((uint64_t)total * cells_w < (1ull << 32) ? __umulhi(cell, 0xFFFFFFFFu / cells_w + 1u) : cell / cells_w);
    const uint32_t cx = cell - cy * cells_w;
    const uint32_t x = cx * 8, y = cy * 8;
    const bool dead = uni((uint32_t)(R.status[timg] != kOk)) != 0;
    constexpr float kC1[8] = {0.98078528f, 0.83146961f, 0.55557023f, 0.19509032f, -0.19509032f, -0.55557023f, -0.83146961f, -0.98078528f};
    constexpr float kC2[8] = {0.92387953f, 0.38268343f, -0.38268343f, -0.92387953f, -0.92387953f, -0.38268343f, 0.38268343f, 0.92387953f};
    constexpr float kA = 0.17677670f;
    // per component and pixel column: the function of x and the factor of the product; per pixel row: the same of y
    float fx[kMaxComp][8], px[kMaxComp][8], fy[kMaxComp][8], py[kMaxComp][8];
    const int16_t* dcp = R.dc + (R.coef_off[timg] >> 6);
    uint32_t plane0 = 0;
#pragma unroll
    for (uint32_t c = 0; c < kMaxComp; c++) {
#pragma unroll
        for (int t = 0; t < 8; t++) { fx[c][t] = 128.f; px[c][t] = 0.f; fy[c][t] = 0.f; py[c][t] = 0.f; }
        if (c < nc) {
            const uint32_t shx = D.hs[c] == D.hmax ? 0u : 1u, shy = D.vs[c] == D.vmax ? 0u : 1u;      // (sampling factors are 1 or 2)
            const uint32_t bcol = (cx * D.hs[c]) >> (D.hmax - 1), brow = (cy * D.vs[c]) >> (D.vmax - 1);
            const uint32_t bw = D.bw[c], bh = D.bh[c];
            const uint32_t tq = D.tq[c] & 3;
            const uint32_t qoff = tq == 0 ? D.qoff[0] : (tq == 1 ? D.qoff[1] : (tq == 2 ? D.qoff[2] : D.qoff[3]));
            const uint32_t wide = tq == 0 ? D.qprec[0] : (tq == 1 ? D.qprec[1] : (tq == 2 ? D.qprec[2] : D.qprec[3]));
            const uint8_t* q = R.rec + qoff;
            uint32_t qs[6], qd[6];                           // the steps, and the divisors (a step of zero predicts nothing)
#pragma unroll
            for (uint32_t k = 0; k < 6; k++) { qs[k] = wide ? ld_be16(q + 2 * k) : q[k]; qd[k] = qs[k] ? qs[k] : 1u; }
            const int16_t* d = dcp + plane0;
            const int m = d[brow * bw + bcol];
            int p1 = 0, p2 = 0, p3 = 0, p4 = 0, p5 = 0;
            if (does[c] && qoff != 0 && bcol < bw && brow < bh) {
                const uint32_t xl = bcol ? bcol - 1 : 0, xr = bcol + 1 < bw ? bcol + 1 : bcol, ya = brow ? brow - 1 : 0, yb = brow + 1 < bh ? brow + 1 : brow;
                const int al = d[ya * bw + xl], a = d[ya * bw + bcol], ar = d[ya * bw + xr];
                const int l = d[brow * bw + xl], r = d[brow * bw + xr];
                const int bl = d[yb * bw + xl], be = d[yb * bw + bcol], br = d[yb * bw + xr];
                if (wide) {
                    p1 = smooth_predict(36, qs[0], l - r, qd[1]); p2 = smooth_predict(36, qs[0], a - be, qd[2]);
                    p3 = smooth_predict(9, qs[0], a + be - 2 * m, qd[3]); p4 = smooth_predict(5, qs[0], (al - ar) - (bl - br), qd[4]);
                    p5 = smooth_predict(9, qs[0], l + r - 2 * m, qd[5]);
                } else {
                    p1 = smooth_predict32(36, qs[0], l - r, qd[1]); p2 = smooth_predict32(36, qs[0], a - be, qd[2]);
                    p3 = smooth_predict32(9, qs[0], a + be - 2 * m, qd[3]); p4 = smooth_predict32(5, qs[0], (al - ar) - (bl - br), qd[4]);
                    p5 = smooth_predict32(9, qs[0], l + r - 2 * m, qd[5]);
                }
            }
            const float F00 = (float)m * (float)qs[0], F01 = (float)p1 * (float)qs[1], F10 = (float)p2 * (float)qs[2];
            const float F20 = (float)p3 * (float)qs[3], F11 = (float)p4 * (float)qs[4], F02 = (float)p5 * (float)qs[5];
            // the eight sample columns and rows of the block ...
            float gx[8], hx[8], gy[8];
#pragma unroll
            for (int t = 0; t < 8; t++) {
                gx[t] = F00 * 0.125f + 128.f + kA * (F01 * kC1[t] + F02 * kC2[t]);
                hx[t] = 0.25f * F11 * kC1[t];
                gy[t] = kA * (F10 * kC1[t] + F20 * kC2[t]);
            }
            // ... and those the cell's pixel columns and rows take them from
            const bool right = shx && (cx & 1u), low = shy && (cy & 1u);
#pragma unroll
            for (int t = 0; t < 8; t++) {
                fx[c][t] = shx ? (right ? gx[4 + (t >> 1)] : gx[t >> 1]) : gx[t];
                px[c][t] = shx ? (right ? hx[4 + (t >> 1)] : hx[t >> 1]) : hx[t];
                fy[c][t] = shy ? (low ? gy[4 + (t >> 1)] : gy[t >> 1]) : gy[t];
                py[c][t] = shy ? (low ? kC1[4 + (t >> 1)] : kC1[t >> 1]) : kC1[t];
            }
            plane0 += bw * bh;
        }
    }
    const uint32_t npx = W - x < 8 ? W - x : 8, nrows = H - y < 8 ? H - y : 8;
    const size_t pitch = (size_t)W * nc;
    uint8_t* wp = out + R.out_off[timg] + (size_t)y * pitch + (size_t)x * nc;
    struct __attribute__((packed, aligned(1))) Words2 { uint32_t a, b; };
    struct __attribute__((packed, aligned(1))) Words4 { uint32_t a, b, c, d; };
    // both chroma components at half resolution both ways (4:2:0): a chroma sample serves a 2 x 2 group of pixels and is
    // evaluated once for it (the same expression on the same values as below, so the pixels do not depend on the path)
    const bool quarter = nc == 3 && D.hs[0] == D.hmax && D.vs[0] == D.vmax && D.hs[1] != D.hmax && D.vs[1] != D.vmax && D.hs[2] != D.hmax && D.vs[2] != D.vmax;
#pragma unroll
    for (int rp = 0; rp < 4; rp++) {
        float u[8], v[8];
#pragma unroll
        for (int t = 0; t < 8; t++) { u[t] = 0.f; v[t] = 0.f; }
        if (quarter && !dead && (uint32_t)(2 * rp) < nrows) {
#pragma unroll
            for (int j = 0; j < 4; j++) {
                u[2 * j] = u[2 * j + 1] = clamp255(fx[1][2 * j] + fy[1][2 * rp] + px[1][2 * j] * py[1][2 * rp]) - 128.f;
                v[2 * j] = v[2 * j + 1] = clamp255(fx[2][2 * j] + fy[2][2 * rp] + px[2][2 * j] * py[2][2 * rp]) - 128.f;
            }
        }
#pragma unroll
        for (int dr = 0; dr < 2; dr++) {
            const int r = 2 * rp + dr;
            if ((uint32_t)r >= nrows) continue;
            uint32_t w[6] = {0, 0, 0, 0, 0, 0};
            if (!dead) {
                if (nc == 3 && !quarter) {
#pragma unroll
                    for (int t = 0; t < 8; t++) {
                        u[t] = clamp255(fx[1][t] + fy[1][r] + px[1][t] * py[1][r]) - 128.f;
                        v[t] = clamp255(fx[2][t] + fy[2][r] + px[2][t] * py[2][r]) - 128.f;
                    }
                }
#pragma unroll
                for (int t = 0; t < 8; t++) {
                    const float s0 = clamp255(fx[0][t] + fy[0][r] + px[0][t] * py[0][r]);
                    if (nc == 1) w[t >> 2] = put_u8(s0, t & 3, w[t >> 2]);
                    else {
                        w[(3 * t) >> 2] = put_u8(s0 + 1.402f * v[t], (3 * t) & 3, w[(3 * t) >> 2]);
                        w[(3 * t + 1) >> 2] = put_u8(s0 - 0.344136f * u[t] - 0.714136f * v[t], (3 * t + 1) & 3, w[(3 * t + 1) >> 2]);
                        w[(3 * t + 2) >> 2] = put_u8(s0 + 1.772f * u[t], (3 * t + 2) & 3, w[(3 * t + 2) >> 2]);
                    }
                }
            }
            uint8_t* rp8 = wp + (size_t)r * pitch;
            if (npx == 8) {
                if (nc == 1) { Words2 e; e.a = w[0]; e.b = w[1]; *reinterpret_cast<Words2*>(rp8) = e; }
                else {
                    Words4 e; e.a = w[0]; e.b = w[1]; e.c = w[2]; e.d = w[3];
                    Words2 f; f.a = w[4]; f.b = w[5];
                    *reinterpret_cast<Words4*>(rp8) = e; *reinterpret_cast<Words2*>(rp8 + 16) = f;
                }
            } else {                                        // the image's last, narrower column of cells
                const uint32_t nb = npx * nc;
                for (uint32_t i = 0; i < nb; i++) {
                    const uint32_t wi = i >> 2;
                    const uint32_t word = wi == 0 ? w[0] : (wi == 1 ? w[1] : (wi == 2 ? w[2] : (wi == 3 ? w[3] : (wi == 4 ? w[4] : w[5]))));
                    rp8[i] = (uint8_t)(word >> (8 * (i & 3)));
                }
            }
        }
    }
}

// --------------------------------------------------------------------------------------
// k_pixel_tail: decode and training tail in one kernel, so that the full-resolution pixels never reach memory.
// One workgroup (128 lanes) per run of MCUs of an MCU row, one lane per block and the samples in two halves as in k_pixel; the pixels of
// the run, rounded as k_pixel rounds them (the tail is defined on the rounded pixels), go to LDS as a word each, and the output
// samples whose two source rows both lie in this MCU row are interpolated from those.  The runs of a row begin at the box's first
// MCU and overlap by one: a run serves the source columns of all its MCUs but the last one, which it holds only as the right-hand
// neighbour (an output sample reads columns xa and xa + 1), and the run that reaches the box's last MCU serves that one too.
// Output rows whose two source rows lie in two MCU rows cannot be served by either: every run leaves its first and last pixel
// row (1/8 of the pixels for 16-row MCUs) in a side buffer, and k_tail_edges interpolates those rows from it afterwards.
//   edge: side buffer, a word per pixel; image i's part starts at edge_off[i] and holds, per MCU row r, its first pixel row at
//         (2 r) * W and its last one at (2 r + 1) * W.
// MCU rows, runs and MCUs that do not touch the image's box are not decoded at all.
// Bound by vector issue at three to four wavefronts per SIMD.  LDS is asked for by what the widest run of the record takes: 21 KB for 21
// MCUs of 4:2:0, 3 KB for pictures of 26 x 26; the pixels of both halves wait in registers and take the samples' place (with room
// for both, 39 KB, 512 photographs took 529 us), and every wavefront finds the output rows and columns for itself by ballots (with
// atomics in LDS: 318).  us a launch, with a workgroup of 256 lanes and 64 KB per MCU row that converted four pixels for every output
// sample, and now: 512 photographs to 224 x 224 at scan group 5 342 / 227, at 10 390 / 290; 2048 of 26 x 26 to 96 311 / 92; 1485 of 57 x 32
// to 160 385 / 126; 2048 of 169 x 126 to 160 622 / 193; 2048 of 64 x 64 to 224 1067 / 270; 300 gray of 300 to 500 180 / 64; 200 of
// 4:4:4 180 / 124; 64 of 1024 x 1024 to 224 123 / 123 (kTailSparse).
// --------------------------------------------------------------------------------------
constexpr int kTailLanes = kPixLanes;
// Colour pictures whose box has this many rows to an output row and more: an output row wants two of them, so a third of the rows and more
// is wanted by nobody, and a lane has a group of one wanted row instead of one of two rows.  us a launch, all rows / the wanted ones: 64 of 1024 x 1024 to 224 x 224
// 133 / 123, to 96 123 / 98; us a call: 512 photographs to 128 500 / 500 (a few boxes above the line), 100 of 700 x 800 to 96 374 / 363.  (From twofold
// on: gray pictures of 400 x 400 to 180 638 / 645, colour ones the same; gray pixels are hardly any work, to 64 625 / 629.)
constexpr int kTailSparse = 3;
struct TailParams { int out_h, out_w; float mean[3], istd[3]; };
// MCUs of a run, runs of an MCU row (whatever its box), and LDS of a workgroup: the samples of half a run, and its pixels in their place
PCR_HD uint32_t tail_run(const ImgDesc& d) { const uint32_t per = pixel_mcus_per_tile(d); return per < d.mcux ? per : d.mcux; }
PCR_HD uint32_t tail_runs(const ImgDesc& d) { const uint32_t per = tail_run(d); return per < d.mcux ? (d.mcux - 2u) / (per - 1u) + 1u : 1u; }
PCR_HD uint32_t tail_lds(const ImgDesc& d) {
    const uint32_t samples = pixel_mcu_samples(blocks_per_mcu(d), pixel_row_groups(d.nc, d.hmax)), pixels = 64u * d.hmax * d.vmax;
    return 4u * tail_run(d) * (samples > pixels ? samples : pixels);
}

// One output sample of every channel from four pixels (bytes 0, 1, 2 of a word).
PCR_D void tail_store(__half* dst, size_t channel, uint32_t nc, uint32_t aa, uint32_t ab, uint32_t ba, uint32_t bb, const TailTap& x, const TailTap& y, const TailParams& P) {
#pragma unroll
    for (uint32_t c = 0; c < kMaxComp; c++) {
        auto of = [c](uint32_t w) { return (float)((w >> (8 * c)) & 255u); };
        if (c < nc) dst[c * channel] = tail_value(of(aa), of(ab), of(ba), of(bb), x, y, P.mean[c], P.istd[c]);
    }
}

// Output samples whose first tap (before the box's edge samples are repeated) can lie at first + from .. first + to - 1: [lo, hi), a few more
// than those.
PCR_D void tail_range(int out, int size, int from, int to, int* lo, int* hi) {
    const float per = (float)out / (float)size;              // (out is 8192 at most, so that what rounding moves is far below one)
    *lo = max(0, (int)floorf((float)from * per) - 2);
    *hi = min(out, (int)floorf(((float)to + 0.5f) * per) + 2);
}

template <bool kRefine, bool kGray>
__global__ void __launch_bounds__(kTailLanes, 4) k_pixel_tail(DevRecord R, const PixelTile* __restrict__ tiles, const ApplyList* __restrict__ lists,
                                                              const int32_t* __restrict__ list_idx, const CropBox* __restrict__ boxes, TailParams P,
                                                              __half* __restrict__ out, uint32_t* __restrict__ edge, const uint64_t* __restrict__ edge_off) {
    extern __shared__ __attribute__((aligned(16))) float tile[];             // samples of half the pixel rows of the run; then its pixels
    __shared__ __attribute__((aligned(16))) float qz[kMaxComp][68];
    __shared__ ApplyList rl[kRefine ? kMaxComp : 1];
    short_kernel_priority();
    const uint32_t item = xcd_major(blockIdx.x, gridDim.x);
    const uint32_t timg = uni(tiles[item].img), mcu0 = uni(tiles[item].mcu0);     // (mcu0: MCU row * MCUs per row + number of the run)
    hand_out_status(R, timg, mcu0);
    const uint32_t tid = threadIdx.x;
    ImgDesc D;
    load_desc(R.img + timg, &D);
    const bool dead = load_const(&R.status[timg]) != kOk;
    const uint64_t coef0 = load_const(&R.coef_off[timg]), edge0 = load_const(&edge_off[timg]);
    CropBox b;
    b.x0 = load_const(&boxes[timg].x0); b.y0 = load_const(&boxes[timg].y0); b.w = load_const(&boxes[timg].w); b.h = load_const(&boxes[timg].h); b.flip = load_const(&boxes[timg].flip);
    wanted_now(D); wanted_now((uint32_t)dead); wanted_now(coef0); wanted_now(edge0);
    wanted_now((uint32_t)b.x0); wanted_now((uint32_t)b.y0); wanted_now((uint32_t)b.w); wanted_now((uint32_t)b.h); wanted_now((uint32_t)b.flip);
    PixGeom G;
    pix_geom(D, &G);
    const uint32_t nc = kGray ? 1u : 3u, W = G.W, H = G.H, mcux = G.mcux, bpm = G.bpm;
    const uint32_t mcu_px_w = 8 * G.hmax, mcu_px_h = 8 * G.vmax;
    if (bpm == 0 || bpm > 12 || G.nc != nc) return;         // (cannot happen for an image the parser accepted)
    const uint32_t gpm = pixel_row_groups(nc, G.hmax), per = pixel_mcus(bpm, gpm), run = per < mcux ? per : mcux;
    const uint32_t my = mcu0 / mcux, seg = mcu0 - my * mcux;
    const uint32_t ylo = my * mcu_px_h, yhi = ylo + mcu_px_h < H ? ylo + mcu_px_h : H;   // pixel rows of this MCU row
    b = clamp_box(b, (int)W, (int)H);
    if ((int)ylo >= b.y0 + b.h || (int)yhi <= b.y0) return;
    const uint32_t mc0 = (uint32_t)b.x0 / mcu_px_w, mc1 = (uint32_t)(b.x0 + b.w - 1) / mcu_px_w;   // MCUs the box touches
    const uint32_t s0 = mc0 + seg * (run - 1);              // the run: MCUs s0 .. s1
    if (seg != 0 && s0 >= mc1) return;                      // (the run before this one reaches the box's last MCU)
    const uint32_t s1 = min(s0 + run - 1, mc1), nm = s1 - s0 + 1;
    const bool last = s1 == mc1;
    // ---- the lane's block and its loads, the tables, as in k_pixel ----
    PixQuant Q;
    pix_quant_where(D, &Q);
    PixSteps steps;
    pix_quant_load(R, Q, nc, tid, &steps);
    const uint32_t m = (tid * recip16(bpm)) >> 16, j = tid - m * bpm;
    const bool mine = !dead && m < nm;
    PixBlock B;
    uint32_t by = 0, bx = 0;
    uint4 v[8];
    int16_t dc = 0;
    if (mine) {
        pix_block(R, G, coef0, j, my, s0 + m, &B, &by, &bx);
        dc = pix_load(B, v);
    }
    if (kRefine) pix_lists(lists, list_idx, timg, nc, rl, tid);
    pix_quant_table(Q, steps, nc, qz, tid, kTailLanes);
    const uint32_t lane = tid & 63u;
    const uint32_t xorg = s0 * mcu_px_w;                    // image column of the run's first pixel
    const int xs = max(b.x0, (int)xorg), xe = last ? b.x0 + b.w : (int)(s1 * mcu_px_w);      // source columns served here: [xs, xe)
    // output rows and columns served here, [lo, hi) x [left, right): every wavefront looks by itself (with lanes of both and atomics in LDS it
    // took longer)
    // Sparse: pixel rows that no output row and no neighbouring MCU row wants are not converted (wanted: a bit per row).
    int lo = 1 << 30, hi = 0, left = 1 << 30, right = 0;
    const bool above = (int)ylo > b.y0, below = (int)yhi < b.y0 + b.h, sparse = !kGray && b.h >= kTailSparse * P.out_h;
    uint32_t wanted = sparse ? (above ? 1u : 0u) | (below ? 1u << (yhi - 1 - ylo) : 0u) : ~0u;
    {
        int o0, o1;
        tail_range(P.out_h, b.h, (int)ylo - b.y0, (int)yhi - b.y0, &o0, &o1);
        for (; o0 < o1; o0 += 64) {
            const TailTap y = tail_row(b, min(o0 + (int)lane, P.out_h - 1), P.out_h);
            uint64_t in = __ballot(o0 + (int)lane < o1 && y.a >= (int)ylo && y.b < (int)yhi);
            if (in) { lo = min(lo, o0 + __builtin_ctzll(in)); hi = o0 + 64 - __builtin_clzll(in); }
            for (; sparse && in; in &= in - 1) {
                const int l = __builtin_ctzll(in);
                wanted |= 1u << (__builtin_amdgcn_readlane(y.a, l) - (int)ylo) | 1u << (__builtin_amdgcn_readlane(y.b, l) - (int)ylo);
            }
        }
        tail_range(P.out_w, b.w, xs - b.x0, xe - b.x0, &o0, &o1);
        for (; o0 < o1; o0 += 64) {
            const int o = min(o0 + (int)lane, P.out_w - 1);
            const TailTap x = tail_tap(o, P.out_w, b.x0, b.w);
            const uint64_t in = __ballot(o0 + (int)lane < o1 && x.a >= xs && x.a < xe);
            if (in) { left = min(left, o0 + __builtin_ctzll(in)); right = o0 + 64 - __builtin_clzll(in); }
        }
        if (b.flip && left < right) { const int r = P.out_w - left; left = P.out_w - right; right = r; }
    }
    __syncthreads();                                        // (the tables)
    float S[64];
    const bool flatb = mine && B.zm <= 1;
    if (mine) {
        const ApplyList* rlc = &rl[kRefine ? B.c : 0];
        asm volatile("" : "+v"(dc), "+v"(v[0].x));            // (see k_pixel)
        if (flatb) S[0] = clamp255((float)pix_dc<kRefine>(R, B, dc, rlc) * qz[B.c][0] + 128.f);
        else pix_samples<kRefine>(R, B, v, dc, qz[B.c], rlc, S);
    }
    // ---- the run's pixels: a lane per group of two pixel rows, the upper half of the rows, then the lower; kept in registers until the
    // samples of both halves have been read, because the pixels take their place ----
    const uint32_t mstride = pixel_mcu_samples(bpm, gpm), pitch = run * mcu_px_w;
    const uint32_t shx0 = G.hs[0] == G.hmax ? 0 : 1, shy0 = G.vs[0] == G.vmax ? 0 : 1;       // sampling factors are 1 or 2
    const uint32_t shx1 = nc > 1 && G.hs[1] != G.hmax, shy1 = nc > 1 && G.vs[1] != G.vmax;
    const uint32_t shx2 = nc > 2 && G.hs[2] != G.hmax, shy2 = nc > 2 && G.vs[2] != G.vmax;
    const uint32_t ppg = kGray ? 8u : 4u, lg = gpm == 4 ? 2u : (gpm == 2 ? 1u : 0u), half_h = mcu_px_h >> 1;
    const uint32_t items = nm * (half_h >> 1) * gpm, rcpn = nm > 1 ? 0xFFFFFFFFu / nm + 1u : 0u;
    constexpr uint32_t kTrips = 3;                          // (24 MCUs of five blocks, 16 x 16 pixels each, are the most items: 384)
    uint32_t px[2][kTrips][2][3];                           // [half][trip][row]: the group's bytes
    auto fetch = [&](uint32_t c, uint32_t mm, uint32_t ly, uint32_t x0, uint32_t shx, uint32_t shy, float s[4]) {
        if (G.flat[c]) {
            const float f = tile[mm * mstride + (G.rb[c] >> 1) + ((x0 >> shx) >> 3) * 8];
            s[0] = s[1] = s[2] = s[3] = f;
        } else four_samples(tile + mm * mstride + (G.rb[c] >> 1) + (ly >> shy) * G.rs[c], x0, shx, s);
    };
    // the pixels of a group in one row (of the half whose samples lie in LDS)
    auto convert = [&](uint32_t mm, uint32_t ly, uint32_t x0, uint32_t w[3]) {
        if (kGray) {
#pragma unroll
            for (uint32_t h = 0; h < 2; h++) {
                float a[4];
                fetch(0, mm, ly, x0 + 4 * h, 0, 0, a);
                w[h] = four_u8(a[0], a[1], a[2], a[3]);
            }
        } else {
            float ys[4], cb[4], cr[4];
            fetch(0, mm, ly, x0, shx0, shy0, ys); fetch(1, mm, ly, x0, shx1, shy1, cb); fetch(2, mm, ly, x0, shx2, shy2, cr);
#pragma unroll
            for (int i = 0; i < 4; i++) { cb[i] -= 128.f; cr[i] -= 128.f; }
            rgb_words(ys, cb, cr, w);
        }
    };
    // Sparse: the wanted rows of each half alone, a lane per group of one row: their numbers, four bits each, and how many groups there are.
    uint32_t row_list[2] = {0, 0}, row_items[2] = {0, 0};
    if (sparse) {
#pragma unroll
        for (uint32_t half = 0; half < 2; half++) {
            uint32_t some = (wanted >> (half * half_h)) & ((1u << half_h) - 1u), n = 0;
            for (; some; some &= some - 1, n++) row_list[half] |= (uint32_t)__builtin_ctz(some) << (4 * n);
            row_items[half] = n * nm * gpm;
        }
    }
    // Where group `it` is: its MCU, the number of its row pair (sparse: of its row in the list), its first pixel.
    struct Place { uint32_t mm, n, x0; };
    auto place = [&](uint32_t it) {
        const uint32_t q = it >> lg, n = nm > 1 ? __umulhi(q, rcpn) : q;
        return Place{q - n * nm, n, (it & (gpm - 1)) * ppg};
    };
#pragma unroll
    for (int half = 0; half < 2; half++) {
        if (half) __syncthreads();                          // (the upper half has been read)
        if (mine) {
            float* const dst = tile + m * mstride + (pick3(B.c, G.rb[0], G.rb[1], G.rb[2]) >> 1) + bx * 8;
            if (half == 0) pix_put_half<0>(S, flatb, B.vs, by, dst, B.hs * 8);
            else pix_put_half<1>(S, flatb, B.vs, by, dst, B.hs * 8);
        }
        __syncthreads();
        if (sparse) {
#pragma unroll
            for (uint32_t e = 0; e < 2 * kTrips; e++) {
                const uint32_t it = tid + e * kTailLanes;
                uint32_t* const w = px[half][e >> 1][e & 1];
                w[0] = w[1] = w[2] = 0;
                if (it >= row_items[half] || dead) continue;
                const Place p = place(it);
                convert(p.mm, (row_list[half] >> (4 * p.n)) & 15u, p.x0, w);
            }
        } else {
#pragma unroll
            for (uint32_t t = 0; t < kTrips; t++) {
                const uint32_t it = tid + t * kTailLanes;
                uint32_t (*const w)[3] = px[half][t];
#pragma unroll
                for (int e = 0; e < 6; e++) w[e / 3][e % 3] = 0;
                if (it >= items || dead) continue;
                const Place p = place(it);
#pragma unroll
                for (uint32_t row = 0; row < 2; row++) convert(p.mm, 2 * p.n + row, p.x0, w[row]);
            }
        }
    }
    __syncthreads();
    uint32_t* const words = reinterpret_cast<uint32_t*>(tile);
    auto leave = [&](const Place& p, uint32_t y, const uint32_t w[3]) {
        uint32_t* const to = words + y * pitch + p.mm * mcu_px_w + p.x0;
        if (kGray) {
#pragma unroll
            for (int h = 0; h < 2; h++) *reinterpret_cast<uint4*>(to + 4 * h) = uint4{w[h] & 255u, (w[h] >> 8) & 255u, (w[h] >> 16) & 255u, w[h] >> 24};
        } else                                              // (a word's top byte is another pixel's)
            *reinterpret_cast<uint4*>(to) = uint4{w[0], __builtin_amdgcn_alignbyte(w[1], w[0], 3), __builtin_amdgcn_alignbyte(w[2], w[1], 2), w[2] >> 8};
    };
    if (sparse) {
#pragma unroll
        for (uint32_t e = 0; e < 4 * kTrips; e++) {
            const uint32_t half = e & 1, slot = e >> 1, it = tid + slot * kTailLanes;
            if (it >= row_items[half]) continue;
            const Place p = place(it);
            leave(p, half * half_h + ((row_list[half] >> (4 * p.n)) & 15u), px[half][slot >> 1][slot & 1]);
        }
    } else {
#pragma unroll
        for (uint32_t e = 0; e < 4 * kTrips; e++) {
            const uint32_t half = e & 1, row = (e >> 1) & 1, t = e >> 2, it = tid + t * kTailLanes;
            if (it >= items) continue;
            const Place p = place(it);
            leave(p, half * half_h + 2 * p.n + row, px[half][t][row]);
        }
    }
    __syncthreads();
    // ---- the first and the last pixel row, for the output rows that need a neighbouring MCU row as well ----
    {
        const int span = xe - xs;
        uint32_t* const e = edge + edge0 + (size_t)(2 * my) * W + xs;
        const uint32_t* const w = words + (xs - (int)xorg);
        for (int x = (int)tid; x < span; x += kTailLanes) {
            if (above) e[x] = w[x];
            if (below) e[W + x] = w[(yhi - 1 - ylo) * pitch + x];
        }
    }
    // ---- the output samples: a lane per column, a wavefront per row; the rows' taps 64 at a time, a lane each, and handed over ----
    const int wave = (int)uni(tid >> 6);
    const size_t channel = (size_t)P.out_h * P.out_w;
    for (int rows0 = lo; rows0 < hi; rows0 += 64) {
        const TailTap mine_y = tail_row(b, min(rows0 + (int)lane, P.out_h - 1), P.out_h);
        const uint32_t ra_l = (uint32_t)(mine_y.a - (int)ylo) * pitch, rb_l = (uint32_t)(mine_y.b - (int)ylo) * pitch;
        const int rows = min(hi - rows0, 64);
        for (int ox = left + (int)lane; ox - (int)lane < right; ox += 64) {
            const TailTap x = tail_col(b, min(ox, P.out_w - 1), P.out_w);
            const uint32_t* const wa = words + min(max(x.a - (int)xorg, 0), (int)pitch - 1);
            const uint32_t* const wb = words + min(max(x.b - (int)xorg, 0), (int)pitch - 1);
            __half* dst = out + (size_t)timg * nc * channel + (size_t)rows0 * P.out_w + ox;
            for (int i = wave; i < rows; i += kTailLanes / 64) {           // (all lanes: the taps come across them)
                auto from = [i](uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, i); };
                const uint32_t ra = from(ra_l), rb = from(rb_l);
                TailTap y;
                y.f = __uint_as_float(from(__float_as_uint(mine_y.f))); y.g = __uint_as_float(from(__float_as_uint(mine_y.g)));
                if (ox < right) tail_store(dst + (size_t)i * P.out_w, channel, nc, wa[ra], wb[ra], wa[rb], wb[rb], x, y, P);
            }
        }
    }
}

// The output rows k_pixel_tail could not serve: their two source rows are the last pixel row of one MCU row and the first
// of the next, both in the side buffer.  One workgroup per (boundary between MCU rows, image); those outside the box leave at once.
// (One per output row and image, most of which had nothing to do: 31.6 us for 512 photographs to 224 x 224 where it takes 18, 103 and 39
// for 2048 pictures of 64 x 64.)
__global__ void __launch_bounds__(64) k_tail_edges(const uint32_t* __restrict__ dims, const uint32_t* __restrict__ mcu_rows_px, uint32_t nc,
                                                   const CropBox* __restrict__ boxes, TailParams P, const uint32_t* __restrict__ edge,
                                                   const uint64_t* __restrict__ edge_off, __half* __restrict__ out) {
    const uint32_t i = blockIdx.y, r = blockIdx.x, lane = threadIdx.x;        // between MCU rows r and r + 1
    const int W = (int)dims[2 * i], H = (int)dims[2 * i + 1];
    const int below = (int)((r + 1) * mcu_rows_px[i]);      // the first pixel row of the lower one
    const CropBox b = clamp_box(boxes[i], W, H);
    if (below <= b.y0 || below >= b.y0 + b.h) return;
    const uint32_t* const rowa = edge + edge_off[i] + (size_t)(2 * r + 1) * W;
    const uint32_t* const rowb = rowa + W;
    const size_t channel = (size_t)P.out_h * P.out_w;
    for (int oy0 = 0; oy0 < P.out_h; oy0 += 64) {
        const TailTap at = tail_row(b, min(oy0 + (int)lane, P.out_h - 1), P.out_h);
        for (uint64_t todo = __ballot(oy0 + (int)lane < P.out_h && at.a + 1 == below && at.b == below); todo; todo &= todo - 1) {
            const int from = __builtin_ctzll(todo);
            TailTap y;
            y.f = __shfl(at.f, from); y.g = __shfl(at.g, from);
            for (int ox = (int)lane; ox < P.out_w; ox += 64) {
                const TailTap x = tail_col(b, ox, P.out_w);
                tail_store(out + (size_t)i * nc * channel + (size_t)(oy0 + from) * P.out_w + ox, channel, nc, rowa[x.a], rowa[x.b], rowb[x.a], rowb[x.b], x, y, P);
            }
        }
    }
}

// --------------------------------------------------------------------------------------
// k_gather: copy regions 1..have of one image back to back, append FF D9 if asked.
// --------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_gather(DevRecord R, uint32_t i, uint32_t have, int add_eoi, uint8_t* dst) {
    uint32_t w = 0;
    for (uint32_t g = 0; g < have; g++) {
        uint32_t p = R.off[(size_t)g * R.n + i], L = R.len[(size_t)g * R.n + i];
        for (uint32_t j = blockIdx.x * 256 + threadIdx.x; j < L; j += gridDim.x * 256) dst[w + j] = R.rec[p + j];
        w += L;
    }
    if (add_eoi && blockIdx.x == 0 && threadIdx.x == 0) { dst[w] = 0xFF; dst[w + 1] = 0xD9; }
}

// --------------------------------------------------------------------------------------
// k_probe_scalar: yardstick for the entropy kernels.  Every wavefront runs `iters` times a chain of 16
// dependent scalar instructions, the same kind of work a wave-uniform decoder is made of; the host
// turns the duration into scalar instructions per second for a given number of wavefronts per CU.
// --------------------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_probe_scalar(uint32_t* out, uint32_t iters, uint32_t seed) {
    uint32_t a = uni(seed + blockIdx.x), b = a * 3u + 1u;
    for (uint32_t i = 0; i < iters; i++) {
        asm volatile(
            "s_add_u32 %0, %0, %1\n s_xor_b32 %1, %1, %0\n s_add_u32 %0, %0, %1\n s_xor_b32 %1, %1, %0\n"
            "s_add_u32 %0, %0, %1\n s_xor_b32 %1, %1, %0\n s_add_u32 %0, %0, %1\n s_xor_b32 %1, %1, %0\n"
            "s_add_u32 %0, %0, %1\n s_xor_b32 %1, %1, %0\n s_add_u32 %0, %0, %1\n s_xor_b32 %1, %1, %0\n"
            "s_add_u32 %0, %0, %1\n s_xor_b32 %1, %1, %0\n s_add_u32 %0, %0, %1\n s_xor_b32 %1, %1, %0\n"
            : "+s"(a), "+s"(b) : : "scc");
    }
    if (threadIdx.x == 0) out[blockIdx.x] = a ^ b;
}

}  // namespace pcr
