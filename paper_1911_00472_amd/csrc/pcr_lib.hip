// C ABI of the PCR decode library (see include/pcr.h) and the host logic behind it: header
// validation, layout of the device buffers, the work lists that map lanes to restart
// intervals, and the kernel launches.  Everything data-dependent runs in the kernels of
// pcr_kernels.h; the host parse done in pcr_open only sizes buffers and rejects bad input early.
#include <hip/hip_runtime.h>
#include <fcntl.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "../../include/pcr.h"
#include "pcr_chains.h"
#include "pcr_kernels.h"
#include "pcr_sequential.h"
#include "pcr_first_split.h"
#include "pcr_hist.h"
#include "pcr_coder.h"
#include "pcr_similarity.h"
#include "pcr_encode.h"

using namespace pcr;

#define HIP_TRY(expr) do { if ((expr) != hipSuccess) { (void)hipGetLastError(); return PCR_E_DEVICE; } } while (0)

namespace {

enum Kind { kDcFirst = 0, kAcFirst = 1, kAcRefine = 2, kSequential = 3, kNumKinds = 4 };
enum SplitBy { kSplitNever = 0, kSplitBySteps = 1, kSplitByTries = 2 };
// Blocks of an MCU of a sequential scan: the tries of a piece (k_split_tries).
uint32_t split_tries_of(const ImgDesc& im, const ScanDesc& sd) {
    uint32_t tries = 0;
    for (int j = 0; j < sd.ns; j++) tries += sd.ns == 1 ? 1u : (uint32_t)im.hs[sd.comp[j]] * im.vs[sd.comp[j]];
    return std::max(1u, tries);
}
// Whether the tries would not fall into step: eight blocks are not enough where a block is of many bits, and what is decoded on outgrows its room (the more
// the longer the scan).  Such units go in steps, and so does, behind the tries, whatever else they leave: 85 ms for four of 1.5 MB at quality 99, 166 for one of 3.2 MB,
// when one wavefront took what the tries left, and 10 and 15 in steps.  ms by tries, and in steps behind them where they left any / in steps / one wavefront:
//                      bits a block:  350 ..                 380 ..                 400 ..                 420 ..                 440 ..
//   4:2:0, 24 to 37 KB       4 of  0.9 / 3.3 / 1.5        1.1 / 1.9 / 1.6        1.4 / 1.9 / 1.7        1.5 / 2.0 / 1.7        2.0 / 2.0 / 1.7
//          52 to 82          4     1.4 / 3.8 / 3.4        1.5 / 4.0 / 3.5        1.6 / 4.0 / 3.6        1.8 / 4.2 / 3.7        2.4 / 4.2 / 3.8
//          93 to 146         4     1.2 / 8.7 / 5.9        1.6 / 6.9 / 6.2        2.3 / 7.0 / 6.3        9.2 / 7.2 / 6.5        8.4 / 7.3 / 6.6
//          230 to 366        4     1.9 / 22 / 15          2.7 / 23 / 16          9.5 / 6.6 / 17         25 / 23 / 16           26 / 25 / 17
//          570 to 910        4     2.9 / 7.2 / 37         3.2 / 7.0 / 38         14 / 10 / 39           12 / 9.9 / 40          17 / 14 / 41
//          2.2 to 3.6 MB     1     9.1 / 10 / 145         13 / 14 / 153          25 / 15 / 153          27 / 20 / 159          28 / 21 / 162
//   4:4:4, 41 to 73 KB       4     1.5 / 3.7 / 3.2        1.8 / 3.7 / 3.3        1.6 / 3.8 / 3.3        1.6 / 3.8 / 3.4        6.0 / 3.9 / 3.6
//          163 to 293        4     2.6 / 5.4 / 13         2.9 / 5.3 / 13         20 / 19 / 13           21 / 19 / 13           16 / 15 / 14
//          1.0 to 1.8 MB     4     3.6 / 6.1 / 76         11 / 8.2 / 80          15 / 9.4 / 82          13 / 10 / 83           15 / 14 / 87
bool split_dense(const ImgDesc& im, const ScanDesc& sd, uint32_t each) {
    const uint64_t blocks = std::max<uint64_t>((uint64_t)split_tries_of(im, sd) * sd.mcus, 1);
    const uint32_t line = each < 100000u ? 445u : (each < 150000u ? 426u : (each < 350000u ? 405u : (each < 1000000u ? 385u : 372u)));
    return 8ull * sd.data_len > line * blocks;
}
// The long sequential scans of a launch: many lanes each, or one wavefront?  k_sequential takes as long as its longest scan until some thousand of them fill the
// scalar units.  k_sequential_split has room for one scan per compute unit (150 KB of LDS), 256 at a time, and a step takes as long as its
// slowest lane.  k_split_tries and what follows use the whole chip for few scans, but decode up to thirteen times what one decoder would.
// ms for n files, by tries / k_sequential_split / k_sequential (the whole call; -: not measured):
//                        n = 1              32             128            512            2048
//   4:2:0, 166 KB    0.9/ 1.9/17     1.1/ 2.4/17    1.9/ 2.3/17    5.0/ 4.6/ -      -  /16.1/ -
//   4:2:0, 50 KB     0.7/ 1.6/5.1    0.9/ 2.1/5.1   0.9/ 2.0/5.1   2.0/ 3.7/ -     8.4/ -  /4.3
//   4:2:0, 19 KB     0.6/ 1.4/1.9    0.8/ 1.6/1.9   0.8/ 1.5/1.9   1.2/ 2.3/1.4    6.4/ -  /1.7
//   4:4:4, 203 KB    0.8/ 1.3/21     1.0/ 1.4/21    1.9/ 1.4/ -    4.8/ 3.1/ -      -  /11.7/ -
//   q 97, 99 KB      1.5/ 6.2/5.3    1.6/ 6.4/5.4   1.6/ 6.4/5.5   4.0/ 7.3/ -      -  /12.6/ -
//   gray, 163 KB     0.8/ 0.8/17     0.9/ 1.2/17    1.1/ 1.1/17    2.6/ 2.2/ -      -  / 8.2/ -
//   2.5 MP, 1.8 MB   3.6/ 6.5/ -     4.9/ 8.0/ -   11.0/ 8.5/ -   45.8/21.4/ -      -
// (steps at quality 97: given up, and decoded by k_sequential behind it.)  What the lines below say follows these figures (in us; kb: the mean of
// the long scans); where every MCU is one block there is one try, and nothing to be had of them.  A record decoded beside others shares
// the compute units with them; the records the process has open (four at most count) are taken as the sign of it, as by
// lanes_pay.  (Without this choice 4096 baseline photographs in four records took 29.1 ms instead of 23.2.)
//
// The tries work in memory of the record (SplitSpace), which it has where some number of open records would have them chosen.
struct SplitLaunch {
    uint32_t units = 0, dense = 0; uint64_t bytes = 0, dense_bytes = 0, tried = 0, blocks = 0, mcu_blocks = 0;       // dense: of the units; tried: bits to be decoded, once per try; blocks, and those of an MCU, of all units
    float work = 0; bool subsampled = false, several = false;       // us by tries with the chip full; some MCUs of several blocks per component, of several blocks
    // `count` units of a scan, of so many bytes each on average; false: they are not long
    bool add(const ImgDesc& im, const ScanDesc& sd, uint32_t each, uint32_t count) {
        if ((uint64_t)each * 8 < kSplitLeastBits) return false;
        const uint32_t tries = split_tries_of(im, sd);
        units += count; bytes += (uint64_t)each * count; blocks += (uint64_t)tries * sd.mcus; mcu_blocks += (uint64_t)tries * count;
        subsampled = subsampled || tries > (uint32_t)im.nc; several = several || tries > 1;
        if (split_dense(im, sd, each)) { dense += count; dense_bytes += (uint64_t)each * count; return true; }
        tried += (uint64_t)tries * each * 8 * count;
        work += (22.f + 4.5f * (float)tries) * 1e-6f * (float)each * (float)count;
        return true;
    }
    // us in steps of so many units, with those of other records beside them.  (Faster the fewer blocks an MCU has and the fewer bits a block: fewer places
    // to be off by, and more blocks to a piece.  ms by tries / in steps, 128 and 300 files of 4:2:0: 50 KB at 247 bits a block 1.0 / 2.0 and 1.6 / 3.2; 98 KB at 193
    // 1.2 / 1.4 and 2.5 / 2.3; 147 KB at 135 1.6 / 1.4 and 2.9 / 2.4; 87 KB at 113 1.1 / 1.4; of 4:2:2, 96 KB at 230 1.0 / 1.2 and 1.9 / 1.8, 99 KB at 150 0.9 / 0.8.)
    float steps(uint32_t count, uint64_t all, float beside) const {
        const float kb = (float)all / (float)count / 1000.f, turns = std::ceil((float)count * beside / 256.f);
        const float long_kb = std::max(0.f, kb - 300.f);     // (a lane's piece is beyond a wrong block then)
        if (!subsampled) return 150.f + turns * (260.f + 4.5f * kb);
        const float a_block = (float)bytes * 8.f / (float)std::max<uint64_t>(blocks, 1), an_mcu = (float)mcu_blocks / (float)units;
        return std::min(1.f, std::max(0.62f, a_block / 270.f)) * std::min(1.f, an_mcu / 6.f) * (550.f + turns * (850.f + 6.f * kb - 3.f * long_kb));
    }
    // room: the tries have memory to work in
    SplitBy by(int open_records, bool room) const {
        if (units == 0) return kSplitNever;
        const float beside = (float)std::min(4, std::max(1, open_records)), n = (float)units * beside, kb = (float)bytes / (float)units / 1000.f;
        const float tries = 150.f + std::ceil((float)(units - dense) * beside / 256.f) * 400.f + beside * work + (dense ? steps(dense, dense_bytes, beside) : 0.f);
        const float in_steps = steps(units, bytes, beside), sequential = 102.f * kb * std::max(1.f, 0.72f + n / 3072.f);
        return room && several && units > dense && tries < in_steps && tries < sequential ? kSplitByTries : (in_steps < sequential ? kSplitBySteps : kSplitNever);
    }
    bool by_tries_perhaps() const {
        for (int open_records = 1; open_records <= 4; open_records++) if (by(open_records, true) == kSplitByTries) return true;
        return false;
    }
    // Pieces are as long as that a launch of few scans fills the chip once, within what the constants say.
    uint32_t piece_bits() const { return (uint32_t)std::min<uint64_t>(kSplitPieceMost, tried / (256 * kSplitLanes)); }
};
// Room for a unit of `bytes` of a scan, in pieces of `least` bits and more.  (More nodes are decoded on than half of those a unit begins with
// hardly ever.)
SplitRoom split_room_of(const ImgDesc& im, const ScanDesc& sd, uint32_t bytes, uint32_t least, bool dense) {
    SplitRoom room{};
    room.tries = split_tries_of(im, sd);
    if (dense) { room.pieces = 1; room.tries = 0; return room; }
    const uint64_t blocks = std::max<uint64_t>((uint64_t)room.tries * sd.mcus, 1);
    room.run_in = (uint32_t)std::min<uint64_t>(kSplitRunInMost, std::max<uint64_t>(kSplitRunInLeast, kSplitRunInBlocks * 8 * (uint64_t)sd.data_len / blocks));
    room.least = std::max(room.run_in, least);
    room.pieces = std::min<uint32_t>(std::min(kSplitPieces, kSplitFirstNodes / room.tries), (uint32_t)((uint64_t)bytes * 8 / room.least + 1));
    const uint32_t first = room.pieces * room.tries;
    room.nodes = std::min(kSplitNodes, first + first / 2 + 1024);
    return room;
}
// Nodes and pieces of several units.
struct SplitSpace {
    uint64_t nodes = 0; uint32_t pieces = 0;
    void add(const SplitRoom& room) { nodes += room.nodes; pieces += room.pieces + 1; }
    bool holds(const SplitSpace& o) const { return o.nodes <= nodes && o.pieces <= pieces; }
};

struct LevelList {
    Unit* d_units = nullptr; uint32_t n = 0; int kind = 0;
    uint32_t level = 0;                                                          // (0-based)
    uint32_t plane_tile = 0, n_plane_tiles = 0, cov_tile = 0, n_cov_tiles = 0;    // AC refinement: the level's share of the plan's lists for the per-block kernels
    LaneJob* d_jobs = nullptr; uint32_t n_jobs = 0;                              // the same units cut into jobs of a lane-per-unit kernel
    uint32_t* d_done = nullptr;                                                  // sequential scans, some of them long: which units have been dealt with by many lanes
    // ... how many those are at most and what they are judged by; by tries, if there is room for them, the rooms of those units, and the most workgroups a unit needs
    SplitLaunch seq;
    SplitRoom* d_rooms = nullptr; uint32_t split_tries = 0, split_stores = 0; bool by_tries = false;
    DcLaunch dc;                                                                 // DC first scans: what decides between lanes and wavefronts
    uint32_t* d_dc_starts = nullptr; uint32_t n_dc_waves = 0;                    // ... wavefronts of lanes, and where they begin if their MCUs are of several shapes
    bool chained = false;                                                        // the plan's chains hold these units too
    LanesLaunch lanes;                                                           // AC scans: what decides between lanes and wavefronts
    FirstSplitLaunch split;                                                      // DC first scans: what decides whether k_first_split goes ahead (d_done: what it has dealt with)
};

struct Plan {                               // launch geometry for one scan group k
    std::vector<LevelList> levels;
    // the scans decoded side by side (k_decode_waves): AC chains first, the DC units (chains of one) behind them
    Unit* d_chain_units = nullptr; UnitChain* d_chains = nullptr; uint32_t n_ac_chains = 0, n_chains = 0, chain_waves = 0;
    uint32_t trio_waves = 0, trio_lds = 0;   // a workgroup's wavefronts and LDS where refinement scans have three wavefronts each (k_decode_trios)
    uint32_t* d_chain_done = nullptr;        // chains of one: which units k_first_split has dealt with
    FirstSplitLaunch split;                  // ... and what decides whether it is launched
    // the AC refinement scans of the call, level after level, and the lists of the per-block kernels
    RefineScan* d_refine = nullptr;
    RefineTile* d_refine_tiles = nullptr;    // k_refine_history: chunks of the padded planes of those scans; behind them, from cov_tile on,
    uint32_t cov_tile = 0, n_cov_tiles = 0;  // k_refine_deal, k_refine_blocks: chunks of the blocks the images cover
    bool chains_built = false;
    ApplyUnit* d_apply = nullptr; ApplyList* d_apply_lists = nullptr; int32_t* d_list_idx = nullptr; uint32_t n_apply = 0, apply_grid_x = 0;
    bool has_ac = false;                     // some scan <= k is an AC scan (else only element 0 of every block is ever touched)
    bool had_ac = false;                     // ... some scan <= k0 (the fidelity an upgrade starts from)
    bool smooths = false;                    // some component of a progressive image has its DC first scan and no other among the scans <= k
    bool dc_complete = true;                 // every component of every image has its first DC scan among the scans <= k
};

// Device memory of a handle comes out of two arenas (one sized by the image and scan counts, one by the
// images themselves): a block that is handed out front to back and re-used as a whole when the handle is
// bound to another record.  An arena grows only when a record needs more than it holds, so that a loader
// that binds record after record of similar size to one handle stops allocating after the first few.
// What does not fit (work lists of a scan group first asked for when the arena is full) is allocated on
// its own and released at the next reset.
struct Arena {
    uint8_t* base = nullptr; size_t cap = 0, used = 0;
    std::vector<void*> extra;
};
constexpr size_t kArenaAlign = 256;
size_t arena_round(size_t bytes) { return (bytes + kArenaAlign - 1) / kArenaAlign * kArenaAlign; }
void arena_release_extra(Arena* a) { for (void* p : a->extra) (void)hipFree(p); a->extra.clear(); }
void arena_free(Arena* a) { arena_release_extra(a); if (a->base) (void)hipFree(a->base); a->base = nullptr; a->cap = a->used = 0; }
// Empties the arena and makes sure it holds at least `bytes`.  Nothing handed out earlier may still be in use.
int arena_reset(Arena* a, size_t bytes) {
    arena_release_extra(a);
    a->used = 0;
    if (a->cap >= bytes) return PCR_OK;
    if (a->base) (void)hipFree(a->base);
    a->base = nullptr; a->cap = 0;
    const size_t want = bytes + bytes / 8;                    // some room for the next, slightly larger record
    if (hipMalloc((void**)&a->base, want) != hipSuccess) {
        (void)hipGetLastError();
        if (hipMalloc((void**)&a->base, bytes) != hipSuccess) { (void)hipGetLastError(); return PCR_E_NOMEM; }
        a->cap = bytes;
    } else a->cap = want;
    return PCR_OK;
}
template <class T> int arena_alloc(Arena* a, T** p, size_t count) {
    *p = nullptr;
    const size_t bytes = arena_round((count ? count : 1) * sizeof(T));
    if (a->used + bytes <= a->cap) { *p = reinterpret_cast<T*>(a->base + a->used); a->used += bytes; return PCR_OK; }
    void* q = nullptr;
    if (hipMalloc(&q, bytes) != hipSuccess) { (void)hipGetLastError(); return PCR_E_NOMEM; }
    a->extra.push_back(q);
    *p = reinterpret_cast<T*>(q);
    return PCR_OK;
}
// Host memory in which tables are put together before they go to the device.  Pinned where its owner binds record after
// record (a loader's slots), and kept there; elsewhere pageable, and given back once the tables are on the device.
struct HostBlock {
    uint8_t* p = nullptr; size_t cap = 0; bool pinned = false;
    void release() { if (p) { if (pinned) (void)hipHostFree(p); else free(p); } p = nullptr; cap = 0; }
    void done() { if (!pinned) release(); }
    // Room for `bytes`, of which the first `keep` are in use; `exact`: and no more is to be expected.
    int reserve(size_t bytes, size_t keep, bool exact = false) {
        if (bytes <= cap) return PCR_OK;
        const size_t want = exact && !pinned ? bytes : std::max<size_t>(bytes + bytes / 2, 1u << 16);
        uint8_t* q = nullptr;
        if (pinned) { if (hipHostMalloc((void**)&q, want, hipHostMallocDefault) != hipSuccess) { (void)hipGetLastError(); return PCR_E_NOMEM; } }
        else if (!(q = (uint8_t*)malloc(want))) return PCR_E_NOMEM;
        if (keep) std::memcpy(q, p, keep);
        release();
        p = q; cap = want;
        return PCR_OK;
    }
};

// Tables on their way into an arena, all of them sent by one copy: a synchronous copy of pageable memory costs about
// 20 us however small it is, and binding a record and planning its decode took 28 of them (0.75 of 1.16 ms of host time
// for a record of 512 photographs).  flush() is synchronous: the data is on the device when it returns, whatever stream
// uses it next; flush_on() is not, and the block must stay as it is until the stream got there.
class Uploads {
    Arena* a_; HostBlock* h_; size_t used_ = 0; int rc_ = PCR_OK;
    struct Item { void* p; size_t at; };
    std::vector<Item> items_;
    int place(uint8_t** base) {
        if (rc_) return rc_;
        if (items_.empty()) return PCR_OK;
        const int rc = arena_alloc(a_, base, used_);
        if (rc) return rc;
        for (const Item& e : items_) { uint8_t* q = *base + e.at; std::memcpy(e.p, &q, sizeof q); }
        items_.clear();
        return PCR_OK;
    }
public:
    Uploads(Arena* a, HostBlock* h) : a_(a), h_(h) {}
    // About so many bytes are to come: the block grows once instead of with every table that does not fit (each time
    // copying what it holds into pages that have to be mapped first).
    void expect(size_t bytes) { if (!rc_) rc_ = h_->reserve(used_ + bytes, used_, true); }
    // Room for `count` entries, to be filled in before anything else is added (null: out of memory, as the flush will say).
    // *p is set by the flush.
    template <class T> T* make(T** p, size_t count) {
        *p = nullptr;
        const size_t room = arena_round(std::max<size_t>(count, 1) * sizeof(T));
        if (!rc_) rc_ = h_->reserve(used_ + room, used_);
        if (rc_) return nullptr;
        T* at = reinterpret_cast<T*>(h_->p + used_);
        items_.push_back(Item{p, used_});
        used_ += room;
        return at;
    }
    template <class T> void add(T** p, const std::vector<T>& v) {
        T* at = make(p, v.size());
        if (at && !v.empty()) std::memcpy(at, v.data(), v.size() * sizeof(T));
    }
    int flush() {
        uint8_t* base = nullptr;
        if (items_.empty() && !rc_) { h_->done(); return PCR_OK; }
        const size_t bytes = used_;
        int rc = place(&base); used_ = 0;
        if (!rc && hipMemcpy(base, h_->p, bytes, hipMemcpyHostToDevice) != hipSuccess) rc = PCR_E_DEVICE;
        h_->done();
        return rc;
    }
    int flush_on(hipStream_t s) {
        uint8_t* base = nullptr;
        if (items_.empty() && !rc_) return PCR_OK;
        const size_t bytes = used_;
        const int rc = place(&base); used_ = 0;
        if (rc) return rc;
        return hipMemcpyAsync(base, h_->p, bytes, hipMemcpyHostToDevice, s) == hipSuccess ? PCR_OK : PCR_E_DEVICE;
    }
};

}  // namespace

constexpr size_t kTimingRing = 64;
struct CallTiming {
    std::vector<hipEvent_t> ev;                // ev[0] = start of the call, ev[i] = end of interval i
    std::vector<uint8_t> stage;                // stage[i] = stage that interval (ev[i-1], ev[i]) belongs to
    size_t used = 0;                           // events recorded by the call that last used this slot
};

// Records this process has open: the default choice between the two shapes of entropy decoder looks at it (lanes_pay).
static std::atomic<int> g_open_records{0};

struct pcr_record {
    pcr_record() { g_open_records.fetch_add(1, std::memory_order_relaxed); }
    ~pcr_record() { g_open_records.fetch_sub(1, std::memory_order_relaxed); }
    pcr_record(const pcr_record&) = delete;
    pcr_record& operator=(const pcr_record&) = delete;
    int device = 0;
    size_t nbytes = 0;
    RecordHeader hdr{};
    std::vector<uint8_t> header;            // host copy of the metadata block
    std::vector<ImgDesc> img;               // host parse (sizes, validation)
    std::vector<ScanDesc> scan;
    std::vector<uint8_t> level;             // [n][G] dependency level of each scan (1-based)
    std::vector<uint64_t> out_off, coef_off, mask_off;
    std::vector<uint32_t> slot_base, slot_cnt;
    uint64_t n_masks = 0; uint32_t n_slots = 0; uint32_t max_level = 0;
    DevRecord d{};
    HostBlock stage;                        // tables on their way to the device
    Arena small, big;                       // descriptor tables (sized by n and G) / everything sized by the images, and the work lists
    uint8_t* d_rec = nullptr;
    PixelTile* d_tiles = nullptr; uint32_t n_tiles = 0;
    PixelTile* d_flat_tiles = nullptr; uint32_t n_flat_tiles = 0;   // runs of 8x8 pixel cells, for decodes of DC scans only
    uint32_t flat_row_cells = 0;                                    // cells per row of the widest image
    PixelTile* d_flat_rows = nullptr; uint32_t n_flat_rows = 0;     // ... and rows of cells (none if an image is too wide for k_pixel_flat_rows)
    uint32_t* d_dims = nullptr;             // [n][2] width, height (for kernels that run without a decode before them)
    bool entry_units = false;               // some scan has units that start at entry points
    bool several_units = false;             // some scan has several units (restart intervals, entry points): lane decoders are worth considering
    int lane_mode = 0;                      // pcr_set_lane_decoders: 0 by the number of units, 1 wherever possible, -1 never
    int last_lane_launches = 0, last_wave_launches = 0;   // AC entropy launches of the last decode call, by decoder shape
    int last_splits = 0, last_wide_splits = 0;            // ... launches of k_first_split, and those with a thousand lanes a unit
    int last_trios = 0;                                   // ... launches of k_decode_trios
    // what the tries of long sequential scans work in, for one launch at a time: the most that a plan from scratch needs of them
    SplitNode* d_nodes = nullptr; uint32_t* d_next = nullptr; SplitPiece* d_pieces = nullptr; SplitSpace split_space;
    int seq_mode = 0;                                     // pcr_set_sequential_decoders
    struct SeqDone { uint32_t* d_done; uint32_t units; };
    int last_seq = 0; std::vector<SeqDone> last_done;     // how the last decode call decoded its sequential scans (SplitBy + 1), its launches by many lanes
    bool last_past = false, last_fill_past = false;       // ... whether its pixels, and the zero fill, were stored past the caches (pixels_past, rows_past, fill_past)
    std::vector<uint32_t> ent_off_h;        // record offset of every scan's entry points (0: none), as uploaded
    std::vector<uint32_t> unit_bits;        // records opened from host bytes: entropy-coded bits of every unit, by slot (else empty)
    // decode fused with the training tail (allocated at its first call): one tile per run of an MCU row, the side buffer of first
    // and last pixel rows, where each image's part of it starts, pixel rows per MCU row of every image
    PixelTile* d_tail_tiles = nullptr; uint32_t n_tail_tiles = 0;
    uint32_t tail_lds = 0, tail_rows = 0;   // LDS of a workgroup; MCU rows of the tallest image
    uint32_t* d_edge = nullptr; uint64_t* d_edge_off = nullptr; uint32_t* d_mcu_px_h = nullptr;
    float2* d_ssim_part = nullptr;          // per-tile sums of the similarity kernels (allocated at their first call)
    uint8_t* d_planes = nullptr;            // rounded samples per component, for pcr_decode_batch_triangle (allocated at its first call)
    uint8_t* d_gather = nullptr; size_t gather_cap = 0;
    std::map<int, Plan> plans;
    bool timing = false;
    int resident_k = 0;                        // scan group whose planes and masks the last pixel decode left behind (0: none)
    bool borrowed = false;                  // record bytes belong to the caller (pcr_open_device)
    // stage timing: one list of events per call, the last kTimingRing calls are kept
    std::vector<CallTiming> ring;
    uint64_t timed_calls = 0;                  // calls recorded since timing was switched on
    CallTiming* cur = nullptr;                 // the call being enqueued
};

namespace {

void compute_levels(pcr_record* r) {
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    r->level.assign((size_t)n * G, 0);
    r->max_level = 0;
    for (uint32_t i = 0; i < n; i++)
        r->max_level = std::max(r->max_level, scan_levels(&r->scan[(size_t)i * G], r->img[i].nscans, &r->level[(size_t)i * G]));
}

// The AC refinement scans of a plan by level, and how many chunks of 256 blocks their padded planes and the blocks they cover have.
struct RefineLevel { std::vector<RefineScan> scans; uint32_t planes = 0, covs = 0; };
uint32_t refine_chunks(const ImgDesc& im, const ScanDesc& sd, bool whole_plane) {
    const int c = sd.comp[0];
    return ((whole_plane ? (uint32_t)im.bw[c] * im.bh[c] : (uint32_t)im.cw[c] * im.ch[c]) + 255u) / 256u;
}
// The work lists of the per-block kernels of refinement scans: one list of each kind for the plan, which a launch behind all levels
// takes whole and a level its share of.
void refine_tiles(const pcr_record* r, const std::vector<RefineLevel>& levels, Plan* plan, Uploads* up) {
    size_t count = 0;
    uint32_t planes = 0, covs = 0;
    std::vector<uint32_t> plane_at, cov_at;
    for (const RefineLevel& l : levels) {
        plane_at.push_back(planes); cov_at.push_back(covs);
        count += l.scans.size(); planes += l.planes; covs += l.covs;
    }
    if (count == 0) return;
    for (LevelList& ll : plan->levels) {
        if (ll.kind != kAcRefine) continue;
        const RefineLevel& l = levels[ll.level];
        ll.plane_tile = plane_at[ll.level]; ll.n_plane_tiles = l.planes; ll.cov_tile = planes + cov_at[ll.level]; ll.n_cov_tiles = l.covs;
    }
    plan->cov_tile = planes; plan->n_cov_tiles = covs;
    if (RefineScan* at = up->make(&plan->d_refine, count))
        for (const RefineLevel& l : levels) at = std::copy(l.scans.begin(), l.scans.end(), at);
    RefineTile* plane = up->make(&plan->d_refine_tiles, (size_t)planes + covs);
    if (!plane) return;                                      // (the flush says so)
    RefineTile* cov = plane + planes;
    uint32_t e = 0;
    for (const RefineLevel& l : levels)
        for (const RefineScan& q : l.scans) {
            const ImgDesc& im = r->img[q.img];
            const ScanDesc& sd = r->scan[(size_t)q.img * r->hdr.G + q.scan];
            for (uint32_t ch = 0, n = refine_chunks(im, sd, true); ch < n; ch++) *plane++ = RefineTile{e, ch};
            for (uint32_t ch = 0, n = refine_chunks(im, sd, false); ch < n; ch++) *cov++ = RefineTile{e, ch};
            e++;
        }
}

// The chains of a plan (once, when a call first wants them).
int build_chains(pcr_record* r, int k0, int k, Plan* plan) {
    if (plan->chains_built) return PCR_OK;
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    ChainSet chains;
    for (uint32_t i = 0; i < n && chains.possible; i++) {
        const uint32_t upto = std::min<uint32_t>(r->img[i].nscans, (uint32_t)k);
        const size_t at = (size_t)i * G;
        chains.add(i, &r->scan[at], &r->slot_cnt[at], &r->ent_off_h[at], (uint32_t)k0, upto);
    }
    const bool in_step = chains.possible;
    if (!in_step) {                                          // the refinement scans follow level by level
        chains = ChainSet();
        for (uint32_t i = 0; i < n; i++) {
            const size_t at = (size_t)i * G;
            chains.add_level_one(i, &r->scan[at], &r->level[at], &r->slot_cnt[at], (uint32_t)k0, std::min<uint32_t>(r->img[i].nscans, (uint32_t)k));
        }
    }
    for (LevelList& l : plan->levels) l.chained = l.kind != kSequential && (in_step || (l.kind != kAcRefine && l.level == 0));
    std::vector<Unit> units; std::vector<UnitChain> list;
    for (auto* set : {&chains.ac, &chains.dc}) {
        std::stable_sort(set->begin(), set->end(), [](const ScanChain& a, const ScanChain& b) { return a.cost > b.cost; });     // the longest first
        uint32_t count = 0, refines = 0;                     // of the chain before: most are alike
        for (const ScanChain& c : *set) {
            if (c.count != count || c.refines != refines) {
                count = c.count; refines = c.refines;
                const uint32_t trios = (uint32_t)__builtin_popcount(refines);
                plan->chain_waves = std::max(plan->chain_waves, count);
                plan->trio_waves = std::max(plan->trio_waves, count + 2 * trios);
                plan->trio_lds = std::max(plan->trio_lds, count * kWaveTabBytes + trios * (uint32_t)sizeof(TrioRings));
            }
            for (uint32_t j = 0; j < c.units; j++) {
                list.push_back(UnitChain{(uint32_t)units.size(), c.count, c.refines, c.waits});
                for (uint32_t a = 0; a < c.count; a++) units.push_back(Unit{c.img, c.scan[a], j, r->slot_base[(size_t)c.img * G + c.scan[a]]});
            }
        }
        if (set == &chains.ac) plan->n_ac_chains = (uint32_t)list.size();
    }
    plan->n_chains = (uint32_t)list.size();
    if (plan->chain_waves == 1)
        for (auto* set : {&chains.ac, &chains.dc})
            for (const ScanChain& c : *set) plan->split.add(r->img[c.img], r->scan[(size_t)c.img * G + c.scan[0]], c.units);
    Uploads up(&r->big, &r->stage);
    if (plan->n_chains) { up.add(&plan->d_chain_units, units); up.add(&plan->d_chains, list); }
    int rc = up.flush();
    if (!rc && (plan->split.pays(true) || plan->split.pays(false))) rc = arena_alloc(&r->big, &plan->d_chain_done, plan->n_chains);
    if (rc) return rc;
    plan->chains_built = true;
    return PCR_OK;
}

// The rooms of a launch's long sequential scans (runs: the longest first), and whether there are any.
template <class Run> int lay_out_split(pcr_record* r, const std::vector<Run>& runs, LevelList* ll, Uploads* up) {
    const uint32_t G = r->hdr.G, bits = ll->seq.piece_bits();
    std::vector<SplitRoom> rooms;
    rooms.reserve(ll->seq.units);
    SplitSpace space;
    uint32_t tries = 0, stores = 0;
    for (size_t e = 0; e < runs.size() && rooms.size() < ll->seq.units; e++) {
        const Run& q = runs[e];
        const ImgDesc& im = r->img[q.img];
        const ScanDesc& sd = r->scan[(size_t)q.img * G + q.scan];
        SplitRoom room = split_room_of(im, sd, q.bytes, bits, r->seq_mode != 3 && split_dense(im, sd, q.bytes));
        const uint32_t per = kSplitLanes / std::max(1u, room.tries);
        tries = std::max(tries, std::max(1u, (room.pieces - 1 + per - 2) / (per - 1)));
        stores = std::max(stores, (room.pieces + kSplitStoreLanes - 1) / kSplitStoreLanes);
        for (uint32_t j = 0; j < q.count; j++) {
            room.node0 = space.nodes; room.piece0 = space.pieces;
            rooms.push_back(room);
            space.add(room);
        }
    }
    if (!r->split_space.holds(space)) {
        if (r->seq_mode != 3) return PCR_OK;                 // (an upgrade's scans may be cut finer than those from scratch: they go without)
        SplitNode* nodes = nullptr; uint32_t* next = nullptr; SplitPiece* pieces = nullptr;
        int rc = arena_alloc(&r->big, &nodes, space.nodes);
        if (!rc) rc = arena_alloc(&r->big, &next, space.nodes);
        if (!rc) rc = arena_alloc(&r->big, &pieces, space.pieces);
        if (rc) return rc;
        r->d_nodes = nodes; r->d_next = next; r->d_pieces = pieces; r->split_space = space;
    }
    up->add(&ll->d_rooms, rooms);
    ll->split_tries = tries; ll->split_stores = stores; ll->by_tries = true;
    return PCR_OK;
}
// What those of any plan from scratch need at most.
SplitSpace split_space_of(const pcr_record* r) {
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    SplitSpace most;
    for (uint32_t k = 1; k <= G; k++)
        for (uint32_t level = 1; level <= r->max_level; level++) {
            auto each = [&](auto&& f) {
                for (uint32_t i = 0; i < n; i++)
                    for (uint32_t g = 0; g < std::min<uint32_t>(k, r->img[i].nscans); g++) {
                        const size_t ig = (size_t)i * G + g;
                        const uint32_t count = r->slot_cnt[ig];
                        if (r->level[ig] == level && count && is_sequential_scan(r->scan[ig])) f(r->img[i], r->scan[ig], r->scan[ig].data_len / count, count);
                    }
            };
            SplitLaunch launch;
            each([&](const ImgDesc& im, const ScanDesc& sd, uint32_t bytes, uint32_t count) { launch.add(im, sd, bytes, count); });
            if (!launch.by_tries_perhaps()) continue;
            SplitSpace space;
            each([&](const ImgDesc& im, const ScanDesc& sd, uint32_t bytes, uint32_t count) {
                if ((uint64_t)bytes * 8 < kSplitLeastBits) return;
                const SplitRoom room = split_room_of(im, sd, bytes, launch.piece_bits(), split_dense(im, sd, bytes));
                for (uint32_t j = 0; j < count; j++) space.add(room);
            });
            most.nodes = std::max(most.nodes, space.nodes); most.pieces = std::max(most.pieces, space.pieces);
        }
    return most;
}

// Launch geometry for decoding scan groups k0+1 .. k (k0 = 0: from scratch) and turning groups 1 .. k into pixels.
int build_plan(pcr_record* r, int k0, int k, Plan** out) {
    const int key = k0 * 256 + k;
    auto it = r->plans.find(key);
    if (it != r->plans.end()) { *out = &it->second; return PCR_OK; }
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    Plan plan;
    // Per (dependency level, kind of scan), the runs of units that belong to one scan (bytes: the scan's mean per unit):
    // ordering a list scan by scan moves whole runs, a few thousand of them, not hundreds of thousands of units.
    struct Run { uint32_t img, scan, count, bytes, shape; };         // (shape: DC first scans)
    std::vector<std::vector<Run>> runs((size_t)r->max_level * kNumKinds);
    std::vector<DcLaunch> dc(r->max_level);
    std::vector<LanesLaunch> lane_launch(runs.size());
    std::vector<FirstSplitLaunch> dc_split(r->max_level);
    std::vector<RefineLevel> refine_levels(r->max_level);
    std::vector<ApplyUnit> apply; uint32_t max_blk = 0;
    // (what the tables below take: every list is rounded up to kArenaAlign, jobs are one per window of scans at least)
    size_t plan_bytes = runs.size() * 6 * kArenaAlign + 2 * kArenaAlign + (size_t)n * kMaxComp * (sizeof(ApplyUnit) + sizeof(int32_t));
    for (uint32_t i = 0; i < n; i++) {
        const uint32_t upto = std::min<uint32_t>(r->img[i].nscans, (uint32_t)k);
        bool refine[kMaxComp] = {false, false, false};
        uint32_t have_dc = 0, carried[kMaxComp] = {0, 0, 0};
        for (uint32_t g = 0; g < upto; g++) {
            const size_t ig = (size_t)i * G + g;
            const ScanDesc& sd = r->scan[ig];
            for (int j = 0; j < sd.ns; j++) carried[sd.comp[j]]++;
            if (sd.Ah > 0) for (int j = 0; j < sd.ns; j++) refine[sd.comp[j]] = true;
            if (sd.Ss == 0 && sd.Ah == 0) for (int j = 0; j < sd.ns; j++) have_dc |= 1u << sd.comp[j];
            const bool seq = is_sequential_scan(sd);
            if (sd.Ss > 0 || seq) { plan.has_ac = true; if (g < (uint32_t)k0) plan.had_ac = true; }
            if (g < (uint32_t)k0) continue;                    // decoded by an earlier call
            if (sd.Ss == 0 && sd.Ah > 0) continue;             // DC refinement has no serial decode
            const int kind = seq ? kSequential : (sd.Ss == 0 ? kDcFirst : (sd.Ah == 0 ? kAcFirst : kAcRefine));
            const uint32_t cnt = r->slot_cnt[ig];
            if (kind == kAcRefine) {
                RefineLevel& l = refine_levels[r->level[ig] - 1];
                const uint32_t planes = refine_chunks(r->img[i], sd, true), covs = refine_chunks(r->img[i], sd, false);
                l.scans.push_back(RefineScan{i, g}); l.planes += planes; l.covs += covs;
                plan_bytes += sizeof(RefineScan) + sizeof(RefineTile) * (planes + covs);
            }
            const size_t li = (size_t)(r->level[ig] - 1) * kNumKinds + kind;
            uint32_t shape = 0;
            // (what the launches are judged by is gathered here, where the descriptors come one after the other: in the order of the runs, by
            // length, it was a cache miss per scan.  First decode of a record of 1024 pictures of 60 to 90 pixels at scan group 6, us till the call
            // returns: 465 and 437)
            if (kind == kDcFirst) { shape = dc_mcu_shape(r->img[i], sd); dc[r->level[ig] - 1].add(r->img[i], sd, cnt); dc_split[r->level[ig] - 1].add(r->img[i], sd, cnt); }
            else if (!seq) lane_launch[li].add(sd, cnt);
            if (cnt) runs[li].push_back(Run{i, g, cnt, sd.data_len / cnt, shape});
            plan_bytes += cnt * sizeof(Unit) + (cnt / kEntropyLanes + 1) * sizeof(LaneJob);   // (more than dc_units_by_shape's starts take)
        }
        if (have_dc != (1u << r->img[i].nc) - 1u) plan.dc_complete = false;
        for (int c = 0; c < r->img[i].nc; c++) if (carried[c] == 1 && (have_dc >> c & 1) && r->img[i].progressive) plan.smooths = true;
        for (int c = 0; c < r->img[i].nc; c++) if (refine[c]) {
            apply.push_back(ApplyUnit{i, (uint32_t)c});
            max_blk = std::max<uint32_t>(max_blk, (uint32_t)r->img[i].bw[c] * r->img[i].bh[c]);
        }
    }
    Uploads up(&r->big, &r->stage);
    up.expect(plan_bytes);
    plan.levels.reserve(runs.size());                                // (the uploads keep pointers to its members)
    std::vector<uint64_t> order;
    for (size_t li = 0; li < runs.size(); li++) {
        auto& rn = runs[li];
        if (rn.empty()) continue;
        std::stable_sort(rn.begin(), rn.end(), [](const Run& a, const Run& b) { return a.bytes > b.bytes; });   // the scans of the longest units first
        plan.levels.emplace_back();
        LevelList& ll = plan.levels.back();
        ll.kind = (int)(li % kNumKinds);
        for (const Run& q : rn) ll.n += q.count;
        Unit* units = up.make(&ll.d_units, ll.n);
        if (!units) return PCR_E_NOMEM;
        std::vector<LaneJob> jobs;
        const bool lanes = ll.kind == kAcFirst || ll.kind == kAcRefine;
        // Jobs of the lane-per-unit kernels.  A wavefront takes as long as its longest lane, and it holds kLaneTabs
        // Huffman tables: the list (scan after scan, the scans ordered by their mean unit) is cut into windows of
        // kLaneTabs scans, the units of a window are ordered by their own length, and every 64 of them are a job.
        // (without the units' own lengths -- a record opened from device memory -- every unit carries its scan's mean,
        // and the scans are in that order already)
        static_assert(kLaneTabs <= 8, "three bits tell the scans of a window apart");
        const bool by_length = lanes && !r->unit_bits.empty();
        uint32_t at = 0;
        if (ll.kind == kDcFirst) {
            ll.dc = dc[li / kNumKinds];
            const std::vector<uint32_t> starts = dc_units_by_shape((uint32_t)rn.size(), [&](uint32_t e) -> const Run& { return rn[e]; }, kEntropyLanes, [&](uint32_t e, uint32_t j) {
                units[at++] = Unit{rn[e].img, rn[e].scan, j, r->slot_base[(size_t)rn[e].img * G + rn[e].scan]};
            });
            ll.n_dc_waves = starts.empty() ? (ll.n + kEntropyLanes - 1) / kEntropyLanes : (uint32_t)starts.size() - 1;
            if (!starts.empty()) up.add(&ll.d_dc_starts, starts);
            ll.split = dc_split[li / kNumKinds];
            if (ll.split.pays(true)) { const int rc = arena_alloc(&r->big, &ll.d_done, ll.n); if (rc) return rc; }
        }
        for (size_t w0 = 0; w0 < rn.size() && ll.kind != kDcFirst; w0 += kLaneTabs) {
            const size_t w1 = std::min(rn.size(), w0 + kLaneTabs);
            const uint32_t first = at;
            if (by_length) {
                order.clear();
                for (size_t e = w0; e < w1; e++) {
                    const uint32_t sb = r->slot_base[(size_t)rn[e].img * G + rn[e].scan];
                    for (uint32_t j = 0; j < rn[e].count; j++)       // the longest first, equal ones in the order of the scans (unit numbers fit 29 bits)
                        order.push_back((uint64_t)(0xFFFFFFFFu - r->unit_bits[sb + j]) << 32 | (uint64_t)(e - w0) << 29 | j);
                }
                std::sort(order.begin(), order.end());
                for (uint64_t o : order) {
                    const Run& q = rn[w0 + (uint32_t)(o >> 29 & 7)];
                    units[at++] = Unit{q.img, q.scan, (uint32_t)o & 0x1FFFFFFFu, r->slot_base[(size_t)q.img * G + q.scan]};
                }
            } else {
                for (size_t e = w0; e < w1; e++) {
                    const uint32_t sb = r->slot_base[(size_t)rn[e].img * G + rn[e].scan];
                    for (uint32_t j = 0; j < rn[e].count; j++) units[at++] = Unit{rn[e].img, rn[e].scan, j, sb};
                }
            }
            if (!lanes) continue;
            LaneJob job{};
            for (size_t e = w0; e < w1; e++) job.key[job.ntab++] = rn[e].img * G + rn[e].scan;
            for (job.first = first; job.first < at; job.first += kEntropyLanes) {
                job.count = std::min<uint32_t>(kEntropyLanes, at - job.first);
                jobs.push_back(job);
            }
        }
        ll.level = (uint32_t)(li / kNumKinds);
        if (!jobs.empty()) {
            ll.lanes = lane_launch[li];
            ll.n_jobs = ll.lanes.jobs = (uint32_t)jobs.size();
            up.add(&ll.d_jobs, jobs);
        }
        if (ll.kind == kSequential) {
            for (const Run& q : rn) if (!ll.seq.add(r->img[q.img], r->scan[(size_t)q.img * G + q.scan], q.bytes, q.count)) break;      // (the longest on average come first)
            int rc = ll.seq.units ? arena_alloc(&r->big, &ll.d_done, ll.n) : PCR_OK;
            if (!rc && ll.seq.units && (ll.seq.by_tries_perhaps() || r->seq_mode == 3)) rc = lay_out_split(r, rn, &ll, &up);
            if (rc) return rc;
        }
    }
    refine_tiles(r, refine_levels, &plan, &up);
    plan.n_apply = (uint32_t)apply.size();
    plan.apply_grid_x = (max_blk * 64 + kApplyChunk - 1) / kApplyChunk;
    if (plan.n_apply) {
        up.add(&plan.d_apply, apply);
        std::vector<int32_t> list_idx((size_t)n * kMaxComp, -1);
        for (size_t e = 0; e < apply.size(); e++) list_idx[(size_t)apply[e].img * kMaxComp + apply[e].comp] = (int32_t)e;
        up.add(&plan.d_list_idx, list_idx);
        const int rc = arena_alloc(&r->big, &plan.d_apply_lists, apply.size()); if (rc) return rc;
    }
    // decodes of DC scans only have pixel kernels, and tiles, of their own
    if (!plan.has_ac && !r->d_flat_tiles) {
        std::vector<PixelTile> tiles, rows;
        tiles.reserve(r->n_flat_tiles); rows.reserve(r->n_flat_rows);
        for (uint32_t i = 0; i < n; i++) {
            const ImgDesc& d = r->img[i];
            for (uint32_t c0 = 0, cells = flat_cells(d.W, d.H); c0 < cells; c0 += kFlatLanes) tiles.push_back(PixelTile{i, c0});
            if (r->n_flat_rows) for (uint32_t cy = 0; cy * 8 < d.H; cy++) rows.push_back(PixelTile{i, cy});
        }
        up.add(&r->d_flat_rows, rows);
        up.add(&r->d_flat_tiles, tiles);
    }
    const int rc = up.flush();
    if (rc) { r->d_flat_tiles = nullptr; return rc; }
    auto ins = r->plans.emplace(key, std::move(plan));
    *out = &ins.first->second;
    return PCR_OK;
}

void free_plans(pcr_record* r) { r->plans.clear(); }        // (their device arrays belong to the arena)

int check_scan_group(const pcr_record* r, int k) {
    if (k < 1 || k > (int)r->hdr.G) return PCR_E_RANGE;
    if (k > (int)r->hdr.k_avail) return PCR_E_TRUNCATED;
    return PCR_OK;
}

// Stage timing.  call_begin records the start event, mark(stage) closes an interval that belongs to
// `stage` (one mark per kernel for the entropy kernels and the pixel kernel, so that a stage's time
// divided by its marks is the average duration of that kernel), call_end files the call.
void mark(pcr_record* r, int stage, hipStream_t s) {
    CallTiming* c = r->cur;
    if (!c) return;
    if (c->used == c->ev.size()) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) { r->cur = nullptr; c->used = 0; return; }
        c->ev.push_back(e); c->stage.push_back(0);
    }
    c->stage[c->used] = (uint8_t)stage;
    (void)hipEventRecord(c->ev[c->used++], s);
}
void call_begin(pcr_record* r, hipStream_t s) {
    r->cur = nullptr;
    if (!r->timing) return;
    if (r->ring.empty()) r->ring.resize(kTimingRing);
    r->cur = &r->ring[r->timed_calls % kTimingRing];
    r->cur->used = 0;
    mark(r, 0, s);
}
void call_end(pcr_record* r) { if (r->cur) { r->timed_calls++; r->cur = nullptr; } }

// adds the per-stage milliseconds and marks of one recorded call; waits for that call to finish
int add_call_times(const CallTiming& c, double* ms, uint32_t* marks) {
    if (c.used < 2) return PCR_OK;
    HIP_TRY(hipEventSynchronize(c.ev[c.used - 1]));
    for (size_t i = 1; i < c.used; i++) {
        float t = 0;
        HIP_TRY(hipEventElapsedTime(&t, c.ev[i - 1], c.ev[i]));
        ms[c.stage[i]] += t; marks[c.stage[i]]++;
    }
    return PCR_OK;
}

// One lane per unit or one wavefront per unit?  (The line: LanesLaunch.)  The library cannot see what else runs on the device; it
// takes the number of records the process has open as the sign of it.
bool lanes_pay(const pcr_record* r, const LevelList& l, bool several) {
    if (!r->several_units || r->lane_mode < 0 || l.n_jobs == 0) return false;
    return r->lane_mode > 0 || l.lanes.by_lanes(l.kind == kAcRefine, several);
}

// The same question for a launch of DC first scans (with AC first scans by lanes they share a launch, see with_ac; the line:
// DcLaunch).  beside: the launch could be part of one of AC scans by wavefronts.
bool dc_lanes_pay(const pcr_record* r, const LevelList& l, bool beside) {
    if (r->lane_mode < 0) return false;
    if (r->lane_mode > 0) return l.n >= (uint32_t)kEntropyLanes;
    return l.dc.by_lanes(g_open_records.load(std::memory_order_relaxed) > 1, beside);
}

// Whether the pixel kernel asks the caches to make no room for its pixels (put_past).
//
// The chip's memory-side cache holds 256 MB.  Planes of a record that fit in it are still there when the pixel kernel reads them, but pixels that
// do not fit beside them push them out as they are written.  Where both fit, or the planes alone do not, or other records' planes and pixels pass through
// the cache meanwhile, nothing is gained, and who reads the pixels next finds them in memory only.  So: a record whose planes fit
// and whose pixels do not fit beside them, with no more than three records open (as by SplitLaunch; of two or three that are decoded at the same time
// some lose), without refinement (which reads masks and records beside the planes), and whole pictures (pixels of boxes are for the training tail, at
// once).  Time past the cache over the time through it: the call alone / with a conversion of all pixels to half precision behind it / with their maximum
//   MB of planes + pixels; in flight    1                         2                         4                         8
//     24 + 24                        0.98 / 1.11 / 1.00       (31 + 24, 80 x 49: 0.92 the kernel, 0.97 the call)
//     96 + 96                        0.99 / 1.16 / 1.05
//    120 + 120                       0.98 / 1.02 / 1.02        0.94 / 0.98 / 0.98        1.00 / 1.00 / 1.01        1.00 / 1.00 / 1.01
//    150 + 150                       0.94 / 0.99 / 0.94        0.99 / 1.00 / 1.02        1.01 / 1.00 / 1.00        1.01 / 1.00 / 1.01
//    159 + 154, odd widths           0.94 / 0.99 / 0.94        1.02 / 1.02 / 1.05        1.05 / 1.02 / 1.05        1.05 / 1.01 / 1.04
//    192 + 192                       0.88 / 0.98 / 0.94        0.95 / 0.97 / 0.93        0.98 / 1.00 / 0.98        0.99 / 1.00 / 0.98
//    192 + 192, 1024 x 1024          0.89 / 0.97 / 0.93        1.00 / 1.01 / 1.02        0.99 / 1.00 / 0.99        1.00 / 1.00 / 1.00
//    202 + 195, odd widths           0.89 / 0.98 / 0.94        0.96 / 0.98 / 0.94        1.02 / 1.01 / 1.02        1.04 / 1.01 / 1.03
//    234 + 234                       0.93 / 0.98 / 0.96        1.02 / 1.00 / 1.01        1.00 / 1.00 / 0.99        1.01 / 1.00 / 0.99
//    255 + 255                       0.96 / 1.00 / 0.98        1.02 / 1.00 / 1.01        1.02 / 1.00 / 1.01        1.01 / 1.00 / 1.01
//    150 + 75, 4:4:4                 1.00 / 1.06 / 1.02        0.99 / 1.04 / 1.02        0.99 / 1.00 / 1.02        0.99 / 1.00 / 1.01
//    210 + 105, 4:4:4                0.94 / 1.00 / 0.95        0.99 / 1.00 / 1.01        0.98 / 1.00 / 0.99        0.99 / 1.00 / 1.00
//    225 + 112, gray                 0.92 / 1.00 / 0.97        0.96 / 1.00 / 0.96        0.98 / 1.00 / 1.00        0.99 / 1.00 / 1.00
//    150 + 150, scan group 10        0.98 / 1.00 / 0.98        0.99 / 1.00 / 1.01        0.99 / 1.00 / 1.00        0.99 / 1.00 / 1.00
//    192 + 192, scan group 10        0.99 / 1.01 / 1.00        0.99 / 1.01 / 1.00        0.99 / 1.00 / 1.00        0.99 / 1.00 / 1.00
// The training tail behind it, from the buffer: 24 + 24 1.08, 96 + 96 1.16, 192 + 192 0.98 (of boxes 1.01), 192 + 96 1.03 (1.07).
bool pixels_past(const pcr_record* r, const Plan* plan, bool boxes) {
    constexpr uint64_t kMB = 1u << 20;
    const uint64_t planes = r->coef_off[r->hdr.n] * sizeof(int16_t), pixels = r->out_off[r->hdr.n];
    return planes <= 256 * kMB && planes + pixels > 280 * kMB && plan->has_ac && !plan->n_apply && !boxes && g_open_records.load(std::memory_order_relaxed) <= 3;
}
// Whether the pixel rows of a DC-only decode (k_pixel_flat_rows), and the zero fill of the coefficient planes, go past it as well: where they do not fit in it
// by themselves and several records' launches have to share it, which four open records are taken as the sign of (as by SplitLaunch).  Zeros that
// do fit in part are still there when the first scans are stored into them, so the fill's line lies higher.  Time past the cache over the time through it;
// in flight: four records at a time / one, three others open and idle (MB of pixels, or of planes)
//   pixel rows   98 0.95 / 0.98   196 0.85 / 0.97   262 0.81 / 0.94 (a conversion to half precision behind it: 0.98 / 1.02)   384 0.77 / 0.87 (0.97 / 0.99)
//     odd widths 234 0.99         320 0.98 / 1.03   469 0.97 / 1.02 (0.99 / 1.01)
//   the fill     183 1.00         192 0.96          234 1.00 / 1.07                 320 0.99 / 1.06   384 0.98 / 1.04   469 0.95 / 1.02 (0.98 / 1.01)
//                703 0.99 / 1.00  938 - / 0.99, two at a time 0.99; 469 at scan group 3 1.00, 8 0.98, 10 0.98 / 1.00, with the training tail 0.95 / 1.00, from a loader
//                0.99; 938 from a loader of two 0.96
bool others_open() { return g_open_records.load(std::memory_order_relaxed) > 3; }
bool rows_past(const pcr_record* r) { return others_open() && r->out_off[r->hdr.n] > (256u << 20); }
bool fill_past(const pcr_record* r) { return others_open() && r->coef_off[r->hdr.n] * sizeof(int16_t) > (400u << 20); }

// Index, marker parse and Huffman tables (of scans k0 .. k-1) on the device.  Small records take the offsets of their
// regions in the same kernel: a launch costs about as much as k_index runs, and a workgroup of k_headers sums at most
// kOwnIndexImages lengths per scan group (the line: see there).
void launch_headers(pcr_record* r, uint32_t k, bool keep_status, uint32_t k0, bool dc_tables, hipStream_t s) {
    const uint32_t n = r->hdr.n;
    const bool own = n <= kOwnIndexImages / 2 || (n <= kOwnIndexImages && k <= (uint32_t)kHeaderWaves);
    if (!own) hipLaunchKernelGGL(k_index, dim3(k), dim3(256), 0, s, r->d, k);
    const uint32_t waves = n <= kHeaderWideImages ? (uint32_t)kHeaderWaves : std::min<uint32_t>(k, n <= kHeaderNarrowImages ? kHeaderWaves : kHeaderWaves / 2);
    hipLaunchKernelGGL(k_headers, dim3(n), dim3(64 * waves), header_lds(k, waves), s, r->d, k, (uint32_t)keep_status, (uint32_t)own, k0, (uint32_t)dc_tables);
}

// Unstuffing of scan groups k0 + 1 .. k and the fills, one launch: the groups with the longest scans first, rows of filling
// workgroups spread evenly between the others (fill_turn) so that they run beside them all the way (as many as unstuff at
// most, or they would go ahead of them; 1024 where that is more: there is room for all at once).
void launch_unstuff(pcr_record* r, uint32_t k0, uint32_t k, FillList fill, ApplyJob lists, bool with_lists, hipStream_t s) {
    const uint32_t n = r->hdr.n, count = k - k0;
    UnstuffPlan P{};
    uint64_t mean[kMaxGroups];
    for (uint32_t g = k0; g < k; g++) {
        const uint8_t* hdr = r->header.data();
        const uint64_t start = g ? ld_le64(hdr + hdr_group_end_pos(g - 1)) : r->hdr.header_bytes;
        mean[g] = (ld_le64(hdr + hdr_group_end_pos(g)) - start) / n;
        uint32_t e = P.count++;
        for (; e > 0 && mean[P.group[e - 1]] < mean[g]; e--) P.group[e] = P.group[e - 1];
        P.group[e] = (uint8_t)g;
    }
    const bool many = n * count <= kUnstuffManyScans && count && mean[P.group[0]] >= kUnstuffManyBytes;
    const uint32_t waves = many ? kUnstuffManyWaves : kUnstuffWaves;
    if (with_lists) lists.groups = ((lists.nau + waves - 1) / waves + kDies - 1) / kDies * kDies;
    uint32_t groups = 0;
    for (uint32_t e = 0; e < count; e++) {
        P.first[e] = groups;
        const bool wide = mean[P.group[e]] >= kUnstuffWide;
        if (wide) P.wide |= 1ull << e;
        groups += wide ? n : (n + waves - 1) / waves;
    }
    P.first[count] = groups;
    size_t pieces = 0;
    for (int f = 0; f < kMaxFills; f++) pieces += fill.n16[f];
    r->last_fill_past = fill_past(r) && pieces > 0;
    fill.past = r->last_fill_past ? 1u : 0u;
    const uint32_t lanes = 64 * waves;                       // (eight pieces per lane, but for the last row)
    fill.rows = fill_rows((uint32_t)std::min<size_t>((pieces + 8 * lanes - 1) / (8 * lanes), std::min<size_t>(many ? 512 : 2048, std::max<size_t>(groups, many ? 256 : 1024))));
    const uint32_t total = lists.groups + groups + kDies * fill.rows;
    if (total == 0) return;
    hipLaunchKernelGGL((many ? k_unstuff<kUnstuffManyWaves> : k_unstuff<kUnstuffWaves>), dim3(total), dim3(lanes), 0, s, r->d, P, fill, fill_period(groups, fill.rows), lists);
}

// Steps 1-5 of the path (index .. entropy decode + refinement) for scans 1..k.
// refine_in_memory: also run k_apply, which leaves the refined coefficients in the planes (the coefficient
// export needs that; the pixel kernel replays the refinement itself from the lists of apply_prep).
// k0 > 0: a fidelity upgrade -- groups 1 .. k0 are in the planes and masks already, only k0+1 .. k are decoded.
int run_entropy_stages(pcr_record* r, int k0, int k, hipStream_t s, bool refine_in_memory, Plan** plan_out) {
    Plan* plan = nullptr;
    int rc = build_plan(r, k0, k, &plan);
    if (rc) return rc;
    *plan_out = plan;
    const uint32_t n = r->hdr.n;
    call_begin(r, s);
    // (decided once per call: the answer depends on how many records the process has open, which another thread may change)
    const int open = g_open_records.load(std::memory_order_relaxed);
    const bool several = open > 1;
    std::vector<char> by_lanes(plan->levels.size(), 0);
    r->last_lane_launches = r->last_wave_launches = r->last_splits = r->last_wide_splits = r->last_trios = 0;
    r->last_past = r->last_fill_past = false; r->last_seq = 0; r->last_done.clear();
    for (size_t li = 0; li < plan->levels.size(); li++) {
        const LevelList& l = plan->levels[li];
        if (l.kind == kSequential) by_lanes[li] = (char)(r->seq_mode == 0 ? l.seq.by(open, l.by_tries) : (l.seq.units == 0 || r->seq_mode == 1 ? kSplitNever : (r->seq_mode == 2 ? kSplitBySteps : (l.by_tries ? kSplitByTries : kSplitNever))));
        else if (l.kind != kDcFirst) {
            by_lanes[li] = lanes_pay(r, l, several) ? 1 : 0;
            if (by_lanes[li]) r->last_lane_launches++; else r->last_wave_launches++;
        }
    }
    // Scans cut by restart markers alone can be decoded side by side, which one launch by lanes between the others rules out: where the launches
    // of a call differ their number of units decides for each, as it does where the fit is unsure.  (20 pictures of 382 x 561 with
    // a marker every MCU row, scan group 6: 253 us a call side by side, 299 with the first scans by lanes.)
    if (!r->entry_units && r->lane_mode == 0 && r->last_lane_launches && r->last_wave_launches) {
        r->last_lane_launches = r->last_wave_launches = 0;
        for (size_t li = 0; li < plan->levels.size(); li++) {
            const LevelList& l = plan->levels[li];
            if (l.kind != kAcFirst && l.kind != kAcRefine) continue;
            by_lanes[li] = r->several_units && l.n_jobs && l.lanes.many(several) ? 1 : 0;
            if (by_lanes[li]) r->last_lane_launches++; else r->last_wave_launches++;
        }
    }
    // Scans side by side where the AC scans are for the wavefront decoders (DC first scans may go to the lanes by themselves);
    // with stage timing on, whose intervals are those of single stages, one after the other.
    bool side_by_side = r->last_wave_launches > 0 && r->last_lane_launches == 0 && !r->timing;
    if (side_by_side && !plan->chains_built) {               // (which copies to the device: not into a stream that is being captured)
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone) side_by_side = false;
        else if ((rc = build_chains(r, k0, k, plan)) != PCR_OK) return rc;
    }
    side_by_side = side_by_side && plan->n_ac_chains > 0;
    // Beside AC first scans that go to the lanes the DC first scans of the same level go there too, in the same launch.
    auto with_ac = [&](size_t li) {
        return plan->levels[li].kind == kDcFirst && li + 1 < plan->levels.size() && plan->levels[li + 1].kind == kAcFirst && plan->levels[li + 1].level == plan->levels[li].level &&
               by_lanes[li + 1] != 0;
    };
    // (the wavefront decoders of DC first scans read pre-built tables, the lane decoder makes its own: when every launch
    // of DC first scans of this call goes to the lanes their tables are not built, and with DC first scans only, none are)
    bool dc_tables = false, dc_beside = side_by_side;
    for (size_t li = 0; li < plan->levels.size(); li++) {
        const LevelList& l = plan->levels[li];
        if (l.kind != kDcFirst) continue;
        by_lanes[li] = with_ac(li) || dc_lanes_pay(r, l, side_by_side && l.chained) ? 1 : 0;
        if (!by_lanes[li]) dc_tables = true;
        if (by_lanes[li] || !l.chained) dc_beside = false;
    }
    launch_headers(r, (uint32_t)k, k0 > 0, dc_tables || plan->has_ac ? (uint32_t)k0 : (uint32_t)k, dc_tables, s);
    mark(r, PCR_STAGE_INDEX_PARSE, s);
    const size_t coef_bytes = r->coef_off[n] * sizeof(int16_t);
    // AC first scans only write the coefficients they decode: everything else must read as zero.  With DC scans
    // only, the pixel kernels read nothing of the planes, so the fill is skipped (the coefficient export shows whole
    // planes and always needs it).  The mask planes need no fill: every entry a kernel reads was written earlier in
    // the same call.  An upgrade keeps the planes; when it brings the first AC scans they are cleared first.
    // The DC first scans write a compact copy of the DC coefficients (one per block), which is what every pixel kernel
    // reads; the planes get them too only for the coefficient export: 2-byte stores 128 bytes apart were measured to
    // cost the DC scan a third of its time and to slow the kernels that run beside it.
    const bool dc_to_planes = refine_in_memory;
    FillList fill{};
    if (k0 == 0 ? (plan->has_ac || refine_in_memory) : (plan->has_ac && !plan->had_ac)) { fill.p[0] = (uint4*)r->d.coef; fill.n16[0] = coef_bytes / 16; }
    if (k0 == 0 && !plan->dc_complete) {                     // a component whose DC scan is not among the scans decoded reads as zero
        fill.p[1] = (uint4*)r->d.dc; fill.n16[1] = (r->coef_off[n] / 64 * sizeof(int16_t) + 15) / 16;
    }
    // (with stage timing on the lists are a launch of their own: the stage that uses them is theirs)
    ApplyJob lists{plan->d_apply, plan->d_apply_lists, plan->n_apply, (uint32_t)k, 0};
    const uint32_t list_groups = (plan->n_apply + kApplyPrepWaves - 1) / kApplyPrepWaves;
    launch_unstuff(r, (uint32_t)k0, (uint32_t)k, fill, lists, !r->timing, s);
    mark(r, PCR_STAGE_UNSTUFF, s);
    const uint32_t* c32 = reinterpret_cast<const uint32_t*>(r->d.clean);
    // (a launch of DC scans alone asks for their tables only: with an AC table's room each, the wavefronts of one record left
    // fewer to those of the others.  Four records of 1024 pictures of 256 x 256 without entry points at scan group 1:
    // 715 us a call with room for an AC table and the words of a stream, 655 with room for the DC tables; gray photographs 1470, 1405.)
    // Long first scans by many lanes each, ahead of the wavefronts, which take what is left: null, or what is not.
    auto split = [&](const FirstSplitLaunch& sp, bool with_dc, const Unit* units, uint32_t n_units, uint32_t* done) -> const uint32_t* {
        if (!done || r->timing || r->lane_mode < 0 || !sp.pays(with_dc)) return nullptr;
        const bool wide = sp.wide(with_dc);
        r->last_splits++; r->last_wide_splits += wide ? 1 : 0;
        if (wide) hipLaunchKernelGGL(k_first_split<1024>, dim3(n_units), dim3(1024), 0, s, r->d, units, done, c32, dc_to_planes ? 1u : 0u);
        else hipLaunchKernelGGL(k_first_split<256>, dim3(n_units), dim3(256), 0, s, r->d, units, done, c32, dc_to_planes ? 1u : 0u);
        return done;
    };
    // Whether the refinement scans of a level, or of all levels in one launch (beside the AC first scans), get three wavefronts a unit.
    auto trios = [&](const LevelList* one, uint32_t groups) {
        TrioLaunch t;
        t.groups = groups; t.chains = !one;
        for (const LevelList& l : plan->levels) {
            if (l.kind == kAcRefine && (!one || one == &l)) t.add(l.lanes);
            if (l.kind == kAcFirst && !one) t.add_beside(l.lanes);
        }
        const bool pays = r->lane_mode >= 0 && t.pays(open);
        r->last_trios += pays ? 1 : 0;
        return pays;
    };
    auto waves = [&](const LevelList& l) {
        const bool dc = l.kind == kDcFirst;
        const uint32_t* had = dc ? split(l.split, true, l.d_units, l.n, l.d_done) : nullptr;
        if (l.kind == kAcRefine && trios(&l, l.n)) {
            hipLaunchKernelGGL((k_decode_trios<kWavesAc, false>), dim3(l.n), dim3(3 * kEntropyLanes), kWaveTabBytes + sizeof(TrioRings), s, r->d, l.d_units, (const UnitChain*)nullptr, c32, 0u, (const uint32_t*)nullptr);
            return;
        }
        hipLaunchKernelGGL((dc ? k_decode_waves<kWavesDc, false> : k_decode_waves<kWavesAc, false>), dim3(l.n), dim3(kEntropyLanes), dc ? kWaveDcTabBytes : kWaveTabBytes, s, r->d, l.d_units,
                           (const UnitChain*)nullptr, c32, dc_to_planes ? 1u : 0u, had);
    };
    if (side_by_side) {
        const uint32_t* had = split(plan->split, dc_beside, plan->d_chain_units, dc_beside ? plan->n_chains : plan->n_ac_chains, plan->d_chain_done);   // (chains of one: unit u is chain u)
        const uint32_t w = plan->chain_waves;                // (chains of several scans are those in which some follow others)
        auto* kernel = w > 1 ? (dc_beside ? k_decode_waves<kWavesDc | kWavesAc, true> : k_decode_waves<kWavesAc, true>)
                             : (dc_beside ? k_decode_waves<kWavesDc | kWavesAc, false> : k_decode_waves<kWavesAc, false>);
        const dim3 groups(dc_beside ? plan->n_chains : plan->n_ac_chains);
        if (plan->trio_waves > w && plan->trio_waves <= kTrioChainWaves && trios(nullptr, groups.x))
            hipLaunchKernelGGL((dc_beside ? k_decode_trios<kWavesDc | kWavesAc, true> : k_decode_trios<kWavesAc, true>), groups, dim3(kEntropyLanes * plan->trio_waves), plan->trio_lds, s, r->d,
                               plan->d_chain_units, plan->d_chains, c32, dc_to_planes ? 1u : 0u, had);
        else
            hipLaunchKernelGGL(kernel, groups, dim3(kEntropyLanes * w), w * kWaveTabBytes, s, r->d, plan->d_chain_units, plan->d_chains, c32, dc_to_planes ? 1u : 0u, had);
    }
    for (size_t li = 0; li < plan->levels.size(); li++) {
        auto& l = plan->levels[li];
        if (side_by_side && l.chained && (l.kind != kDcFirst || dc_beside)) continue;
        const dim3 block(kEntropyLanes);
        if (with_ac(li) && !r->timing) {                     // (timed, each stage has a launch, and an interval, of its own)
            const auto& ac = plan->levels[++li];
            hipLaunchKernelGGL(k_first_lanes, dim3(l.n_dc_waves + ac.n_jobs), block, 0, s, r->d, l.d_units, l.n, l.d_dc_starts, l.n_dc_waves, ac.d_units, ac.d_jobs, c32, dc_to_planes ? 1u : 0u);
        }
        else if (l.kind == kDcFirst) {
            if (by_lanes[li]) hipLaunchKernelGGL(k_dc_first_lanes, dim3(l.n_dc_waves), block, 0, s, r->d, l.d_units, l.n, l.d_dc_starts, c32, dc_to_planes ? 1u : 0u);
            else waves(l);
            mark(r, PCR_STAGE_DC_FIRST, s);
        }
        else if (l.kind == kSequential) {
            const uint32_t lanes = by_lanes[li] == kSplitByTries ? l.seq.units : (by_lanes[li] ? l.n : 0u);
            if (by_lanes[li] == kSplitByTries) {
                hipLaunchKernelGGL(k_split_tries, dim3(lanes, l.split_tries), dim3(kSplitLanes), 0, s, r->d, l.d_units, l.d_rooms, r->d_nodes, r->d_next, c32);
                hipLaunchKernelGGL(k_split_settle, dim3(lanes), dim3(kSplitLanes), 0, s, r->d, l.d_units, l.d_rooms, r->d_nodes, r->d_next, r->d_pieces, l.d_done, c32);
                hipLaunchKernelGGL(k_split_store, dim3(lanes, l.split_stores), dim3(kSplitStoreLanes), 0, s, r->d, l.d_units, l.d_rooms, r->d_pieces, l.d_done, c32);
            }
            if (lanes) hipLaunchKernelGGL(k_sequential_split, dim3(lanes), dim3(kSplitLanes), 0, s, r->d, l.d_units, l.d_done, by_lanes[li] == kSplitByTries ? 1u : 0u, c32);
            if (lanes) r->last_done.push_back(pcr_record::SeqDone{l.d_done, l.seq.units});
            r->last_seq = std::max(r->last_seq, by_lanes[li] + 1);
            hipLaunchKernelGGL(k_sequential, dim3(l.n), block, 0, s, r->d, l.d_units, (const uint32_t*)l.d_done, lanes, c32);
            mark(r, PCR_STAGE_SEQUENTIAL, s);
        }
        else if (l.kind == kAcFirst) {
            if (by_lanes[li]) hipLaunchKernelGGL(k_ac_first_lanes, dim3(l.n_jobs), block, 0, s, r->d, l.d_units, l.d_jobs, c32);
            else waves(l);
            mark(r, PCR_STAGE_AC_FIRST, s);
        }
        else if (by_lanes[li]) {
            if (l.n_plane_tiles) hipLaunchKernelGGL(k_refine_history, dim3(l.n_plane_tiles), dim3(256), 0, s, r->d, plan->d_refine, plan->d_refine_tiles + l.plane_tile);
            mark(r, PCR_STAGE_REFINE_BLOCKS, s);
            hipLaunchKernelGGL(k_ac_refine_lanes, dim3(l.n_jobs), block, 0, s, r->d, l.d_units, l.d_jobs, c32);
            mark(r, PCR_STAGE_AC_REFINE, s);
            if (l.n_cov_tiles) hipLaunchKernelGGL(k_refine_deal, dim3(l.n_cov_tiles), dim3(256), 0, s, r->d, plan->d_refine, plan->d_refine_tiles + l.cov_tile);
            mark(r, PCR_STAGE_REFINE_BLOCKS, s);
        }
        else {
            waves(l);
            mark(r, PCR_STAGE_AC_REFINE, s);
            if (l.n_cov_tiles && !side_by_side) hipLaunchKernelGGL(k_refine_blocks, dim3(l.n_cov_tiles), dim3(256), 0, s, r->d, plan->d_refine, plan->d_refine_tiles + l.cov_tile);
            mark(r, PCR_STAGE_REFINE_BLOCKS, s);
        }
    }
    // The blocks of all refinement scans the wavefronts have walked, in one launch: of an earlier refinement scan a later one needs
    // what the wavefronts themselves leave (kRefNz, kRefHist).  (A launch behind every level held up the next one: 256 pictures
    // of 17 to 320 pixels with entry points at scan group 10 358 us a call with two launches of 26, 345 with one.)
    if (side_by_side && plan->n_cov_tiles)
        hipLaunchKernelGGL(k_refine_blocks, dim3(plan->n_cov_tiles), dim3(256), 0, s, r->d, plan->d_refine, plan->d_refine_tiles + plan->cov_tile);
    if (plan->n_apply) {
        if (r->timing) hipLaunchKernelGGL(k_apply_prep, dim3(list_groups), dim3(64 * kApplyPrepWaves), 0, s, r->d, lists);
        if (refine_in_memory)
            hipLaunchKernelGGL(k_apply, dim3(plan->apply_grid_x, plan->n_apply), dim3(256), 0, s, r->d, plan->d_apply, plan->d_apply_lists);
    }
    if (plan->n_apply) mark(r, PCR_STAGE_REFINE_APPLY, s);
    if (hipGetLastError() != hipSuccess) { r->cur = nullptr; return PCR_E_DEVICE; }
    return PCR_OK;
}

// Images in groups of about this many bytes of what the host codes or puts together from: so much is pinned for it, or what a single image takes.
// (The device's tables, bit counts and offsets of all images come back at once, 5.7 KB an image, as the symbol counts do where the host codes, 20 KB.)
constexpr size_t kTranscodePinned = 64u << 20;

// Cuts images 0 .. n - 1 into such groups: offset[i] is where image i begins, offset[n] the end.  Returns the first images of the groups
// and n; *most: the longest group.
std::vector<uint32_t> transcode_groups(const std::vector<uint64_t>& offset, size_t unit, size_t* most) {
    const uint32_t n = (uint32_t)offset.size() - 1;
    std::vector<uint32_t> group(1, 0);
    *most = 0;
    for (uint32_t i = 0; i < n; i++) {
        if (i > group.back() && (offset[i + 1] - offset[group.back()]) * unit > kTranscodePinned) group.push_back(i);
        *most = std::max<size_t>(*most, (offset[i + 1] - offset[group.back()]) * unit);
    }
    group.push_back(n);
    return group;
}

// Files first .. last - 1 by up to `threads` threads: write(i, where, room, &size) writes file i where there is room for it, or says
// why not.
template <class Write> int transcode_write(uint32_t first, uint32_t last, uint32_t threads, void* out, const uint64_t* out_off, uint64_t* written, int* status, const Write& write) {
    std::atomic<uint32_t> next(first);
    auto work = [&]() {
        for (;;) {
            const uint32_t i = next.fetch_add(1);
            if (i >= last) break;
            size_t size = 0;
            const size_t room = (size_t)(out_off[i + 1] - out_off[i]);
            status[i] = write(i, (uint8_t*)out + out_off[i], room, &size);
            written[i] = size;
            if (!status[i] && size > room) status[i] = PCR_E_RANGE;
        }
    };
    return enc::on_threads(std::min(threads, last - first), work) ? PCR_OK : PCR_E_NOMEM;
}

// Device and pinned memory of a call, given back when what it has enqueued is done.
struct CallMemory {
    hipStream_t stream;
    std::vector<void*> dev, host;
    explicit CallMemory(hipStream_t s) : stream(s) {}
    CallMemory(const CallMemory&) = delete;
    CallMemory& operator=(const CallMemory&) = delete;
    ~CallMemory() { (void)hipStreamSynchronize(stream); for (void* p : dev) (void)hipFree(p); for (void* p : host) (void)hipHostFree(p); }
    template <class T> T* device(size_t count) {
        void* p = nullptr;
        dev.reserve(dev.size() + 1);
        if (hipMalloc(&p, count * sizeof(T) + 1) != hipSuccess) return nullptr;
        dev.push_back(p);
        return (T*)p;
    }
    template <class T> T* pinned(size_t count) {
        void* p = nullptr;
        host.reserve(host.size() + 1);
        if (hipHostMalloc(&p, count * sizeof(T) + 1, hipHostMallocDefault) != hipSuccess) return nullptr;
        host.push_back(p);
        return (T*)p;
    }
};

// The files by the device's coder (pcr_coder.h), without restart markers.  frames[i]: what read_frame said of file i, kOk for all
// that are to be written.
struct SourceFrame { int rc; ImgDesc img; enc::Frame frame; };
bool same_frame(const ImgDesc& a, const ImgDesc& b) {
    bool same = a.nc == b.nc && (a.nc == 1 || a.nc == 3) && a.mcux == b.mcux && a.mcuy == b.mcuy;
    for (int c = 0; same && c < a.nc; c++)
        same = a.hs[c] == b.hs[c] && a.vs[c] == b.vs[c] && a.bw[c] == b.bw[c] && a.bh[c] == b.bh[c] && a.cw[c] == b.cw[c] && a.ch[c] == b.ch[c];
    return same;
}
int transcode_on_device(pcr_record* r, const void* const* files, const std::vector<SourceFrame>& frames, uint32_t threads, void* out, const uint64_t* out_off, uint64_t* written,
                               int* status, hipStream_t s) {
    const uint32_t n = r->hdr.n;
    const size_t scans = (size_t)n * kScriptScansMax;
    CallMemory M(s);
    uint32_t* d_hist = M.device<uint32_t>((size_t)n * kHistPerImage);
    ScanMarks* d_marks = M.device<ScanMarks>(scan_marks_of_image(r->coef_off[n], n));
    uint32_t* d_raw = M.device<uint32_t>(scans);
    uint32_t* d_codes = M.device<uint32_t>(scans * 2 * 256);
    uint64_t* d_off = M.device<uint64_t>(scans + 1);
    const size_t spec_bytes = arena_round(scans * 2 * sizeof(CodeSpec));     // (tables and bit counts come back together)
    uint8_t *d_made = M.device<uint8_t>(spec_bytes + scans * sizeof(uint64_t)), *made = M.pinned<uint8_t>(spec_bytes + scans * sizeof(uint64_t));
    if (!d_hist || !d_marks || !d_raw || !d_codes || !d_off || !d_made || !made) return PCR_E_NOMEM;
    CodeSpec* d_specs = reinterpret_cast<CodeSpec*>(d_made);
    uint64_t* d_bits = reinterpret_cast<uint64_t*>(d_made + spec_bytes);
    const ImgDesc* d_img = r->d.img;
    const int16_t* d_coef = r->d.coef;
    hipLaunchKernelGGL(k_symbol_hist, dim3(n, kScriptScansMax), dim3(kHistLanes), 0, s, d_img, d_coef, r->d.coef_off, 0u, d_hist, d_marks, d_raw);
    hipLaunchKernelGGL(k_code_tables, dim3(n, kScriptScansMax), dim3(128), 0, s, d_img, (const uint32_t*)d_hist, (const uint32_t*)d_raw, d_specs, d_codes, d_bits);
    if (hipGetLastError() != hipSuccess || hipMemcpyAsync(made, d_made, spec_bytes + scans * sizeof(uint64_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) return PCR_E_DEVICE;
    const CodeSpec* specs = reinterpret_cast<const CodeSpec*>(made);
    const uint64_t* bits = reinterpret_cast<const uint64_t*>(made + spec_bytes);
    std::vector<uint64_t> at(n + 1, 0);                        // words of the images
    for (uint32_t i = 0; i < n; i++) {
        at[i + 1] = at[i];
        for (int g = 0; g < kScriptScansMax; g++) at[i + 1] += (bits[(size_t)i * kScriptScansMax + g] + 31) / 32;
    }
    size_t most;
    const std::vector<uint32_t> group = transcode_groups(at, sizeof(uint32_t), &most);
    most /= sizeof(uint32_t);
    uint32_t *d_words = M.device<uint32_t>(most), *words = M.pinned<uint32_t>(most);
    uint64_t* off = M.pinned<uint64_t>(scans + 1);
    if (!d_words || !words || !off) return PCR_E_NOMEM;
    for (size_t e = 0; e + 1 < group.size(); e++) {
        const uint32_t first = group[e], last = group[e + 1];
        const size_t mine = (size_t)(last - first) * kScriptScansMax;
        off[0] = 0;
        for (size_t q = 0; q < mine; q++) off[q + 1] = off[q] + (bits[(size_t)first * kScriptScansMax + q] + 31) / 32;
        if (hipMemcpyAsync(d_off, off, (mine + 1) * sizeof(uint64_t), hipMemcpyHostToDevice, s) != hipSuccess) return PCR_E_DEVICE;
        hipLaunchKernelGGL(k_code_scans, dim3(last - first, kScriptScansMax), dim3(kCodeLanes), 0, s, d_img, d_coef, r->d.coef_off, (const ScanMarks*)d_marks, (const uint32_t*)d_codes,
                           (const uint64_t*)d_off, first, d_words);
        if (hipGetLastError() != hipSuccess || (off[mine] && hipMemcpyAsync(words, d_words, off[mine] * sizeof(uint32_t), hipMemcpyDeviceToHost, s) != hipSuccess) ||
            hipStreamSynchronize(s) != hipSuccess) return PCR_E_DEVICE;
        // (a thread for every two megabytes: more of them take longer to start than to do it)
        const uint32_t useful = (uint32_t)std::min<uint64_t>(threads, 1 + off[mine] * sizeof(uint32_t) / (2u << 20));
        const int rc = transcode_write(first, last, useful, out, out_off, written, status, [&](uint32_t i, uint8_t* dst, size_t room, size_t* size) {
            const SourceFrame& F = frames[i];
            if (F.rc) return F.rc;
            const size_t scan = (size_t)i * kScriptScansMax;
            *size = enc::assemble_progressive((const uint8_t*)files[i], F.img, F.frame, specs + 2 * scan, bits + scan, words, off + (size_t)(i - first) * kScriptScansMax, dst, room);
            return (int)kOk;
        });
        if (rc) return rc;
    }
    return PCR_OK;
}

// The files by the host's coder: coefficients (and, device_counts, symbol counts) to pinned memory (30 MB of coefficients took 10 ms
// through pageable memory), the files coded by several threads straight from there.
int transcode_on_host(pcr_record* r, const void* const* files, const size_t* sizes, uint32_t restart_interval, bool device_counts, uint32_t threads, void* out, const uint64_t* out_off,
                             uint64_t* written, int* status, hipStream_t s) {
    const uint32_t n = r->hdr.n;
    size_t most;
    const std::vector<uint32_t> group = transcode_groups(r->coef_off, sizeof(int16_t), &most);
    const size_t counts_of = device_counts ? (size_t)n * kHistPerImage : 0;
    CallMemory M(s);
    int16_t *host = M.pinned<int16_t>(most / sizeof(int16_t)), *d_coef = M.device<int16_t>((size_t)r->coef_off[n]);
    uint32_t *hist = M.pinned<uint32_t>(counts_of), *d_hist = M.device<uint32_t>(counts_of);
    if (!host || !d_coef || !hist || !d_hist) return PCR_E_NOMEM;
    hipLaunchKernelGGL(k_export_natural, dim3(2048), dim3(256), 0, s, r->d.coef, d_coef, (size_t)r->coef_off[n]);
    if (device_counts)
        hipLaunchKernelGGL(k_symbol_hist, dim3(n, kScriptScansMax), dim3(kHistLanes), 0, s, (const ImgDesc*)r->d.img, (const int16_t*)r->d.coef, r->d.coef_off, restart_interval, d_hist,
                           (ScanMarks*)nullptr, (uint32_t*)nullptr);
    if (hipGetLastError() != hipSuccess) return PCR_E_DEVICE;
    if (device_counts && hipMemcpyAsync(hist, d_hist, counts_of * sizeof(uint32_t), hipMemcpyDeviceToHost, s) != hipSuccess) return PCR_E_DEVICE;
    for (size_t e = 0; e + 1 < group.size(); e++) {
        const uint32_t first = group[e], last = group[e + 1];
        const uint64_t at = r->coef_off[first];
        if (hipMemcpyAsync(host, d_coef + at, (size_t)(r->coef_off[last] - at) * sizeof(int16_t), hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return PCR_E_DEVICE;
        const int rc = transcode_write(first, last, threads, out, out_off, written, status, [&](uint32_t i, uint8_t* dst, size_t room, size_t* size) {
            std::vector<uint8_t> bytes;
            const int made = enc::transcode_progressive((const uint8_t*)files[i], sizes[i], host + (r->coef_off[i] - at), (size_t)(r->coef_off[i + 1] - r->coef_off[i]), restart_interval, &bytes,
                                                        device_counts ? hist + (size_t)i * kHistPerImage : nullptr);
            *size = bytes.size();
            if (!made && bytes.size() <= room) memcpy(dst, bytes.data(), bytes.size());
            return made;
        });
        if (rc) return rc;
    }
    return PCR_OK;
}

}  // namespace

extern "C" {

// Host-side validation of the metadata block: region lengths must tile every available group and
// agree with the per-image scan counts.  hdr: host copy of the first header_bytes bytes.
static int validate_index(const uint8_t* hdr, const RecordHeader& h, std::vector<uint32_t>* off, std::vector<uint32_t>* len, std::vector<uint32_t>* nsc) {
    const uint32_t n = h.n, G = h.G;
    off->assign((size_t)G * n, 0); len->assign((size_t)G * n, 0); nsc->assign(n, 0);
    uint64_t start = h.header_bytes;
    for (uint32_t g = 0; g < h.k_avail; g++) {
        uint64_t pos = start;
        for (uint32_t i = 0; i < n; i++) {
            uint32_t L = ld_le32(hdr + hdr_len_pos(n, G, g, i));
            (*off)[(size_t)g * n + i] = (uint32_t)pos; (*len)[(size_t)g * n + i] = L; pos += L;
        }
        if (h.version == 2)                                       // the group's entry points lie behind its regions
            for (uint32_t i = 0; i < n; i++) pos += entry_bytes(ld_le16(hdr + hdr_ecount_pos(n, G, g, i)));
        if (pos != ld_le64(hdr + hdr_group_end_pos(g))) return PCR_E_FORMAT;
        start = pos;
    }
    for (uint32_t i = 0; i < n; i++) {
        (*nsc)[i] = ld_le32(hdr + hdr_nscans_pos(n, G, i));
        if ((*nsc)[i] == 0 || (*nsc)[i] > G) return PCR_E_FORMAT;
        for (uint32_t g = 0; g < h.k_avail; g++)
            if ((g < (*nsc)[i]) != ((*len)[(size_t)g * n + i] != 0)) return PCR_E_FORMAT;
    }
    return PCR_OK;
}

// What a bind clears, one launch of it.  (ptr: of an arena, whose pieces are rounded up to more than 16 bytes.)
static void add_fill(BindFill* F, void* ptr, size_t bytes, uint32_t word) { F->p[F->count] = (uint4*)ptr; F->n16[F->count] = (bytes + 15) / 16; F->word[F->count++] = word; }
static int launch_fill(const BindFill& F, hipStream_t s) {
    size_t most = 0;
    for (uint32_t f = 0; f < F.count; f++) most = std::max<size_t>(most, F.n16[f]);
    const uint32_t groups = (uint32_t)std::min<size_t>(2048, (most + 1023) / 1024 + 1);       // (four pieces a lane)
    hipLaunchKernelGGL(k_bind_fill, dim3(groups), dim3(256), 0, s, F);
    return hipGetLastError() == hipSuccess ? PCR_OK : PCR_E_DEVICE;
}

// Everything after the image/scan descriptors are known (r->img, r->scan filled, r->d.rec set):
// dependency levels, buffer layout, the buffers themselves (out of r->big), their initial contents.
// Fills are enqueued on s, with those in `fill` in one launch; the caller synchronises s before anything else uses the handle.
static int finish_open(pcr_record* r, BindFill fill, hipStream_t s) {
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    const size_t nbytes = r->nbytes;
    for (uint32_t i = 0; i < n; i++) if (r->img[i].status != kOk) return r->img[i].status;
    compute_levels(r);
    r->out_off.assign(n + 1, 0); r->coef_off.assign(n + 1, 0);
    r->mask_off.assign((size_t)n * G, 0); r->slot_base.assign((size_t)n * G, 0); r->slot_cnt.assign((size_t)n * G, 0);
    std::vector<PixelTile> tiles;
    uint32_t flat_tiles = 0, flat_rows = 0;                       // (listed when a plan first needs them)
    bool rows_fit = true;
    r->flat_row_cells = 0;
    uint64_t nm = 0; uint64_t ns = 0; bool long_scans = false;
    std::vector<uint32_t> tab_idx((size_t)n * G, 0); uint32_t ntabs = 0;
    std::vector<uint32_t> dctab_idx((size_t)n * G, 0); uint32_t ndctabs = 0;
    r->several_units = r->entry_units = false;
    // version 2: where the entry points of every scan lie (behind the regions of the scan's group)
    std::vector<uint32_t> ent_off((size_t)n * G, 0), ent_cnt((size_t)n * G, 0);
    if (r->hdr.version == 2) {
        const uint8_t* hdr = r->header.data();
        for (uint32_t g = 0; g < r->hdr.k_avail; g++) {
            uint64_t all = 0;
            for (uint32_t i = 0; i < n; i++) all += entry_bytes(ld_le16(hdr + hdr_ecount_pos(n, G, g, i)));
            uint64_t at = ld_le64(hdr + hdr_group_end_pos(g)) - all;                   // (validate_index: this is where the regions end)
            for (uint32_t i = 0; i < n; i++) {
                const uint32_t field = ld_le16(hdr + hdr_ecount_pos(n, G, g, i));
                ent_off[(size_t)i * G + g] = (uint32_t)at; ent_cnt[(size_t)i * G + g] = entry_count(field);
                at += entry_bytes(field);
            }
        }
    }
    for (uint32_t i = 0; i < n; i++) {
        const ImgDesc& d = r->img[i];
        r->out_off[i + 1] = r->out_off[i] + (uint64_t)d.W * d.H * d.nc;
        uint64_t cc = 0;
        for (int c = 0; c < d.nc; c++) {
            const uint64_t elems = (uint64_t)d.bw[c] * d.bh[c] * 64;
            if (elems >= (1ull << 32)) return PCR_E_UNSUPPORTED;       // the decoders index a plane with 32 bits
            cc += elems;
        }
        if (cc >= (1ull << 32)) return PCR_E_UNSUPPORTED;               // ... and an image's planes together
        r->coef_off[i + 1] = r->coef_off[i] + cc;
        for (uint32_t g = 0; g < d.nscans; g++) {
            const size_t ig = (size_t)i * G + g;
            const ScanDesc& sd = r->scan[ig];
            if (sd.Ss > 0) {
                r->mask_off[ig] = nm;
                nm += sd.Ah ? ref_words((uint64_t)d.bw[sd.comp[0]] * d.bh[sd.comp[0]]) : 0;   // one record per block of a refinement scan
                tab_idx[ig] = ntabs++;                       // (first scans use theirs only when the tables are built ahead)
            }
            uint32_t cnt = sd.ri ? (sd.mcus + sd.ri - 1) / sd.ri : 1;
            const bool serial = !(d.progressive && sd.Ss == 0 && sd.Ah > 0);          // (DC refinement is read in place, without units)
            if (sd.ri == 0 && serial && ent_cnt[ig] > 0) cnt = 1 + ent_cnt[ig];         // units start at the entry points
            else ent_off[ig] = 0;
            if (ent_off[ig]) r->entry_units = true;
            if (d.progressive && sd.Ss == 0 && sd.Ah == 0) { dctab_idx[ig] = ndctabs; ndctabs += kMaxComp; }
            long_scans = long_scans || (sd.data_len * 8ull >= kSplitLeastBits && is_sequential_scan(sd));
            if (cnt > 1 && (sd.Ss > 0 || d.progressive)) r->several_units = true;
            r->slot_base[ig] = (uint32_t)ns; r->slot_cnt[ig] = cnt;
            ns += cnt + 1;
        }
        const uint32_t per = pixel_mcus_per_tile(d), mcus = (uint32_t)d.mcux * d.mcuy;       // runs of MCUs, one lane per block
        for (uint32_t m0 = 0; m0 < mcus; m0 += per) tiles.push_back(PixelTile{i, m0});
        flat_tiles += (flat_cells(d.W, d.H) + kFlatLanes - 1) / kFlatLanes;
        rows_fit = rows_fit && flat_rows_fit(d.W);
        r->flat_row_cells = std::max(r->flat_row_cells, ((uint32_t)d.W + 7) >> 3);
        flat_rows += (d.H + 7u) / 8u;
    }
    if (ns >= (1ull << 32)) return PCR_E_UNSUPPORTED;
    r->n_masks = nm; r->n_slots = (uint32_t)ns; r->n_tiles = (uint32_t)tiles.size(); r->n_flat_tiles = flat_tiles;
    if (!rows_fit) flat_rows = 0;
    r->n_flat_rows = flat_rows; r->d_flat_tiles = r->d_flat_rows = nullptr;

    DevRecord& d = r->d;
    const size_t padded = nbytes + 1024;      // slack: bit readers look ahead
    // what the buffers below take, plus room for the work lists of a few scan groups (16 bytes per unit,
    // 12 per image and component, ...): anything beyond that is allocated on its own
    size_t need = arena_round(padded) + arena_round(r->coef_off[n] * sizeof(int16_t)) + arena_round((r->coef_off[n] / 64 + 1) * sizeof(int16_t)) + arena_round((nm + 2) * sizeof(uint64_t)) +
                  arena_round((ns + 1) * sizeof(uint32_t)) + 2 * arena_round((n + 1) * sizeof(uint64_t)) +
                  4 * arena_round(((size_t)n * G + 1) * sizeof(uint64_t)) + arena_round((tiles.size() + 1) * sizeof(PixelTile)) + arena_round((flat_tiles + 1ull) * sizeof(PixelTile)) + arena_round((flat_rows + 1ull) * sizeof(PixelTile)) + arena_round((n + 1) * 8) +
                  arena_round(((size_t)ntabs + 1) * sizeof(AcTab)) + arena_round(((size_t)ndctabs + 1) * sizeof(DcTab)) + arena_round(((size_t)n * G + 1) * sizeof(uint32_t)) + arena_round(((size_t)n * G + 1) * sizeof(uint32_t));
    need += 8 * ((ns + (size_t)n * G) * sizeof(Unit) + (size_t)n * kMaxComp * 64) + (1u << 20);
    need += 8 * (r->coef_off[n] / 64 / 256 + (size_t)n * G) * 2 * sizeof(RefineTile);     // (the tile lists of the refinement helpers: one entry per 256 blocks)
    r->last_done.clear();
    r->d_nodes = nullptr; r->d_next = nullptr; r->d_pieces = nullptr;
    r->split_space = long_scans ? split_space_of(r) : SplitSpace();
    const SplitSpace space = r->split_space;
    const size_t tries_need = space.nodes ? arena_round(space.nodes * sizeof(SplitNode)) + arena_round(space.nodes * sizeof(uint32_t)) + arena_round(space.pieces * sizeof(SplitPiece)) : 0;
    int rc = arena_reset(&r->big, need + tries_need);
    if (rc && tries_need) { r->split_space = SplitSpace(); rc = arena_reset(&r->big, need); }      // (long sequential scans are decoded without it as well)
    if (!rc && r->split_space.nodes) {
        rc = arena_alloc(&r->big, &r->d_nodes, space.nodes);
        if (!rc) rc = arena_alloc(&r->big, &r->d_next, space.nodes);
        if (!rc) rc = arena_alloc(&r->big, &r->d_pieces, space.pieces);
    }
    if (!rc) rc = arena_alloc(&r->big, &d.clean, padded);
    if (!rc) rc = arena_alloc(&r->big, &d.coef, r->coef_off[n]);
    if (!rc) rc = arena_alloc(&r->big, &d.dc, r->coef_off[n] / 64 + 8);              // (+8: cleared in 16-byte units)
    if (!rc) rc = arena_alloc(&r->big, &d.masks, nm + 2);
    if (!rc) rc = arena_alloc(&r->big, &d.ivl_start, ns);
    uint64_t *d_coef_off = nullptr, *d_out_off = nullptr, *d_mask_off = nullptr; uint32_t *d_sb = nullptr, *d_sc = nullptr;
    std::vector<uint32_t> dims((size_t)n * 2);
    for (uint32_t i = 0; i < n; i++) { dims[2 * i] = (uint32_t)r->img[i].W; dims[2 * i + 1] = (uint32_t)r->img[i].H; }
    uint32_t *d_tab_idx = nullptr, *d_dctab_idx = nullptr, *d_ent_off = nullptr;
    Uploads up(&r->big, &r->stage);
    up.add(&d_coef_off, r->coef_off);
    up.add(&d_out_off, r->out_off);
    up.add(&d_mask_off, r->mask_off);
    up.add(&d_sb, r->slot_base);
    up.add(&d_sc, r->slot_cnt);
    up.add(&r->d_tiles, tiles);
    up.add(&r->d_dims, dims);
    up.add(&d_tab_idx, tab_idx);
    up.add(&d_dctab_idx, dctab_idx);
    up.add(&d_ent_off, ent_off);
    if (!rc) rc = up.flush_on(s);
    r->ent_off_h = std::move(ent_off); r->unit_bits.clear();
    if (!rc) rc = arena_alloc(&r->big, &d.dctabs, (size_t)ndctabs);
    if (!rc) rc = arena_alloc(&r->big, &d.tabs, (size_t)ntabs);
    d.dctab_idx = d_dctab_idx;
    d.ent_off = d_ent_off;
    d.tab_idx = d_tab_idx;
    d.coef_off = d_coef_off; d.out_off = d_out_off; d.mask_off = d_mask_off; d.slot_base = d_sb; d.slot_cnt = d_sc;
    // (the refinement records need no initial contents: every word a kernel reads was written earlier in the same
    // call, or by the call an upgrade builds on; consumers skip blocks outside the scans' own grids)
    if (!rc) {
        add_fill(&fill, d.clean, padded, 0xFFFFFFFFu);
        add_fill(&fill, d.ivl_start, (ns ? ns : 1) * sizeof(uint32_t), 0);
        rc = launch_fill(fill, s);
    }
    return rc;
}

// Buffers the index and parse kernels write (out of r->small); needed before the descriptors exist.  *fill: what is to be cleared.
static int alloc_descriptor_buffers(pcr_record* r, BindFill* fill) {
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    DevRecord& d = r->d;
    const size_t ng = (size_t)G * n;
    int rc = arena_reset(&r->small, arena_round((ng + 1) * sizeof(uint32_t)) + arena_round((n + 1) * sizeof(ImgDesc)) +
                                    arena_round((ng + 1) * sizeof(ScanDesc)) + arena_round((n + 1) * sizeof(int32_t)));
    if (!rc) rc = arena_alloc(&r->small, &d.off, ng);
    if (!rc) rc = arena_alloc(&r->small, &d.img, n);
    if (!rc) rc = arena_alloc(&r->small, &d.scan, ng);
    if (!rc) rc = arena_alloc(&r->small, &d.status, n);
    if (!rc) { add_fill(fill, d.off, ng * sizeof(uint32_t), 0); add_fill(fill, d.scan, ng * sizeof(ScanDesc), 0); add_fill(fill, d.img, (size_t)n * sizeof(ImgDesc), 0); }
    d.n = n; d.G = G; d.nbytes = r->nbytes;
    d.len = (const uint32_t*)(d.rec + hdr_len_pos(n, G, 0, 0));
    d.nscans = (const uint32_t*)(d.rec + hdr_nscans_pos(n, G, 0));
    return rc;
}

// Entropy-coded bits of every unit, for records whose bytes the host has: the entry points say where the units of a scan
// start (the lane-per-unit kernels put units of like length into one wavefront).  Scans cut by restart markers, whose
// intervals only the unstuff kernel finds, get their mean.
static void measure_units(pcr_record* r, const uint8_t* bytes, size_t nbytes) {
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    size_t slots = 0;
    for (size_t ig = 0; ig < (size_t)n * G; ig++) slots = std::max<size_t>(slots, (size_t)r->slot_base[ig] + r->slot_cnt[ig] + 1);
    r->unit_bits.assign(slots, 0);
    for (uint32_t i = 0; i < n; i++) {
        for (uint32_t g = 0; g < r->img[i].nscans && g < r->hdr.k_avail; g++) {
            const size_t ig = (size_t)i * G + g;
            const uint32_t cnt = r->slot_cnt[ig], sb = r->slot_base[ig], eo = r->ent_off_h[ig];
            const uint64_t all = (uint64_t)r->scan[ig].data_len * 8;
            const uint32_t stride = entry_stride(ld_le16(r->header.data() + hdr_ecount_pos(n, G, g, i)));
            if (eo && cnt > 1 && (size_t)eo + (size_t)stride * (cnt - 1) <= nbytes) {
                uint64_t prev = 0;
                for (uint32_t j = 0; j < cnt; j++) {
                    const uint64_t end = j + 1 < cnt ? ld_le32(bytes + eo + (size_t)stride * j + 4) : std::max<uint64_t>(all, prev);
                    r->unit_bits[sb + j] = (uint32_t)std::min<uint64_t>(end > prev ? end - prev : 0, 0xFFFFFFFFu);
                    prev = std::max(prev, end);
                }
            } else {
                for (uint32_t j = 0; j < cnt; j++) r->unit_bits[sb + j] = (uint32_t)(all / std::max<uint32_t>(cnt, 1));
            }
        }
    }
}

// Marker parse of every image: layout, work sizes, early rejection.
static int parse_on_host(pcr_record* r, const uint8_t* bytes, const std::vector<uint32_t>& off, const std::vector<uint32_t>& len, const std::vector<uint32_t>& nsc) {
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    r->img.resize(n); r->scan.assign((size_t)n * G, ScanDesc{});
    for (uint32_t i = 0; i < n; i++) {
        parse_image(bytes, off.data(), len.data(), n, i, nsc[i], r->hdr.k_avail, &r->img[i], &r->scan[(size_t)i * G]);
        if (r->img[i].status) return r->img[i].status;
    }
    return PCR_OK;
}

int pcr_open(const void* bytes_, size_t nbytes, int device_id, pcr_record** out) {
    if (!bytes_ || !out) return PCR_E_ARG;
    const uint8_t* bytes = (const uint8_t*)bytes_;
    RecordHeader h;
    int rc = parse_record_header(bytes, nbytes, &h);
    if (rc) return rc;
    if (nbytes >= (1ull << 32)) return PCR_E_UNSUPPORTED;
    if (h.k_avail == 0) return PCR_E_TRUNCATED;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device_id < 0 || device_id >= ndev) { (void)hipGetLastError(); return PCR_E_DEVICE; }
    HIP_TRY(hipSetDevice(device_id));

    pcr_record* r = new (std::nothrow) pcr_record();
    if (!r) return PCR_E_NOMEM;
    r->device = device_id; r->nbytes = nbytes; r->hdr = h;
    const uint32_t n = h.n, G = h.G;
    r->header.assign(bytes, bytes + h.header_bytes);
    std::vector<uint32_t> off, len, nsc;
    rc = validate_index(r->header.data(), h, &off, &len, &nsc);
    if (!rc) rc = parse_on_host(r, bytes, off, len, nsc);
    if (!rc && hipMalloc((void**)&r->d_rec, nbytes + 64) != hipSuccess) { (void)hipGetLastError(); rc = PCR_E_NOMEM; }
    if (!rc && hipMemcpy(r->d_rec, bytes, nbytes, hipMemcpyHostToDevice) != hipSuccess) rc = PCR_E_DEVICE;
    BindFill fill{};
    if (!rc) { r->d.rec = r->d_rec; fill.tail = r->d_rec + nbytes; rc = alloc_descriptor_buffers(r, &fill); }
    if (!rc) rc = finish_open(r, fill, nullptr);
    if (!rc) measure_units(r, bytes, nbytes);
    if (!rc && hipStreamSynchronize(nullptr) != hipSuccess) rc = PCR_E_DEVICE;
    if (rc) { (void)hipGetLastError(); pcr_close(r); return rc; }
    r->stage.done();
    *out = r;
    return PCR_OK;
}

// Binds handle r (fresh, or one whose earlier work has finished) to record bytes in device memory.  Without a host copy of
// them (host null): header checks on the host, index and marker parse ON THE DEVICE, and only the small descriptor tables
// come back.  With one, everything is read from it, while the bytes may still be on their way to the device (enqueued on s
// before), and 64 bytes behind them are cleared.  Then the buffer layout.  Everything is enqueued on s, which is synchronised
// before returning.  On failure the handle holds no record (pcr_close is all that may follow).
static int bind_bytes(pcr_record* r, const void* d_bytes, size_t nbytes, const uint8_t* host, hipStream_t s);
static int bind_device(pcr_record* r, const void* d_bytes, size_t nbytes, const uint8_t* host, hipStream_t s) {
    auto holds_nothing = [&]() {                             // until the bind succeeds: no images, and layouts of no images
        r->hdr = RecordHeader{}; r->n_tiles = 0; r->n_flat_tiles = 0; r->n_flat_rows = 0;
        r->out_off.assign(1, 0); r->coef_off.assign(1, 0);
    };
    r->plans.clear(); r->resident_k = 0;
    holds_nothing();
    r->d_dims = nullptr; r->d_ssim_part = nullptr; r->d_planes = nullptr;
    r->d_tail_tiles = nullptr; r->n_tail_tiles = 0; r->d_edge = nullptr; r->d_edge_off = nullptr; r->d_mcu_px_h = nullptr;
    int rc = bind_bytes(r, d_bytes, nbytes, host, s);
    if (hipStreamSynchronize(s) != hipSuccess && !rc) rc = PCR_E_DEVICE;
    r->stage.done();
    if (rc) { (void)hipGetLastError(); holds_nothing(); }
    return rc;
}
static int bind_bytes(pcr_record* r, const void* d_bytes, size_t nbytes, const uint8_t* host, hipStream_t s) {
    // fixed part of the header, then the whole metadata block
    uint8_t fixed[24];
    if (host) std::memcpy(fixed, host, 24);
    else {
        HIP_TRY(hipMemcpyAsync(fixed, d_bytes, 24, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
    }
    if (fixed[0] != 'P' || fixed[1] != 'C' || fixed[2] != 'R' || fixed[3] != '1') return PCR_E_FORMAT;
    const uint64_t header_bytes = ld_le64(fixed + 16);
    if (header_bytes < 24 || header_bytes > (1ull << 31)) return PCR_E_FORMAT;
    if (header_bytes > nbytes) return PCR_E_TRUNCATED;
    r->header.resize(header_bytes);
    if (host) std::memcpy(r->header.data(), host, header_bytes);
    else {
        HIP_TRY(hipMemcpyAsync(r->header.data(), d_bytes, header_bytes, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
    }
    RecordHeader h;
    int rc = parse_record_header(r->header.data(), nbytes, &h);
    if (!rc && h.k_avail == 0) rc = PCR_E_TRUNCATED;
    if (rc) return rc;
    r->nbytes = nbytes; r->hdr = h;
    const uint32_t n = h.n, G = h.G;
    std::vector<uint32_t> off, len, nsc;
    rc = validate_index(r->header.data(), h, &off, &len, &nsc);
    if (rc) return rc;
    r->d.rec = (const uint8_t*)d_bytes;
    BindFill fill{};
    rc = alloc_descriptor_buffers(r, &fill);
    if (rc) return rc;
    if (host) {
        fill.tail = (uint8_t*)d_bytes + nbytes;              // (a loader's own buffer)
        rc = parse_on_host(r, host, off, len, nsc);
        if (rc) return rc;
    } else {
        rc = launch_fill(fill, s);
        if (rc) return rc;
        fill = BindFill{};
        launch_headers(r, h.k_avail, false, h.k_avail, false, s);          // (no tables: where they go is not laid out yet)
        r->img.resize(n); r->scan.resize((size_t)n * G);
        HIP_TRY(hipMemcpyAsync(r->img.data(), r->d.img, n * sizeof(ImgDesc), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipMemcpyAsync(r->scan.data(), r->d.scan, (size_t)n * G * sizeof(ScanDesc), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
    }
    // (the units are not measured: ordering them takes longer than it saves where a record is decoded once)
    return finish_open(r, fill, s);
}

static int check_device_bytes(const void* d_bytes, size_t nbytes, int* device) {
    if (!d_bytes) return PCR_E_ARG;
    if (((uintptr_t)d_bytes & 15) != 0) return PCR_E_ARG;              // header tables are read as aligned words
    if (nbytes < 24) return PCR_E_TRUNCATED;
    if (nbytes >= (1ull << 32)) return PCR_E_UNSUPPORTED;
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, d_bytes) != hipSuccess) { (void)hipGetLastError(); return PCR_E_ARG; }
    if (attr.type != hipMemoryTypeDevice) return PCR_E_ARG;
    *device = attr.device;
    return PCR_OK;
}

int pcr_open_device(const void* d_bytes, size_t nbytes, void* stream, pcr_record** out) {
    if (!out) return PCR_E_ARG;
    int device = 0;
    int rc = check_device_bytes(d_bytes, nbytes, &device);
    if (rc) return rc;
    HIP_TRY(hipSetDevice(device));
    pcr_record* r = new (std::nothrow) pcr_record();
    if (!r) return PCR_E_NOMEM;
    r->device = device; r->borrowed = true;
    rc = bind_device(r, d_bytes, nbytes, nullptr, (hipStream_t)stream);
    if (rc) { pcr_close(r); return rc; }
    *out = r;
    return PCR_OK;
}

int pcr_rebind_device(pcr_record* r, const void* d_bytes, size_t nbytes, void* stream) {
    if (!r) return PCR_E_ARG;
    int device = 0;
    int rc = check_device_bytes(d_bytes, nbytes, &device);
    if (rc) return rc;
    if (device != r->device) return PCR_E_ARG;
    HIP_TRY(hipSetDevice(device));
    if (!r->borrowed && r->d_rec) { (void)hipFree(r->d_rec); }             // the handle's own copy of its first record
    r->d_rec = nullptr; r->borrowed = true;
    return bind_device(r, d_bytes, nbytes, nullptr, (hipStream_t)stream);
}

void pcr_close(pcr_record* r) {
    if (!r) return;
    (void)hipSetDevice(r->device);
    (void)hipDeviceSynchronize();
    free_plans(r);
    arena_free(&r->small); arena_free(&r->big); r->stage.release();
    if (!r->borrowed && r->d_rec) (void)hipFree(r->d_rec);
    if (r->d_gather) (void)hipFree(r->d_gather);
    for (auto& c : r->ring) for (auto& e : c.ev) (void)hipEventDestroy(e);
    delete r;
}

int pcr_num_images(const pcr_record* r, int* n) { if (!r || !n) return PCR_E_ARG; *n = (int)r->hdr.n; return PCR_OK; }
int pcr_num_scan_groups(const pcr_record* r, int* G) { if (!r || !G) return PCR_E_ARG; *G = (int)r->hdr.G; return PCR_OK; }
int pcr_available_scan_groups(const pcr_record* r, int* k) { if (!r || !k) return PCR_E_ARG; *k = (int)r->hdr.k_avail; return PCR_OK; }

int pcr_group_end_offset(const pcr_record* r, int k, uint64_t* off) {
    if (!r || !off) return PCR_E_ARG;
    if (k < 1 || k > (int)r->hdr.G) return PCR_E_RANGE;
    *off = ld_le64(r->header.data() + hdr_group_end_pos((uint32_t)k - 1));
    return PCR_OK;
}

int pcr_image_info(const pcr_record* r, int i, int* w, int* h, int* c, int32_t* label) {
    if (!r) return PCR_E_ARG;
    if (i < 0 || i >= (int)r->hdr.n) return PCR_E_RANGE;
    if (w) *w = r->img[i].W;
    if (h) *h = r->img[i].H;
    if (c) *c = r->img[i].nc;
    if (label) *label = (int32_t)ld_le32(r->header.data() + hdr_label_pos(r->hdr.G, (uint32_t)i));
    return PCR_OK;
}

int pcr_output_layout(const pcr_record* r, uint64_t* offsets) {
    if (!r || !offsets) return PCR_E_ARG;
    if (r->out_off.size() != (size_t)r->hdr.n + 1) {           // a handle without a record (n = 0) has the one entry 0
        if (r->hdr.n) return PCR_E_ARG;
        offsets[0] = 0;
        return PCR_OK;
    }
    std::memcpy(offsets, r->out_off.data(), r->out_off.size() * sizeof(uint64_t));
    return PCR_OK;
}

int pcr_coef_layout(const pcr_record* r, uint64_t* offsets) {
    if (!r || !offsets) return PCR_E_ARG;
    if (r->coef_off.size() != (size_t)r->hdr.n + 1) {
        if (r->hdr.n) return PCR_E_ARG;
        offsets[0] = 0;
        return PCR_OK;
    }
    std::memcpy(offsets, r->coef_off.data(), r->coef_off.size() * sizeof(uint64_t));
    return PCR_OK;
}

int pcr_index(const pcr_record* r, uint64_t* off, uint32_t* len) {
    if (!r || !off || !len) return PCR_E_ARG;
    HIP_TRY(hipSetDevice(r->device));
    const uint32_t n = r->hdr.n, G = r->hdr.G, k = r->hdr.k_avail;
    hipLaunchKernelGGL(k_index, dim3(k), dim3(256), 0, 0, r->d, k);
    std::vector<uint32_t> o((size_t)G * n);
    HIP_TRY(hipMemcpy(o.data(), r->d.off, o.size() * sizeof(uint32_t), hipMemcpyDeviceToHost));
    std::vector<uint32_t> l((size_t)G * n);
    HIP_TRY(hipMemcpy(l.data(), r->d.len, l.size() * sizeof(uint32_t), hipMemcpyDeviceToHost));
    for (size_t e = 0; e < (size_t)k * n; e++) { off[e] = o[e]; len[e] = l[e]; }
    return PCR_OK;
}

int pcr_reassemble(pcr_record* r, int i, int k, uint8_t* dst, size_t cap, size_t* len) {
    if (!r || !len) return PCR_E_ARG;
    if (i < 0 || i >= (int)r->hdr.n) return PCR_E_RANGE;
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    const uint32_t n = r->hdr.n, G = r->hdr.G;
    const uint32_t ns = ld_le32(r->header.data() + hdr_nscans_pos(n, G, (uint32_t)i));
    const uint32_t have = std::min<uint32_t>(ns, (uint32_t)k);
    size_t total = 0;
    for (uint32_t g = 0; g < have; g++) total += ld_le32(r->header.data() + hdr_len_pos(n, G, g, (uint32_t)i));
    const int add_eoi = have < ns;
    total += add_eoi ? 2 : 0;
    if (!dst) { *len = total; return PCR_OK; }
    if (cap < total) return PCR_E_RANGE;
    HIP_TRY(hipSetDevice(r->device));
    if (r->gather_cap < total) {
        if (r->d_gather) (void)hipFree(r->d_gather);
        r->d_gather = nullptr; r->gather_cap = 0;
        if (hipMalloc((void**)&r->d_gather, total) != hipSuccess) return PCR_E_NOMEM;
        r->gather_cap = total;
    }
    hipLaunchKernelGGL(k_index, dim3(k), dim3(256), 0, 0, r->d, (uint32_t)k);
    hipLaunchKernelGGL(k_gather, dim3(64), dim3(256), 0, 0, r->d, (uint32_t)i, have, add_eoi, r->d_gather);
    HIP_TRY(hipMemcpy(dst, r->d_gather, total, hipMemcpyDeviceToHost));
    *len = total;
    return PCR_OK;
}

int pcr_set_lane_decoders(pcr_record* r, int mode) {
    if (!r || mode < -1 || mode > 1) return PCR_E_ARG;
    r->lane_mode = mode;
    return PCR_OK;
}

int pcr_set_sequential_decoders(pcr_record* r, int mode) {
    if (!r || mode < 0 || mode > 3) return PCR_E_ARG;
    if (mode != r->seq_mode) free_plans(r);                  // (their rooms are laid out for the mode)
    r->seq_mode = mode;
    return PCR_OK;
}
int pcr_last_sequential_decoders(pcr_record* r, int* by, uint32_t* counts, uint32_t* rounds) {
    if (!r || !by || !counts || !rounds) return PCR_E_ARG;
    *by = r->last_seq; counts[0] = counts[1] = counts[2] = rounds[0] = rounds[1] = 0;
    HIP_TRY(hipSetDevice(r->device));
    std::vector<uint32_t> done;
    for (const pcr_record::SeqDone& l : r->last_done) {
        done.resize(l.units);
        HIP_TRY(hipMemcpy(done.data(), l.d_done, l.units * sizeof(uint32_t), hipMemcpyDeviceToHost));
        for (uint32_t v : done) {
            const uint32_t how = v == 0 ? 2u : (v > kSplitInSteps ? 1u : 0u);
            counts[how]++;
            if (how < 2) rounds[how] = std::max(rounds[how], v - 1 - how * kSplitInSteps);
        }
    }
    return PCR_OK;
}

int pcr_last_decoder_shapes(pcr_record* r, int* lane_launches, int* wavefront_launches) {
    if (!r || !lane_launches || !wavefront_launches) return PCR_E_ARG;
    *lane_launches = r->last_lane_launches; *wavefront_launches = r->last_wave_launches;
    return PCR_OK;
}

int pcr_last_refine_trios(pcr_record* r, int* launches) {
    if (!r || !launches) return PCR_E_ARG;
    *launches = r->last_trios;
    return PCR_OK;
}
int pcr_last_past_stores(pcr_record* r, int* past) {
    if (!r || !past) return PCR_E_ARG;
    *past = r->last_past ? 1 : 0;
    return PCR_OK;
}
int pcr_last_past_fills(pcr_record* r, int* past) {
    if (!r || !past) return PCR_E_ARG;
    *past = r->last_fill_past ? 1 : 0;
    return PCR_OK;
}
int pcr_last_first_splits(pcr_record* r, int* launches, int* wide_launches) {
    if (!r || !launches || !wide_launches) return PCR_E_ARG;
    *launches = r->last_splits; *wide_launches = r->last_wide_splits;
    return PCR_OK;
}

int pcr_enable_stage_timing(pcr_record* r, int on) {
    if (!r) return PCR_E_ARG;
    r->timing = on != 0;
    r->timed_calls = 0;                        // switching on (again) starts a new history
    return PCR_OK;
}

int pcr_last_stage_ms(pcr_record* r, float* ms) {
    if (!r || !ms) return PCR_E_ARG;
    if (!r->timing || r->timed_calls == 0) return PCR_E_ARG;
    HIP_TRY(hipSetDevice(r->device));
    double sum[PCR_NUM_STAGES] = {}; uint32_t marks[PCR_NUM_STAGES] = {};
    int rc = add_call_times(r->ring[(r->timed_calls - 1) % kTimingRing], sum, marks);
    if (rc) return rc;
    for (int s = 0; s < PCR_NUM_STAGES; s++) ms[s] = (float)sum[s];
    return PCR_OK;
}

int pcr_stage_ms_history(pcr_record* r, double* sum_ms, uint32_t* launches, uint32_t* calls) {
    if (!r || !sum_ms || !launches || !calls) return PCR_E_ARG;
    if (!r->timing) return PCR_E_ARG;
    HIP_TRY(hipSetDevice(r->device));
    for (int s = 0; s < PCR_NUM_STAGES; s++) { sum_ms[s] = 0; launches[s] = 0; }
    const uint64_t have = r->timed_calls < kTimingRing ? r->timed_calls : kTimingRing;
    for (uint64_t j = 0; j < have; j++) {
        int rc = add_call_times(r->ring[(r->timed_calls - 1 - j) % kTimingRing], sum_ms, launches);
        if (rc) return rc;
    }
    *calls = (uint32_t)have;
    return PCR_OK;
}

int pcr_decode_coefficients(pcr_record* r, int k, int16_t* d_coef, void* stream) {
    if (!r || !d_coef) return PCR_E_ARG;
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    HIP_TRY(hipSetDevice(r->device));
    hipStream_t s = (hipStream_t)stream;
    Plan* plan = nullptr;
    r->resident_k = 0;                                       // k_apply refines the planes in place: nothing to upgrade from afterwards
    rc = run_entropy_stages(r, 0, k, s, true, &plan);
    if (rc) return rc;
    call_end(r);
    hipLaunchKernelGGL(k_export_natural, dim3(2048), dim3(256), 0, s, r->d.coef, d_coef, (size_t)r->coef_off[r->hdr.n]);
    if (hipGetLastError() != hipSuccess) return PCR_E_DEVICE;
    return PCR_OK;
}

// k0 = 0: from scratch; k0 > 0: on top of the planes and masks a previous call left for scan group k0
static int decode_to_pixels(pcr_record* r, int k0, int k, uint8_t* out, size_t cap, void* stream, int32_t* d_status, const CropBox* boxes = nullptr,
                            bool smooth = false) {
    if (cap < r->out_off[r->hdr.n]) return PCR_E_RANGE;
    HIP_TRY(hipSetDevice(r->device));
    hipStream_t s = (hipStream_t)stream;
    Plan* plan = nullptr;
    r->resident_k = 0;
    int rc = run_entropy_stages(r, k0, k, s, false, &plan);
    if (rc) return rc;
    // smoothing: with DC first scans only, a kernel of its own; otherwise the predicted coefficients go into the planes
    // for the pixel kernel and are taken out again after it (where there is a component to predict at all: the two
    // launches took 150 of the 1550 us of 2048 pictures of 132 x 133 at scan group 10, to find that there is none)
    DevRecord d = r->d;
    d.status_out = d_status;
    const bool smooth_flat = smooth && !plan->has_ac && !plan->n_apply && !boxes;
    if (smooth_flat || !plan->smooths) smooth = false;
    const bool by_rows = !smooth_flat && !plan->n_apply && !plan->has_ac && !smooth && r->n_flat_rows && !boxes;     // DC scans only: every block is flat
    r->last_past = by_rows ? rows_past(r) : pixels_past(r, plan, boxes != nullptr);
    if (smooth) hipLaunchKernelGGL(k_smooth<false>, dim3(kSmoothGroups, r->hdr.n), dim3(256), 0, s, r->d);
    if (smooth_flat)
        hipLaunchKernelGGL(k_pixel_smooth_flat, dim3(r->n_flat_tiles), dim3(kFlatLanes), 0, s, d, r->d_flat_tiles, out);
    else if (plan->n_apply)
        hipLaunchKernelGGL((k_pixel<true, false>), dim3(r->n_tiles), dim3(kPixLanes), 0, s, d, r->d_tiles, out, plan->d_apply_lists, plan->d_list_idx, boxes, 0u);
    else if (plan->has_ac || smooth)
        hipLaunchKernelGGL((k_pixel<false, false>), dim3(r->n_tiles), dim3(kPixLanes), 0, s, d, r->d_tiles, out, (const ApplyList*)nullptr, (const int32_t*)nullptr, boxes, r->last_past ? 1u : 0u);
    else if (by_rows)
        hipLaunchKernelGGL(k_pixel_flat_rows, dim3(r->n_flat_rows), dim3(kFlatRowLanes), flat_rows_lds(r->flat_row_cells), s, d, r->d_flat_rows, out, r->flat_row_cells, r->last_past ? 1u : 0u);
    else
        hipLaunchKernelGGL(k_pixel_flat, dim3(r->n_flat_tiles), dim3(kFlatLanes), 0, s, d, r->d_flat_tiles, out, boxes);
    if (smooth) hipLaunchKernelGGL(k_smooth<true>, dim3(kSmoothGroups, r->hdr.n), dim3(256), 0, s, r->d);
    mark(r, PCR_STAGE_PIXEL, s);
    call_end(r);
    if (hipGetLastError() != hipSuccess) return PCR_E_DEVICE;
    r->resident_k = k;
    return PCR_OK;
}

int pcr_decode_batch(pcr_record* r, int k, uint8_t* out, size_t cap, void* stream, int32_t* d_status) {
    if (!r || !out) return PCR_E_ARG;
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    return decode_to_pixels(r, 0, k, out, cap, stream, d_status);
}

int pcr_decode_batch_smooth(pcr_record* r, int k, uint8_t* out, size_t cap, void* stream, int32_t* d_status) {
    if (!r || !out) return PCR_E_ARG;
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    return decode_to_pixels(r, 0, k, out, cap, stream, d_status, nullptr, true);
}

int pcr_decode_batch_triangle(pcr_record* r, int k, uint8_t* out, size_t cap, void* stream, int32_t* d_status) {
    if (!r || !out) return PCR_E_ARG;
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    const uint32_t n = r->hdr.n;
    if (cap < r->out_off[n]) return PCR_E_RANGE;
    HIP_TRY(hipSetDevice(r->device));
    if (!r->d_planes) {                                      // one byte per coefficient slot
        rc = arena_alloc(&r->big, &r->d_planes, (size_t)r->coef_off[n] + 16);
        if (rc) return rc;
    }
    hipStream_t s = (hipStream_t)stream;
    Plan* plan = nullptr;
    r->resident_k = 0;
    rc = run_entropy_stages(r, 0, k, s, false, &plan);
    if (rc) return rc;
    DevRecord d = r->d;
    d.status_out = d_status;
    if (plan->n_apply)
        hipLaunchKernelGGL((k_pixel<true, true>), dim3(r->n_tiles), dim3(kPixLanes), 0, s, d, r->d_tiles, r->d_planes, plan->d_apply_lists, plan->d_list_idx, (const CropBox*)nullptr, 0u);
    else
        hipLaunchKernelGGL((k_pixel<false, true>), dim3(r->n_tiles), dim3(kPixLanes), 0, s, d, r->d_tiles, r->d_planes, (const ApplyList*)nullptr, (const int32_t*)nullptr, (const CropBox*)nullptr, 0u);
    uint32_t items = 1;
    for (uint32_t i = 0; i < n; i++) items = std::max(items, (((uint32_t)r->img[i].W + 3) / 4) * (uint32_t)r->img[i].H);
    hipLaunchKernelGGL(k_triangle_rgb, dim3((items + 255) / 256, n), dim3(256), 0, s, r->d, (const uint8_t*)r->d_planes, out);
    mark(r, PCR_STAGE_PIXEL, s);
    call_end(r);
    if (hipGetLastError() != hipSuccess) return PCR_E_DEVICE;
    r->resident_k = k;
    return PCR_OK;
}

int pcr_resident_scan_group(const pcr_record* r, int* k) {
    if (!r || !k) return PCR_E_ARG;
    *k = r->resident_k;
    return PCR_OK;
}

int pcr_upgrade_batch(pcr_record* r, int k, uint8_t* out, size_t cap, void* stream, int32_t* d_status) {
    if (!r || !out) return PCR_E_ARG;
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    if (r->resident_k < 1 || k < r->resident_k) return PCR_E_ARG;
    return decode_to_pixels(r, r->resident_k, k, out, cap, stream, d_status);
}

int pcr_crop_resize_batch(pcr_record* r, const uint8_t* d_pixels, const pcr_crop* d_crops, int out_h, int out_w,
                          const float* mean, const float* inv_std, void* d_out_f16, size_t out_capacity, void* stream) {
    if (!r || !d_pixels || !d_crops || !mean || !inv_std) return PCR_E_ARG;
    if (out_h < 1 || out_w < 1 || out_h > 8192 || out_w > 8192) return PCR_E_RANGE;      // (the kernel's fractions stay inside 32 bits)
    if (!d_out_f16) return PCR_E_ARG;
    const uint32_t n = r->hdr.n;
    if (n == 0 || !r->d_dims) return PCR_E_ARG;
    const int C = r->img[0].nc;
    for (uint32_t i = 1; i < n; i++) if (r->img[i].nc != C) return PCR_E_UNSUPPORTED;    // one tensor, one channel count
    if (out_capacity < (size_t)n * C * out_h * out_w * sizeof(__half)) return PCR_E_RANGE;
    HIP_TRY(hipSetDevice(r->device));
    static_assert(sizeof(pcr_crop) == sizeof(CropBox), "crop box layout");
    if (n > 65535) return PCR_E_UNSUPPORTED;                  // (images are the grid's third dimension)
    const dim3 grid(((uint32_t)out_w + 31) / 32, ((uint32_t)out_h + 7) / 8, n);
    hipLaunchKernelGGL(k_crop_resize, grid, dim3(256), 0, (hipStream_t)stream, r->d_dims, r->d.out_off, d_pixels, reinterpret_cast<const CropBox*>(d_crops),
                       out_h, out_w, C, mean[0], C > 1 ? mean[1] : 0.f, C > 2 ? mean[2] : 0.f,
                       inv_std[0], C > 1 ? inv_std[1] : 1.f, C > 2 ? inv_std[2] : 1.f, reinterpret_cast<__half*>(d_out_f16));
    if (hipGetLastError() != hipSuccess) return PCR_E_DEVICE;
    return PCR_OK;
}

// Tiles, side buffer and tables of the fused decode + tail (once per bound record).
static int prepare_fused_tail(pcr_record* r) {
    if (r->d_tail_tiles) return PCR_OK;
    const uint32_t n = r->hdr.n;
    std::vector<PixelTile> tiles; std::vector<uint64_t> eoff(n + 1, 0); std::vector<uint32_t> mh(n);
    r->tail_lds = 0; r->tail_rows = 1;
    for (uint32_t i = 0; i < n; i++) {
        const ImgDesc& d = r->img[i];
        for (uint32_t my = 0; my < d.mcuy; my++) for (uint32_t run = 0, runs = tail_runs(d); run < runs; run++) tiles.push_back(PixelTile{i, my * d.mcux + run});
        eoff[i + 1] = eoff[i] + (uint64_t)2 * d.mcuy * d.W;
        mh[i] = 8u * d.vmax;
        r->tail_lds = std::max(r->tail_lds, tail_lds(d)); r->tail_rows = std::max<uint32_t>(r->tail_rows, d.mcuy);
    }
    PixelTile* dt = nullptr;
    Uploads up(&r->big, &r->stage);
    up.add(&r->d_edge_off, eoff);
    up.add(&r->d_mcu_px_h, mh);
    up.add(&dt, tiles);
    int rc = arena_alloc(&r->big, &r->d_edge, (size_t)eoff[n]);
    if (!rc) rc = up.flush();
    if (rc) return rc;
    r->d_tail_tiles = dt; r->n_tail_tiles = (uint32_t)tiles.size();
    return PCR_OK;
}

int pcr_decode_crop_batch(pcr_record* r, int k, const pcr_crop* d_crops, uint8_t* d_pixels, size_t pixel_capacity, int out_h, int out_w,
                          const float* mean, const float* inv_std, void* d_out_f16, size_t out_capacity, void* stream, int32_t* d_status) {
    if (!r || !d_crops || !mean || !inv_std) return PCR_E_ARG;
    if (!d_pixels) {
        // No working buffer: decode and tail in one kernel, the full-resolution pixels stay on the chip.
        int rc = check_scan_group(r, k);
        if (rc) return rc;
        if (out_h < 1 || out_w < 1 || out_h > 8192 || out_w > 8192) return PCR_E_RANGE;
        if (!d_out_f16 || !r->d_dims) return PCR_E_ARG;
        const uint32_t n = r->hdr.n;
        const int C = r->img[0].nc;
        for (uint32_t i = 1; i < n; i++) if (r->img[i].nc != C) return PCR_E_UNSUPPORTED;
        if (n > 65535) return PCR_E_UNSUPPORTED;
        if (out_capacity < (size_t)n * C * out_h * out_w * sizeof(__half)) return PCR_E_RANGE;
        HIP_TRY(hipSetDevice(r->device));
        rc = prepare_fused_tail(r);
        if (rc) return rc;
        hipStream_t s = (hipStream_t)stream;
        Plan* plan = nullptr;
        r->resident_k = 0;
        rc = run_entropy_stages(r, 0, k, s, false, &plan);
        if (rc) return rc;
        DevRecord d = r->d;
        d.status_out = d_status;
        TailParams P;
        P.out_h = out_h; P.out_w = out_w;
        for (int c = 0; c < 3; c++) { P.mean[c] = c < C ? mean[c] : 0.f; P.istd[c] = c < C ? inv_std[c] : 1.f; }
        static_assert(sizeof(pcr_crop) == sizeof(CropBox), "crop box layout");
        const CropBox* boxes = reinterpret_cast<const CropBox*>(d_crops);
        auto* kernel = plan->n_apply ? (C == 1 ? k_pixel_tail<true, true> : k_pixel_tail<true, false>) : (C == 1 ? k_pixel_tail<false, true> : k_pixel_tail<false, false>);
        hipLaunchKernelGGL(kernel, dim3(r->n_tail_tiles), dim3(kTailLanes), r->tail_lds, s, d, r->d_tail_tiles, plan->n_apply ? (const ApplyList*)plan->d_apply_lists : nullptr,
                           plan->n_apply ? (const int32_t*)plan->d_list_idx : nullptr, boxes, P, reinterpret_cast<__half*>(d_out_f16), r->d_edge, r->d_edge_off);
        if (r->tail_rows > 1)
            hipLaunchKernelGGL(k_tail_edges, dim3(r->tail_rows - 1, n), dim3(64), 0, s, r->d_dims, r->d_mcu_px_h, (uint32_t)C, boxes, P, r->d_edge, r->d_edge_off,
                           reinterpret_cast<__half*>(d_out_f16));
        mark(r, PCR_STAGE_PIXEL, s);
        call_end(r);
        if (hipGetLastError() != hipSuccess) return PCR_E_DEVICE;
        r->resident_k = k;
        return PCR_OK;
    }
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    // argument checks of the tail before anything is enqueued (it repeats them)
    if (out_h < 1 || out_w < 1 || out_h > 8192 || out_w > 8192) return PCR_E_RANGE;
    if (!d_out_f16 || !r->d_dims) return PCR_E_ARG;
    const uint32_t n = r->hdr.n;
    const int C = r->img[0].nc;
    for (uint32_t i = 1; i < n; i++) if (r->img[i].nc != C) return PCR_E_UNSUPPORTED;
    if (n > 65535) return PCR_E_UNSUPPORTED;
    if (out_capacity < (size_t)n * C * out_h * out_w * sizeof(__half)) return PCR_E_RANGE;
    rc = decode_to_pixels(r, 0, k, d_pixels, pixel_capacity, stream, d_status, reinterpret_cast<const CropBox*>(d_crops));
    if (rc) return rc;
    return pcr_crop_resize_batch(r, d_pixels, d_crops, out_h, out_w, mean, inv_std, d_out_f16, out_capacity, stream);
}

// Rows per tile and tiles of the picture that needs most, for the similarity kernels.
static void ssim_layout(const pcr_record* r, uint32_t* rows, uint32_t* tiles_max) {
    const uint32_t n = r->hdr.n;
    for (uint32_t pick : kSsimRowChoices) {
        uint32_t t = 1;
        for (uint32_t i = 0; i < n; i++) t = std::max(t, ssim_tiles_all((uint32_t)r->img[i].W, (uint32_t)r->img[i].H, pick));
        *rows = pick; *tiles_max = t;
        if (ssim_rows_suit(n, t)) return;
    }
}
static int launch_ssim(pcr_record* r, const uint8_t* d_a, const uint8_t* d_b, float2* part, uint32_t rows, uint32_t tmax, float* d_scores, hipStream_t s) {
    const uint32_t n = r->hdr.n;
    const uint32_t every = ssim_workgroups(tmax);
    if ((uint64_t)every * n >= (1ull << 31)) return PCR_E_UNSUPPORTED;
    if (r->img[0].nc == 3) hipLaunchKernelGGL(k_ssim_tiles<3>, dim3(every * n), dim3(64), 0, s, r->d_dims, r->d.out_off, d_a, d_b, part, n, tmax, every, rows);
    else hipLaunchKernelGGL(k_ssim_tiles<1>, dim3(every * n), dim3(64), 0, s, r->d_dims, r->d.out_off, d_a, d_b, part, n, tmax, every, rows);
    hipLaunchKernelGGL(k_ssim_score, dim3(n), dim3(64), 0, s, r->d_dims, part, tmax, rows, d_scores);
    return hipGetLastError() == hipSuccess ? PCR_OK : PCR_E_DEVICE;
}

int pcr_msssim_batch(pcr_record* r, const uint8_t* d_a, const uint8_t* d_b, float* d_scores, void* stream) {
    if (!r || !d_a || !d_b || !d_scores) return PCR_E_ARG;
    const uint32_t n = r->hdr.n;
    if (n == 0 || !r->d_dims) return PCR_E_ARG;
    const int C = r->img[0].nc;
    if (C != 1 && C != 3) return PCR_E_UNSUPPORTED;
    for (uint32_t i = 1; i < n; i++) if (r->img[i].nc != C) return PCR_E_UNSUPPORTED;
    if (n > 65535) return PCR_E_UNSUPPORTED;                  // (images are the grid's second dimension)
    HIP_TRY(hipSetDevice(r->device));
    uint32_t rows, tmax;
    ssim_layout(r, &rows, &tmax);
    if (!r->d_ssim_part) {
        int rc = arena_alloc(&r->big, &r->d_ssim_part, (size_t)n * tmax);
        if (rc) return rc;
    }
    return launch_ssim(r, d_a, d_b, r->d_ssim_part, rows, tmax, d_scores, (hipStream_t)stream);
}

// ---- similarity scores without any allocation ----
// The per-tile sums of the similarity kernels in a fixed array of the code object instead of the handle's
// arena, for callers that must not allocate (HIP graph capture, serving loops).  Every GPU holds its own copy
// of the array at its own address; host code never uses the array's name as an address, only the pointer
// hipGetSymbolAddress returned for that device.
constexpr size_t kStaticSsimTiles = 512 * 1024;                       // 4 MiB of float2 per device
static __device__ __align__(256) float2 scratch[kStaticSsimTiles];
constexpr int kStaticMaxDevices = 64;
static std::mutex g_scratch_mu;
static float2* g_scratch_ptr[kStaticMaxDevices] = {};

// the array's address on `device` (which must be current), looked up once per device
static int static_scratch(int device, float2** p) {
    if (device < 0 || device >= kStaticMaxDevices) return PCR_E_DEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* q = nullptr;
        if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) { (void)hipGetLastError(); return PCR_E_DEVICE; }
        g_scratch_ptr[device] = reinterpret_cast<float2*>(q);
    }
    *p = g_scratch_ptr[device];
    return PCR_OK;
}

int pcr_msssim_batch_static(pcr_record* r, const uint8_t* d_a, const uint8_t* d_b, float* d_scores, void* stream) {
    if (!r || !d_a || !d_b || !d_scores) return PCR_E_ARG;
    const uint32_t n = r->hdr.n;
    if (n == 0 || !r->d_dims) return PCR_E_ARG;
    const int C = r->img[0].nc;
    if (C != 1 && C != 3) return PCR_E_UNSUPPORTED;
    for (uint32_t i = 1; i < n; i++) if (r->img[i].nc != C) return PCR_E_UNSUPPORTED;
    if (n > 65535) return PCR_E_UNSUPPORTED;
    // (the limit is stated, and stays, in tiles of 32 x 32 window positions, of which the kernels' tiles are fewer)
    uint32_t limit = 1, rows, tmax;
    for (uint32_t i = 0; i < n; i++) limit = std::max(limit, ssim_limit_tiles((uint32_t)r->img[i].W, (uint32_t)r->img[i].H));
    if ((uint64_t)n * limit > kStaticSsimTiles) return PCR_E_RANGE;   // the record's tile sums do not fit the fixed array
    HIP_TRY(hipSetDevice(r->device));
    float2* part = nullptr;
    int rc = static_scratch(r->device, &part);
    if (rc) return rc;
    // (nothing to clear: every entry k_ssim_score reads is written by k_ssim_tiles in the same call)
    ssim_layout(r, &rows, &tmax);
    return launch_ssim(r, d_a, d_b, part, rows, tmax, d_scores, (hipStream_t)stream);
}

// ---- record creation (host only) ----
int pcr_scan_ends(const void* jpeg, size_t nbytes, uint64_t* ends, int max_ends, int* n_scans) {
    if (!jpeg || !ends || !n_scans || max_ends < 1) return PCR_E_ARG;
    const int s = enc::scan_ends((const uint8_t*)jpeg, nbytes, ends, max_ends);
    if (s <= 0) return PCR_E_FORMAT;
    *n_scans = s;
    return PCR_OK;
}

int pcr_record_size(const void* const* files, const size_t* sizes, uint32_t n, uint64_t* record_bytes, uint32_t* scan_groups) {
    if (!files || !sizes || !record_bytes) return PCR_E_ARG;
    enc::RecordPlan P;
    const int rc = enc::plan_record(files, sizes, n, &P);
    if (rc) return rc;
    *record_bytes = P.total;
    if (scan_groups) *scan_groups = P.G;
    return PCR_OK;
}

int pcr_record_write(const void* const* files, const size_t* sizes, const int32_t* labels, uint32_t n, void* out, size_t capacity, uint64_t* written) {
    if (!files || !sizes || !out) return PCR_E_ARG;
    enc::RecordPlan P;
    const int rc = enc::plan_record(files, sizes, n, &P);
    if (rc) return rc;
    if (written) *written = P.total;
    if (capacity < P.total) return PCR_E_RANGE;
    enc::write_record(P, files, labels, (uint8_t*)out);
    return PCR_OK;
}

int pcr_record_write_indexed(const void* const* files, const size_t* sizes, const int32_t* labels, uint32_t n, uint32_t entry_interval,
                             void* out, size_t capacity, uint64_t* written) {
    if (!files || !sizes || !out) return PCR_E_ARG;
    if (entry_interval < 1 || entry_interval > (1u << 20)) return PCR_E_RANGE;
    enc::IndexedPlan Q;
    const int rc = enc::plan_record_indexed(files, sizes, n, entry_interval, &Q);
    if (rc) return rc;
    if (written) *written = Q.P.total;
    if (capacity < Q.P.total) return PCR_E_RANGE;
    enc::write_record_indexed(Q, files, labels, (uint8_t*)out);
    return PCR_OK;
}

int pcr_transcode_progressive(const void* src_jpeg, size_t src_bytes, const int16_t* coef, size_t coef_count, uint32_t restart_interval,
                              void* out, size_t capacity, uint64_t* written) {
    if (!src_jpeg || !coef || !written) return PCR_E_ARG;
    std::vector<uint8_t> bytes;
    bytes.reserve(src_bytes + src_bytes / 4 + 1024);
    const int rc = enc::transcode_progressive((const uint8_t*)src_jpeg, src_bytes, coef, coef_count, restart_interval, &bytes);
    if (rc) return rc;
    *written = bytes.size();
    if (!out || capacity < bytes.size()) return PCR_E_RANGE;
    memcpy(out, bytes.data(), bytes.size());
    return PCR_OK;
}

int pcr_transcode_progressive_counted(const void* src_jpeg, size_t src_bytes, const int16_t* coef, size_t coef_count, uint32_t restart_interval,
                                      const uint32_t* counts, void* out, size_t capacity, uint64_t* written) {
    if (!src_jpeg || !coef || !written || !counts) return PCR_E_ARG;
    std::vector<uint8_t> bytes;
    bytes.reserve(src_bytes + src_bytes / 4 + 1024);
    const int rc = enc::transcode_progressive((const uint8_t*)src_jpeg, src_bytes, coef, coef_count, restart_interval, &bytes, counts);
    if (rc) return rc;
    *written = bytes.size();
    if (!out || capacity < bytes.size()) return PCR_E_RANGE;
    memcpy(out, bytes.data(), bytes.size());
    return PCR_OK;
}

int pcr_transcode_symbol_counts(const void* src_jpeg, size_t src_bytes, const int16_t* coef, size_t coef_count, uint32_t restart_interval,
                                uint32_t* counts) {
    if (!src_jpeg || !coef || !counts) return PCR_E_ARG;
    return enc::transcode_progressive((const uint8_t*)src_jpeg, src_bytes, coef, coef_count, restart_interval, nullptr, nullptr, counts);
}

// The batch of pcr_transcode_progressive(_counted) for the files a record was made of: one decode for coefficients, then the
// files, coded on the device where it counts the symbols too and no restart markers are asked for.
int pcr_transcode_batch(pcr_record* r, const void* const* files, const size_t* sizes, uint32_t n, uint32_t restart_interval, int device_counts, int threads,
                        void* out, const uint64_t* out_off, uint64_t* written, void* stream) {
    if (!r || !files || !sizes || !out || !out_off || !written || n != r->hdr.n || threads < 1) return PCR_E_ARG;
    if (restart_interval > 65535) return PCR_E_RANGE;
    const int k = (int)r->hdr.k_avail;
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    HIP_TRY(hipSetDevice(r->device));
    hipStream_t s = (hipStream_t)stream;
    Plan* plan = nullptr;
    r->resident_k = 0;                                       // the planes are refined in place, as for the coefficient export
    rc = run_entropy_stages(r, 0, k, s, true, &plan);
    if (rc) return rc;
    call_end(r);
    try {
    // (files whose frames are not those of the record's images are coded by their own: on the host, which has no others)
    bool on_device = device_counts && restart_interval == 0;
    std::vector<SourceFrame> frames(on_device ? n : 0);
    for (uint32_t i = 0; on_device && i < n; i++) {
        SourceFrame& F = frames[i];
        F.rc = enc::read_frame((const uint8_t*)files[i], sizes[i], nullptr, (size_t)(r->coef_off[i + 1] - r->coef_off[i]), &F.img, &F.frame);
        if (F.rc == kOk) on_device = same_frame(F.img, r->img[i]);
    }
    std::vector<int> status(n, PCR_OK);
    rc = on_device ? transcode_on_device(r, files, frames, (uint32_t)threads, out, out_off, written, status.data(), s)
                   : transcode_on_host(r, files, sizes, restart_interval, device_counts != 0, (uint32_t)threads, out, out_off, written, status.data(), s);
    if (rc) { (void)hipGetLastError(); return rc; }
    for (uint32_t i = 0; i < n; i++) if (status[i] && status[i] != PCR_E_RANGE) return status[i];
    for (uint32_t i = 0; i < n; i++) if (status[i]) return status[i];
    } catch (const std::bad_alloc&) { return PCR_E_NOMEM; }
    return PCR_OK;
}

int pcr_symbol_histograms(pcr_record* r, uint32_t restart_interval, uint32_t* d_hist, void* stream) {
    if (!r || !d_hist) return PCR_E_ARG;
    if (restart_interval > 65535) return PCR_E_RANGE;
    const int k = (int)r->hdr.k_avail;
    int rc = check_scan_group(r, k);
    if (rc) return rc;
    HIP_TRY(hipSetDevice(r->device));
    hipStream_t s = (hipStream_t)stream;
    Plan* plan = nullptr;
    r->resident_k = 0;                                       // the planes are refined in place, as for the coefficient export
    rc = run_entropy_stages(r, 0, k, s, true, &plan);
    if (rc) return rc;
    call_end(r);
    static_assert(PCR_HIST_ENTRIES == kHistPerImage, "header and kernel agree on the layout of the counts");
    hipLaunchKernelGGL(k_symbol_hist, dim3(r->hdr.n, kScriptScansMax), dim3(kHistLanes), 0, s, (const ImgDesc*)r->d.img, (const int16_t*)r->d.coef, r->d.coef_off,
                       restart_interval, d_hist, (ScanMarks*)nullptr, (uint32_t*)nullptr);
    if (hipGetLastError() != hipSuccess) return PCR_E_DEVICE;
    return PCR_OK;
}

int pcr_select_scan_group(pcr_record* r, float min_mean_score, uint8_t* d_work_a, uint8_t* d_work_b, size_t work_capacity, float* d_scores,
                          float* mean_by_group, int* scan_group, void* stream) {
    if (!r || !d_work_a || !d_work_b || !d_scores || !scan_group) return PCR_E_ARG;
    const uint32_t n = r->hdr.n;
    const int top = (int)r->hdr.k_avail;
    if (n == 0 || top < 1) return PCR_E_ARG;
    if (mean_by_group) for (int g = 0; g < (int)r->hdr.G; g++) mean_by_group[g] = -1.0f;
    int rc = pcr_decode_batch(r, top, d_work_b, work_capacity, stream, nullptr);              // the reference pictures
    if (rc) return rc;
    std::vector<float> host(n);
    *scan_group = top;
    for (int k = 1; k < top; k++) {
        rc = k == 1 ? pcr_decode_batch(r, 1, d_work_a, work_capacity, stream, nullptr) : pcr_upgrade_batch(r, k, d_work_a, work_capacity, stream, nullptr);
        if (!rc) rc = pcr_msssim_batch(r, d_work_a, d_work_b, d_scores, stream);
        if (rc) return rc;
        if (hipMemcpyAsync(host.data(), d_scores, n * sizeof(float), hipMemcpyDeviceToHost, (hipStream_t)stream) != hipSuccess ||
            hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return PCR_E_DEVICE;
        double sum = 0; uint32_t cnt = 0;
        for (uint32_t i = 0; i < n; i++) if (host[i] == host[i]) { sum += host[i]; cnt++; }   // (images too small to score are NaN)
        const float mean = cnt ? (float)(sum / cnt) : 1.0f;
        if (mean_by_group) mean_by_group[k - 1] = mean;
        if (mean >= min_mean_score) { *scan_group = k; return PCR_OK; }
    }
    if (mean_by_group) mean_by_group[top - 1] = 1.0f;
    return PCR_OK;
}

int pcr_probe_scalar_issue_rate(int device_id, int waves_per_cu, double* ginst_per_s) {
    if (!ginst_per_s || waves_per_cu < 1 || waves_per_cu > 32) return PCR_E_ARG;
    HIP_TRY(hipSetDevice(device_id));
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, device_id));
    const uint32_t grid = (uint32_t)prop.multiProcessorCount * (uint32_t)waves_per_cu, iters = 20000;
    uint32_t* d_out = nullptr;
    if (hipMalloc((void**)&d_out, grid * sizeof(uint32_t)) != hipSuccess) return PCR_E_NOMEM;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = PCR_OK;
    float ms = 0;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) rc = PCR_E_DEVICE;
    for (int rep = 0; rep < 2 && rc == PCR_OK; rep++) {          // the first launch warms up
        (void)hipEventRecord(e0, nullptr);
        hipLaunchKernelGGL(k_probe_scalar, dim3(grid), dim3(64), 0, nullptr, d_out, iters, 1u);
        (void)hipEventRecord(e1, nullptr);
        if (hipEventSynchronize(e1) != hipSuccess || hipGetLastError() != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = PCR_E_DEVICE;
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipFree(d_out);
    if (rc == PCR_OK) *ginst_per_s = (double)grid * iters * 16.0 / (ms * 1e-3) / 1e9;
    return rc;
}

int pcr_prefix_length(const void* first_bytes, size_t nbytes, int k, uint64_t* need) {
    if (!first_bytes || !need) return PCR_E_ARG;
    const uint8_t* b = (const uint8_t*)first_bytes;
    if (nbytes < 24) { *need = 24; return PCR_E_TRUNCATED; }
    if (b[0] != 'P' || b[1] != 'C' || b[2] != 'R' || b[3] != '1') return PCR_E_FORMAT;
    if (ld_le32(b + 4) != 1 && ld_le32(b + 4) != 2) return PCR_E_UNSUPPORTED;
    const uint32_t G = ld_le32(b + 12);
    if (k < 1 || (uint32_t)k > G) return PCR_E_RANGE;
    const size_t pos = hdr_group_end_pos((uint32_t)k - 1);
    if (nbytes < pos + 8) { *need = pos + 8; return PCR_E_TRUNCATED; }
    *need = ld_le64(b + pos);
    return PCR_OK;
}

// ---- loader: re-used pinned staging buffers, device buffers, streams and handles ----
struct pcr_loader_slot {
    void* host = nullptr; uint8_t* dev = nullptr; hipStream_t stream = nullptr; pcr_record* rec = nullptr;
};
struct pcr_loader {
    int device = 0; size_t slot_bytes = 0;
    std::vector<pcr_loader_slot> slots;
    // token bucket: `rate` bytes are granted per second, at most `burst` are saved up
    double rate = 0, burst = 0, tokens = 0;
    std::chrono::steady_clock::time_point last;
};

int pcr_loader_create(int device_id, int slots, size_t slot_bytes, pcr_loader** out) {
    if (!out || slots < 1 || slots > 16 || slot_bytes < 24 || slot_bytes >= (1ull << 32)) return PCR_E_ARG;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device_id < 0 || device_id >= ndev) { (void)hipGetLastError(); return PCR_E_DEVICE; }
    HIP_TRY(hipSetDevice(device_id));
    pcr_loader* ld = new (std::nothrow) pcr_loader();
    if (!ld) return PCR_E_NOMEM;
    ld->device = device_id; ld->slot_bytes = slot_bytes; ld->slots.resize((size_t)slots);
    ld->last = std::chrono::steady_clock::now();
    int rc = PCR_OK;
    for (auto& sl : ld->slots) {
        if (hipHostMalloc(&sl.host, slot_bytes, hipHostMallocDefault) != hipSuccess) { rc = PCR_E_NOMEM; break; }
        if (hipMalloc((void**)&sl.dev, slot_bytes + 64) != hipSuccess) { rc = PCR_E_NOMEM; break; }
        if (hipStreamCreateWithFlags(&sl.stream, hipStreamNonBlocking) != hipSuccess) { rc = PCR_E_DEVICE; break; }
    }
    if (rc) { (void)hipGetLastError(); pcr_loader_destroy(ld); return rc; }
    *out = ld;
    return PCR_OK;
}

void pcr_loader_destroy(pcr_loader* ld) {
    if (!ld) return;
    (void)hipSetDevice(ld->device);
    for (auto& sl : ld->slots) {
        if (sl.stream) (void)hipStreamSynchronize(sl.stream);
        if (sl.rec) pcr_close(sl.rec);
        if (sl.stream) (void)hipStreamDestroy(sl.stream);
        if (sl.dev) (void)hipFree(sl.dev);
        if (sl.host) (void)hipHostFree(sl.host);
    }
    delete ld;
}

static pcr_loader_slot* loader_slot(pcr_loader* ld, int slot) {
    return (ld && slot >= 0 && (size_t)slot < ld->slots.size()) ? &ld->slots[(size_t)slot] : nullptr;
}

int pcr_loader_staging(pcr_loader* ld, int slot, void** host, size_t* capacity) {
    pcr_loader_slot* sl = loader_slot(ld, slot);
    if (!sl || !host) return PCR_E_ARG;
    *host = sl->host;
    if (capacity) *capacity = ld->slot_bytes;
    return PCR_OK;
}

int pcr_loader_stream(pcr_loader* ld, int slot, void** hip_stream) {
    pcr_loader_slot* sl = loader_slot(ld, slot);
    if (!sl || !hip_stream) return PCR_E_ARG;
    *hip_stream = (void*)sl->stream;
    return PCR_OK;
}

int pcr_loader_set_rate(pcr_loader* ld, double bytes_per_second, double burst_bytes) {
    if (!ld || bytes_per_second < 0 || burst_bytes < 0) return PCR_E_ARG;
    ld->rate = bytes_per_second; ld->burst = burst_bytes; ld->tokens = 0;
    ld->last = std::chrono::steady_clock::now();
    return PCR_OK;
}

// blocks until the bucket holds `bytes` tokens (a request larger than the burst size waits for the whole amount)
static void loader_take_tokens(pcr_loader* ld, double bytes) {
    if (ld->rate <= 0) return;
    for (;;) {
        const auto now = std::chrono::steady_clock::now();
        ld->tokens += std::chrono::duration<double>(now - ld->last).count() * ld->rate;
        ld->last = now;
        const double cap = std::max(ld->burst, bytes);
        if (ld->tokens > cap) ld->tokens = cap;
        if (ld->tokens >= bytes) { ld->tokens -= bytes; return; }
        std::this_thread::sleep_for(std::chrono::duration<double>((bytes - ld->tokens) / ld->rate));
    }
}

int pcr_loader_upload(pcr_loader* ld, int slot, size_t nbytes, pcr_record** rec) {
    pcr_loader_slot* sl = loader_slot(ld, slot);
    if (!sl) return PCR_E_ARG;
    if (nbytes < 24) return PCR_E_TRUNCATED;
    if (nbytes > ld->slot_bytes) return PCR_E_RANGE;
    HIP_TRY(hipSetDevice(ld->device));
    HIP_TRY(hipStreamSynchronize(sl->stream));                // the slot's buffers and handle are free again
    loader_take_tokens(ld, (double)nbytes);
    HIP_TRY(hipMemcpyAsync(sl->dev, sl->host, nbytes, hipMemcpyHostToDevice, sl->stream));
    // (the handle is laid out from the host's bytes while the copy runs; bind_device waits for the copy)
    const bool fresh = !sl->rec;
    if (fresh) {
        sl->rec = new (std::nothrow) pcr_record();
        if (!sl->rec) { (void)hipStreamSynchronize(sl->stream); return PCR_E_NOMEM; }
        sl->rec->device = ld->device; sl->rec->borrowed = true; sl->rec->stage.pinned = true;
    }
    const int rc = bind_device(sl->rec, sl->dev, nbytes, (const uint8_t*)sl->host, sl->stream);
    if (rc && fresh) { pcr_close(sl->rec); sl->rec = nullptr; }
    if (rc) return rc;
    if (rec) *rec = sl->rec;
    return PCR_OK;
}

// pread until `count` bytes are in or the file ends; returns the bytes read, or -1
static ssize_t read_fully(int fd, uint8_t* dst, size_t count, off_t at) {
    size_t got = 0;
    while (got < count) {
        const ssize_t r = pread(fd, dst + got, count - got, at + (off_t)got);
        if (r < 0) return -1;
        if (r == 0) break;
        got += (size_t)r;
    }
    return (ssize_t)got;
}

int pcr_loader_read_file(pcr_loader* ld, int slot, const char* path, int k, size_t* nbytes, pcr_record** rec) {
    pcr_loader_slot* sl = loader_slot(ld, slot);
    if (!sl || !path) return PCR_E_ARG;
    HIP_TRY(hipSetDevice(ld->device));
    HIP_TRY(hipStreamSynchronize(sl->stream));                // the staging buffer is free again
    const int fd = open(path, O_RDONLY | O_CLOEXEC);
    if (fd < 0) return PCR_E_ARG;
    uint8_t* host = (uint8_t*)sl->host;
    const size_t head = std::min<size_t>(24 + 8 * 64, ld->slot_bytes);
    const ssize_t got = read_fully(fd, host, head, 0);
    int rc = got < 0 ? PCR_E_ARG : PCR_OK;
    uint64_t need = 0;
    if (!rc) rc = pcr_prefix_length(host, (size_t)got, k, &need);   // (a file that ends inside its header: TRUNCATED)
    if (!rc && need > ld->slot_bytes) rc = PCR_E_RANGE;
    if (!rc && need > (uint64_t)got) {
        const ssize_t more = read_fully(fd, host + got, (size_t)(need - (uint64_t)got), (off_t)got);
        if (more < 0) rc = PCR_E_ARG;
        else if ((uint64_t)got + (uint64_t)more < need) rc = PCR_E_TRUNCATED;
    }
    (void)close(fd);
    if (rc) return rc;
    if (nbytes) *nbytes = (size_t)need;
    return pcr_loader_upload(ld, slot, (size_t)need, rec);
}

int pcr_loader_decode(pcr_loader* ld, int slot, int k, uint8_t* out, size_t cap, int32_t* d_status) {
    pcr_loader_slot* sl = loader_slot(ld, slot);
    if (!sl || !sl->rec) return PCR_E_ARG;
    return pcr_decode_batch(sl->rec, k, out, cap, (void*)sl->stream, d_status);
}

int pcr_loader_decode_crop(pcr_loader* ld, int slot, int k, const pcr_crop* d_crops, uint8_t* d_pixels, size_t pixel_capacity, int out_h, int out_w,
                           const float* mean, const float* inv_std, void* d_out_f16, size_t out_capacity, int32_t* d_status) {
    pcr_loader_slot* sl = loader_slot(ld, slot);
    if (!sl || !sl->rec) return PCR_E_ARG;
    return pcr_decode_crop_batch(sl->rec, k, d_crops, d_pixels, pixel_capacity, out_h, out_w, mean, inv_std, d_out_f16, out_capacity,
                                 (void*)sl->stream, d_status);
}

int pcr_loader_wait(pcr_loader* ld, int slot) {
    pcr_loader_slot* sl = loader_slot(ld, slot);
    if (!sl) return PCR_E_ARG;
    HIP_TRY(hipSetDevice(ld->device));
    HIP_TRY(hipStreamSynchronize(sl->stream));
    return PCR_OK;
}

const char* pcr_strerror(int code) {
    switch (code) {
        case PCR_OK: return "ok";
        case PCR_E_ARG: return "invalid argument";
        case PCR_E_FORMAT: return "malformed record or JPEG stream";
        case PCR_E_TRUNCATED: return "record bytes do not reach the requested scan group";
        case PCR_E_UNSUPPORTED: return "unsupported JPEG feature or record size";
        case PCR_E_RANGE: return "index or capacity out of range";
        case PCR_E_NOMEM: return "out of memory";
        case PCR_E_DEVICE: return "HIP device error";
        default: return "unknown error";
    }
}

}  // extern "C"
