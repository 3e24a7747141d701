// Which scans of an image may be decoded by one launch, and in what order the others follow.  Host code; needs nothing of HIP.
//
// Two scans of a component whose bands overlap have to be decoded in file order: a refinement scan reads what the scans
// before it made of a block, and a first scan over coefficients that an earlier scan of the component holds (T.81 rules it
// out, files have it) stores over them.  Scans of different components, or of bands that do not meet, are independent.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "pcr_format.h"

namespace pcr {

// Level of each of an image's scans: 1 + the highest level of an earlier scan it has to follow.  Returns the highest one.
inline uint32_t scan_levels(const ScanDesc* s, uint32_t count, uint8_t* level) {
    uint32_t most = 0;
    for (uint32_t g = 0; g < count; g++) {
        uint32_t lv = 1;
        for (uint32_t q = 0; q < g; q++) {
            bool share = false;
            for (int a = 0; a < s[g].ns; a++) for (int b = 0; b < s[q].ns; b++) if (s[g].comp[a] == s[q].comp[b]) share = true;
            if (share && s[q].Ss <= s[g].Se && s[g].Ss <= s[q].Se) lv = std::max<uint32_t>(lv, level[q] + 1u);
        }
        level[g] = (uint8_t)lv;
        most = std::max(most, lv);
    }
    return most;
}

// A chain: scans whose interval j is decoded by the wavefronts of one workgroup (k_decode_waves).  units: intervals;
// count: scans; byte w of waits: the earlier scans of the chain that scan w follows through the image.
constexpr uint32_t kChainWaves = 8;
struct ScanChain { uint32_t img, cost, units, count, scan[kChainWaves]; uint64_t waits; };

// The chains of a launch that takes all scans of a call (add), or, where some of them cannot keep in step, only those that
// wait for nothing (add_level_one).
//
// In step: the AC scans of one component in file order, each refinement scan following the scans it builds on.  Interval j
// of each of them has to cover the same blocks, so restart intervals must agree; entry points, which every scan has at
// places of its own, rule it out where one of the scans builds on another.  ONLY REFINEMENT SCANS WAIT: the symbol loop of
// the first scans asks for no block, and DC first scans are workgroups of their own.  A first scan that would have to
// follow an earlier scan of the call therefore rules it out too, and all is decoded level by level.
struct ChainSet {
    std::vector<ScanChain> ac, dc;
    bool possible = true;

    static ScanChain alone(uint32_t i, uint32_t g, const ScanDesc& sd, uint32_t units) {
        ScanChain c{};
        c.img = i; c.cost = sd.data_len / std::max(1u, units) * (sd.Ah ? 2u : 1u);     // (a byte of a refinement scan takes a wavefront about twice as long)
        c.units = units; c.count = 1; c.scan[0] = g;
        return c;
    }

    // Scans k0 .. upto - 1 of image i: scan descriptors, units and entry points (0: none) of its scans.
    void add(uint32_t i, const ScanDesc* s, const uint32_t* units, const uint32_t* entries, uint32_t k0, uint32_t upto) {
        std::vector<uint32_t> comp_scans[kMaxComp];
        uint32_t dc_seen = 0;                                  // components whose DC some scan of the call has brought
        for (uint32_t g = k0; g < upto; g++) {
            if (is_sequential_scan(s[g])) possible = false;
            else if (s[g].Ss > 0) comp_scans[s[g].comp[0]].push_back(g);
            else if (s[g].Ah == 0) {
                for (int a = 0; a < s[g].ns; a++) {
                    const uint32_t bit = 1u << s[g].comp[a];
                    if (dc_seen & bit) possible = false;
                    dc_seen |= bit;
                }
                dc.push_back(alone(i, g, s[g], units[g]));
            }
        }
        for (const auto& v : comp_scans) if (!v.empty()) add_component(i, s, units, entries, v);
    }
    void add_level_one(uint32_t i, const ScanDesc* s, const uint8_t* level, const uint32_t* units, uint32_t k0, uint32_t upto) {
        for (uint32_t g = k0; g < upto; g++) {
            if (is_sequential_scan(s[g]) || s[g].Ah > 0 || level[g] != 1) continue;
            (s[g].Ss > 0 ? ac : dc).push_back(alone(i, g, s[g], units[g]));
        }
    }

private:
    void add_component(uint32_t i, const ScanDesc* s, const uint32_t* units, const uint32_t* entries, const std::vector<uint32_t>& scans) {
        const uint32_t first = scans[0];
        std::vector<uint32_t> waits(scans.size(), 0);
        bool ordered = false, same = scans.size() <= kChainWaves;
        for (size_t a = 0; a < scans.size(); a++) {
            const ScanDesc& A = s[scans[a]];
            if (a > 0) same = same && A.ri == s[first].ri && units[scans[a]] == units[first] && entries[scans[a]] == 0 && entries[first] == 0;
            for (size_t b = 0; b < a; b++) {
                const ScanDesc& B = s[scans[b]];
                if (B.Ss > A.Se || A.Ss > B.Se) continue;
                ordered = true;
                same = same && A.Ah > 0;
                if (b < 32) waits[a] |= 1u << b;
            }
        }
        if (!ordered) { for (uint32_t g : scans) ac.push_back(alone(i, g, s[g], units[g])); return; }
        if (!same) { possible = false; return; }
        ScanChain c{};
        c.img = i; c.units = units[first]; c.count = (uint32_t)scans.size();
        for (size_t a = 0; a < scans.size(); a++) {
            c.scan[a] = scans[a];
            c.cost = std::max(c.cost, alone(i, scans[a], s[scans[a]], units[scans[a]]).cost);
            c.waits |= (uint64_t)waits[a] << (8 * a);
        }
        ac.push_back(c);
    }
};

}  // namespace pcr
