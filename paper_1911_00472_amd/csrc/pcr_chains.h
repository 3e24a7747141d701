// Which scans of an image may be decoded by one launch, and in what order the others follow; and which decoder a launch of DC
// first scans is for.  Host code; needs nothing of HIP.
//
// Two scans of a component whose bands overlap have to be decoded in file order: a refinement scan reads what the scans
// before it made of a block, and a first scan over coefficients that an earlier scan of the component holds (T.81 rules it
// out, files have it) stores over them.  Scans of different components, or of bands that do not meet, are independent.
#pragma once
#include <algorithm>
#include <cstdint>
#include <utility>
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
// count: scans; refines: those of them that are refinement scans, a bit each (noted where the descriptors come one after the other: looked up again in the
// order of the chains, by length, it took 20 of 600 us of a plan of 2048 pictures); byte w of waits: the earlier scans of the chain that
// scan w follows through the image.
constexpr uint32_t kChainWaves = 8;
struct ScanChain { uint32_t img, cost, units; uint16_t count, refines; uint32_t scan[kChainWaves]; uint64_t waits; };

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
        c.units = units; c.count = 1; c.refines = sd.Ah > 0 ? 1 : 0; c.scan[0] = g;
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
        c.img = i; c.units = units[first]; c.count = (uint16_t)scans.size();
        for (size_t a = 0; a < scans.size(); a++) {
            c.scan[a] = scans[a];
            if (s[scans[a]].Ah > 0) c.refines |= (uint16_t)(1u << a);
            c.cost = std::max(c.cost, alone(i, scans[a], s[scans[a]], units[scans[a]]).cost);
            c.waits |= (uint64_t)waits[a] << (8 * a);
        }
        ac.push_back(c);
    }
};

// The larger of a launch's longest unit so far and of a scan of `all` in `units` units, on average (divided only where it is larger: records
// have tens of thousands of scans).
inline void longest_of(uint32_t* longest, uint64_t all, uint32_t units) {
    if (all >= ((uint64_t)*longest + 1) * units) *longest = (uint32_t)(all / units);
}

// A launch of first scans by wavefronts, and whether k_first_split -- many lanes for every unit -- goes ahead of it.
//
// The wavefronts take as long as the longest unit, 7.5 ns a bit and 60 a block of an AC scan, 75 a block of a DC scan, and more
// with many of them; the lanes some 35 us, what a DC scan takes to fall into step (longest where its MCUs have many blocks),
// and what the workgroups cost that find no room at once.  us a call of plain records, wavefronts / lanes:
//                                          one picture     32            256           1024
//   4:2:0, quality 90, noisy, scan group 5
//      64 x 64                              94 / 90      101 / 103     105 / 115     134 / 222
//      100 x 100                           148 / 101     162 / 142     176 / 174     219 / 292
//      128 x 128                           196 / 130     214 / 151     231 / 190     278 / 321
//   the same at 2, 128 x 128               125 / 129     126 / 148     143 / 184     190 / 254
//   less noise, at 5, 256 x 256            299 / 161     334 / 200     386 / 307     506 / 500
//   quality 75, smooth, at 5, 256 x 256    174 / 165     187 / 273     237 / 274     356 / 458
//      400 x 400                           340 / 155     352 / 208     435 / 301
//      700 x 700                           899 / 166     947 / 252
//   4:4:4, quality 95, at 5, 200 x 200     873 / 237     921 / 270    1012 / 377    1124 / 728
//   gray, at 3, 300 x 300                  658 / 107     717 / 122     774 / 168
//   scan group 1: 4:2:0 256 x 256          174 / 154     181 / 189     186 / 258     246 / 300
//      400 x 400                           332 / 139     339 / 172     365 / 240
//   4:4:4 200 x 200                        222 / 101     230 / 150     245 / 162     289 / 187
//   gray 300 x 300                         190 / 77      200 / 99      207 / 104
// DC scans of MCUs of more than three blocks that take more than six bits a block (strong, coarse contrasts: few symbols in a piece, codes of luma and chroma
// of like lengths) do not fall into step in a scan or two of a hundred, and then the launch by wavefronts is as long as without: photographs of
// 7.8 bits a block at scan group 1, 128 of them 583 / 735, 1024 699 / 876, where those of 3.7 to 5.4 bits a block are the gains above.
// 1024 lanes a unit instead of 256 are better only for very long units: 1000 x 1000 at quality 90, noisy, scan group 5 401 / 673 us a
// call (8264 by wavefronts), 32 of them 491 / 801; 4:4:4 200 x 200 as above 243 / 237.
struct FirstSplitLaunch {
    uint32_t units = 0, ac_bits = 0, ac_blocks = 0, dc_units = 0, dc_blocks = 0, dc_per_mcu = 0;      // bits, blocks: of the longest unit
    uint64_t ac_visits = 0, dc_visits = 0, dc_bits = 0;       // blocks of all units
    void add(const ImgDesc& img, const ScanDesc& sd, uint32_t count) {
        if (sd.Ah != 0 || is_sequential_scan(sd) || count == 0) return;
        uint32_t per_mcu = sd.ns > 1 ? 0u : 1u;
        for (int j = 0; j < sd.ns && sd.ns > 1; j++) per_mcu += (uint32_t)img.hs[sd.comp[j]] * img.vs[sd.comp[j]];
        if (sd.Ss > 0) {
            units += count; ac_visits += (uint64_t)sd.mcus;
            longest_of(&ac_bits, (uint64_t)sd.data_len * 8, count); longest_of(&ac_blocks, (uint64_t)sd.mcus * per_mcu, count);
        } else {
            dc_units += count; dc_visits += (uint64_t)sd.mcus * per_mcu; dc_bits += (uint64_t)sd.data_len * 8;
            longest_of(&dc_blocks, (uint64_t)sd.mcus * per_mcu, count); dc_per_mcu = std::max(dc_per_mcu, per_mcu);
        }
    }
    // with_dc: the DC scans are part of the launch
    bool pays(bool with_dc) const {
        const float n = (float)(units + (with_dc ? dc_units : 0u)), dc = with_dc ? (float)dc_blocks : 0.f, seen = (float)ac_visits + (with_dc ? (float)dc_visits : 0.f);
        if (n == 0.f) return false;
        const float in_step = dc_per_mcu > 3 ? 120.f : (dc_per_mcu > 1 ? 60.f : 30.f);
        const float waves = std::max(0.0075f * (float)ac_bits + 0.06f * (float)ac_blocks, 0.075f * dc) + 0.0001f * (float)ac_visits + (with_dc ? 0.00004f * (float)dc_visits : 0.f);
        // (what does not fall into step the wavefronts decode behind the lanes)
        const float again = dc_per_mcu > 3 && dc_bits > 6 * dc_visits ? 0.075f * dc : 0.f;
        const float lanes = 35.f + std::max(std::min(in_step, 0.1f * dc), 0.0008f * (float)ac_bits) + 0.028f * n + 0.00004f * seen + again;
        return lanes < waves;
    }
    bool wide(bool with_dc) const { return units + (with_dc ? dc_units : 0u) <= 512 && ac_bits >= 131072; }
};

// A launch of DC first scans, and whether it goes to the lane decoders instead of to a wavefront per unit.
//
// A lane decodes a DC symbol with a fifth of the instructions a wavefront spends on it, but a launch of lanes takes as long as
// its longest unit, however few there are, and the wavefronts' time a symbol only grows once they fill the scalar units.  So
// what decides is the launch's blocks over those of its longest unit: `full`, the number of units where all are alike.  us a call
// by wavefronts / by lanes (units and blocks as a plan counts them: a record written with an entry every 64 MCUs has one every 32
// in DC first scans):
//   scan group 1, one record open; full =           2048         4096         6144         8192
//     cut into units of   32 blocks (gray)           61 / 69      67 / 71                   72 / 66
//                         96 (4:4:4)                 78 / 91      88 / 92                  106 / 93
//                        192 (4:2:0)                 89 / 110    112 / 118    131 / 127    151 / 134
//                        384                        124 / 155    161 / 171    224 / 214    271 / 237
//                       3072                                     908 / 991   1180 / 1175  1504 / 1333
//     whole scans of       9 blocks (gray)           81 / 96     112 / 117    149 / 148    190 / 177
//                        216                        129 / 140    208 / 196    261 / 233    341 / 289
//                        384                        165 / 189    235 / 226    331 / 303    444 / 379
//                        864                        230 / 289    401 / 405    535 / 507    695 / 609
//                       3750                        743 / 1031  1178 / 1274  1539 / 1528  2006 / 1787
//     of many sizes, the longest of  384 blocks     174 / 199    288 / 276    422 / 364                (full: 2012, 4029, 6044)
//                                   1536            452 / 573    588 / 675    849 / 851                (2793, 3724, 5587)
//   the same where wavefronts would decode them beside the AC scans of the call, in one launch, and lanes behind it (scan group 2):
//     cut into units of  192 blocks                 134 / 177    182 / 210                 328 / 325
//     whole scans of     384                                     416 / 465                 737 / 735
//     of many sizes, up to 726 blocks                            624 / 704                1154 / 1152  (3978, 7957)
//   four records open, scan group 1, whole scans; units of each and full: 2048, 2048        4096, 4096          6144, 6144
//     of 384 blocks                                 453 / 472    823 / 724   1188 / 977
//     of 1536                                      1043 / 1238  1912 / 1785
//     of many sizes, up to  384 blocks              295 / 348    547 / 478    767 / 648                (full: 1007, 2012, 3021)
//                           720                     360 / 513    556 / 659    852 / 795                (734, 1468, 2202)
//                          1260                     536 / 826    847 / 1058  1339 / 1294               (1061, 2122, 3183)
struct DcLaunch {
    uint32_t units = 0, scans = 0, longest = 0;               // longest: blocks of the longest unit
    uint64_t blocks = 0;
    void add(const ImgDesc& img, const ScanDesc& sd, uint32_t n) {
        uint32_t per_mcu = 0;
        for (int j = 0; j < sd.ns; j++) per_mcu += sd.ns > 1 ? (uint32_t)img.hs[sd.comp[j]] * img.vs[sd.comp[j]] : 1u;
        if (n == 0) return;
        units += n; scans++; blocks += (uint64_t)sd.mcus * per_mcu;
        longest = std::max(longest, (n == 1 ? sd.mcus : (sd.mcus + n - 1) / n) * per_mcu);
    }
    // several: the process has more than one record open; beside: the launch could be part of one of AC scans by wavefronts
    bool by_lanes(bool several, bool beside) const {
        const uint64_t full = blocks / std::max(1u, longest);
        if (several) return units >= 4096 && full >= (longest <= 768 ? 2000u : 3000u);
        if (beside) return full >= 8192;
        const bool cut = units >= 2 * scans;
        return full >= (cut || longest < 64 || longest > 768 ? 6144u : longest <= 384 ? 3584u : 4608u);
    }
};

// A launch of AC scans (first scans, or refinement scans of one level) of records with several units a scan, and whether a lane
// decodes a unit, 64 of them a wavefront, or a wavefront does.
//
// Wavefronts are bound by the scalar instructions of all units, lanes by the symbols of the longest unit one after the other, with a
// fifth of the instructions in total.  What decides is the launch's bits and blocks against those of its longest unit: the figures
// below are a fit (non-negative, of the difference) to what calls of 49 sizes of one record took at three or four scan groups
// each.  us a call by wavefronts / by lanes, one record open (units of the launch of first scans, thousands):
//                                              scan group 2             5                       6                       10
//   340 x 340, quality 90, noisy, entries 64   5.6  193 / 186    14  243 / 325     421 / 598      715 / 1004
//                                             11    275 / 222    29  382 / 370     718 / 706     1267 / 1214
//                                             22    467 / 313    57  689 / 488    1308 / 844     2359 / 1394
//   the same at quality 85, entries 32         4.8  135 / 123    12  150 / 146     231 / 250      364 / 413
//                                             11    183 / 151    28  218 / 170     363 / 287      625 / 474
//                                             22    267 / 182    56  337 / 202     619 / 347     1114 / 559
//   700 x 700, quality 80, entries 64          5.4  180 / 166    12  199 / 175     313 / 308      530 / 554
//                                             11    245 / 198    25  260 / 207     470 / 363      861 / 630
//   340 x 340, 4:4:4, quality 88, entries 64   5.6  223 / 193    22  303 / 286     462 / 496      993 / 1021
//                                             11    353 / 255    45  570 / 376     858 / 682     1895 / 1306
//   128 x 128, quality 85, entries 64          2.3  142 / 161     6  170 / 192     254 / 374      410 / 683
//                                              5.5  198 / 178    14  238 / 224     395 / 418      693 / 763
// A record decoded beside others leaves them what it does not use, in part (they share hardware queues): its own work counts half as
// much again.  (Over 50 sizes of two and four records that loses 1 % against the better of the two, counted as often as there are
// records 3 to 5 %.)  Where the fit says less than its error, and for units of more than a hundred blocks, their number decides:
// 8192 with others open and 32768 without; so it does for refinement scans whose wavefronts of lanes would be a quarter empty (2048
// pictures of 82 x 120 at scan group 7: 481 us a call with those by wavefronts, 535 by lanes).
struct LanesLaunch {
    uint32_t units = 0, jobs = 0, longest_bits = 0, longest_blocks = 0;      // of the scan whose units are longest on average
    uint64_t bits = 0, blocks = 0;
    void add(const ScanDesc& sd, uint32_t n) {
        if (n == 0) return;
        units += n; bits += (uint64_t)sd.data_len * 8; blocks += sd.mcus;
        longest_of(&longest_bits, (uint64_t)sd.data_len * 8, n); longest_of(&longest_blocks, sd.mcus, n);
    }
    bool many(bool several) const { return units >= (several ? 8192u : 32768u) && units >= 32u * jobs; }     // (jobs half full at least)
    bool by_lanes(bool refine, bool several) const {
        const bool many = this->many(several);
        if (blocks > 100ull * units || (refine && units < 50u * jobs)) return many;
        const float much = several ? 1.5f : 1.f, mbit = much * (float)bits * 1e-6f, kblk = much * (float)blocks * 1e-3f;
        const float gain = refine ? 1.2f * mbit + 0.22f * kblk - 0.058f * (float)longest_bits - 1.1f * (float)longest_blocks - 10.f
                                  : 1.75f * mbit + 0.064f * kblk - 0.041f * (float)longest_bits - 0.029f * (float)longest_blocks - 0.011f * much * (float)jobs + 15.f;
        const float unsure = several ? 30.f : (refine ? 25.f : 12.f);
        return gain > (many ? -unsure : unsure);
    }
};

// A launch of refinement scans by wavefronts (of one level, or of all where the scans of a component are decoded side by side), and
// whether their units have three wavefronts each (pcr_refine_trio.h).
//
// Three take two thirds of the time of one while the launch takes as long as its longest unit, and up to half as much again once the launches
// of all records in flight fill the chip.  So what decides is `full`: what the launch asks of the chip over its longest unit, in bits, a block counted as
// 14 and the start of a workgroup as 800 where it is of a chain (it brings tables, and takes the room of the widest one, whatever is in it), as 100 where it is of a unit, first scans
// beside the refinement scans by half of theirs (they keep one wavefront).  Where the line lies depends on the records decoded at a time, of which
// the records the process has open are all that is known: a program may keep several open and decode them one after another, each when the
// last one is done.  Three wavefronts gain most there, so the lines for several are no lower than that what is lost where all are in flight
// stays within 4 %.  us a call by one wavefront a unit / by three (n pictures a record; full), calls of all records issued without waiting for any:
//                                                  one record              two                    four
//   plain records (all scans side by side)
//     300 to 500 pixels, scan group 10   n 400    5716 / 4123  (702)     7412 / 5881         14404 / 12175
//                                          512    5860 / 4256  (900)     7703 / 6954         14917 / 14470
//                                          640    6038 / 4394  (1123)    8332 / 8474         15914 / 16912
//                                          800    6223 / 4906  (1402)    9053 / 10544
//                                         1024    6456 / 6344  (1796)   10218 / 13394
//     96 x 96, 4:4:4, scan group 6         700     304 / 285   (1256)     591 / 553            825 / 899
//                                         1200     349 / 396   (2132)     543 / 687           1116 / 1420
//     192 x 192, 4:4:4, 6                  700     897 / 798   (1085)    1377 / 1430          2071 / 2709
//     128 x 128, gray, 6                   550     496 / 400   (1111)     726 / 742           1431 / 1468
//                                          900     571 / 650   (1803)     919 / 1095          1562 / 1981
//     64 x 64, 10                          400     213 / 188   (988)      265 / 274            525 / 544
//     24 x 24, 8                           250     115 / 112   (1357)      130 / 132            253 / 265
//                                          900     121 / 137   (4666)     161 / 192            324 / 389
//   a marker every MCU row, 256 x 256, 10   16     160 / 150   (1179)     187 / 206            334 / 373
//                                           32     170 / 208   (2442)     232 / 312            444 / 617
//   entry points every 64 MCUs (level by level)
//     17 to 320 pixels, 10                  64     243 / 228    (949)     284 / 284            520 / 529
//                                          128     271 / 280   (1675)     335 / 364            649 / 739
// and calls that set out together and are waited for together:
//     300 to 500 pixels, scan group 10   n 512    5674 / 4132   (945)     8780 / 7165         14515 / 14170
//                                          600    5880 / 4282  (1090)     9000 / 7853         15355 / 16027
//                                          640    5911 / 4329  (1182)     9122 / 8320         15787 / 16927
//                                          720    5984 / 4538  (1290)     9453 / 9360
//     256 x 256, 10                        500    1673 / 1255   (882)     2721 / 2387          4696 / 4626
//                                          600    1720 / 1378  (1055)     2906 / 2752          5029 / 5387
//     192 x 192, 4:4:4, 6                  700     825 / 727   (1145)     1369 / 1344          2386 / 2596; of 500 (818) 2035 / 2000
//     128 x 128, gray, 6                   550     493 / 395    (966)      797 / 728           1354 / 1347
//     64 x 64, 10                          500     211 / 191                314 / 318            546 / 586
//   a marker every MCU row, 256 x 256, 10   16     159 / 153                225 / 234            364 / 394
//   entry points, level by level, two launches a call (the larger full)
//     17 to 320 pixels, every 64, 10        64     246 / 231   (949)      343 / 329            541 / 539
//     429 x 559, gray, every 32, 6           4     140 / 134   (889)      191 / 184            289 / 288
//                                            6     142 / 140              198 / 200            308 / 322
//     300 x 300, 4:4:4, every 128, 8        20     214 / 205              301 / 285            481 / 462
// (With lines of 950 for two and three records, 700 from four on and 500 a workgroup three records of 512 photographs, decoded one after another, took 5241 instead of 4155.)
struct TrioLaunch {
    uint64_t work = 0, beside = 0; uint32_t longest = 0, groups = 0; bool chains = false;      // groups: workgroups of the launch; chains: each of a chain of scans, not of a unit
    void add(const LanesLaunch& l) {
        work += l.bits + 14 * l.blocks;
        longest = std::max(longest, l.longest_bits + 14 * l.longest_blocks);
    }
    void add_beside(const LanesLaunch& l) { beside += l.bits + 14 * l.blocks; }
    bool pays(int open_records) const {
        const uint64_t line = open_records <= 1 ? 1500 : (open_records <= 3 ? 1170 : 1025);
        return longest > 0 && work + beside / 2 + (chains ? 800ull : 100ull) * groups <= line * (longest + 70);
    }
};

// The MCUs of a DC scan, as far as lanes that decode them in step have to agree on them.
inline uint32_t dc_mcu_shape(const ImgDesc& img, const ScanDesc& sd) {
    uint32_t f[2 * kMaxComp] = {1, 1, 1, 1, 1, 1};
    for (int j = 0; j < sd.ns && sd.ns > 1; j++) { f[2 * j] = img.hs[sd.comp[j]]; f[2 * j + 1] = img.vs[sd.comp[j]]; }
    return dc_shape(sd.ns, f[0], f[1], f[2], f[3], f[4], f[5]);
}

// The units of a launch of DC first scans: of n runs, run e has run(e).count units, all of MCUs of run(e).shape; emit(e, unit) is called for
// each of them in the order of the launch.  A wavefront of `lanes` lanes takes shapes one after the other, so where there are
// several no wavefront gets more than one: returns the unit at which each begins, and their number at the end (empty: one
// shape, a wavefront every `lanes` units).  Otherwise the order is that of the runs.  8192 pictures of 77 to 192 pixels a
// side in four samplings, whole scans, scan group 1: 1204 us a call with the shapes as they come, 639 when a trip of the lane
// decoder took a symbol of each lane whatever its shape; now 701 by lanes (and by wavefronts, to which they go).
template <class RunOf, class Emit>
std::vector<uint32_t> dc_units_by_shape(uint32_t n, RunOf run, uint32_t lanes, Emit emit) {
    struct Group { uint32_t shape; std::vector<std::pair<uint32_t, uint32_t>> units; };
    std::vector<Group> groups;
    std::vector<uint32_t> starts;
    bool one = true;
    for (uint32_t e = 1; e < n; e++) one = one && run(e).shape == run(0).shape;
    if (!one) starts.push_back(0);
    auto wavefront = [&](Group& g) {
        if (g.units.empty()) return;
        for (const auto& u : g.units) emit(u.first, u.second);
        starts.push_back(starts.back() + (uint32_t)g.units.size());
        g.units.clear();
    };
    for (uint32_t e = 0; e < n; e++) {
        const uint32_t count = run(e).count, shape = run(e).shape;
        if (one) { for (uint32_t j = 0; j < count; j++) emit(e, j); continue; }
        size_t g = 0;
        while (g < groups.size() && groups[g].shape != shape) g++;
        if (g == groups.size()) groups.push_back(Group{shape, {}});
        for (uint32_t j = 0; j < count; j++) {
            groups[g].units.emplace_back(e, j);
            if (groups[g].units.size() == lanes) wavefront(groups[g]);
        }
    }
    for (Group& g : groups) wavefront(g);
    return starts;
}

}  // namespace pcr
