// CPU build of the walks of k_first_split and k_sequential_split (pcr_first_split.h, pcr_sequential.h) on look-ups whose entries no code has, codes of no bits among them: every
// walk ends.  Prints how far behind the end it was given each of them stopped.  Test-only.
#include <cstdio>
#include <cstring>
#include <vector>
#include "../../paper_1911_00472_amd/csrc/pcr_first_split.h"

using namespace pcr;

int main() {
    constexpr uint32_t kBits = 40000;
    std::vector<uint32_t> words(kBits / 32 + 64);
    LaneRing ring;
    FirstTables T;
    static SplitTables Q;
    const uint32_t fills[] = {0u, 0xFFFFFFFFu, 0x20002000u, 0x40004000u, 0x80008000u, 0xA000A000u, 0x01010101u, 0x0F0F0F0Fu, 0xFF00FF00u, 0x00F000F0u};
    for (uint32_t fill : fills)
        for (uint32_t data = 0; data < 3; data++) {
            uint32_t seed = 12345;
            for (auto& w : words) { seed = seed * 1664525u + 1013904223u; w = data == 0 ? 0u : (data == 1 ? ~0u : seed); }
            auto fill_with = [&](void* p, size_t bytes) { for (size_t e = 0; e + 4 <= bytes; e += 4) memcpy((char*)p + e, &fill, 4); };
            LaneTab* tab = reinterpret_cast<LaneTab*>(T.piece);
            fill_with(tab, sizeof *tab);
            for (uint32_t& l : tab->limit) l = 65536;          // (all codes are in the look-up: an index beyond it is a read of elsewhere)
            tab->sh2 = 0;
            SplitScan S{words.data(), kBits, 0, 0, 0, 0, 0, 1, 0, 8, 1, 1, 1, 1, 1, 1, 8, 8, 8, 0, 0, 0};
            SplitState to{0, 0};
            uint32_t blocks = 0;
            LaneLookup code;
            code.init(tab);
            std::vector<int16_t> plane(64 * 64), dense(64);
            first_ac_walk<false>(code, S, 1, 63, 1, SplitState{7, 1}, kBits - 100, &ring, 0, &to, &blocks, nullptr, 0, 0, 0);
            printf("%08x %u ac %d", fill, data, (int)(to.pos - (kBits - 100)));
            first_ac_walk<true>(code, S, 1, 63, 1, SplitState{7, 1}, kBits - 100, &ring, 0, &to, &blocks, plane.data(), 64 * 64, 0, 64);
            SplitSums sums{0, 0, 0, 0};
            fill_with(T.piece, sizeof T.piece);
            first_dc_walk<false>(reinterpret_cast<const DcTab*>(T.piece), S, 1, SplitState{7, 0}, kBits - 100, &ring, 0, &to, &sums, nullptr, nullptr, 0, 0);
            printf(" dc %d", (int)(to.pos - (kBits - 100)));
            sums = SplitSums{0, 0, 0, 0};
            first_dc_walk<true>(reinterpret_cast<const DcTab*>(T.piece), S, 1, SplitState{7, 0}, kBits - 100, &ring, 0, &to, &sums, plane.data(), dense.data(), 64 * 64, 64);
            fill_with(&Q, sizeof Q);
            for (CanonCode& c : Q.code)
                for (uint32_t l = 0; l < 17; l++) { c.lim[l] = l < 16 ? 0u : fill & 65535u; c.first[l] = 0; }       // (codes of sixteen bits, or none)
            S.dc_tabs = 0; S.ac_tabs = 3; S.hs0 = S.vs0 = 1;
            sums = SplitSums{0, 0, 0, 0};
            split_walk<false>(S, Q, SplitState{7, 0}, kBits - 100, &ring, 0, &to, &sums, nullptr, nullptr, 0, 0, 0);
            printf(" whole %d", (int)(to.pos - (kBits - 100)));
            sums = SplitSums{0, 0, 0, 0};
            split_walk<true>(S, Q, SplitState{7, 0}, kBits - 100, &ring, 0, &to, &sums, plane.data(), dense.data(), 64 * 64, 0, 64);
            printf("\n"); fflush(stdout);
        }
    printf("walks end\n");
    return 0;
}
