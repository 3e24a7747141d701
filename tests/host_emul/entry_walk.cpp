// CPU build of the record writer's walk over AC scans (pcr_encode.h: walk_first_block, walk_refine_block) against one that takes a bit
// after the other and a position after the other, on streams of valid codes and on noise: position, non-zero positions and run after every
// block, with the bit-scan instructions and without.  Test-only.
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>
#include "../../paper_1911_00472_amd/csrc/pcr_encode.h"

using namespace pcr;
using namespace pcr::enc;

struct Bits {
    const uint8_t* d; uint64_t pos;
    uint32_t one() { const uint32_t b = (d[pos >> 3] >> (7 - (pos & 7))) & 1u; pos++; return b; }
    uint32_t take(uint32_t n) { uint32_t v = 0; while (n--) v = v << 1 | one(); return v; }
};
// the symbol at the head of the stream, -1: none
static int symbol(Bits* b, const uint8_t* dht) {
    int code = 0, first = 0, at = 0;
    for (int l = 1; l <= 16; l++) {
        code = code << 1 | (int)b->one();
        const int n = dht[l - 1];
        if (code < first + n) return at + code - first < 256 ? dht[16 + at + code - first] : -1;
        at += n; first = (first + n) << 1;
    }
    return -1;
}
static int plain_block(Bits* b, const uint8_t* dht, uint64_t* h, int Ss, int Se, bool refine) {
    int k = Ss, run = 0;
    while (k <= Se) {
        const int s = symbol(b, dht);
        if (s < 0) return -1;
        int r = s >> 4; const int size = s & 15;
        if (size == 0 && r < 15) { run = (1 << r) + (int)b->take((uint32_t)r); break; }
        if (!refine) {
            k += r;
            if (size) { if (k > Se) return -1; b->take((uint32_t)size); *h |= 1ull << k; }
            k++;
            continue;
        }
        if (size > 1) return -1;
        if (size) b->one();
        uint64_t fresh = 0;
        for (; k <= Se; k++) {
            if (*h >> k & 1) { b->one(); continue; }
            if (r-- == 0) { fresh = 1ull << k; k++; break; }
        }
        if (size && !fresh) return -1;
        if (size) *h |= fresh;
    }
    if (refine && run) for (; k <= Se; k++) if (*h >> k & 1) b->one();
    return run;
}

int main() {
    std::mt19937 rng(7);
    if (!walk_bmi2()) printf("no bmi2 here\n");
    size_t blocks = 0, runs = 0, refused = 0;
    for (int t = 0; t < 4000; t++) {
        const bool refine = t & 1;
        // a code: lengths that fill the code space but for the last code, symbols of the kind of scan (and, now and then, others)
        uint8_t dht[16 + 256] = {0};
        std::vector<uint8_t> syms;
        for (int r = 0; r < 16; r++) for (int s = 0; s < (refine ? 2 : 11); s++) syms.push_back((uint8_t)(r << 4 | s));
        if (t % 7 == 0) syms.push_back(refine ? 0x35 : 0x0F);
        std::shuffle(syms.begin(), syms.end(), rng);
        auto rank = [&](uint8_t s) { return (s >> 4) + 2 * (s & 15) + ((t & 2) && (s & 15) == 0 && s != 0xF0 ? 12 : 0); };      // (runs have short codes, or long ones)
        std::stable_sort(syms.begin(), syms.end(), [&](uint8_t a, uint8_t b) { return rank(a) < rank(b); });
        size_t left = syms.size(), at = 0;
        for (uint32_t l = 1, room = 2; l <= 16 && left > 0; l++, room *= 2) {
            const uint32_t most = l < 16 ? (room > 2 ? room - 2 : 0) : room - 1;      // (codes stay over for the longer ones)
            uint32_t n = std::min<uint32_t>({most, (uint32_t)left, (uint32_t)(rng() % (1 + room / (1 + t % 3)))});
            if (l == 16) n = std::min<uint32_t>(room - 1, (uint32_t)left);
            dht[l - 1] = (uint8_t)std::min<uint32_t>(n, 255);
            n = dht[l - 1];
            memcpy(dht + 16 + at, syms.data() + at, n);
            at += n; left -= n; room -= n;
        }
        AcTab tab; actab_build(&tab, dht);
        WalkTable W; W.build(&tab, refine);
        std::vector<uint8_t> d(4096 + kWalkPad, 0xFF);
        for (size_t i = 0; i < 4096; i++) d[i] = (uint8_t)(t % 5 == 4 ? rng() & rng() : rng());
        const int Ss = 1 + (int)(rng() % 20) * (t % 3 == 0), Se = t % 4 == 0 ? Ss + (int)(rng() % (64 - Ss)) : 63;
        const uint64_t band = (Se >= 63 ? ~0ull : (1ull << (Se + 1)) - 1) & ~((1ull << Ss) - 1);
        uint64_t pos = rng() % 64;
        while (pos < 4096 * 8) {
            uint64_t h0 = ((uint64_t)rng() << 32 | rng()) & ((uint64_t)rng() << 32 | rng()) & ((uint64_t)rng() << 32 | rng());
            if (!refine) h0 = 0;
            Bits b{d.data(), pos};
            uint64_t want = h0;
            const int run = plain_block(&b, dht, &want, Ss, Se, refine);
            for (int bmi2 = 0; bmi2 < (refine && walk_bmi2() ? 2 : 1); bmi2++) {
                uint64_t p = pos, h = h0;
                const int got = !refine ? walk_first_block(d.data(), W, &p, &h, (uint32_t)Ss, (uint32_t)Se)
                                        : (bmi2 ? walk_refine_block<true>(d.data(), W, &p, &h, band) : walk_refine_block<false>(d.data(), W, &p, &h, band));
                if (got != run || (run >= 0 && (p != b.pos || h != want))) {
                    printf("differs: %d refine %d bmi2 %d at %llu: run %d %d, position %llu %llu\n", t, refine, bmi2, (unsigned long long)pos, got, run, (unsigned long long)p, (unsigned long long)b.pos);
                    return 1;
                }
            }
            blocks++; runs += run > 0; refused += run < 0;
            pos = run < 0 ? pos + 1 + rng() % 97 : b.pos;
        }
    }
    printf("%zu blocks, %zu end in a run, %zu refused\nwalks agree\n", blocks, runs, refused);
    return 0;
}
