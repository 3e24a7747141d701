// Multi-scale structural similarity of two batches of decoded pictures (the fidelity estimate of the paper's
// Section 6.4: how close the picture of scan group k is to the full one), on the device.
//
// The measure is the published one (Wang, Simoncelli and Bovik 2003): on luma, an 11 x 11 Gaussian window of
// sigma 1.5 at every position where it fits, C1 = (0.01*255)^2, C2 = (0.03*255)^2; the contrast-structure term
// averaged at scales 1 .. M-1 and luminance x contrast-structure at scale M, combined as a product of powers
// with the published exponents; each further scale is the 2 x 2 average of the one before.  M = 5, or as many
// scales as keep the smaller side at least 11 samples (with fewer than five, the exponents used are rescaled to
// sum to 1); a negative scale mean counts as 0.
//
// Layout of the work: ONE WAVEFRONT per strip of 64 columns (54 window positions) and up to 128 rows of window positions
// of one scale of one picture.  A lane owns a column and walks down it: it makes the two samples of its column, and adds
// them to the eleven windows that are open in its column -- a chain of eleven fused multiply-adds per moment that also
// moves every open window on by one (a[t] = a[t-1] + g[t] v), so the column pass takes no memory at all.  Every fourth
// row the four finished rows of column sums go through LDS, and the lanes finish them as four neighbouring window
// positions each: sixteen values per moment, read as four 16-byte vectors, make 4 x 11 taps.
// Four moments are enough: with s = a + b and d = a - b (a, b: the two pictures) the terms are
//   (2 cov + C2) / (var_a + var_b + C2)             = (var_s - var_d + 2 C2) / (var_s + var_d + 2 C2),
//   (2 mu_a mu_b + C1) / (mu_a^2 + mu_b^2 + C1)     = (mu_s^2 - mu_d^2 + 2 C1) / (mu_s^2 + mu_d^2 + 2 C1),
// and only the term a scale contributes is computed (contrast-structure below the last scale, the product at it).
// A sample of scale j is the mean of an aligned 2^j x 2^j block of the picture (what j rounds of 2 x 2 averaging
// give), taken straight from the uint8 pixels with exact integer sums, so no pyramid is ever stored.  Samples are
// centred on 128 before squaring, which keeps the fp32 variances (a difference of two large numbers) accurate.
// Bound by the issue of vector instructions and, behind it, by the rate at which the loads are taken (with the loads left
// out in a copy, the kernel took 1.27 ms where it took 1.56).  1024 pictures of 300..500 pixels a side, ms: 1.64 before the
// following; 1.56 with a workgroup per wavefront; 1.46 with the open windows moved on by the multiply-add itself (fma_apart)
// and its factors in vector registers; 1.45 with two rows of pixels in flight at the largest scale; 1.34 with one load per
// block of three and six bytes instead of two; 1.31 with strips of 128 rows.  652 million vector instructions (838).
// A version before all these -- a workgroup per 32 x 32 tile, five moments, both passes through LDS, 84 LDS reads and 210
// operations per window position -- took 5.3 ms.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "pcr_kernels.h"

namespace pcr {

constexpr int kSsimScales = 5, kSsimWin = 11, kSsimCols = 64 - (kSsimWin - 1);     // window positions across a strip

__host__ __device__ inline int ssim_scale_count(uint32_t W, uint32_t H) {
    const uint32_t m = W < H ? W : H;
    if (m < (uint32_t)kSsimWin) return 0;
    int M = 1;
    while (M < kSsimScales && (m >> M) >= (uint32_t)kSsimWin) M++;
    return M;
}
// Tiles (strips of `rows` window positions down) of scale j of a W x H picture (j below its scale count), and how many
// lie side by side.
__host__ __device__ inline uint32_t ssim_tiles(uint32_t W, uint32_t H, int j, uint32_t rows, uint32_t* across) {
    const uint32_t ow = (W >> j) - (kSsimWin - 1), oh = (H >> j) - (kSsimWin - 1);
    *across = (ow + kSsimCols - 1) / kSsimCols;
    return *across * ((oh + rows - 1) / rows);
}
__host__ __device__ inline uint32_t ssim_tiles_all(uint32_t W, uint32_t H, uint32_t rows) {
    uint32_t t = 0, across;
    for (int j = 0, M = ssim_scale_count(W, H); j < M; j++) t += ssim_tiles(W, H, j, rows, &across);
    return t;
}
// Rows per tile: ten rows are walked down before the first window is complete, so tall tiles waste less, but tiles of very
// different heights leave the last wave of wavefronts ragged.  1024 photographs, ms: 192 rows 1.27, 128 1.28, 96 1.29,
// 64 1.32, 32 1.43.  A launch wants eight wavefronts per SIMD (8192); few or small pictures are cut finer to have them.  us in strips
// of 128 / 32 rows: 10 of 1024 x 1024 351 / 261, 30 471 / 398, 500 of 128 x 128 77 / 87, 100 photographs 255 / 273.
constexpr uint32_t kSsimRowChoices[3] = {128, 64, 32};
inline bool ssim_rows_suit(uint32_t n, uint32_t tiles_max) { return (uint64_t)n * tiles_max >= 8192; }

// Workgroups per picture: one for each tile, and one more where that is a multiple of four.  Workgroups are dealt out to a die's 32
// compute units in turn, and with such a number the long tiles of pictures of one size -- of the smallest scales, whose rows are
// sixteen of pixels -- came to the same few units again and again.  us a call for n tiles a picture and n + 1: 220 pictures of
// 375 x 500 (40 tiles of 128 rows) 570 / 427, of 350 x 350 (60 of 64) 343 / 273, 90 of 512 x 512 (108) 304 / 275, 300 of 128 x 128
// (16 of 32) 76 / 61.  With n + 2 and n + 4 375 x 500 took 472 and 549; numbers that are twice an odd one are left alone (100 of
// 200 x 200, 34 tiles: 66 / 76; 200: 120 / 114; 400 of 100 x 100, 10: 49 / 53).
inline uint32_t ssim_workgroups(uint32_t tiles_max) { return tiles_max % 4 == 0 ? tiles_max + 1 : tiles_max; }

// What the entry point that allocates nothing counts its limit in: tiles of 32 x 32 window positions of all scales.
inline uint32_t ssim_limit_tiles(uint32_t W, uint32_t H) {
    uint32_t t = 0;
    for (int j = 0, M = ssim_scale_count(W, H); j < M; j++) {
        const uint32_t ow = (W >> j) - (kSsimWin - 1), oh = (H >> j) - (kSsimWin - 1);
        t += ((ow + 31) / 32) * ((oh + 31) / 32);
    }
    return t;
}

// sums of the bytes of 2^j pixels of one row, per channel
struct SsimSum { uint32_t c0, c1, c2; };
template <class T> __device__ inline T ssim_load(const uint8_t* p) { struct __attribute__((packed, aligned(1))) U { T v; }; return reinterpret_cast<const U*>(p)->v; }
__device__ inline void ssim_add4(SsimSum* s, uint32_t w0, uint32_t w1, uint32_t w2) {       // four RGB pixels in twelve bytes
    s->c0 = __builtin_amdgcn_udot4(w2, 0x00000100u, __builtin_amdgcn_udot4(w1, 0x00010000u, __builtin_amdgcn_udot4(w0, 0x01000001u, s->c0, false), false), false);
    s->c1 = __builtin_amdgcn_udot4(w2, 0x00010000u, __builtin_amdgcn_udot4(w1, 0x01000001u, __builtin_amdgcn_udot4(w0, 0x00000100u, s->c1, false), false), false);
    s->c2 = __builtin_amdgcn_udot4(w2, 0x01000001u, __builtin_amdgcn_udot4(w1, 0x00000100u, __builtin_amdgcn_udot4(w0, 0x00010000u, s->c2, false), false), false);
}
// The bytes of the block of one sample of scale J that lie in kRows rows of it (C channels), as loaded.  Three and six
// bytes are loaded as four and eight that begin kBack bytes ahead of the block (the buffer's last block ends at its end):
// one instruction instead of two.  The pointers a strip walks down are set back by that for every lane but the one whose
// column starts at the buffer's first byte; skip is what lies ahead of the block in the words, in bits.
template <int C, int J, int kRows>
struct SsimRaw {
    static constexpr int kBytes = C << J, kWords = (kBytes + 3) / 4, kBack = kBytes == 3 || kBytes == 6 ? 4 * kWords - kBytes : 0;
    uint32_t w[kRows][kWords];
    __device__ inline void load(const uint8_t* p, uint32_t pitch) {
#pragma unroll
        for (int r = 0; r < kRows; r++) {
            const uint8_t* q = p + (size_t)r * pitch;
            if (kBytes == 1) w[r][0] = q[0];
            else if (kBytes == 2) w[r][0] = ssim_load<uint16_t>(q);
            else if (kBytes == 3) w[r][0] = ssim_load<uint32_t>(q);
            else if (kBytes == 6) { const uint2 t = ssim_load<uint2>(q); w[r][0] = t.x; w[r][kWords - 1] = t.y; }
            else {
                constexpr int kVec = kWords % 4 == 0 ? 4 : (kWords % 3 == 0 ? 3 : 1);
                struct V { uint32_t e[kVec]; };
#pragma unroll
                for (int v = 0; v < kWords / kVec; v++) {
                    const V t = ssim_load<V>(q + 4 * kVec * v);
#pragma unroll
                    for (int e = 0; e < kVec; e++) w[r][kVec * v + e] = t.e[e];
                }
            }
        }
    }
    __device__ inline void add_to(SsimSum* s, uint32_t skip) const {
#pragma unroll
        for (int r = 0; r < kRows; r++) {
            if (C == 1) {
#pragma unroll
                for (int q = 0; q < kWords; q++) s->c0 = __builtin_amdgcn_udot4(w[r][q], 0x01010101u, s->c0, false);
            } else if (kBytes == 3) {
                const uint32_t v = w[r][0] >> skip;
                s->c0 += v & 255u; s->c1 += (v >> 8) & 255u; s->c2 += (v >> 16) & 255u;
            } else if (kBytes == 6) {
                const uint32_t v0 = __builtin_amdgcn_alignbit(w[r][kWords - 1], w[r][0], skip), v1 = w[r][kWords - 1] >> skip;
                s->c0 = __builtin_amdgcn_udot4(v0, 0x01000001u, s->c0, false);
                s->c1 = __builtin_amdgcn_udot4(v1, 0x00000001u, __builtin_amdgcn_udot4(v0, 0x00000100u, s->c1, false), false);
                s->c2 = __builtin_amdgcn_udot4(v1, 0x00000100u, __builtin_amdgcn_udot4(v0, 0x00010000u, s->c2, false), false);
            } else {
#pragma unroll
                for (int q = 0; q + 2 < kWords; q += 3) ssim_add4(s, w[r][q], w[r][q + 1], w[r][q + 2]);
            }
        }
    }
};
template <int C>
__device__ inline float ssim_luma(const SsimSum& s, float inv_area) {
    if (C == 3) return (0.299f * (float)s.c0 + 0.587f * (float)s.c1 + 0.114f * (float)s.c2) * inv_area - 128.0f;
    return (float)s.c0 * inv_area - 128.0f;
}
// A constant in a vector register.  A multiply-add with an operand from a scalar register issues every four cycles, one
// with all of them from vector registers every other cycle if a second wavefront has such an instruction ready (single
// instructions, four wavefronts a SIMD: 4.2 and 2.3 cycles).
__device__ inline float in_vgpr(float c) {
    float v;
    asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(c));
    return v;
}
// g v + a in a register of its own (the compiler adds to a's register and then moves all open windows on by one with a
// copy each)
__device__ inline float fma_apart(float g, float v, float a) {
    float d;
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "v"(g), "v"(v), "v"(a));
    return d;
}
// num / den, den > 0 far from the ends of the range: one refinement of the reciprocal, exact where num == den.  (Against the
// definition in double precision over 36 sizes and channel counts and eight kinds of pairs of pictures, in strips of 128 rows,
// the scores' relative error is 3.8e-8 in the mean and 4.7e-7 at worst; in strips of 96 3.7e-8 and 4.7e-7.)
__device__ inline float ssim_ratio(float num, float den) {
    const float r = __builtin_amdgcn_rcpf(den), q = num * r;
    return __builtin_fmaf(__builtin_fmaf(-q, den, num), r, q);
}

constexpr int kSsimRowLen = 80;            // columns of a row in LDS: 64, and what the last lanes' vectors run over
struct SsimRows { float v[4][4][kSsimRowLen]; };       // [moment][row][column]

// One strip: rows_in rows of samples of scale J whose column starts at A and B (rows of the pictures pitch bytes apart);
// ow, x0: window positions across the scale and the strip's first; last: the scale contributes the product of both terms.
// Returns this lane's share of the sum.
template <int C, int J>
__device__ inline float ssim_strip(const uint8_t* A, const uint8_t* B, uint32_t pitch, uint32_t rows_in, uint32_t x0, uint32_t ow, bool last, bool at_start, SsimRows* L, uint32_t lane) {
    // the window: exp(-(t - 5)^2 / (2 1.5^2)), normalised (symmetric)
    const float g0 = in_vgpr(0.0010283801f), g1 = in_vgpr(0.0075987582f), g2 = in_vgpr(0.036000773f), g3 = in_vgpr(0.10936069f),
                g4 = in_vgpr(0.21300554f), g5 = in_vgpr(0.26601172f);
    const float g[kSsimWin] = {g0, g1, g2, g3, g4, g5, g4, g3, g2, g1, g0};
    constexpr float inv_area = 1.0f / (float)(1 << (2 * J));
    // Rows of pixels in flight: at the largest scale (three quarters of the work) the pixels of the next two rows of samples
    // are under way while this row's are added to the windows; at the smaller ones a block is more registers than that is
    // worth (with a second row in flight at scale 1 as well the kernel spills at four wavefronts a SIMD).
    constexpr bool kAhead = J == 0;
    constexpr int kRows = J == 0 ? 1 : (J == 4 ? 2 : (J == 3 ? 4 : 1 << J));
    const uint32_t rows_out = rows_in - (kSsimWin - 1);
    float ms[kSsimWin], md[kSsimWin], ss[kSsimWin], dd[kSsimWin];     // open windows of the column: [rows of the window behind it]
#pragma unroll
    for (int q = 0; q < kSsimWin; q++) ms[q] = md[q] = ss[q] = dd[q] = 0.f;
    const uint32_t hrow = lane >> 4, hcol = (lane & 15u) * 4; // the finishing pass: row of the four, first of four positions
    float sum = 0.f;
    const size_t down = (size_t)pitch << J;
    // a row of samples, and what it adds to the open windows; the finished row of column sums, if there is one, to LDS
    auto sums = [&](const SsimSum& sa, const SsimSum& sb, uint32_t y) {
        const float va = ssim_luma<C>(sa, inv_area), vb = ssim_luma<C>(sb, inv_area);
        const float s = va + vb, d = va - vb, s2 = s * s, d2 = d * d;
#pragma unroll
        for (int q = kSsimWin - 1; q > 0; q--) {
            ms[q] = fma_apart(g[q], s, ms[q - 1]); md[q] = fma_apart(g[q], d, md[q - 1]);
            ss[q] = fma_apart(g[q], s2, ss[q - 1]); dd[q] = fma_apart(g[q], d2, dd[q - 1]);
        }
        ms[0] = g[0] * s; md[0] = g[0] * d; ss[0] = g[0] * s2; dd[0] = g[0] * d2;
        if (y < (uint32_t)(kSsimWin - 1)) return;
        const uint32_t r = (y - (kSsimWin - 1)) & 3u;
        L->v[0][r][lane] = ms[kSsimWin - 1]; L->v[1][r][lane] = md[kSsimWin - 1];
        L->v[2][r][lane] = ss[kSsimWin - 1]; L->v[3][r][lane] = dd[kSsimWin - 1];
    };
    SsimRaw<C, J, kRows> ra, rb, ra2, rb2;
    const uint32_t back = at_start ? 0u : (uint32_t)ra.kBack, skip = 8 * back;
    A -= back; B -= back;
    if (kAhead) {
        ra.load(A, pitch); rb.load(B, pitch);
        A += down; B += down;                                 // (a strip has eleven rows of samples at the least)
        ra2.load(A, pitch); rb2.load(B, pitch);
    }
    constexpr uint32_t kStep = kAhead ? 2 : 1;
    for (uint32_t y = 0; y < rows_in; y += kStep) {
        uint32_t y1 = y;                                      // the last row of this trip
        if (kAhead) {
            SsimSum sa{0, 0, 0}, sb{0, 0, 0};
            ra.add_to(&sa, skip); rb.add_to(&sb, skip);
            if (y + 2 < rows_in) { A += down; B += down; }    // (the last row once more: its bytes are there)
            ra.load(A, pitch); rb.load(B, pitch);
            sums(sa, sb, y);
            if (y + 1 < rows_in) {
                SsimSum sc{0, 0, 0}, sd{0, 0, 0};
                ra2.add_to(&sc, skip); rb2.add_to(&sd, skip);
                if (y + 3 < rows_in) { A += down; B += down; }
                ra2.load(A, pitch); rb2.load(B, pitch);
                sums(sc, sd, ++y1);
            }
        } else {
            SsimSum sa{0, 0, 0}, sb{0, 0, 0};
            // (Where this loop begins is fixed: it is nearly all instructions of eight bytes, and how they lie on the lines they are
            // fetched by is 4 to 12 % of a launch of few pictures.  10 of 1024 x 1024 at a multiple of 64 bytes 268 us, four bytes past
            // one 242; 30 of 512 x 512 182 and 170.)
#pragma unroll 1
            [[clang::code_align(64)]] for (int r = 0; r < (1 << J); r += kRows) {
                asm volatile("s_nop 0");
                ra.load(A + (size_t)r * pitch, pitch); rb.load(B + (size_t)r * pitch, pitch);
                ra.add_to(&sa, skip); rb.add_to(&sb, skip);
            }
            A += down; B += down;
            sums(sa, sb, y);
        }
        if (y1 < (uint32_t)(kSsimWin - 1)) continue;
        const uint32_t r = y1 - (kSsimWin - 1);
        if ((r & 3) != 3 && r + 1 != rows_out) continue;
        wave_sync();                                          // window rows r & ~3 .. r of the tile are in LDS
        float m[4][4];                                        // [moment][position]
#pragma unroll
        for (int f = 0; f < 4; f++) {
            float v[16];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const float4 x = *reinterpret_cast<const float4*>(&L->v[f][hrow][hcol + 4 * q]);
                v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
            }
#pragma unroll
            for (int o = 0; o < 4; o++) {
                float acc = g[0] * v[o];
#pragma unroll
                for (int q = 1; q < kSsimWin; q++) acc = __builtin_fmaf(g[q], v[o + q], acc);
                m[f][o] = acc;
            }
        }
#pragma unroll
        for (int o = 0; o < 4; o++) {
            const float m2 = m[0][o] * m[0][o], e2 = m[1][o] * m[1][o];
            const float var_s = m[2][o] - m2, var_d = m[3][o] - e2, c2 = 2.0f * 58.5225f;
            float v = ssim_ratio(var_s - var_d + c2, var_s + var_d + c2);
            if (last) {
                const float ps = m[0][o] + 256.0f, p2 = ps * ps, c1 = 2.0f * 6.5025f;
                v *= ssim_ratio(p2 - e2 + c1, p2 + e2 + c1);
            }
            const uint32_t x = hcol + o;
            sum += (x < (uint32_t)kSsimCols && x0 + x < ow && (r & ~3u) + hrow < rows_out) ? v : 0.f;
        }
        wave_sync();
    }
    return sum;
}

// part[i * tiles_max + t] = (sum of contrast-structure, sum of luminance x contrast-structure; only the one its scale
// contributes) over the window positions of tile t of picture i; tiles are numbered scale by scale.
// Workgroups: `every` per picture (ssim_workgroups), those beyond tiles_max have nothing to do.
template <int C>
__global__ void __launch_bounds__(64, 4) k_ssim_tiles(const uint32_t* __restrict__ dims, const uint64_t* __restrict__ out_off,
                                                    const uint8_t* __restrict__ pa, const uint8_t* __restrict__ pb,
                                                    float2* __restrict__ part, uint32_t n, uint32_t tiles_max, uint32_t every, uint32_t rows) {
    // (a workgroup of one wavefront: with four to a workgroup the strips of a workgroup waited for its tallest before
    // the next workgroup had its LDS: twelve wavefronts a compute unit on average instead of fourteen, 1.64 ms and 1.56)
    __shared__ __attribute__((aligned(16))) SsimRows buf;
    const uint32_t lane = threadIdx.x;
    // (every die works through a contiguous eighth of the pictures: the scales of a picture read the same pixels)
    const uint32_t item = xcd_major(blockIdx.x, gridDim.x), i = item / every;
    if (i >= n) return;
    uint32_t t = item - i * every;
    const uint32_t W = dims[2 * i], H = dims[2 * i + 1];
    const int M = ssim_scale_count(W, H);
    const uint32_t slot = t;
    uint32_t across = 1;
    int j = 0;
    for (; j < M; j++) {
        const uint32_t cnt = ssim_tiles(W, H, j, rows, &across);
        if (t < cnt) break;
        t -= cnt;
    }
    if (j >= M) return;
    const uint32_t Wj = W >> j, Hj = H >> j, ow = Wj - (kSsimWin - 1), oh = Hj - (kSsimWin - 1);
    const uint32_t ox = (t % across) * kSsimCols, oy = (t / across) * rows;
    const uint32_t rows_in = (oh - oy < rows ? oh - oy : rows) + (kSsimWin - 1);
    const uint32_t X = ox + lane < Wj ? ox + lane : Wj - 1;  // (columns past the picture only reach positions past it)
    const uint32_t pitch = W * C;
    const size_t at = out_off[i] + (size_t)(oy << j) * pitch + (size_t)(X << j) * C;
    const uint8_t *A = pa + at, *B = pb + at;
    const bool last = j == M - 1;
    float sum = 0.f;
    switch (j) {
        case 0: sum = ssim_strip<C, 0>(A, B, pitch, rows_in, ox, ow, last, at == 0, &buf, lane); break;
        case 1: sum = ssim_strip<C, 1>(A, B, pitch, rows_in, ox, ow, last, at == 0, &buf, lane); break;
        case 2: sum = ssim_strip<C, 2>(A, B, pitch, rows_in, ox, ow, last, at == 0, &buf, lane); break;
        case 3: sum = ssim_strip<C, 3>(A, B, pitch, rows_in, ox, ow, last, at == 0, &buf, lane); break;
        default: sum = ssim_strip<C, 4>(A, B, pitch, rows_in, ox, ow, last, at == 0, &buf, lane); break;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    if (lane == 0) part[(size_t)i * tiles_max + slot] = last ? make_float2(0.f, sum) : make_float2(sum, 0.f);
}

// One wavefront per picture: the scale means from the tile sums (in double, in a fixed order), then the
// product of powers.  A picture too small for the window scores NaN.
__global__ void __launch_bounds__(64) k_ssim_score(const uint32_t* __restrict__ dims, const float2* __restrict__ part, uint32_t tiles_max,
                                                   uint32_t rows, float* __restrict__ scores) {
    const double weight[kSsimScales] = {0.0448, 0.2856, 0.3001, 0.2363, 0.1333};
    const uint32_t i = blockIdx.x, lane = threadIdx.x;
    const uint32_t W = dims[2 * i], H = dims[2 * i + 1];
    const int M = ssim_scale_count(W, H);
    if (M == 0) { if (lane == 0) scores[i] = __builtin_nanf(""); return; }
    double wsum = 0;
    for (int j = 0; j < M; j++) wsum += weight[j];
    if (M == kSsimScales) wsum = 1.0;                       // all five scales: the exponents as published (they sum to 1.0001)
    double score = 1.0;
    uint32_t first = 0;
    for (int j = 0; j < M; j++) {
        uint32_t across;
        const uint32_t cnt = ssim_tiles(W, H, j, rows, &across);
        double cs = 0, lcs = 0;
        for (uint32_t t = lane; t < cnt; t += 64) {
            const float2 p = part[(size_t)i * tiles_max + first + t];
            cs += (double)p.x; lcs += (double)p.y;
        }
        for (int d = 32; d > 0; d >>= 1) { cs += __shfl_down(cs, d); lcs += __shfl_down(lcs, d); }
        const double positions = (double)((W >> j) - (kSsimWin - 1)) * (double)((H >> j) - (kSsimWin - 1));
        double term = (j == M - 1 ? lcs : cs) / positions;
        if (!(term > 0.0)) term = 0.0;
        score *= pow(term, weight[j] / wsum);
        first += cnt;
    }
    if (lane == 0) scores[i] = (float)score;
}

}  // namespace pcr
