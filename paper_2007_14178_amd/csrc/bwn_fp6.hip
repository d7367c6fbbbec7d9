// Binary-Weight-Network convolution (Sec. II-A, Eq. 1) on the matrix instruction for 6- and 4-bit
// operands (v_mfma_scale_f32_32x32x64_f8f6f4, four times the bf16 instruction's rate): the 32
// channels of one packed word at one position are a block with one power of two as its scale, and
// every value x of the block is a sum of five FP6 (E2M3) digits,
//
//   x = s * (d0 + d1 2^-4 + d2 2^-9 + d3 2^-14 + d4 2^-19) + e,   |e| <= 2^-22 s,
//
// each digit what the ones before it left over, rounded to four significant bits.  s is chosen so that
// the block's largest magnitude lies in [3.875, 7.75) s (E2M3 ends at 7.5, and 7.75 still rounds to it with a
// remainder of 0.25): |e| is about half an ulp of the block's largest value, and values from about that one's
// binade up have no error at all.  The differences are exact in fp32.  The weights are +-1 in FP4, so the
// products are exact; the powers of the digits ride on the filters' scale, s on the input's, and the sum is
// accumulated in fp32: five instructions per 64 channels where the bf16 terms of csrc/bwn_split.hip need twelve
// of the same length.
//
//   bwn_fp6_kernel: a workgroup (1..8 waves) owns 32 * NF filters x one tile of 32 consecutive output pixels of one
//   image per wave.  Per chunk of G words the rows under the pixels (whole rows: one run of the plane per
//   channel) are read, a position and word per lane, cut into digits in registers and laid into LDS as
//   [word][position][5 digits x 24 bytes, scale]; the last position is zeros, which is where padding and
//   the pixels past the last one read.  The filters' words of the chunk lie beside it as [tap][word][filter].
//   A step multiplies two (tap, word) blocks, one per lane half: NF * 5 matrix instructions.  What a step's
//   matrix instructions used is loaded again for the next one right behind its last use, and the sign words
//   of the next step become FP4 codes between them.  The chunk's staging stands between two barriers; the two or
//   more workgroups on a compute unit fill each other's.
//
//   Two shapes of workgroup more, where estimates of all say so (search_fp6_plan).  Splits: the waves of a pixel tile have filters
//   of their own and share the tile's digits, so that a block is cut for more filters (128x384x13x13 F=384 3x3 105 -> 91 us).
//   Stagers: three or four waves that only stage, into two buffers, a chunk ahead of the others, the next round's loads in
//   flight while a round is cut: layers that leave units with one workgroup, whose chunk's chain nothing else hides
//   (32x512x7x7 F=512 3x3 41 -> 29 us, 1x256x14x14 F=256 3x3 19 -> 13.5; 200 drawn layers with both 1.17 times as fast).
//
//   Bound by: the matrix pipe at the card's power (6.3 PFLOP/s of this pair of formats in a loop of random digits, 9.0 of
//   zeros; an instruction takes 32 cycles; the first layer above with nothing but its matrix instructions and stores takes 83 us),
//   then by the digits' conversions (about 1200 cycles per 64 blocks, again for every filter group) and the wait for a chunk's loads, which other workgroups fill in part.
//   Passes against the bf16 terms: 128x384x13x13 F=384 3x3 177 -> 104 us; loops of launches: 128x512x28x28 F=512 3x3
//   1300 -> 706 us, 16x128x56x56 F=128 7x7 291 -> 116, 1x256x14x14 F=256 3x3 48 -> 23.
//   Relative error against 64-bit sums 5.2e-7 -> 2.6e-7 (fewer roundings of the sum: five per 64 channels, not twelve).
// Of the bf16 form's over five layers from 1x1 on 96 channels to 7x7 on 256: 0.43 to 0.66 for normal, positive, rectified and
// log-normal values (sigma 4) and channels of 1 to 2^-96, but for the log-normal ones with one tap (1.14), whose sums are one value
// each; 0.73 to 0.97 beside a channel of 1e4.  It is the larger where two such channels of one block cancel (1.1 to 6.7 times).
//   Inputs that are not finite give NaN in every window that holds them (the block's scale is NaN).
//   Scales end at 2^-103: below, a value's error is at most 2^-125, and no digit's product leaves the normal range.  Sums
// are of half the products, so that the first digit of a value in fp32's top 1/32, which rounds to 2^128, is inside it.
#include <algorithm>
#include <atomic>

#include "xnor_internal.hpp"

namespace xnor {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v32f __attribute__((ext_vector_type(32)));
typedef uint32_t v6u __attribute__((ext_vector_type(6)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kPosBytes = 136;     // five digits, the scale, four bytes so that 32 lanes' 8-byte accesses at
                                   // consecutive positions touch every bank once (17 bank pairs apart)
constexpr int kDigits = 5;
constexpr int kMaxWaves = 8;
constexpr int kMinScale = 24;      // exponent field of the smallest scale, 2^-103
constexpr size_t kLds = 160 * 1024;

struct Fp6Params {
    const float *I;
    const uint32_t *Wpk;
    const float *alpha;
    float *out;
    int C, H, W, F, kh, kw, sh, sw, ph, pw, OH, OW, Cw;
    int G;                         // words per chunk (the last chunk of an odd number of words has one)
    int splits, tiles;             // waves that share a pixel tile, each with filters of its own; pixel tiles of a workgroup
    uint32_t inv_splits;
    int stagers;                   // STAGERS: waves that only stage
    int wgs;                       // workgroups of an image (per filter group)
    int fgroups, units;            // filter groups, of splits * 32 * NF filters; N * wgs
    uint32_t inv_row;              // of a row's words in LDS, splits * 32 * NF
    int words_bytes;               // of a chunk's filter words in LDS
    int positions;                 // staged positions there is room for; the zero position is the next one
};

// Power of the digit t against the block's scale: 0, -4, -9, -14, -19.
__device__ constexpr int digit_exp(int t) { return t == 0 ? 0 : 1 - 5 * t; }

// Both conversions write their result over several cycles while they still read: the result may not share registers
// with an operand (the early clobber), and the next instruction may not read it at once (the wait states).
__device__ inline v6u to_fp6(const v16f &even, const v16f &odd, float scale)
{
    v6u r;
    asm("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, %3\n\ts_nop 1" : "=&v"(r) : "v"(even), "v"(odd), "v"(scale));
    return r;
}

__device__ inline v32f from_fp6(const v6u &d, float scale)
{
    v32f r;
    asm("v_cvt_scalef32_pk32_f32_fp6 %0, %1, %2\n\ts_nop 1" : "=&v"(r) : "v"(d), "v"(scale));
    return r;
}

// Sign words -> FP4 codes, four registers of eight: register j's code n is the sign of channel 4 n + 3 - j, a shift and
// one three-input operation a register (bit 1 is +1.0 = 0x2, bit 0 is -1.0 = 0xa): 7 instructions a word where
// expand_word takes 11, 2 to 7 % of a layer with two and more filter tiles a wave.
__device__ inline v4i sign_codes(uint32_t w)
{
    auto codes = [](uint32_t v) { return (int)((~v & 0x88888888u) | 0x22222222u); };
    return (v4i){codes(w), codes(w << 1), codes(w << 2), codes(w << 3)};
}

// The block's values in the order of those codes: field 2i of a digit is even[i], channel channel_of(i) of the word,
// field 2i + 1 is odd[i], the channel four behind it.
struct Block {
    v16f even, odd;
};
__device__ constexpr int channel_of(int i) { return 8 * (i & 3) + 3 - (i >> 2); }

// `src` is the image's rows, `lane` the byte offset of the lane's block, `first` the bytes before the chunk's first
// channel, `plane` those of a channel's plane; `nvalid` of the block's channels are there.
__device__ inline void load_block(Block &b, __amdgpu_buffer_rsrc_t src, int lane, int first, int plane, bool whole, int nvalid)
{
    if (whole) {                   // (uniform)
        auto load = [&](int c) __attribute__((always_inline)) {
            return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(src, lane, first + c * plane, 0));
        };
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            b.even[i] = load(channel_of(i));
            b.odd[i] = load(channel_of(i) + 4);
        }
    } else {                       // the last word of C % 32 channels: reads stay inside, the rest is zero
        auto load = [&](int c) __attribute__((always_inline)) {
            const float v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(src, lane + min(c, nvalid - 1) * plane, first, 0));
            return c < nvalid ? v : 0.f;
        };
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            b.even[i] = load(channel_of(i));
            b.odd[i] = load(channel_of(i) + 4);
        }
    }
}

// The block's digits and scale to `at` (where `keep`: lanes past the last position take part in the arithmetic only).
__device__ inline void split_block(Block &b, char *at, bool keep)
{
    float m = 0.f;                 // (propagates NaN)
#pragma unroll
    for (int i = 0; i < 16; ++i)
        m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(b.even[i])), fabsf(b.odd[i]));
    const uint32_t bits = __float_as_uint(m);
    // the exponent, one more from 1.9375 times the power of two up, less two
    const uint32_t scale = (bits & 0x7fffffffu) >= 0x7f800000u ? 255u
                           : (uint32_t)max((int)((bits + (1u << 19)) >> 23) - 2, kMinScale);
    if (keep) *reinterpret_cast<uint32_t *>(at + 120) = scale;
#pragma unroll
    for (int t = 0; t < kDigits; ++t) {
        const float s = __uint_as_float((scale + digit_exp(t)) << 23);
        const v6u d = to_fp6(b.even, b.odd, s);
        if (keep) {
            v2u *o = reinterpret_cast<v2u *>(at + 24 * t);
            o[0] = (v2u){d[0], d[1]};
            o[1] = (v2u){d[2], d[3]};
            o[2] = (v2u){d[4], d[5]};
        }
        if (t + 1 < kDigits) {
            // (half of the digit, subtracted twice: from 1.9375 * 2^127 up the first one is 4.0 * 2^126, which is no float)
            const v32f back = from_fp6(d, __uint_as_float((scale - 1 + digit_exp(t)) << 23));
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                b.even[i] = fmaf(-2.f, back[2 * i], b.even[i]);
                b.odd[i] = fmaf(-2.f, back[2 * i + 1], b.odd[i]);
            }
        }
    }
}

// SPLITS: more than one split, or stagers.
template <int NF, bool SPLITS, bool STAGERS>
struct Fp6Wave {
    static constexpr int kFilters = 32 * NF;

    // Half of digit T of the pixels' blocks against one filter tile.  The digits' powers are the bytes of two registers.
    template <int T>
    static __device__ __attribute__((always_inline)) inline void product(v16f &acc, const v4i &a, const v6u &d, int scale)
    {
        constexpr int powers = T < 4 ? (126 + digit_exp(0)) | (126 + digit_exp(1)) << 8 | (126 + digit_exp(2)) << 16 | (126 + digit_exp(3)) << 24
                                     : 126 + digit_exp(4);
        const v8i b = {(int)d[0], (int)d[1], (int)d[2], (int)d[3], (int)d[4], (int)d[5], 0, 0};
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(__builtin_shufflevector(a, a, 0, 1, 2, 3, -1, -1, -1, -1), b, acc, 4, 2,
                                                              T & 3, powers, 0, scale);
    }
    template <int T>
    static __device__ __attribute__((always_inline)) inline void digit(v16f (&acc)[NF], const v4i (&A)[NF], const v6u &d, int scale)
    {
#pragma unroll
        for (int f = 0; f < NF; ++f) product<T>(acc[f], A[f], d, scale);
    }

    // One chunk's steps: two (tap, word) blocks each.  With two words in the chunk lane half h takes word h of the
    // step's tap, with one the word of tap 2 * step + h.
    static __device__ __attribute__((always_inline)) inline void steps(v16f (&acc)[NF], const Fp6Params &p, const char *dig, const uint32_t *words,
                                                                       int row, bool two, int iy, int ix, int row0, int half, int col)
    {
        const int taps = p.kh * p.kw, nsteps = two ? taps : (taps + 1) >> 1;
        const int word_bytes = (p.positions + 1) * kPosBytes, zero = p.positions * kPosBytes;
        const int group = two && half ? word_bytes : 0;
        // The lane's tap: its row and column in the image, its column in the window, its place.  (With scalars for the two
        // halves' walks a step of one filter tile waits for the scalar chain: 46x45x7x7 F=98 7x7 18.0 -> 20.8 us.)
        int y = iy, x = ix, kx = 0, to = ((iy - row0) * p.W + ix) * kPosBytes;
        const int y_end = iy + p.kh, back = (p.W - p.kw + 1) * kPosBytes;
        auto next_tap = [&]() __attribute__((always_inline)) {
            const bool wrap = kx + 1 == p.kw;
            to += wrap ? back : kPosBytes;
            x = wrap ? ix : x + 1;
            kx = wrap ? 0 : kx + 1;
            y += wrap ? 1 : 0;
        };
        if (!two && half) next_tap();
        auto place = [&]() __attribute__((always_inline)) {
            const bool in = y < y_end & (unsigned)y < (unsigned)p.H & (unsigned)x < (unsigned)p.W;
            const int at = in ? to : zero;
            next_tap();
            if (!two) next_tap();
            return dig + (at + group);
        };
        v6u B[kDigits];
        auto read_digit = [&](int t, const char *at) __attribute__((always_inline)) {
            const v2u *o = reinterpret_cast<const v2u *>(at + 24 * t);
            const v2u a = o[0], b = o[1], c = o[2];
            B[t] = (v6u){a.x, a.y, b.x, b.y, c.x, c.y};
        };
        const uint32_t *wat = words + half * row + col;
        uint32_t wnext[NF];
        auto read_words = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < NF; ++f) wnext[f] = wat[32 * f];
            wat += 2 * row;
        };
        v4i A[NF];
        auto expand = [&](int f) __attribute__((always_inline)) { A[f] = sign_codes(wnext[f]); };
        const char *at = place();
#pragma unroll
        for (int t = 0; t < kDigits; ++t) read_digit(t, at);
        int scale = *reinterpret_cast<const int *>(at + 120);
        read_words();
#pragma unroll
        for (int f = 0; f < NF; ++f) expand(f);
        for (int s = 0; s < nsteps; ++s) {
            // the next step's place (past the last step: the zero position, and two rows of words that nothing filled)
            at = place();
            read_words();
            const int scale_next = *reinterpret_cast<const int *>(at + 120);
            digit<0>(acc, A, B[0], scale);
            read_digit(0, at);
            __builtin_amdgcn_sched_barrier(0);
            digit<1>(acc, A, B[1], scale);
            read_digit(1, at);
            __builtin_amdgcn_sched_barrier(0);
            digit<2>(acc, A, B[2], scale);
            read_digit(2, at);
            __builtin_amdgcn_sched_barrier(0);
            digit<3>(acc, A, B[3], scale);
            read_digit(3, at);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                product<4>(acc[f], A[f], B[4], scale);
                expand(f);
                __builtin_amdgcn_sched_barrier(0);
            }
            read_digit(4, at);
            __builtin_amdgcn_sched_barrier(0);
            scale = scale_next;
        }
    }

    static __device__ __attribute__((always_inline)) inline void run(const Fp6Params &p)
    {
        extern __shared__ __attribute__((aligned(16))) char smem[];
        const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int taps = p.kh * p.kw;
        const int word_bytes = (p.positions + 1) * kPosBytes;
        const int G = p.G;
        // one buffer for a chunk, or two taken in turn: digits, filter words
        const int dig_bytes = G * word_bytes;
        const int buffer = dig_bytes + p.words_bytes;

        // a unit's filter groups run one behind the other on one XCD (workgroup ids go round the eight)
        const int k = blockIdx.x >> 3, fg = k % p.fgroups, unit = (k / p.fgroups) * 8 + (blockIdx.x & 7);
        if (unit >= p.units) return;
        const int n = unit / p.wgs, all_waves = nt >> 6, waves = STAGERS ? all_waves - p.stagers : all_waves;
        const int tiles = SPLITS ? p.tiles : waves, tile = SPLITS ? (int)quot((uint32_t)wave, p.inv_splits) : wave;
        const bool stager = STAGERS && wave >= waves;
        const int OHW = p.OH * p.OW, HW = p.H * p.W;
        const int px0 = (unit - n * p.wgs) * tiles * 32, px1 = min(OHW, px0 + tiles * 32) - 1;
        const int row0 = max(0, px0 / p.OW * p.sh - p.ph);
        const int row1 = min(p.H - 1, px1 / p.OW * p.sh - p.ph + p.kh - 1);
        const int npos = max(0, row1 - row0 + 1) * p.W;       // <= p.positions
        // the workgroup's filters; the wave's (none of them may exist)
        const int row_words = SPLITS ? p.splits * kFilters : kFilters, f_wg = fg * row_words;
        const int f0 = SPLITS ? f_wg + (wave - tile * p.splits) * kFilters : f_wg, nfil = min(kFilters, p.F - f0);

        const int px = px0 + tile * 32 + col;
        const int oy = px / p.OW, ox = px - oy * p.OW;
        const int iy = px < OHW ? oy * p.sh - p.ph : -128, ix = ox * p.sw - p.pw;

        // (bytes of an image < 2^31, so every offset is)
        const __amdgpu_buffer_rsrc_t in = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(p.I + (size_t)n * p.C * HW + (size_t)row0 * p.W), 0, 0x7fffffff, 0x00027000);
        const int plane = HW * 4;
        const int nchunks = (p.Cw + G - 1) / G;
        for (int i = tid; i < G * (kPosBytes / 4); i += nt) {
            const int at = (i / (kPosBytes / 4)) * word_bytes + p.positions * kPosBytes;
            reinterpret_cast<uint32_t *>(smem + at)[i % (kPosBytes / 4)] = 0;
            if constexpr (STAGERS) reinterpret_cast<uint32_t *>(smem + buffer + at)[i % (kPosBytes / 4)] = 0;
        }

        // staging rounds of a chunk by `count` waves from `first` on: 64 * count blocks each, the positions of its first word and then
        // those of its second
        auto words_in = [&](int ch) { return min(G, p.Cw - ch * G); };
        auto place_of = [&](int i, int &g, int &pos) __attribute__((always_inline)) {
            g = i >= npos ? 1 : 0;
            pos = i - (g ? npos : 0);
        };
        auto load_round = [&](Block &b, int ch, int i) __attribute__((always_inline)) {
            int g, pos;
            place_of(i, g, pos);
            if (i < npos * words_in(ch))
                load_block(b, in, pos * 4 + g * 32 * plane, ch * G * 32 * plane, plane, (ch + 1) * G * 32 <= p.C, p.C - 32 * (ch * G + g));
        };
        // Filter words go from memory into LDS without a register, 64 lanes' words side by side, in rows of the filters'
        // words (tap, word).  Filters past the last one, whose outputs are not stored, read the last one's
        // words; a row past the last one, that one's.  (A filter's words side by side, so that 64 lanes touch a few
        // lines and not one each, cost the loop an address per tile and were slower: 114 for 102 us at
        // 128x384x13x13 F=384 3x3.)
        const __amdgpu_buffer_rsrc_t wsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint32_t *>(p.Wpk + (size_t)f_wg * taps * p.Cw), 0, 0x7fffffff, 0x00027000);
        const int f_last = min(row_words, p.F - f_wg) - 1;
        auto load_words = [&](int ch, char *words, int first, int count) __attribute__((always_inline)) {
            const bool two = words_in(ch) == 2;
            const int rows = two ? 2 * taps : taps;
            auto *to = (__attribute__((address_space(3))) char *)words;
            for (int item = first; item * 64 < rows * row_words; item += count) {
                const int i = item * 64 + lane, r = SPLITS ? (int)quot((uint32_t)i, p.inv_row) : i / kFilters, f = i - r * row_words, row = min(r, rows - 1);
                const int tap = two ? row >> 1 : row, g = two ? row & 1 : 0;
                const int at = (min(f, f_last) * taps + tap) * (p.Cw * 4) + g * 4;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wsrc, (__attribute__((address_space(3))) void *)(to + item * 256), 4, at,
                                                         ch * G * 4, 0, 0);
            }
        };
        auto stage = [&](int ch, int first, int count) __attribute__((always_inline)) {
            char *const to = smem + (STAGERS ? (ch & 1) * buffer : 0);
            load_words(ch, to + dig_bytes, first, count);
            const int blocks = npos * words_in(ch);
            for (int r = 0; r < blocks; r += 64 * count) {
                const int i = r + 64 * first + lane;
                int g, pos;
                place_of(i, g, pos);
                Block cur;
                load_round(cur, ch, i);
                split_block(cur, to + g * word_bytes + pos * kPosBytes, i < blocks);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): the words are in LDS
        };

        v16f acc[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][r] = 0.f;
        auto multiply = [&](int ch) __attribute__((always_inline)) {
            const char *const dig = smem + (STAGERS ? (ch & 1) * buffer : 0);
            if (px0 + tile * 32 < OHW && nfil > 0)
                steps(acc, p, dig, reinterpret_cast<const uint32_t *>(dig + dig_bytes) + (f0 - f_wg), row_words, words_in(ch) == 2, iy, ix, row0, half, col);
        };

        if constexpr (STAGERS) {
            stage(0, wave, all_waves);
            __syncthreads();
            if (stager) {
                // a round's loads are in flight while the round before is cut into digits, up to the chunk's end; lanes past the last block
                // load that one
                const int first = wave - waves, round = 64 * p.stagers;
                auto load_ahead = [&](Block &b, int ch, int r) __attribute__((always_inline)) {
                    const int i = min(r + 64 * first + lane, npos * words_in(ch) - 1);
                    load_round(b, ch, i);
                };
                Block next;
                if (nchunks > 1 && npos > 0) load_ahead(next, 1, 0);
                for (int ch = 1; ch < nchunks; ++ch) {
                    char *const to = smem + (ch & 1) * buffer;
                    load_words(ch, to + dig_bytes, first, p.stagers);
                    const int blocks = npos * words_in(ch);
                    for (int r = 0; r < blocks; r += round) {
                        Block cur = next;
                        const bool last = r + round >= blocks;
                        if (!last || ch + 1 < nchunks) load_ahead(next, last ? ch + 1 : ch, last ? 0 : r + round);
                        __builtin_amdgcn_sched_barrier(0);
                        const int i = r + 64 * first + lane;
                        int g, pos;
                        place_of(i, g, pos);
                        split_block(cur, to + g * word_bytes + pos * kPosBytes, i < blocks);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the words are in LDS (and the next round's values in registers)
                    __syncthreads();                     // chunk ch is there, chunk ch - 1 has been read
                }
                return;
            }
            for (int ch = 0; ch < nchunks; ++ch) {
                multiply(ch);
                if (ch + 1 < nchunks) __syncthreads();
            }
        } else {
            for (int ch = 0; ch < nchunks; ++ch) {
                __syncthreads();                         // the chunk before has been read
                stage(ch, wave, all_waves);
                __syncthreads();
                multiply(ch);
            }
        }

        // accumulator register r of a lane: filter row 8*(r/4) + 4*half + r%4 of the tile, pixel column `col`
        if (px < OHW && nfil > 0) {
            float *dst = p.out + ((size_t)n * p.F + f0) * OHW + px;
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 32 * f + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (row < nfil) dst[(size_t)row * OHW] = (acc[f][r] + acc[f][r]) * p.alpha[f0 + row];
                }
        }
    }
};

template <int NF, bool SPLITS, bool STAGERS>
__global__ __launch_bounds__(64 * kMaxWaves, STAGERS ? 4 : 3) void bwn_fp6_kernel(Fp6Params p)
{
    Fp6Wave<NF, SPLITS, STAGERS>::run(p);
}

struct Fp6Plan {
    bool ok;
    int nf, G, splits, stagers, waves, wgs, positions;
    size_t lds;
    double cycles;                 // about what the launch takes (see kRouteCosts)
};

// LDS of a workgroup: the staged positions of G words and the zero position; the filter words of G * taps rows, up to
// whole steps, and of two steps that are read ahead of use (the rows' last 64 words may reach into these).
size_t fp6_words_bytes(const Geom &g, int filters, int G)
{
    const int taps = g.kh * g.kw, steps = G == 2 ? taps : (taps + 1) / 2;
    return (size_t)(steps + 2) * 8 * filters;
}
size_t fp6_lds(const Geom &g, int filters, int G, int positions, int buffers)
{
    return buffers * ((size_t)G * (positions + 1) * kPosBytes + fp6_words_bytes(g, filters, G));
}

// Most positions that a workgroup of `tiles` tiles stages: whole rows under the output rows it can touch.
long long fp6_positions(const Geom &g, int tiles)
{
    const long long orows = std::min(g.OH, (32 * tiles + g.OW - 2) / g.OW + 1);
    return std::min((long long)g.H, (orows - 1) * g.sh + g.kh) * g.W;
}

// About what a launch takes on its busiest compute unit, in cycles: `busiest` workgroups, in batches of those
// that a unit holds.  A batch is through when its matrix instructions and conversions are, on the SIMD that
// has most of its waves, or when one workgroup's chain is: load, convert, barrier, multiply.
struct Fp6Costs {
    double contended;              // matrix instructions beside others', at the card's power
    double convert, load;          // a round of blocks: the conversions; the wait for its loads
    double chunk, words;           // barriers and the first operands; an instruction of filter words
    double stores, launch;         // outputs of a filter tile
};
// Between a layer's own shapes of workgroup: a fit to 2700 timed launches of 45 layers (1 to 128 images, 32 to 512 channels and
// filters, 1x1 to 7x7, 7 to 64 wide); the shape taken is 2 % slower than the best of the up to 64 on average, 20 % at most.
constexpr Fp6Costs kPlanCosts = {1.3, 1850, 2100, 3300, 320, 1900, 0};
// Between the two forms, with split_cycles of csrc/bwn_split.hip: a fit to which is the faster one, over the shapes taken of 13000
// layers (1 to 128 images, 1 to 512 channels, 4 to 512 filters, 1x1 to 7x7, 4 to 420 wide, strides 1 to 4).
constexpr Fp6Costs kRouteCosts = {2.4, 800, 2500, 0, 0, 3500, 8800};

double fp6_cost(const Fp6Costs &c, const Geom &g, int nf, int G, int waves, int positions, size_t lds, long long busiest)
{
    constexpr double kSteps = 430;                        // into the steps, per chunk
    const int taps = g.kh * g.kw, nt = 64 * waves;
    double mfma = 0, convert = 0, wait = 0;
    auto chunks = [&](int n, int words) {
        const int steps = words == 2 ? taps : (taps + 1) / 2, rounds = ceil_div((long long)positions * words, nt);
        mfma += n * (steps * nf * kDigits * 32 + kSteps);
        convert += n * rounds * c.convert;
        wait += n * (c.chunk + rounds * c.load + c.words * taps * words * nf * 0.5 / waves);
    };
    chunks(g.Cw / G, G);
    if (g.Cw % G) chunks(1, 1);
    const double alone = mfma + convert + wait + c.stores * nf;
    // registers hold three waves on a SIMD, four with one filter tile (with two filter tiles four as well, as the other estimate below
    // has it; this one's constants were fitted with three); of workgroups of five to eight waves, which put two on some SIMD, one or two
    const int per_simd = nf == 1 ? 4 : 3;
    const int held = std::max(1, std::min((int)(kLds / lds), waves > 4 ? per_simd / 2 : 4 * per_simd / waves));
    auto batch = [&](long long n) {
        return std::max(alone, ceil_div(n * waves, 4) * (mfma * c.contended + convert) + wait / n);
    };
    const long long full = busiest / held, rest = busiest % held;
    return c.launch + full * batch(held) + (rest ? batch(rest) : 0.0);
}

// The same of a workgroup of `splits` x `t` multiplying waves and `stagers` that only stage.  A fit to 257000 timed launches of 1269 layers
// (every shape of each: 1 to 128 images, 32 to 512 channels and filters, 1x1 to 7x7, 7 to 70 wide, strides 1 and 2), for the
// time of the shape taken.  Against the shapes above alone it is 0.83 of the time on average (the best shapes of all 0.79); a shape
// that it takes is more than 3 % slower in 1.3 % of the layers and more than 10 % in 0.3 %; without the margin, or with stagers beside
// more filters a wave, more pixel tiles or more workgroups than units, where their waves and LDS cost what they save, in 3 % and 1.3 %.
constexpr int kMaxSplits = 4;
constexpr double kSplitMargin = 0.75;
double fp6_split_cost(const Geom &g, int nf, int G, int splits, int t, int stagers, int positions, size_t lds, long long busiest)
{
    constexpr double kContended = 1.06, kConvert = 2520, kLoad = 1210, kChunk = 9520, kWords = 324, kStores = 2245, kSteps = 194;
    constexpr double kStage = 0.81 * kConvert + 35, kStaged = 2330, kHandOver = 4510, kFirst = 1077, kMixed = 0.87;
    const int taps = g.kh * g.kw, waves = splits * t, all = waves + stagers;
    double mfma = 0, convert = 0, wait = 0, alone = kStores * nf;
    auto chunks = [&](int n, int words) {
        const double steps = (words == 2 ? taps : (taps + 1) / 2) * nf * kDigits * 32 + kSteps;
        const double filter_words = kWords * taps * words * nf * splits * 0.5;
        const int rounds = ceil_div((long long)positions * words, 64 * (stagers ? stagers : waves));
        mfma += n * steps;
        convert += (double)n * rounds * kConvert * (stagers ? stagers : waves);
        if (stagers) {
            alone += n * std::max(steps + kHandOver, rounds * kStage + filter_words / stagers + kStaged);
            wait += n * 30;
        } else {
            const double w = kChunk + rounds * kLoad + filter_words / waves;
            alone += n * (steps + rounds * kConvert + w);
            wait += n * w;
        }
    };
    chunks(g.Cw / G, G);
    if (g.Cw % G) chunks(1, 1);
    double less = 1.0;
    if (stagers) {
        const int rounds = ceil_div((long long)positions * G, 64 * all);
        alone += rounds * (kConvert + kLoad) + kFirst;
        wait += rounds * kLoad + kFirst;
        less += 0.033 * std::max(0, ceil_div((long long)positions * G, 64 * stagers) - 1) + 0.26 * std::max(0LL, busiest - 1);
    }
    const int per_simd = nf <= (stagers ? 3 : 2) ? 4 : 3;
    const long long held = std::max<long long>(1, std::min<long long>((long long)(kLds / lds), all > 4 ? per_simd / 2 : 4 * per_simd / all));
    auto batch = [&](long long n) {
        return n == 0 ? 0.0 : std::max(alone, n * waves / 4.0 * mfma * kContended + n * convert / 4 * (stagers ? kMixed : 1.0) + wait / n);
    };
    return less * ((busiest / held) * batch(held) + batch(busiest % held));
}

Fp6Plan search_fp6_plan(const Geom &g, int cus)
{
    Fp6Plan pl{};
    const long long OHW = (long long)g.OH * g.OW, taps = (long long)g.kh * g.kw;
    if (taps > 64 || OHW > (1 << 24) || (long long)g.C * g.H * g.W >= (1LL << 29)) return pl;     // (32-bit byte offsets)
    if ((long long)g.F * taps * g.Cw >= (1LL << 29)) return pl;
    const int tiles = ceil_div(OHW, 32);
    // Workgroups that the busiest compute unit gets: a unit's filter groups run on one XCD (with 36 units and seven groups 35 workgroups
    // on its 32 compute units).
    auto busiest_of = [&](int wgs, int filters) {
        const long long per_xcd = ((long long)g.N * wgs + 7) / 8 * ceil_div(g.F, filters);
        return (long long)ceil_div(per_xcd, std::max(1, cus / 8));
    };
    auto consider = [&](double &best, Fp6Plan &to, int nf, int G, int splits, int t, int stagers) {
        const long long positions = fp6_positions(g, t);
        if (positions > (long long)(kLds / kPosBytes)) return;
        const size_t lds = fp6_lds(g, 32 * nf * splits, G, (int)positions, stagers ? 2 : 1);
        if (lds > kLds) return;
        const int wgs = ceil_div(tiles, t);
        const long long all = (long long)g.N * wgs * ceil_div(g.F, 32 * nf * splits);
        if (all > 0x7ffffff0LL) return;
        // (only in launches of at most a workgroup a unit, on the XCD that has most of them: of 7800 drawn layers 101 had one more there
        // and take 0.78 of their time with the shapes that this leaves, 11 of them up to 1.2 times it)
        if (stagers && (all > cus || busiest_of(wgs, 32 * nf * splits) > 1)) return;
        const bool one = &to == &pl;
        const double cost = one ? fp6_cost(kPlanCosts, g, nf, G, t, (int)positions, lds, (all + cus - 1) / cus)
                                : fp6_split_cost(g, nf, G, splits, t, stagers, (int)positions, lds, (all + cus - 1) / cus);
        if (best >= 0 && cost >= best) return;
        best = cost;
        to = {true, nf, G, splits, stagers, splits * t, wgs, (int)positions, lds, 0.0};
    };
    auto shapes = [&](auto with) {
        for (int nf = 4; nf >= 1; --nf)
            if (nf == 1 || 32 * (nf - 1) < g.F)
                for (int G = std::min(2, g.Cw); G >= 1; --G) with(nf, G);
    };
    double best = -1.0;
    shapes([&](int nf, int G) {
        for (int t = std::min(kMaxWaves, tiles); t >= 1; --t) consider(best, pl, nf, G, 1, t, 0);
    });
    if (pl.ok) {
        pl.cycles = fp6_cost(kRouteCosts, g, pl.nf, pl.G, pl.waves, pl.positions, pl.lds, busiest_of(pl.wgs, 32 * pl.nf));
        // A shape with splits or stagers, where it is the better one by a margin.  Without stagers two splits in 2, 4 or 8 waves, as the estimate
        // was fitted for: with the other numbers of both it would choose differently in 2 % of 7800 drawn layers, 0.91 of the time on
        // average and up to 1.35 times.  The route to this form or the other keeps the estimate of the shape without.
        Fp6Plan other{};
        double least = -1.0;
        shapes([&](int nf, int G) {
            for (int splits = 1; splits <= kMaxSplits && (splits == 1 || 32 * nf * (splits - 1) < g.F); ++splits)
                for (int t = std::min(kMaxWaves / splits, tiles); t >= 1; --t) {
                    const int waves = splits * t;
                    if (splits == 2 && (waves == 2 || waves == 4 || waves == 8)) consider(least, other, nf, G, splits, t, 0);
                    if (waves <= 4 && (nf == 1 || (nf == 2 && t <= 2)))
                        for (int stagers = 3; stagers <= 4; ++stagers) consider(least, other, nf, G, splits, t, stagers);
                }
        });
        const double one = fp6_split_cost(g, pl.nf, pl.G, 1, pl.waves, 0, pl.positions, pl.lds,
                                          ((long long)g.N * pl.wgs * ceil_div(g.F, 32 * pl.nf) + cus - 1) / cus);
        // (of one word all is staged at once: half a microsecond slower)
        if (other.ok && g.Cw > 1 && least < kSplitMargin * one) {
            other.cycles = pl.cycles;
            return other;
        }
    }
    return pl;
}

const Fp6Plan &make_fp6_plan(const Geom &g)
{
    static thread_local PlanMemo<Fp6Plan> memo;
    const int cus = compute_units();
    return memo.get(g, cus, [&] { return search_fp6_plan(g, cus); });
}

template <int NF, bool SPLITS, bool STAGERS>
hipError_t start_fp6(const Fp6Plan &pl, const Fp6Params &p, unsigned blocks, hipStream_t st)
{
    if (pl.lds > 64 * 1024) {
        // raise the kernel's dynamic-LDS limit once per device
        static std::atomic<unsigned long long> raised{0};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return hipGetLastError();
        const unsigned long long bit = 1ull << (dev & 63);
        if (!(raised.load() & bit)) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&bwn_fp6_kernel<NF, SPLITS, STAGERS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
            if (e != hipSuccess) return e;
            raised.fetch_or(bit);
        }
    }
    bwn_fp6_kernel<NF, SPLITS, STAGERS><<<dim3(blocks), dim3(64 * (pl.waves + pl.stagers)), pl.lds, st>>>(p);
    return hipGetLastError();
}

template <bool SPLITS>
hipError_t start_shape(const Fp6Plan &pl, const Fp6Params &p, unsigned blocks, hipStream_t st)
{
    switch (pl.nf) {
        case 4: return start_fp6<4, SPLITS, false>(pl, p, blocks, st);
        case 3: return start_fp6<3, SPLITS, false>(pl, p, blocks, st);
        case 2: return start_fp6<2, SPLITS, false>(pl, p, blocks, st);
        default: return start_fp6<1, SPLITS, false>(pl, p, blocks, st);
    }
}

hipError_t launch_fp6_plan(const Fp6Plan &pl, const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g,
                           float *out, hipStream_t st)
{
    Fp6Params p;
    p.I = I; p.Wpk = Wpk; p.alpha = alpha; p.out = out;
    p.C = g.C; p.H = g.H; p.W = g.W; p.F = g.F; p.kh = g.kh; p.kw = g.kw;
    p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw; p.OH = g.OH; p.OW = g.OW; p.Cw = g.Cw;
    p.G = pl.G;
    p.splits = pl.splits;
    p.tiles = pl.waves / pl.splits;
    p.inv_splits = reciprocal((unsigned long long)pl.splits);
    p.wgs = pl.wgs;
    p.fgroups = ceil_div(g.F, 32 * pl.nf * pl.splits);
    p.inv_row = reciprocal(32ull * pl.nf * pl.splits);
    p.positions = pl.positions;
    const long long units = (long long)g.N * pl.wgs, blocks = (units + 7) / 8 * 8 * p.fgroups;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    p.units = (int)units;
    const unsigned b = (unsigned)blocks;
    p.stagers = pl.stagers;
    p.words_bytes = (int)fp6_words_bytes(g, 32 * pl.nf * pl.splits, pl.G);
    if (pl.stagers) return pl.nf == 1 ? start_fp6<1, true, true>(pl, p, b, st) : start_fp6<2, true, true>(pl, p, b, st);
    return pl.splits > 1 ? start_shape<true>(pl, p, b, st) : start_shape<false>(pl, p, b, st);
}

}  // namespace

bool bwn_fp6_supports(const Geom &g) { return make_fp6_plan(g).ok; }
double bwn_fp6_cycles(const Geom &g) { return make_fp6_plan(g).cycles; }
bool bwn_fp6_plan(const Geom &g, int cus, Fp6Shape *out)
{
    const Fp6Plan pl = search_fp6_plan(g, cus > 0 ? cus : compute_units());
    if (!pl.ok) return false;
    *out = {pl.nf, pl.G, pl.splits, pl.waves / pl.splits, pl.stagers, pl.lds, (long long)g.N * pl.wgs * ceil_div(g.F, 32 * pl.nf * pl.splits)};
    return true;
}

hipError_t launch_bwn_fp6(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g, float *out,
                          hipStream_t st)
{
    const Fp6Plan &pl = make_fp6_plan(g);
    if (!pl.ok) return hipErrorInvalidValue;
    return launch_fp6_plan(pl, I, Wpk, alpha, g, out, st);
}

}  // namespace xnor
