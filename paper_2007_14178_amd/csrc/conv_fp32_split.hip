// Real-valued fp32 convolution (the float comparison of Sec. IV, Table I) on the 16-bit matrix
// instructions.  Both operands are split into three bf16 terms, x = hi + mid + lo, each the nearest
// bf16 to what the terms before it left over (3 x 8 significand bits hold all 24 of an fp32, both
// differences are exact: |mid| <= 2^-8, |lo| <= 2^-17 of x's leading bit).  With r = mid + lo a product is
//   hi*hi + hi*mid + hi*lo + mid*hi + lo*hi + r*r,
// the first five on the bf16 instruction and the last one, at most 2^-16 of the whole, on the f16 one with r
// rounded to f16's 11 bits (2^-29 of the whole lost on average, of either sign; 2^-26 at most): six matrix instructions per 16
// channels where bf16 alone takes eight (mid*mid, mid*lo and lo*mid in place of r*r).
//   f16's range is kept by powers of two: a filter tile's chunk of 16 channels is multiplied by the one that brings its largest
// magnitude to 2^23 .. 2^24, a workgroup's input by the one that brings the largest of its first chunk to 2^18 .. 2^19, and a
// chain's sum is divided by both where it joins the output's.  Scaled values of 2^-6 to 2^24 and zeros are held.  A wave that
// meets others (a filter decayed to 2^-30 of its neighbours, an input value 2^-25 or 2^5 of the first chunk's largest) takes the eight
// products from that chunk on, which need no range: such a layer is as fast as with eight products everywhere, where forming the
// outputs that could matter by the plain sum took three times as long (us, eight products in chains of one tap / this with six
// products only and such outputs by the plain sum, the images' magnitudes read beforehand / this):
//                                          ordinary values       one filter of 1e-11     the lower half zero, one value of 1e-12
//   128 x 512 x 28 x 28 F=512 3x3     3285 / 2690 / 2510      3360 / 8820 / 2620 to 2810      2800 / 6990 / 2200
//   16 x 128 x 56 x 56 F=128 5x5       327 / 251 / 245         326 / 790 / 273                 291 / 949 / 227
//   32 x 512 x 56 x 56 F=64 1x1        103 / 122 / 90
//   32 x 256 x 56 x 56 F=16 2x2        131 / 161 / 118
//
// What the sum loses.  The products of two taps x 16 channels form a chain of their own that starts at zero,
// small products first, and joins the output's sum in one addition: the large sum is rounded once per 32
// terms (the fp32 matrix instruction rounds it once per two, and six products in one chain with it were
// no better).  The instructions shift what they add to the exponent of the largest and drop the rest towards
// minus infinity, which left every output the same amount too low (0.27e-6 of their root mean square for 7 x 7 x 416
// terms): the weights of every other chain are therefore stored negated and its sum is subtracted.  Measured
// against 64-bit sums over layers of 32 to 384 channels, 1 x 1 to 5 x 5, normal, positive, constant, log-normal values and values,
// channels and filters of very different sizes: 0.65 to 0.94 of the error of chains of one tap with eight products
// (1 x 1, where a chain has one tap: the same), which had 0.17 to 0.57 of that of the kernels without a workspace.
//
//   split_filters_kernel: filters -> the A operands of the convolution in its order, into the
//   caller's workspace, 8 bytes per weight: [filter tile of 32][chunk of 16 channels][tap][hi, mid, lo, r]
//   [lane] of 16 bytes (lane = filter lane % 32, channels 8 * (lane / 32) .. + 7).
//   conv_fp32_split_kernel: workgroup = 4 waves = 128 filters x up to 4 tiles of 32 output pixels of
//   one image (64 filters x up to 8 tiles for layers of at most 64 filters); wave = 64 filters x up
//   to two tiles (a third one's accumulators would leave no registers for the chains).  Per chunk of 16 channels
//   the input under the pixels is fetched a chunk ahead (buffer loads: outside the image they give the zeros of
//   the padding), split and staged in LDS as [position][term][16 channels] (144 bytes a position: sixteen
//   lanes' 16-byte reads at consecutive positions touch distinct banks).  A B operand is one 16-byte LDS read per
//   lane and feeds three matrix instructions on average, an A operand is one 16-byte load per lane from the L2
//   and feeds as many; each is fetched again into its registers behind its last use, 7 (LDS) and 15 (L2) matrix
//   instructions ahead of its next one.
//   Nothing in a chunk's steps branches: the fetch past the last chunk reads from an empty buffer.  (A branch around it let the
//   compiler move the additions of chains and the magnitudes' maxima behind it; it spilled 25 to 280 registers then.)
//   Bound by power as much as by time: a register-only loop of the bf16 instruction on random operands keeps 1.74 GHz, this
//   1.77.  One wave per SIMD with four tiles (half the filter loads) was slower.
//
// Pairs (layers of many terms, see takes_pairs): both operands as two f16 terms, x = h + l, each the nearest f16 to what is
// left, and three products of them on the f16 instruction, l * h + h * l + h * h: half the matrix instructions.  A pair holds
// 22 significant bits and a sign, all of x in three values of four and all but its last bit in the others; with l * l left
// out a product is off by 8e-8 of itself on average.  The sums make up for it: a chain takes all taps of a chunk up to nine or ten,
// where the six products' takes two (the rounding of the outputs' sums is the larger part of a long sum's error).  Against
// 64-bit sums, normal values, six products / pairs:
//   3 x 3, 128, 256, 512 channels: 1.23e-7 1.67e-7 2.30e-7 / 1.59e-7 1.67e-7 1.82e-7;  5 x 5, 64, 128, 512: 1.36e-7 1.86e-7
//   3.59e-7 / 1.63e-7 1.74e-7 2.30e-7;  positive values 0.95e-7 to 3.0e-7 / 0.63e-7 to 1.5e-7.
// us: 128 x 512 x 28 x 28 F=512 3x3 2360 -> 1320, 16 x 128 x 56 x 56 F=128 5x5 247 -> 146, 1 x 512 x 13 x 13 F=64 3x3 92 -> 74.
//   Powers of two for f16's range: a filter tile's chunk has its own, and so has a workgroup's chunk of the input: its largest
// magnitude is found when its values arrive, a chunk ahead of their commit.  Low terms are stored times 2^11, as large as their
// high ones, so that values of 2^-21 of their chunk's largest are still within 2^-23 of themselves.  The sums have that factor,
// too: h * h gets it from its operands, multiplied by 2^5 and 2^6 in their registers behind the other two products.  (Stored as
// they are, low terms leave f16's normal range from 2^-17 of the largest on: an output that only values of 2^-20 of their
// neighbours' size go into had 2.5 to 4.2 times the error of three terms, and has 0.79 to 0.94 of it so.  The multiplications
// cost 4 % at the first layer above, 2 % at the second, and 2.4 % on average over 100 drawn layers.)
//   Smaller values are held in part, within 2^-45 of the largest.  What all of them can do to an output is bounded by their number
// (3 in 10^7 of normal values); a wave forms the few outputs below 2^22 times that one by one, in 64 bits.  Where there are
// more of them, or a value without a power of two (infinite, NaN, of 2^-46 or 2^68), or an output that came out infinite, NaN or
// below 2^-120, the workgroup's outputs are formed from three terms as in the layers without pairs.  Log-normal values (sigma 4)
// and filters of 2^-16 or 1e-11 of their neighbours stop at once, at 1.02 to 1.14 times that form's time; where it shows in
// the outputs alone (such a value somewhere in a workgroup and filters or windows of zeros) the workgroup takes 1.6 times it.
//   Errors against those of three terms by kind of values (3 x 3 on 288 and 512 channels, 5 x 5 on 128): normal 0.79 to 0.96, half
// of them zeros 0.79 to 0.98, positive 0.47 to 0.52, constant 0.33 to 0.44, channels of 2^-(c % 16) 0.82 to 0.97, log-normal
// (sigma 2) 0.82 to 0.96, 90 % zeros 0.73 to 0.87.  Larger ones are left where few terms are: 99 % zeros 1.09 to 1.24 (a
// product alone is within 2^-21, that of three terms within 2^-23); and constant values in one window with others of 2^16 of
// their size, whose largest error is 0.6 to 2.2 times (the chain that holds those is the longer one).
//   conv_fp32_split_kernel<.., PAIR> has the tiles and the staging of the other forms, 80 bytes a position.  The A operands
// are a ring of three taps (two where the window's taps are no multiple of three) in registers, an operand fetched again behind
// its last use, 26 (14) matrix instructions ahead; those fetched in a chunk's last tap are waited for at its end, with the values of the chunk
// after the next, for their magnitudes.  What it measured at the first layer: pairs with the six products' loop
// 1435 us, with one buffer descriptor for an image in place of one a plane and without a load at the head of a chunk 1355, with the
// ring, and granules for the positions that there are (240; 384 had been handled), 1275 (matrix pipe busy 63 % of the cycles at 1.72 GHz), with the high terms' multiplications 1320;
// a loop of the matrix instructions alone takes 895 us, at the card's power.  Timing-only builds: without A loads
// 12 % shorter, without B reads 9, without commits 15.
//
// FLUSH: where the layer would otherwise run one thread per output, whose sums are formed from short
// chains, that is still the less exact of the two.  This form keeps two accumulators per output: the
// matrix instructions sum two taps of a chunk, then that sum is added to the other accumulator and what the
// addition rounded off is where the next chain starts from (0.43 of the error of one thread per output).  It has no
// registers for a fourth term: three, unscaled, and eight products (all but lo*lo, below 2^-32 of the whole).
//
// What the split cannot hold goes by the fp32 matrix instruction instead (plain_tiles), a wave's outputs at
// a time: all outputs of a workgroup that stages an infinity, a NaN or a value too large for bf16 or the scale (it leaves
// the loop at the chunk that has one), outputs that came out infinite or NaN, and outputs so small that bits of a value
// below 2^-133, bf16's last one, could matter to them (only where a (scaled) input or weight below 2^-110 was seen, see
// `doubtful`).  The instructions themselves keep subnormals.
// A launch whose every output goes that way: see plain_tiles.
#include <algorithm>
#include <atomic>
#include <type_traits>
#include <utility>

#include "xnor_internal.hpp"

namespace xnor {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kChan = 16;              // channels per chunk = the reduction length of one matrix instruction
// Terms of a split operand: hi, mid, lo in bf16, and but for the form with short chains (see FLUSH) mid + lo in f16.
constexpr int terms(bool flush) { return flush ? 3 : 4; }
constexpr int pos_bytes(bool flush) { return terms(flush) * 32 + 16; }         // see above
constexpr int operand_bytes(bool flush) { return terms(flush) * 1024; }        // the A operands of a (filter tile, chunk, tap)
// Granules (8 channels of one position) a thread fetches ahead per chunk: three, or four where 32 pixels stage more
// positions than that (the form with short chains has no such variant).
constexpr int kGranules = 3, kMostGranules = 4;
constexpr int max_pos(int granules) { return granules * 128; }   // staged positions of a workgroup
constexpr int kWaveTiles = 2;          // pixel tiles per wave
// Chains of the form without short ones: the taps of a chunk two and two, the last one alone where their number is odd.
// (The other form counts the taps of all chunks in a row.)
__device__ inline bool chain_negated(bool flush, int chunk, int tap, int taps)
{
    return (flush ? (chunk * taps + tap) >> 1 : chunk * ((taps + 1) / 2) + (tap >> 1)) & 1;
}
constexpr int kMaxTaps = 49;           // 7 x 7; the filter pass holds 32 x 8 channels x taps in LDS
constexpr size_t kLdsShared = 80 * 1024;  // two workgroups per compute unit

struct Fp32SplitParams {
    const float *I;
    const float *Wt;
    const unsigned char *Wx;       // split filters
    const uint32_t *wstat;         // one word per (filter tile, 8 channels): kTinyBit | largest magnitude
    const int *wexp;               // per (filter tile, chunk): kUnheld | the power of two its weights are stored times + kExpBias
    const unsigned char *Wp;       // pairs: split filters, the power of two of each (filter tile, chunk), and per (filter tile,
    const int *pexp;               //   8 channels) the weights that a pair holds in part, kNotHeld and more where none do
    const uint32_t *plow;
    float *out;
    int N, C, H, W, F, kh, kw, sh, sw, ph, pw, OH, OW;
    int nchunks, ftiles;
    int fwaves;                    // waves along the filters: 2 or 1 (64 filters each)
    int fgroups, groups;           // workgroups along the filters, along the pixels of an image
    int tiles;                     // pixel tiles per workgroup (tw == 0), or tx * ty
    int tw;                        // 0: a tile is 32 consecutive pixels; else tiles of tw x 32 / tw pixels
    int tx, ty, gx;                // tw > 0: tiles of a workgroup along x and y, workgroups along x
    int pitch, npos;               // staged positions per row, in all
    uint32_t inv_pitch;
};

constexpr int kRaw = 0x00027000;             // (buffer descriptor: a plain buffer of dwords)
constexpr uint32_t kOutside = 0xfffffff0u;   // (an offset beyond any buffer: the load is 0)
constexpr uint32_t kTinyBit = 0x80000000u;
constexpr float kTiny = 0x1p-110f;
constexpr float kDoubt = 0x1p-104f;
constexpr uint32_t kHuge = 0x7f7f8000u << 1;              // (doubled bits) from here on bf16 rounds to infinity
constexpr uint32_t kInfBits = 0x7f800000u;

// The power of two that brings a largest magnitude (its bits) to 2^23 .. 2^24 for weights, to 2^18 .. 2^19 for inputs (see
// above), as far as values of ordinary size behind tiny ones stay in fp32's range and what divides by two of them does (2^60 each).
constexpr int kTopW = 23, kMostW = 59, kTopX = 18, kMostX = 40, kLeast = -60;
constexpr int kExpBias = 256, kUnheld = 1024;
__device__ inline int scale_of(uint32_t top, int to, int most) { return top == 0 ? 0 : max(kLeast, min(most, to + 127 - (int)(top >> 23))); }
constexpr float kHeldLow = 0x1p-6f, kHeldTop = 0x1p24f;   // scaled values whose mid + lo f16 holds to 11 bits
// 2^e for e >= -149, infinite from 2^128 on
__device__ inline uint32_t power_bits(int e)
{
    return e > 127 ? kInfBits : e > -127 ? (uint32_t)(e + 127) << 23 : 1u << max(0, e + 149);
}

// Pairs: a chunk's largest magnitude is brought to 2^kPairTopW (weights) or 2^kPairTopX (input) and up to twice that, by at most
// 2^kPairMost or 2^-kPairMostDown.  The low term is stored times 2^kPairShift, and the high ones are multiplied by 2^kPairUpW and
// 2^kPairUpX, which make 2^kPairShift, for their product.  A scaled value below kPairLow that is not zero counts as held in part: kPairLoss
// of it may be lost.
constexpr int kPairTopW = 9, kPairTopX = 8, kPairUpW = 14 - kPairTopW, kPairUpX = 14 - kPairTopX, kPairShift = kPairUpW + kPairUpX;
constexpr int kPairMost = 54, kPairMostDown = 60;
constexpr float kPairLow = 0x1p-13f;
constexpr int kPairLossExp = -25 - kPairShift;
constexpr uint32_t kNotHeld = 1u << 20, kPairMostLow = 1024, kPairMostLowW = 64;    // (of a workgroup's input, of its weights)
constexpr int kPairShareExp = 22;       // an output stands where such values can change it by at most 2^-kPairShareExp of itself
static_assert(kPairShift == 11, "a low term is as large as its high one");
constexpr int kPairFew = 4;             // doubtful outputs that a wave forms one by one
constexpr float kPairLeast = 0x1p-120f;
constexpr int kPairPosBytes = 2 * 32 + 16, kPairOperandBytes = 2 * 1024;
// Taps of a chunk in a chain.
__host__ __device__ constexpr int pair_chain_taps(int taps) { return taps % 3 == 0 ? 9 : 10; }
__device__ inline int pair_chains(int taps) { return (taps + pair_chain_taps(taps) - 1) / pair_chain_taps(taps); }
__device__ inline bool pair_chain_negated(int chunk, int tap, int taps)
{
    return (chunk * pair_chains(taps) + tap / pair_chain_taps(taps)) & 1;
}
// the power of two for a largest magnitude (its bits), `held`: there is one
__device__ inline int pair_exp(int to, uint32_t top, bool &held)
{
    const int e = to + 127 - (int)(top >> 23);
    held = top == 0 || (e >= -kPairMostDown && e <= kPairMost);
    return top == 0 ? kPairMost : e;
}

// two fp32 -> two bf16 in one dword, to nearest even (one v_cvt_pk_bf16_f32)
__device__ inline uint32_t pack_bf16(float a, float b)
{
    const floatx2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// two fp32 -> two f16 in one dword, to nearest even (one v_cvt_pk_f16_f32)
__device__ inline uint32_t pack_f16(float a, float b)
{
    const floatx2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, halfx2));
}
// half of eight f16 (0: the first four) times 2^N
template <int N, int HALF>
__device__ inline void scale_f16(uint4 &v)
{
    auto times = [](uint32_t t) __attribute__((always_inline)) {
        return __builtin_bit_cast(uint32_t, __builtin_bit_cast(halfx2, t) * (halfx2)(_Float16)(1 << N));
    };
    uint32_t &x = HALF ? v.z : v.x, &y = HALF ? v.w : v.y;
    x = times(x);
    y = times(y);
}
// what the f16 pair `t` leaves of (a, b), times 2^kPairShift, for (a, b) given so; exact
__device__ inline void leave_pair_f16(float &a, float &b, uint32_t t)
{
    const halfx2 h = __builtin_bit_cast(halfx2, t);
    a = fmaf(-(float)(1 << kPairShift), (float)h.x, a);
    b = fmaf(-(float)(1 << kPairShift), (float)h.y, b);
}
// what the bf16 pair `t` leaves of (a, b); exact
__device__ inline void subtract_pair(float &a, float &b, uint32_t t)
{
    a -= __uint_as_float(t << 16);
    b -= __uint_as_float(t & 0xffff0000u);
}

// 32 filters x 8 channels x all taps per workgroup: a read in runs (a filter's channels are one run in
// memory) into LDS, then per (tap, filter) eight values from LDS, split, and 16-byte writes of 32 lanes side by
// side.  4 bytes read and 8 (6) written per weight.  The chunk's other eight channels are read for their
// magnitudes alone: the chunk has one power of two.
template <bool FLUSH, bool PAIR>
__global__ __launch_bounds__(kThreads) void split_filters_kernel(const float *__restrict__ Wt, int F, int C, int taps, int nchunks, int ftiles,
                                                                 uint32_t inv_run, unsigned char *__restrict__ Wx, unsigned char *__restrict__ Wp)
{
    extern __shared__ float wl[];
    __shared__ uint32_t stat[5];
    const int octs = 2 * nchunks;
    if (threadIdx.x < 5) stat[threadIdx.x] = threadIdx.x == 1 || threadIdx.x == 3 ? 0xffffffffu : 0u;
    __syncthreads();
    uint32_t top = 0, low = 0xffffffffu;         // of the magnitudes' bits; low: less one (0 - 1 wraps to the top)
    constexpr int kBatch = 8;                    // loads of a thread in flight
    const int ft = blockIdx.x / octs, oc = blockIdx.x - ft * octs;
    const int run = 8 * taps, pitch = run | 1;                     // (odd: filters fall into distinct banks)
    // values of the run that exist, in this half of the chunk and in the other
    const int live = max(0, min(8, C - 8 * oc)) * taps, live2 = FLUSH ? 0 : max(0, min(8, C - 8 * (oc ^ 1))) * taps;
    uint32_t finite = 0, low2 = 0xffffffffu;     // of both halves: the largest that is finite, the smallest
    for (int i0 = threadIdx.x; i0 < 32 * run; i0 += kBatch * kThreads) {
        float v[kBatch], o[kBatch];
        int at[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int idx = min(i0 + k * kThreads, 32 * run - 1);
            const int f = (int)quot((uint32_t)idx, inv_run), i = idx - f * run, fg = 32 * ft + f;
            const float *src = Wt + (size_t)min(fg, F - 1) * C * taps;
            const bool in = fg < F && i < live, in2 = fg < F && i < live2;
            at[k] = f * pitch + i;
            v[k] = src[in ? 8 * oc * taps + i : 0];
            v[k] = in ? v[k] : 0.f;
            if constexpr (!FLUSH) {
                o[k] = src[in2 ? 8 * (oc ^ 1) * taps + i : 0];
                o[k] = in2 ? o[k] : 0.f;
            }
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            wl[at[k]] = v[k];                                      // (the last value again: the same to the same place)
            const uint32_t u = __float_as_uint(v[k]) & ~kTinyBit;
            top = max(top, u);
            low = min(low, u - 1u);
            if constexpr (!FLUSH) {
                const uint32_t u2 = __float_as_uint(o[k]) & ~kTinyBit;
                finite = max(finite, max(u < kInfBits ? u : 0u, u2 < kInfBits ? u2 : 0u));
                low2 = min(low2, min(u - 1u, u2 - 1u));
            }
        }
    }
#pragma unroll
    for (int m = 1; m < 64; m *= 2) {
        top = max(top, (uint32_t)__shfl_xor((int)top, m));
        low = min(low, (uint32_t)__shfl_xor((int)low, m));
        if constexpr (!FLUSH) {
            finite = max(finite, (uint32_t)__shfl_xor((int)finite, m));
            low2 = min(low2, (uint32_t)__shfl_xor((int)low2, m));
        }
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&stat[0], top);
        atomicMin(&stat[1], low);
        if constexpr (!FLUSH) {
            atomicMax(&stat[2], finite);
            atomicMin(&stat[3], low2);
        }
    }
    __syncthreads();
    const int e = FLUSH ? 0 : scale_of(stat[2], kTopW, kMostW);
    unsigned char *const dst = Wx + ((size_t)ft * nchunks + (oc >> 1)) * taps * operand_bytes(FLUSH) + (oc & 1) * 512;
    bool pair_held = false;
    const int pe = PAIR ? pair_exp(kPairTopW, stat[2], pair_held) : 0;
    unsigned char *const pdst = Wp + ((size_t)ft * nchunks + (oc >> 1)) * taps * kPairOperandBytes + (oc & 1) * 512;
    uint32_t lows = 0;
    for (int i = threadIdx.x; i < 32 * taps; i += kThreads) {
        const int f = i & 31, t = i >> 5;
        const bool negated = chain_negated(FLUSH, oc >> 1, t, taps);               // (every other chain: see above)
        const float factor = negated ? -ldexpf(1.f, e) : ldexpf(1.f, e);
        uint32_t h[4], m[4], l[4], r[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float a = factor * wl[f * pitch + (2 * k) * taps + t], b = factor * wl[f * pitch + (2 * k + 1) * taps + t];
            h[k] = pack_bf16(a, b);
            subtract_pair(a, b, h[k]);
            r[k] = pack_f16(a, b);
            m[k] = pack_bf16(a, b);
            subtract_pair(a, b, m[k]);
            l[k] = pack_bf16(a, b);
        }
        uint4 *o = reinterpret_cast<uint4 *>(dst + (size_t)t * operand_bytes(FLUSH) + f * 16);
        o[0] = make_uint4(h[0], h[1], h[2], h[3]);
        o[64] = make_uint4(m[0], m[1], m[2], m[3]);
        o[128] = make_uint4(l[0], l[1], l[2], l[3]);
        if constexpr (!FLUSH) o[192] = make_uint4(r[0], r[1], r[2], r[3]);
        if constexpr (PAIR) {
            const float by = pair_chain_negated(oc >> 1, t, taps) ? -ldexpf(1.f, pe) : ldexpf(1.f, pe);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float a = by * wl[f * pitch + (2 * k) * taps + t], b = by * wl[f * pitch + (2 * k + 1) * taps + t];
                lows += (wl[f * pitch + (2 * k) * taps + t] != 0.f && fabsf(a) < kPairLow) + (wl[f * pitch + (2 * k + 1) * taps + t] != 0.f && fabsf(b) < kPairLow);
                h[k] = pack_f16(a, b);
                a *= (float)(1 << kPairShift);
                b *= (float)(1 << kPairShift);
                leave_pair_f16(a, b, h[k]);
                l[k] = pack_f16(a, b);
            }
            uint4 *q = reinterpret_cast<uint4 *>(pdst + (size_t)t * kPairOperandBytes + f * 16);
            q[0] = make_uint4(h[0], h[1], h[2], h[3]);
            q[64] = make_uint4(l[0], l[1], l[2], l[3]);
        }
    }
    if constexpr (PAIR) {
        if (lows) atomicAdd(&stat[4], lows);
        __syncthreads();
        if (threadIdx.x == 0) {
            // (stat[0], unlike stat[2], has the infinities and the NaN of this half)
            int *const pexps = reinterpret_cast<int *>(Wp + (size_t)ftiles * nchunks * taps * kPairOperandBytes);
            if ((oc & 1) == 0) pexps[ft * nchunks + (oc >> 1)] = pe;
            reinterpret_cast<uint32_t *>(pexps + ftiles * nchunks)[blockIdx.x] = pair_held && stat[0] < kInfBits ? min(stat[4], kNotHeld) : kNotHeld;
        }
    }
    if (threadIdx.x == 0) {
        uint32_t *stats = reinterpret_cast<uint32_t *>(Wx + (size_t)ftiles * nchunks * taps * operand_bytes(FLUSH));
        stats[blockIdx.x] = stat[0] | (stat[1] < __float_as_uint(ldexpf(kTiny, -e)) - 1u ? kTinyBit : 0u);
        if (!FLUSH && (oc & 1) == 0)
            reinterpret_cast<int *>(stats + ftiles * octs)[ft * nchunks + (oc >> 1)] =
                (e + kExpBias) | (e == kLeast || stat[3] < __float_as_uint(ldexpf(kHeldLow, -e)) - 1u ? kUnheld : 0);
    }
}

// The outputs of a wave's tiles by the plain sum, on the fp32 matrix instruction: per tap chains of 32
// channels, each added to the output's sum where the tap is inside the image (an infinite weight over padding adds
// nothing).  `put(i, j, r, v)` takes the value of accumulator register r of filter tile i and pixel tile j.
//   The filters come from the workspace, hi + mid + lo, which is the weight again; a lane whose weights are not
//   all held there (infinite, NaN, too large for bf16 or so small that bits are missing) reads its own from the
//   layer's filters.  32 x 256 x 28 x 28 F=256 3x3 takes 0.19 ms, with one NaN in the input 0.42, all NaN 0.58, with a third
//   of the filters at 1e-36 0.60, below 1e-44 0.87 (0.45 for any without a workspace; 15 to 36 ms where lanes formed
//   such outputs one by one).  The operands of a (tap, chunk) step are loaded a step ahead: a lane of half h holds channels
//   8 h .. 8 h + 7 of the chunk, and a matrix instruction takes one of either half.
template <int NT, bool FLUSH, class Pixel, class Put>
__device__ __attribute__((always_inline)) void plain_tiles(const Fp32SplitParams &p, int n, int f0, Pixel pixel_of, Put put)
{
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    const int HW = p.H * p.W, taps = p.kh * p.kw;
    const float *img = p.I + (size_t)n * p.C * HW;
    const uint32_t *stats = p.wstat;
    int ft[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) ft[i] = min((f0 >> 5) + i, p.ftiles - 1);
    int y[NT], x[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        int oy, ox;
        pixel_of(j, oy, ox);
        y[j] = oy * p.sh - p.ph;
        x[j] = ox * p.sw - p.pw;
    }
    auto inside = [&](int j, int t, int &at) -> bool {
        const int ky = t / p.kw, iy = y[j] + ky, ix = x[j] + t - ky * p.kw;
        const bool in = (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W;
        at = in ? iy * p.W + ix : 0;
        return in;
    };
    uint4 raw[2][3];
    float bn[NT][8];
    auto fetch = [&](int t, int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint4 *src = reinterpret_cast<const uint4 *>(p.Wx + (((size_t)ft[i] * p.nchunks + ch) * taps + t) * operand_bytes(FLUSH)) + lane;
            raw[i][0] = src[0];
            raw[i][1] = src[64];
            raw[i][2] = src[128];
        }
        const int c0 = ch * kChan + 8 * half;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            int at;
            inside(j, t, at);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float v = img[(size_t)(c0 + k < p.C ? c0 + k : 0) * HW + at];
                bn[j][k] = c0 + k < p.C ? v : 0.f;
            }
        }
    };
    floatx16 total[2][NT], part[2][NT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) { total[i][j] = floatx16{}; part[i][j] = floatx16{}; }
    fetch(0, 0);
    for (int t = 0, ch = 0; t < taps;) {
        const float sgn = chain_negated(FLUSH, ch, t, taps) ? -1.f : 1.f;
        float w[2][8], b[NT][8];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            bool held = true;
            const float back = FLUSH ? sgn : sgn * ldexpf(1.f, kExpBias - (p.wexp[ft[i] * p.nchunks + ch] & ~kUnheld));
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const auto term = [&](int q) {
                    const uint32_t u = (k >> 1) == 0 ? raw[i][q].x : (k >> 1) == 1 ? raw[i][q].y : (k >> 1) == 2 ? raw[i][q].z : raw[i][q].w;
                    return __uint_as_float(k & 1 ? u & 0xffff0000u : u << 16);
                };
                const float hi = term(0);
                held &= fabsf(hi) >= kTiny && fabsf(hi) < INFINITY;
                w[i][k] = back * ((hi + term(1)) + term(2));
            }
            // (uniform) does the operand hold all weights as they are, but for zeros?
            const uint32_t s0 = stats[(ft[i] * p.nchunks + ch) * 2], s1 = stats[(ft[i] * p.nchunks + ch) * 2 + 1];
            const bool all_held = ((s0 | s1) & kTinyBit) == 0 && max(s0 & ~kTinyBit, s1 & ~kTinyBit) < (kHuge >> 1);
            if (!all_held && !held) {
                const int f = ft[i] * 32 + col, c0 = ch * kChan + 8 * half;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    w[i][k] = f < p.F && c0 + k < p.C ? p.Wt[((size_t)f * p.C + c0 + k) * taps + t] : 0.f;
            }
        }
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int k = 0; k < 8; ++k) b[j][k] = bn[j][k];
        const int tap = t;
        const bool add = (ch & 1) || ch + 1 == p.nchunks;
        if (++ch == p.nchunks) { ch = 0; ++t; }
        if (t < taps) fetch(t, ch);
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) part[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[i][k], b[j][k], part[i][j], 0, 0, 0);
        if (add) {
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                int at;
                const bool in = inside(j, tap, at);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        total[i][j][r] += in ? part[i][j][r] : 0.f;
                        part[i][j][r] = 0.f;
                    }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) put(i, j, r, total[i][j][r]);
}

// f(0) .. f(31), each number a constant
template <class F, int... M>
__device__ __attribute__((always_inline)) inline void for_each_of(F f, std::integer_sequence<int, M...>)
{
    (f(std::integral_constant<int, M>{}), ...);
}
template <class F>
__device__ __attribute__((always_inline)) inline void for_units(F f) { for_each_of(f, std::make_integer_sequence<int, 32>{}); }

// The products of a (tap, 16 channels) step in their order, small ones first: the terms of filters and input (0 .. 3: hi, mid, lo,
// r = mid + lo), and which term's registers are free behind each.
template <int PRODUCTS>
struct Order;
template <>
struct Order<6> {      // r*r, hi*lo, hi*mid, lo*hi, mid*hi, hi*hi
    int a[6] = {3, 0, 0, 2, 1, 0}, b[6] = {3, 2, 1, 0, 0, 0};
    int load_a[6] = {3, -1, -1, 2, 1, 0}, read_b[6] = {3, 2, 1, -1, -1, 0};
};
template <>
struct Order<8> {      // mid*lo, lo*mid, lo*hi, hi*lo, mid*mid, mid*hi, hi*mid, hi*hi
    int a[8] = {1, 2, 2, 0, 1, 1, 0, 0}, b[8] = {2, 1, 0, 2, 1, 0, 1, 0};
    int load_a[8] = {3, -1, 2, -1, -1, 1, -1, 0}, read_b[8] = {3, -1, -1, 2, -1, -1, 1, 0};
};

// The output pixel of lane column `col` in tile j of the workgroup, clamped to the image for the reads, and whether it exists.
__device__ __attribute__((always_inline)) inline bool tile_pixel(const Fp32SplitParams &p, int t0, int X0, int Y0, int tw_shift, int j, int col, int &oy, int &ox)
{
    if (p.tw == 0) {
        const int OHW = p.OH * p.OW, px = (t0 + j) * 32 + col, pxc = min(px, OHW - 1);
        oy = pxc / p.OW;
        ox = pxc - oy * p.OW;
        return px < OHW;
    }
    const int jy = j / p.tx, jx = j - jy * p.tx;
    oy = Y0 + jy * (32 >> tw_shift) + (col >> tw_shift);
    ox = X0 + jx * p.tw + (col & (p.tw - 1));
    const bool in = oy < p.OH && ox < p.OW;
    oy = min(oy, p.OH - 1);
    ox = min(ox, p.OW - 1);
    return in;
}

// Largest of a wave's values, in every lane.
__device__ inline uint32_t wave_max(uint32_t v)
{
    auto step = [&](auto ctrl) __attribute__((always_inline)) {
        v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, decltype(ctrl)::value, 0xf, 0xf, false));
    };
    step(std::integral_constant<int, 0x111>{});      // within a row of 16: 1, 2, 4 and 8 lanes on
    step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{});
    step(std::integral_constant<int, 0x118>{});
    step(std::integral_constant<int, 0x142>{});      // a row's last lane to the next row, then to the upper half
    step(std::integral_constant<int, 0x143>{});
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// A wave's work in the form with pairs: false where the workgroup's outputs are to be formed from three terms after all (the
// same for all its waves).  Arguments as for split_wave; fw0: the workgroup's first filter.
template <int NT, int GRAN, int RING>
__device__ __attribute__((always_inline)) bool pair_wave(const Fp32SplitParams &p, int n, int f0, int fw0, int t0, int X0, int Y0,
                                                         int oy0, int iy0, int ix0, int rows, int tile0)
{
    // LDS: two input buffers, taken in turn by the chunks, each [npos][high, low][16 channels]
    extern __shared__ unsigned char lds_raw[];
    constexpr int kGran = GRAN, kTiles = NT > 0 ? NT : 1;
    const int tile_bytes = p.npos * kPairPosBytes;
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    const int OHW = p.OH * p.OW, taps = p.kh * p.kw, HW = p.H * p.W;
    const int tw_shift = p.tw ? 31 - __builtin_clz((unsigned)p.tw) : 5;
    auto pixel_of = [&](int j, int &oy, int &ox) -> bool { return tile_pixel(p, t0, X0, Y0, tw_shift, j, col, oy, ox); };
    int base[kTiles];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        int oy, ox;
        pixel_of(tile0 + j, oy, ox);
        base[j] = ((oy - oy0) * p.sh * p.pitch + (ox * p.sw - p.pw - ix0)) * kPairPosBytes + half * 16;
    }
    // Words behind the buffers: the waves' largest magnitudes of a chunk, by its parity; how many values of even and of odd chunks
    // are held in part; is there an output to be formed again?
    uint32_t *const words = reinterpret_cast<uint32_t *>(lds_raw + 2 * tile_bytes);

    // Staging, granules and the places of values as in split_wave.
    const float *img = p.I + (size_t)n * p.C * HW;
    const int tl = threadIdx.x & 127;
    const int oct = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 7);
    uint32_t voff[kGran];
    int wr_off[kGran];
#pragma unroll
    for (int q = 0; q < kGran; ++q) {
        const int pos = min(q * 128 + tl, p.npos - 1);
        wr_off[q] = pos * kPairPosBytes + oct * 16;
        const uint32_t r = quot((uint32_t)pos, p.inv_pitch);
        const int xw = (int)((uint32_t)pos - r * (uint32_t)p.pitch);
        const int iy = iy0 + (int)r, ix = ix0 + xw;
        const bool ok = (int)r < rows && (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W;
        voff[q] = ok ? (uint32_t)(iy * p.W + ix) * 4u : kOutside;
    }
    float first[kGran][8], nxt[kGran][8];
    // (a channel past the last one reads that one again: its weights are zeros, and its largest magnitude is counted already)
    const auto image = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(img), 0, p.C * HW * 4, kRaw);
    auto prefetch = [&](float (&to)[kGran][8], int ch) __attribute__((always_inline)) {
        const int c0 = ch * kChan + 8 * oct;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int at = min(c0 + k, p.C - 1) * (HW * 4);
#pragma unroll
            for (int q = 0; q < kGran; ++q) to[q][k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(image, (int)voff[q], at, 0));
        }
    };
    // a chunk's largest magnitude, this wave's part, for the scale of its commit
    auto put_top = [&](float (&of)[kGran][8], int ch) __attribute__((always_inline)) {
        float m = 0.f;                           // (propagates NaN)
#pragma unroll
        for (int q = 0; q < kGran; ++q)
#pragma unroll
            for (int k = 0; k < 8; k += 2)
                m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(of[q][k])), fabsf(of[q][k + 1]));
        const uint32_t top = wave_max(__float_as_uint(m) & ~kTinyBit);
        if (lane == 0) words[4 * (ch & 1) + (threadIdx.x >> 6)] = top;
    };
    // The power of two of the chunk to be committed next, of the one being multiplied, the smallest so far; the first as a factor, with and
    // without that of the low terms.
    int xexp = 0, xexp_now = 0, xleast = kPairMost;
    float xscale = 1.f, xscale_low = 1.f;
    uint32_t xlow = 0;                           // below it a (doubled) value is held in part
    auto take_scale = [&](const uint4 &t) __attribute__((always_inline)) -> bool {
        const uint32_t top = __builtin_amdgcn_readfirstlane((int)max(max(t.x, t.y), max(t.z, t.w)));
        bool held;
        xexp = pair_exp(kPairTopX, top, held);
        held = held && top < kInfBits;
        xleast = min(xleast, xexp);
        xscale = __uint_as_float((uint32_t)(127 + xexp) << 23);
        xscale_low = __uint_as_float((uint32_t)(127 + kPairShift + xexp) << 23);
        xlow = (__float_as_uint(kPairLow) - ((uint32_t)xexp << 23)) << 1;
        return held;
    };
    auto tops_of = [&](int ch) __attribute__((always_inline)) { return *reinterpret_cast<const uint4 *>(words + 4 * (ch & 1)); };
    constexpr int kPieces = 2 * kGran + 1, kUnits = 6;
    float pv[4];
    uint32_t ph[2], pu[4], lows = 0;
    auto commit_unit = [&](float (&from)[kGran][8], auto piece_c, auto unit_c, int ch) __attribute__((always_inline)) {
        constexpr int S = decltype(piece_c)::value, U = decltype(unit_c)::value;
        if constexpr (S < 2 * kGran) {
            constexpr int q = S >> 1, hf = S & 1;
            if constexpr (U == 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) pv[k] = from[q][4 * hf + k] * xscale;
            } else if constexpr (U == 1) {       // (0 less one wraps to the top)
#pragma unroll
                for (int k = 0; k < 4; ++k) pu[k] = (__float_as_uint(from[q][4 * hf + k]) << 1) - 1u;
            } else if constexpr (U == 2) {
                lows += min(min(pu[0], pu[1]), min(pu[2], pu[3])) < xlow - 1u;       // (four at most)
                ph[0] = pack_f16(pv[0], pv[1]);
                ph[1] = pack_f16(pv[2], pv[3]);
            } else if constexpr (U == 3) {
#pragma unroll
                for (int k = 0; k < 4; ++k) pv[k] = from[q][4 * hf + k] * xscale_low;
            } else if constexpr (U == 4) {
                leave_pair_f16(pv[0], pv[1], ph[0]);
                leave_pair_f16(pv[2], pv[3], ph[1]);
            } else if constexpr (U == 5) {
                uint2 *dst = reinterpret_cast<uint2 *>(lds_raw + (ch & 1) * tile_bytes + wr_off[q] + hf * 8);
                dst[0] = make_uint2(ph[0], ph[1]);
                dst[4] = make_uint2(pack_f16(pv[0], pv[1]), pack_f16(pv[2], pv[3]));
            }
        } else if constexpr (U == 0) {
            prefetch(nxt, ch + 1);
        }
    };
    auto commit_piece = [&](float (&from)[kGran][8], auto piece_c, int ch) __attribute__((always_inline)) {
        commit_unit(from, piece_c, std::integral_constant<int, 0>{}, ch);
        commit_unit(from, piece_c, std::integral_constant<int, 1>{}, ch);
        commit_unit(from, piece_c, std::integral_constant<int, 2>{}, ch);
        commit_unit(from, piece_c, std::integral_constant<int, 3>{}, ch);
        commit_unit(from, piece_c, std::integral_constant<int, 4>{}, ch);
        commit_unit(from, piece_c, std::integral_constant<int, 5>{}, ch);
    };
    auto commit_rest = [&](float (&of)[kGran][8], int from, int ch) __attribute__((always_inline)) {
        if (from <= 0) commit_piece(of, std::integral_constant<int, 0>{}, ch);
        if (from <= 1) commit_piece(of, std::integral_constant<int, 1>{}, ch);
        if constexpr (kGran > 1) {
            if (from <= 2 && p.npos > 128) commit_piece(of, std::integral_constant<int, 2>{}, ch);
            if (from <= 3 && p.npos > 128) commit_piece(of, std::integral_constant<int, 3>{}, ch);
        }
        if constexpr (kGran > 2) {
            if (from <= 4 && p.npos > 256) commit_piece(of, std::integral_constant<int, 4>{}, ch);
            if (from <= 5 && p.npos > 256) commit_piece(of, std::integral_constant<int, 5>{}, ch);
        }
        static_assert(kGran <= 3, "two lines per granule");
    };

    // The A operands of both filter tiles walk linearly through the workspace: a ring of RING taps, an operand fetched again behind
    // its last use.
    const int ft0 = f0 >> 5, ft1 = min(ft0 + 1, p.ftiles - 1);
    const int per_tile = p.nchunks * taps * kPairOperandBytes;      // (all of them less than 2 GiB)
    const auto operands = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(p.Wp), 0, p.ftiles * per_tile, kRaw);
    int wx = ft0 * per_tile;                     // of the next tap to be fetched (past the last one: that one again, unused)
    const int wx_last = wx + per_tile - kPairOperandBytes, to_second = (ft1 - ft0) * per_tile, lane16 = lane * 16;
    uint4 a[RING][2][2];                         // [tap][filter tile][high, low]
    auto load_a = [&](int slot, int i, int term) __attribute__((always_inline)) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(operands, lane16 + term * 1024, wx + (i ? to_second : 0), 0);
        a[slot][i][term] = make_uint4(v.x, v.y, v.z, v.w);
    };
    auto next_a = [&]() __attribute__((always_inline)) { wx = min(wx + kPairOperandBytes, wx_last); };

    // the powers of two of both filter tiles in 64 chunks, a lane each
    uint32_t wexps = 0;
    auto load_exps = [&](int ch) __attribute__((always_inline)) {
        const int c = min(ch + lane, p.nchunks - 1);
        wexps = (uint32_t)(p.pexp[ft0 * p.nchunks + c] + kExpBias) | (uint32_t)(p.pexp[ft1 * p.nchunks + c] + kExpBias) << 16;
    };

    prefetch(first, 0);
    prefetch(nxt, 1);
    load_exps(0);
    if constexpr (NT > 0) {
#pragma unroll
        for (int slot = 0; slot < RING; ++slot) {
#pragma unroll
            for (int k = 0; k < 4; ++k) load_a(slot, k & 1, 1 - (k >> 1));
            next_a();
        }
    }
    // the workgroup's filters: weights held in part, the smallest power of two
    uint32_t partly = 0;
    int wleast = kPairMost;
    {
        const int fa = fw0 >> 5, fb = min(fa + 2 * p.fwaves, p.ftiles);
        for (int i = fa * 2 * p.nchunks + lane; i < fb * 2 * p.nchunks; i += 64) partly = min(partly + p.plow[i], kNotHeld);
        for (int i = fa * p.nchunks + lane; i < fb * p.nchunks; i += 64) wleast = min(wleast, p.pexp[i]);
        wleast = 512 - (int)wave_max((uint32_t)(512 - wleast));
#pragma unroll
        for (int m = 1; m < 64; m *= 2) partly = min(partly + (uint32_t)__shfl_xor((int)partly, m), kNotHeld);
        partly = __builtin_amdgcn_readfirstlane((int)partly);
    }
    put_top(first, 0);
    if (threadIdx.x < 3) words[8 + threadIdx.x] = 0;
    __syncthreads();
    bool stop = partly >= kPairMostLowW;         // (uniform over the workgroup)
    stop |= !take_scale(tops_of(0));
    xexp_now = xexp;
    commit_rest(first, 0, 0);
    put_top(nxt, 1);
    if (lows) atomicAdd(&words[8], 4 * lows);
    lows = 0;
    __syncthreads();

    static_assert(NT <= 2, "where the operands are scaled");
    floatx16 acc[2][kTiles], chain[2][kTiles];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) { acc[i][j][r] = 0.f; chain[i][j][r] = 0.f; }
    uint32_t counts[2] = {(uint32_t)__builtin_amdgcn_readfirstlane((int)words[8]), 0};
    uint32_t sign = 0;                           // that the current chain's weights are stored with
    for (int ch = 0; ch < p.nchunks && !stop; ++ch) {
        const bool more = ch + 1 < p.nchunks;
        int pc = more ? 0 : kPieces;             // the next piece of chunk ch + 1 to commit
        if constexpr (NT > 0) {
            const unsigned char *tile_r = lds_raw + (ch & 1) * tile_bytes;
            auto read_b = [&](uint4 &to, int term, int byte_off) __attribute__((always_inline)) {
                to = *reinterpret_cast<const uint4 *>(tile_r + byte_off + 32 * term);
            };
            uint4 bh[kTiles], bl[kTiles];        // of the current tap
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                read_b(bh[j], 0, base[j]);
                read_b(bl[j], 1, base[j]);
            }
            if (more) stop |= !take_scale(tops_of(ch + 1));
            if ((ch & 63) == 0 && ch > 0) load_exps(ch);
            const uint32_t exps = (uint32_t)__builtin_amdgcn_readlane((int)wexps, ch & 63);
            const uint32_t e0 = (uint32_t)(127 - kPairShift + kExpBias - xexp_now - (int)(exps & 0xffffu)) << 23, e1 = (uint32_t)(127 - kPairShift + kExpBias - xexp_now - (int)(exps >> 16)) << 23;
            // a chain joins the output's sum, without the scales and the sign of its operands
            auto settle = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const float by = __uint_as_float((i ? e1 : e0) ^ sign);
#pragma unroll
                    for (int j = 0; j < NT; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            acc[i][j][r] = fmaf(by, chain[i][j][r], acc[i][j][r]);
                            chain[i][j][r] = 0.f;
                        }
                }
                sign ^= 0x80000000u;
            };
            const int row_step = (p.pitch - p.kw + 1) * kPairPosBytes;
            int kx = 0, off = 0, left = taps, in_chain = pair_chain_taps(taps);
            // A tap, its operands in slot `slot` of the ring, with pieces FIRST .. FIRST + COUNT - 1 of the commit: high * low, low * high (in
            // the order that leaves the fetches more time: the first first, for B's, or last, for A's in the shorter ring), high * high of all
            // tiles, the high operands scaled for the last behind their other product, no more vector instructions to a unit than issue under a
            // matrix instruction, an operand fetched again behind its last use, the next tap's place found between.  (100 drawn layers 2.2 %
            // faster than with all of an operand's scaling in one unit, commits in five units and the first order alone; with either order for both
            // rings the other one's layers are 2 % slower.)
            constexpr int kHighLow = RING == 2 ? 1 : 0, kLowHigh = 1 - kHighLow;
            auto tap_body = [&](auto slot_c, auto first_c, auto count_c) __attribute__((always_inline)) {
                constexpr int slot = decltype(slot_c)::value, FIRST = decltype(first_c)::value, COUNT = decltype(count_c)::value;
                __builtin_amdgcn_sched_barrier(0);
                auto unit = [&](auto m_c) __attribute__((always_inline)) {
                    constexpr int M = decltype(m_c)::value;
                    if constexpr (M < 6 * NT) {
                        constexpr int P = M / (2 * NT), j = M % (2 * NT) / 2, i = M & 1, ta = P == kLowHigh ? 1 : 0;
                        chain[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a[slot][i][ta]), __builtin_bit_cast(halfx8, P == kHighLow ? bl[j] : bh[j]),
                                                                             chain[i][j], 0, 0, 0);
                        if constexpr (M == 1) {
                            const bool wrap = kx + 1 == p.kw;
                            --left;
                            kx = wrap ? 0 : kx + 1;
                            off = left > 0 ? off + (wrap ? row_step : kPairPosBytes) : 0;
                        }
                        if constexpr (j == NT - 1 && P != kHighLow) load_a(slot, i, ta);
                        if constexpr (i == 1 && P == kHighLow) read_b(bl[j], 1, base[j] + off);
                        if constexpr (i == 1 && P == 2) read_b(bh[j], 0, base[j] + off);
                        // (x, y: the unit behind a high operand's other product; halves in units of their own where those come before its third)
                        constexpr int x = M - (2 * NT * kHighLow + 2 * (NT - 1)), y = M - (2 * NT * kLowHigh + 1);
                        constexpr bool a_halves = 2 * NT * kHighLow + 2 * NT < 4 * NT, b_halves = 2 * NT * kLowHigh + 3 < 4 * NT;
                        if constexpr (x == 0 || x == 1) {
                            scale_f16<kPairUpW, 0>(a[slot][x][0]);
                            if constexpr (!a_halves) scale_f16<kPairUpW, 1>(a[slot][x][0]);
                        }
                        if constexpr (a_halves && (x == 2 || x == 3)) scale_f16<kPairUpW, 1>(a[slot][x - 2][0]);
                        if constexpr (b_halves && y >= 1 && y <= 2 * NT) scale_f16<kPairUpX, (y - 1) & 1>(bh[(y - 1) / 2]);
                        if constexpr (!b_halves && y >= 0 && y % 2 == 0 && y / 2 < NT) {
                            scale_f16<kPairUpX, 0>(bh[y / 2]);
                            scale_f16<kPairUpX, 1>(bh[y / 2]);
                        }
                        constexpr int piece = M / kUnits, u = M % kUnits;
                        if constexpr (piece < COUNT) commit_unit(nxt, std::integral_constant<int, FIRST + piece>{}, std::integral_constant<int, u>{}, ch + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                for_units(unit);
                next_a();
            };
            // RING taps, with the pieces from FIRST on, NT to a tap
            auto body = [&](auto first_c) __attribute__((always_inline)) {
                constexpr int FIRST = decltype(first_c)::value;
                using std::integral_constant;
                tap_body(integral_constant<int, 0>{}, integral_constant<int, FIRST>{}, integral_constant<int, std::max(0, std::min(NT, kPieces - FIRST))>{});
                tap_body(integral_constant<int, 1>{}, integral_constant<int, FIRST + NT>{}, integral_constant<int, std::max(0, std::min(NT, kPieces - FIRST - NT))>{});
                if constexpr (RING == 3)
                    tap_body(integral_constant<int, 2>{}, integral_constant<int, FIRST + 2 * NT>{}, integral_constant<int, std::max(0, std::min(NT, kPieces - FIRST - 2 * NT))>{});
                in_chain -= RING;
                if (in_chain == 0 && left > 0) { settle(); in_chain = pair_chain_taps(taps); }
            };
            constexpr int kPer = RING * NT;
            if (more) {
                if (left >= RING) { body(std::integral_constant<int, 0>{}); pc = std::min(kPer, kPieces); }
                if constexpr (kPer < kPieces) if (left >= RING) { body(std::integral_constant<int, kPer>{}); pc = std::min(2 * kPer, kPieces); }
                if constexpr (2 * kPer < kPieces) if (left >= RING) { body(std::integral_constant<int, 2 * kPer>{}); pc = std::min(3 * kPer, kPieces); }
                if constexpr (3 * kPer < kPieces) if (left >= RING) { body(std::integral_constant<int, 3 * kPer>{}); pc = std::min(4 * kPer, kPieces); }
            }
            while (left >= RING) body(std::integral_constant<int, kPieces>{});
            if constexpr (RING == 2) {
                if (left > 0) {                  // one tap: the ring turns by one
                    tap_body(std::integral_constant<int, 0>{}, std::integral_constant<int, kPieces>{}, std::integral_constant<int, 0>{});
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint4 t = a[0][k >> 1][k & 1];
                        a[0][k >> 1][k & 1] = a[1][k >> 1][k & 1];
                        a[1][k >> 1][k & 1] = t;
                    }
                }
            }
            settle();
        } else {
            if (more) stop |= !take_scale(tops_of(ch + 1));
        }
        if (pc < kPieces) {                      // what the chunk's steps did not carry
            commit_rest(nxt, pc, ch + 1);
            prefetch(nxt, ch + 2);
        }
        xexp_now = xexp;
        if (lows) { atomicAdd(&words[8 + ((ch + 1) & 1)], 4 * lows); lows = 0; }
        if (more) put_top(nxt, ch + 2);
        __syncthreads();                         // chunk ch has been read, chunk ch + 1 is written
        // (written before the barrier, and again only behind the next one)
        counts[(ch + 1) & 1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)words[8 + ((ch + 1) & 1)]);
        stop |= counts[0] + counts[1] >= kPairMostLow;
    }
    // What values held in part can do to an output, times 2^kPairShareExp.
    const uint32_t count = partly + counts[0] + counts[1];
    const float doubtful = (float)count * ldexpf(1.f, kPairShareExp + kPairLossExp + std::max(kPairTopW, kPairTopX) + 1 - xleast - wleast);
    bool again = stop;
    uint32_t few[kTiles];
    int number = 0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        int oy, ox;
        few[j] = 0;
        if (pixel_of(tile0 + j, oy, ox)) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float v = fabsf(acc[i][j][r]);
                    const int f = f0 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (f < p.F) {
                        again |= !(v <= 3.402823466e38f) || (v < kPairLeast && v > 0.f);
                        few[j] |= v < doubtful ? 1u << (16 * i + r) : 0u;
                    }
                }
        }
        number += __builtin_popcount(few[j]);
    }
    if (__any(number != 0)) {
#pragma unroll
        for (int m = 1; m < 64; m *= 2) number += __shfl_xor(number, m);
        again |= number > kPairFew;
    }
    if (__any(again) && lane == 0) words[10] = 1;
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane((int)words[10]) != 0) return false;
    float *dst = p.out + (size_t)n * p.F * OHW;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        int oy, ox;
        if (pixel_of(tile0 + j, oy, ox)) {
            const int px = oy * p.OW + ox;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int f = f0 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (f < p.F) dst[(size_t)f * OHW + px] = acc[i][j][r];
                }
        }
    }
    // (none of them but by chance where values are of one size)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        for (unsigned long long who; (who = __ballot(few[j] != 0)) != 0;) {
            const int l = __builtin_ctzll(who);
            const int bit = __builtin_ctz(__builtin_amdgcn_readlane((int)few[j], l));
            int oy, ox;
            pixel_of(tile0 + j, oy, ox);
            oy = __builtin_amdgcn_readlane(oy, l);
            ox = __builtin_amdgcn_readlane(ox, l);
            const int r = bit & 15, f = f0 + (bit >> 4) * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
            const float *w = p.Wt + (size_t)f * p.C * taps;
            double sum = 0.;                     // (a lane a channel, loads of four channels in flight)
            for (int t = 0; t < taps; ++t) {
                const int ky = t / p.kw, iy = oy * p.sh - p.ph + ky, ix = ox * p.sw - p.pw + t - ky * p.kw;
                if ((unsigned)iy >= (unsigned)p.H || (unsigned)ix >= (unsigned)p.W) continue;
                for (int c = lane; c < p.C; c += 256) {
                    float x[4], y[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int ck = min(c + 64 * k, p.C - 1);
                        x[k] = img[(size_t)ck * HW + iy * p.W + ix];
                        y[k] = w[(size_t)ck * taps + t];
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) sum = fma(c + 64 * k < p.C ? (double)x[k] : 0., (double)y[k], sum);
                }
            }
#pragma unroll
            for (int m = 1; m < 64; m *= 2) sum += __shfl_xor(sum, m);
            if (lane == l) {
                dst[(size_t)f * OHW + oy * p.OW + ox] = (float)sum;
                few[j] &= few[j] - 1;
            }
        }
    }
    return true;
}

// The work of one wave with NT pixel tiles (0: it only takes part in the staging).  X0, Y0: the output
// pixel of the workgroup's first tile (tw > 0); ix0, iy0: the input position of the staged block's corner.
template <int NT, bool FLUSH, int GRAN>
__device__ __attribute__((always_inline)) void split_wave(const Fp32SplitParams &p, int n, int f0, int t0, int X0, int Y0,
                                                          int oy0, int iy0, int ix0, int rows, int tile0)
{
    // LDS: two input buffers, taken in turn by the chunks, each [npos][term][16 channels]
    extern __shared__ unsigned char lds_raw[];
    constexpr int kGran = GRAN, kPosBytes = pos_bytes(FLUSH), kOperandBytes = operand_bytes(FLUSH);
    const int tile_bytes = p.npos * kPosBytes;
    const int lane = threadIdx.x & 63;
    const int col = lane & 31, half = lane >> 5;
    const int OHW = p.OH * p.OW;
    const int taps = p.kh * p.kw;
    const int HW = p.H * p.W;
    const int tw_shift = p.tw ? 31 - __builtin_clz((unsigned)p.tw) : 5;
    auto pixel_of = [&](int j, int &oy, int &ox) -> bool { return tile_pixel(p, t0, X0, Y0, tw_shift, j, col, oy, ox); };
    int base[NT > 0 ? NT : 1];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        int oy, ox;
        pixel_of(tile0 + j, oy, ox);
        base[j] = ((oy - oy0) * p.sh * p.pitch + (ox * p.sw - p.pw - ix0)) * kPosBytes + half * 16;
    }

    floatx16 acc[2][NT > 0 ? NT : 1], sum[2][FLUSH && NT > 0 ? NT : 1], tapsum[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[i][j][r] = 0.f;
                if (FLUSH) sum[i][j][r] = 0.f;
            }
#pragma unroll
    for (int r = 0; r < 16; ++r) tapsum[1][r] = 0.f;
    float sgn = 1.f;                             // FLUSH: of the current chain's weights
    int chain = 2;                               // ... taps until the next flush
    // FLUSH: a chain joins the output's sum, what the addition rounds off starts the next one
    auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float s = fmaf(sgn, acc[i][j][r], sum[i][j][r]);
                    acc[i][j][r] = fmaf(sgn, s - sum[i][j][r], -acc[i][j][r]);
                    sum[i][j][r] = s;
                }
        sgn = -sgn;
    };
    // else: a finished chain joins the output's sum, times what its operands are not scaled by and its sign
    // (a quarter of its registers)
    auto settle = [&](int i, int j, uint32_t factor, int quarter) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 4 * quarter; r < 4 * quarter + 4; ++r) acc[i][j][r] = fmaf(__uint_as_float(factor), tapsum[i][r], acc[i][j][r]);
    };
    // Largest and smallest non-zero magnitude of what is staged, less one (FLUSH: of all, doubled bits; else: of a chunk, scaled)
    uint32_t xtop = 0, xlow = 0xffffffffu;
    float xmax = 0.f;
    int xexp = 0;                                // else: the power of two that the workgroup's input is staged times
    float xscale = 1.f;

    const float *img = p.I + (size_t)n * p.C * HW;

    // Staging.  A granule is eight channels of one staged position: thread t takes the positions
    // q * 128 + t % 128 (q < kGran) of channel octet t / 128, the same for a whole wave, so the address
    // of a value is a scalar base (the channel's plane) plus a lane offset kept in registers.  A
    // position past the last one repeats the last one (the same bytes to the same place), one outside
    // the image loads from past the buffer's end, which gives zero: no branch, and nothing waits for a
    // load before the next is issued.
    const int tl = threadIdx.x & 127;
    const int oct = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 7);
    uint32_t voff[kGran];
    int wr_off[kGran];
#pragma unroll
    for (int q = 0; q < kGran; ++q) {
        const int pos = min(q * 128 + tl, p.npos - 1);
        wr_off[q] = pos * kPosBytes + oct * 16;
        const uint32_t r = quot((uint32_t)pos, p.inv_pitch);
        const int xw = (int)((uint32_t)pos - r * (uint32_t)p.pitch);
        const int iy = iy0 + (int)r, ix = ix0 + xw;
        const bool ok = (int)r < rows && (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W;
        voff[q] = ok ? (uint32_t)(iy * p.W + ix) * 4u : kOutside;
    }
    float nxt[kGran][8];
    auto prefetch = [&](int ch) __attribute__((always_inline)) {
        const int c0 = ch * kChan + 8 * oct;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            // (scalar; a channel past the last one: an empty buffer, every load is 0)
            const int c = min(c0 + k, p.C - 1);
            const auto buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(img + (size_t)c * HW), 0, c0 + k < p.C ? HW * 4 : 0, kRaw);
#pragma unroll
            for (int q = 0; q < kGran; ++q) nxt[q][k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(buf, (int)voff[q], 0, 0));
        }
    };
    // The commit of chunk `ch` into buffer ch % 2 comes in pieces, each laid among the matrix
    // instructions of one step of the chunk before, in units small enough to fit behind one
    // instruction: piece s < 2 * kGran splits and writes one half (four channels) of granule s / 2, the
    // last one issues the loads of chunk ch + 1 into the registers just freed.
    constexpr int kPieces = 2 * kGran + 1;
    float pv[4];
    uint32_t ph[2], pm[2], pl[2], pr[2];
    // Words behind the input buffers.  By the chunks, in turn: FLUSH: has a value been too large?  Else: number + 1 of the last
    // chunk with a value whose mid + lo f16 does not hold (kTinyBit: with one that is not finite); then the largest and the
    // smallest of such values and the waves' largest of the first chunk.
    uint32_t *const words = reinterpret_cast<uint32_t *>(lds_raw + 2 * tile_bytes);
    auto commit_unit = [&](auto piece_c, auto unit_c, int ch) __attribute__((always_inline)) {
        constexpr int S = decltype(piece_c)::value, U = decltype(unit_c)::value;
        if constexpr (S < 2 * kGran) {
            constexpr int q = S >> 1, hf = S & 1;
            if constexpr (U == 0 || U == 3) {
                constexpr int k = U ? 2 : 0;
                pv[k] = nxt[q][4 * hf + k];
                pv[k + 1] = nxt[q][4 * hf + k + 1];
                if constexpr (FLUSH) {
                    const uint32_t a = __float_as_uint(pv[k]) << 1, b = __float_as_uint(pv[k + 1]) << 1;
                    xtop = max(max(xtop, a), b);
                    xlow = min(min(xlow, a - 1u), b - 1u);
                } else {
                    pv[k] *= xscale;
                    pv[k + 1] *= xscale;
                    xmax = __builtin_elementwise_maximum(__builtin_elementwise_maximum(xmax, fabsf(pv[k])), fabsf(pv[k + 1]));   // (keeps NaN)
                    xlow = min(xlow, min((__float_as_uint(pv[k]) << 1) - 1u, (__float_as_uint(pv[k + 1]) << 1) - 1u));
                }
            } else if constexpr (U == 1 || U == 4) {
                constexpr int e = U == 4;
                ph[e] = pack_bf16(pv[2 * e], pv[2 * e + 1]);
                subtract_pair(pv[2 * e], pv[2 * e + 1], ph[e]);
                if constexpr (!FLUSH) pr[e] = pack_f16(pv[2 * e], pv[2 * e + 1]);
            } else if constexpr (U == 2 || U == 5) {
                constexpr int e = U == 5;
                pm[e] = pack_bf16(pv[2 * e], pv[2 * e + 1]);
                subtract_pair(pv[2 * e], pv[2 * e + 1], pm[e]);
                pl[e] = pack_bf16(pv[2 * e], pv[2 * e + 1]);
            } else if constexpr (U == 6) {
                uint2 *dst = reinterpret_cast<uint2 *>(lds_raw + (ch & 1) * tile_bytes + wr_off[q] + hf * 8);
                dst[0] = make_uint2(ph[0], ph[1]);
                dst[4] = make_uint2(pm[0], pm[1]);
                dst[8] = make_uint2(pl[0], pl[1]);
                if constexpr (!FLUSH) dst[12] = make_uint2(pr[0], pr[1]);
            }
        } else if constexpr (U == 0) {
            prefetch(ch + 1);      // (past the last chunk: no channel, every load is 0 without a read)
        }
    };
    auto commit_piece = [&](auto piece_c, int ch) __attribute__((always_inline)) {
        commit_unit(piece_c, std::integral_constant<int, 0>{}, ch);
        commit_unit(piece_c, std::integral_constant<int, 1>{}, ch);
        commit_unit(piece_c, std::integral_constant<int, 2>{}, ch);
        commit_unit(piece_c, std::integral_constant<int, 3>{}, ch);
        commit_unit(piece_c, std::integral_constant<int, 4>{}, ch);
        commit_unit(piece_c, std::integral_constant<int, 5>{}, ch);
        commit_unit(piece_c, std::integral_constant<int, 6>{}, ch);
    };
    // pieces `from` .. kPieces - 1 of chunk ch, one after the other (granules without a position of their own: none)
    auto commit_rest = [&](int from, int ch) __attribute__((always_inline)) {
        if (from <= 0) commit_piece(std::integral_constant<int, 0>{}, ch);
        if (from <= 1) commit_piece(std::integral_constant<int, 1>{}, ch);
        if constexpr (kGran > 1) {
            if (from <= 2 && p.npos > 128) commit_piece(std::integral_constant<int, 2>{}, ch);
            if (from <= 3 && p.npos > 128) commit_piece(std::integral_constant<int, 3>{}, ch);
        }
        if constexpr (kGran > 2) {
            if (from <= 4 && p.npos > 256) commit_piece(std::integral_constant<int, 4>{}, ch);
            if (from <= 5 && p.npos > 256) commit_piece(std::integral_constant<int, 5>{}, ch);
        }
        if constexpr (kGran > 3) {
            if (from <= 6 && p.npos > 384) commit_piece(std::integral_constant<int, 6>{}, ch);
            if (from <= 7 && p.npos > 384) commit_piece(std::integral_constant<int, 7>{}, ch);
        }
        if (from < kPieces) commit_piece(std::integral_constant<int, kPieces - 1>{}, ch);
        static_assert(kPieces <= 9, "one line per piece");
    };

    // The A operands of both filter tiles walk linearly through the workspace, chunk by chunk and tap by tap.
    const int ft0 = f0 >> 5, ft1 = min(ft0 + 1, p.ftiles - 1);
    const size_t per_tile = (size_t)p.nchunks * taps * kOperandBytes;
    const unsigned char *wx0 = p.Wx + ft0 * per_tile, *wx1 = p.Wx + ft1 * per_tile;
    // FLUSH: those of the next tap are loaded at the head of a tap.
    int steps_left = p.nchunks * taps - 1;       // taps still to be fetched
    uint4 fa[FLUSH ? 2 : 1][3], fan[FLUSH ? 2 : 1][3];
    auto load_next = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            fan[0][t] = reinterpret_cast<const uint4 *>(wx0)[t * 64 + lane];
            fan[FLUSH][t] = reinterpret_cast<const uint4 *>(wx1)[t * 64 + lane];
        }
        const int d = steps_left > 0 ? kOperandBytes : 0;          // (the last one is fetched again, unused)
        wx0 += d; wx1 += d; --steps_left;
    };
    // else: a chain's taps at a time, each operand loaded again for the next chain behind its last use, in the
    // order of their uses: twelve matrix instructions or more ahead.
    int taps_left = p.nchunks * taps;            // from the chain on whose operands the pointers stand at
    int second = taps_left > 1 ? kOperandBytes : 0;
    uint4 a[2][2][4];                            // [tap of the chain][filter tile][hi, mid, lo, mid + lo]
    auto load_a = [&](int tap, int i, int term) __attribute__((always_inline)) {
        a[tap][i][term] = reinterpret_cast<const uint4 *>((i ? wx1 : wx0) + (tap ? second : 0))[term * 64 + lane];
    };
    auto next_chain = [&](int n) __attribute__((always_inline)) {   // n taps on (past the last chain: the last tap again, unused)
        const int d = min(n, taps_left - 1);
        wx0 += d * kOperandBytes; wx1 += d * kOperandBytes; taps_left -= d;
        second = taps_left > 1 ? kOperandBytes : 0;
    };
    // What a chain's sum is to be multiplied by, in bits: per filter tile for this chunk and, of the second tile, for the
    // chain that is still to be settled; the sign is that of the current chain's weights, turned at its head.
    uint32_t factor[2] = {0, 0}, pending = 0, sign = 0x80000000u;

    prefetch(0);
    if constexpr (NT > 0) {
        if constexpr (FLUSH) {
            load_next();
        } else {
#pragma unroll
            for (int t = 3; t >= 0; --t)
#pragma unroll
                for (int k = 0; k < 4; ++k) load_a(k >> 1, k & 1, t);
        }
    }
    // else: does what was committed for chunk `ch` have a value that f16 does not hold?
    auto check_held = [&](int ch) __attribute__((always_inline)) {
        if (!(xmax < kHeldTop) || xlow < (__float_as_uint(kHeldLow) << 1) - 1u) {
            atomicMax(&words[ch & 1], ((uint32_t)ch + 1u) | (xmax < INFINITY ? 0u : kTinyBit));
            atomicMax(&words[2], __float_as_uint(xmax));
            atomicMin(&words[3], xlow);
        }
        xmax = 0.f;
        xlow = 0xffffffffu;
    };
    if constexpr (FLUSH) {
        if (threadIdx.x < 2) words[threadIdx.x] = 0;
        __syncthreads();
    } else {
        uint32_t top = 0;
#pragma unroll
        for (int q = 0; q < kGran; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t u = __float_as_uint(nxt[q][k]) & ~kTinyBit;
                top = max(top, u < kInfBits ? u : 0u);
            }
#pragma unroll
        for (int m = 1; m < 64; m *= 2) top = max(top, (uint32_t)__shfl_xor((int)top, m));
        if (threadIdx.x < 4) words[threadIdx.x] = threadIdx.x == 3 ? 0xffffffffu : 0u;
        if (lane == 0) words[4 + (threadIdx.x >> 6)] = top;
        __syncthreads();
        top = __builtin_amdgcn_readfirstlane((int)max(max(words[4], words[5]), max(words[6], words[7])));
        xexp = top == 0 ? kTopX : scale_of(top, kTopX, kMostX);
        xscale = __uint_as_float(power_bits(xexp));
    }
    commit_rest(0, 0);
    if constexpr (FLUSH) {
        if (xtop >= kHuge) words[0] = 1;
    } else {
        check_held(0);
    }
    __syncthreads();
    bool by_plain_sum = false;                 // (uniform over the workgroup)
    int ch = 0;
    int wexp0 = 0, wexp1 = 0;                    // else: the present chunk's words of both filter tiles
    auto one_chunk = [&](auto products_c) __attribute__((always_inline)) {
        // (written before the barrier behind which it is read, and again only behind the next one)
        const uint32_t flag = FLUSH ? words[ch & 1] : words[ch & 1] & kTinyBit;
        const bool more = ch + 1 < p.nchunks;
        int pc = more ? 0 : kPieces;                     // the next piece of chunk ch + 1 to commit
        if constexpr (NT > 0 && FLUSH) {
            // The flat sequence of (tap, pixel tile) steps, sixteen matrix instructions each; a step's
            // three B operands are read one step ahead, and the chunk's first steps carry one piece
            // of the next chunk's commit each.
            const unsigned char *tile_r = lds_raw + (ch & 1) * tile_bytes;
            auto read3 = [&](uint4 (&b)[3], int byte_off) __attribute__((always_inline)) {
                const uint4 *src = reinterpret_cast<const uint4 *>(tile_r + byte_off);
                b[0] = src[0];
                b[1] = src[2];
                b[2] = src[4];
            };
            const int row_step = (p.pitch - p.kw + 1) * kPosBytes;
            int off = 0, kx = 0;                         // byte offset and window column of the current tap
            uint4 bc[3], bn[3];
            read3(bc, base[0]);
            auto step = [&](auto piece_c, int j, int next_off) __attribute__((always_inline)) {
                constexpr int S = decltype(piece_c)::value;
                read3(bn, next_off);
                __builtin_amdgcn_sched_barrier(0);
                auto unit = [&](auto m_c) __attribute__((always_inline)) {
                    // filter tile and product of the M-th instruction: the tiles' chains run side by side, the
                    // first tile's one instruction ahead
                    constexpr int M = decltype(m_c)::value;
                    constexpr int i = M == 0 ? 0 : M == 15 ? 1 : (M & 1) ^ 1, P = M == 0 ? 0 : M == 15 ? 7 : i ? (M >> 1) - 1 : (M + 1) >> 1;
                    // mid*lo, lo*mid, lo*hi, hi*lo, mid*mid, mid*hi, hi*mid, hi*hi
                    constexpr int ta = P == 0 ? 1 : P == 1 ? 2 : P == 2 ? 2 : P == 3 ? 0 : P == 4 ? 1 : P == 5 ? 1 : 0;
                    constexpr int tb = P == 0 ? 2 : P == 1 ? 1 : P == 2 ? 0 : P == 3 ? 2 : P == 4 ? 1 : P == 5 ? 0 : P == 6 ? 1 : 0;
                    const bf16x8 wa = __builtin_bit_cast(bf16x8, fa[i][ta]), xb = __builtin_bit_cast(bf16x8, bc[tb]);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, xb, acc[i][j], 0, 0, 0);
                    if constexpr (S >= 0) commit_unit(piece_c, m_c, ch + 1);
                    __builtin_amdgcn_sched_barrier(0);
                };
                unit(std::integral_constant<int, 0>{});
                unit(std::integral_constant<int, 1>{});
                unit(std::integral_constant<int, 2>{});
                unit(std::integral_constant<int, 3>{});
                unit(std::integral_constant<int, 4>{});
                unit(std::integral_constant<int, 5>{});
                unit(std::integral_constant<int, 6>{});
                unit(std::integral_constant<int, 7>{});
                unit(std::integral_constant<int, 8>{});
                unit(std::integral_constant<int, 9>{});
                unit(std::integral_constant<int, 10>{});
                unit(std::integral_constant<int, 11>{});
                unit(std::integral_constant<int, 12>{});
                unit(std::integral_constant<int, 13>{});
                unit(std::integral_constant<int, 14>{});
                unit(std::integral_constant<int, 15>{});
#pragma unroll
                for (int t = 0; t < 3; ++t) bc[t] = bn[t];
            };
            // one tap: its NT steps, the first of them with piece FIRST of the commit (-1: no pieces)
            auto tap_body = [&](auto first_c, int tap) __attribute__((always_inline)) {
                constexpr int FIRST = decltype(first_c)::value;
#pragma unroll
                for (int t = 0; t < 3; ++t) { fa[0][t] = fan[0][t]; fa[1][t] = fan[1][t]; }
                load_next();
                const bool wrap = kx + 1 == p.kw, further = tap + 1 < taps;
                const int off_n = further ? off + (wrap ? row_step : kPosBytes) : off;
                kx = wrap ? 0 : kx + 1;
                step(std::integral_constant<int, (FIRST >= 0 && FIRST < kPieces) ? FIRST : -1>{}, 0, NT > 1 ? base[NT > 1 ? 1 : 0] + off : base[0] + off_n);
                if constexpr (NT > 1) step(std::integral_constant<int, (FIRST >= 0 && FIRST + 1 < kPieces) ? FIRST + 1 : -1>{}, 1, base[0] + off_n);
                static_assert(NT <= 2, "one line per step");
                off = off_n;
                if (--chain == 0) { flush(); chain = 2; }
            };
            int tap = 0;
            if (more) {
                if (tap < taps) { tap_body(std::integral_constant<int, 0>{}, tap); ++tap; }
                if constexpr (1 * NT < kPieces) if (tap < taps) { tap_body(std::integral_constant<int, 1 * NT>{}, tap); ++tap; }
                if constexpr (2 * NT < kPieces) if (tap < taps) { tap_body(std::integral_constant<int, 2 * NT>{}, tap); ++tap; }
                if constexpr (3 * NT < kPieces) if (tap < taps) { tap_body(std::integral_constant<int, 3 * NT>{}, tap); ++tap; }
                if constexpr (4 * NT < kPieces) if (tap < taps) { tap_body(std::integral_constant<int, 4 * NT>{}, tap); ++tap; }
                if constexpr (5 * NT < kPieces) if (tap < taps) { tap_body(std::integral_constant<int, 5 * NT>{}, tap); ++tap; }
                if constexpr (6 * NT < kPieces) if (tap < taps) { tap_body(std::integral_constant<int, 6 * NT>{}, tap); ++tap; }
                static_assert(kPieces <= 7, "one line per tap that carries pieces");
                pc = min(tap * NT, kPieces);
            }
            for (; tap < taps; ++tap) tap_body(std::integral_constant<int, -1>{}, tap);
        } else if constexpr (NT > 0) {
            // The sequence of (chain, pixel tile) steps, twelve or sixteen matrix instructions a tap; a step's B operands
            // are read during the step before, each behind the last use of its register, and the chunk's first
            // steps carry the pieces of the next chunk's commit.
            factor[0] = power_bits(kExpBias - xexp - (wexp0 & ~kUnheld));
            factor[1] = power_bits(kExpBias - xexp - (wexp1 & ~kUnheld));
            const unsigned char *tile_r = lds_raw + (ch & 1) * tile_bytes;
            auto read_b = [&](uint4 &to, int term, int byte_off) __attribute__((always_inline)) {
                to = *reinterpret_cast<const uint4 *>(tile_r + byte_off + 32 * term);
            };
            const int row_step = (p.pitch - p.kw + 1) * kPosBytes;
            int kx = 0;                                  // window column of the last tap that has an offset
            int off[2], off_n[2];                        // byte offsets of the chain's taps and of the next one's
            auto next_tap = [&](int o) -> int {
                const bool wrap = kx + 1 == p.kw;
                kx = wrap ? 0 : kx + 1;
                return o + (wrap ? row_step : kPosBytes);
            };
            off[0] = 0;
            off[1] = taps > 1 ? next_tap(0) : 0;
            uint4 b[2][4];                               // [tap of the chain][hi, mid, lo, mid + lo]
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int k = 3; k >= 0; --k) read_b(b[t][k], k, base[0] + off[t]);
            // TAPS taps of tile j, with pieces FIRST .. FIRST + COUNT - 1 of the commit; `to` the next step's tile
            auto step = [&](auto taps_c, auto first_c, auto count_c, auto j_c, int to0, int to1) __attribute__((always_inline)) {
                constexpr int TAPS = decltype(taps_c)::value, FIRST = decltype(first_c)::value, COUNT = decltype(count_c)::value;
                constexpr int j = decltype(j_c)::value;
                __builtin_amdgcn_sched_barrier(0);
                auto unit = [&](auto m_c) __attribute__((always_inline)) {
                    // filter tile, product and tap of the M-th instruction: one tile's chain after the other's, so that
                    // a chain's sum is settled under the instructions of the next one, four values to each
                    constexpr int M = decltype(m_c)::value, PRODUCTS = decltype(products_c)::value, LEN = PRODUCTS * TAPS;
                    if constexpr (M < 2 * LEN) {
                        constexpr int i = M / LEN, at = M % LEN, P = at / TAPS, tap = at % TAPS;
                        constexpr Order<PRODUCTS> O{};
                        constexpr int ta = O.a[P], tb = O.b[P];
                        const floatx16 none = {};
                        if constexpr (ta == 3) {
                            tapsum[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a[tap][i][ta]), __builtin_bit_cast(halfx8, b[tap][tb]),
                                                                               at == 0 ? none : tapsum[i], 0, 0, 0);
                        } else {
                            tapsum[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[tap][i][ta]), __builtin_bit_cast(bf16x8, b[tap][tb]),
                                                                                at == 0 ? none : tapsum[i], 0, 0, 0);
                        }
                        if constexpr (at > 0 && at < 5) {
                            if constexpr (i == 0) settle(1, j > 0 ? j - 1 : NT - 1, pending, at - 1);   // (of the step before)
                            else settle(0, j, factor[0] ^ sign, at - 1);
                        }
                        if constexpr (M == 2 * LEN - 1) pending = factor[1] ^ sign;
                        if constexpr (j == NT - 1 && O.load_a[P] >= 0) {
                            load_a(tap, i, O.load_a[P]);
                            if constexpr (TAPS == 1) load_a(1, i, O.load_a[P]);
                        }
                        if constexpr (i == 1 && O.read_b[P] >= 0) {
                            constexpr int term = O.read_b[P];
                            read_b(b[tap][term], term, tap ? to1 : to0);
                            if constexpr (TAPS == 1) read_b(b[1][term], term, to1);
                        }
                        // (behind the instructions without such values)
                        constexpr int piece = TAPS == 2 ? i : 0, unit = TAPS == 2 ? at - 5 : M - 5;
                        if constexpr (unit >= 0 && piece < COUNT) commit_unit(std::integral_constant<int, FIRST + piece>{}, std::integral_constant<int, unit>{}, ch + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                for_units(unit);
            };
            // one chain of TAPS taps: its NT steps, with up to PER pieces of the commit each from FIRST on
            constexpr int kPer = 2;                      // (a step has room for two)
            int left = taps;                             // taps from this chain on
            auto chain_body = [&](auto taps_c, auto first_c, auto per_c) __attribute__((always_inline)) {
                constexpr int TAPS = decltype(taps_c)::value, FIRST = decltype(first_c)::value, PER = decltype(per_c)::value;
                constexpr int C0 = std::max(0, std::min(PER, kPieces - FIRST)), C1 = std::max(0, std::min(PER, kPieces - FIRST - PER));
                next_chain(TAPS);
                sign ^= 0x80000000u;
                left -= TAPS;
                // (past the last tap: any staged position, read and not used)
                off_n[0] = left > 0 ? next_tap(off[TAPS - 1]) : 0;
                off_n[1] = left > 1 ? next_tap(off_n[0]) : off_n[0];
                using std::integral_constant;
                if constexpr (NT == 1) {
                    step(taps_c, first_c, integral_constant<int, C0>{}, integral_constant<int, 0>{}, base[0] + off_n[0], base[0] + off_n[1]);
                } else {
                    constexpr int J = NT - 1;
                    step(taps_c, first_c, integral_constant<int, C0>{}, integral_constant<int, 0>{}, base[J] + off[0], base[J] + off[TAPS - 1]);
                    step(taps_c, integral_constant<int, FIRST + C0>{}, integral_constant<int, C1>{}, integral_constant<int, J>{}, base[0] + off_n[0], base[0] + off_n[1]);
                }
                static_assert(NT <= 2, "one line per step");
                off[0] = off_n[0];
                off[1] = off_n[1];
            };
            constexpr std::integral_constant<int, 1> one{};
            constexpr std::integral_constant<int, 2> two{};
            constexpr std::integral_constant<int, kPieces> none_left{};
            constexpr std::integral_constant<int, kPer> per{};
            if (more) {
                constexpr int kA = kPer * NT, kB = 2 * kA, kC = 3 * kA;
                if (left > 1) { chain_body(two, std::integral_constant<int, 0>{}, per); pc = std::min(kA, kPieces); }
                if (left > 1) { chain_body(two, std::integral_constant<int, kA>{}, per); pc = std::min(kB, kPieces); }
                if constexpr (kB < kPieces) if (left > 1) { chain_body(two, std::integral_constant<int, kB>{}, per); pc = std::min(kC, kPieces); }
                if constexpr (kC < kPieces) if (left > 1) { chain_body(two, std::integral_constant<int, kC>{}, per); pc = std::min(4 * kA, kPieces); }
                if (taps == 1) { chain_body(one, std::integral_constant<int, 0>{}, one); pc = NT; }
            }
            while (left > 1) chain_body(two, none_left, per);
            if (left > 0) chain_body(one, none_left, per);
        }
        if (pc < kPieces) commit_rest(pc, ch + 1);       // what the chunk's steps did not carry
        if constexpr (FLUSH) {
            if (more && xtop >= kHuge) words[(ch + 1) & 1] = 1;
        } else {
            if (more) check_held(ch + 1);
        }
        __syncthreads();                                 // chunk ch has been read, chunk ch + 1 is written
        by_plain_sum = __builtin_amdgcn_readfirstlane((int)flag) != 0;
        ++ch;
    };
    if constexpr (FLUSH || NT == 0) {
        while (ch < p.nchunks && !by_plain_sum) one_chunk(std::integral_constant<int, 8>{});
    } else {
        // six products up to the first chunk with a value that f16 does not hold, eight from there on
        // (scalar loads: vector loads at the head of a chunk wait for all loads before them)
        typedef const __attribute__((address_space(4))) int *Words;
        const Words w0 = (Words)(uintptr_t)(p.wexp + ft0 * p.nchunks), w1 = (Words)(uintptr_t)(p.wexp + ft1 * p.nchunks);
        auto take_exps = [&]() __attribute__((always_inline)) {
            wexp0 = w0[ch];
            wexp1 = w1[ch];
        };
        auto held = [&]() __attribute__((always_inline)) -> bool {
            take_exps();
            return ((wexp0 | wexp1) & kUnheld) == 0 && (__builtin_amdgcn_readfirstlane((int)words[ch & 1]) & 0x7fffffff) != ch + 1;
        };
        while (ch < p.nchunks && !by_plain_sum && held()) one_chunk(std::integral_constant<int, 6>{});
        while (ch < p.nchunks && !by_plain_sum) {
            take_exps();
            one_chunk(std::integral_constant<int, 8>{});
        }
    }

    if constexpr (NT > 0 && !FLUSH) {
#pragma unroll
        for (int k = 0; k < 4; ++k) settle(1, NT - 1, pending, k);
    }

    // Below which magnitude an output is doubtful.
    // A (scaled) value of 2^-110 and above is held in full; of a smaller one up to 2^-134 is lost.  The losses add up
    // to at most 2^-134 * Nred * (max |x| + max |w|), and an output of 2^30 times that is not touched by them.
    if constexpr (FLUSH) {
        uint32_t *const wgstat = reinterpret_cast<uint32_t *>(lds_raw);    // (nothing staged is used past the last barrier)
#pragma unroll
        for (int s = 1; s < 64; s *= 2) {
            xtop = max(xtop, (uint32_t)__shfl_xor((int)xtop, s));
            xlow = min(xlow, (uint32_t)__shfl_xor((int)xlow, s));
        }
        if (lane == 0) { wgstat[2 * (threadIdx.x >> 6)] = xtop; wgstat[2 * (threadIdx.x >> 6) + 1] = xlow; }
        __syncthreads();
        if constexpr (NT == 0) return;
        xtop = max(max(wgstat[0], wgstat[2]), max(wgstat[4], wgstat[6]));
        xlow = min(min(wgstat[1], wgstat[3]), min(wgstat[5], wgstat[7]));
    }
    if constexpr (NT == 0) return;
    uint32_t wtop = 0, wtiny = 0;
    for (int i = lane; i < 2 * p.nchunks; i += 64) {
        const uint32_t s0 = p.wstat[ft0 * 2 * p.nchunks + i], s1 = p.wstat[ft1 * 2 * p.nchunks + i];
        wtop = max(wtop, max(s0 & ~kTinyBit, s1 & ~kTinyBit));
        wtiny |= s0 | s1;
    }
    const bool wlost = __any((wtiny & kTinyBit) != 0);
    if constexpr (!FLUSH) {
        xmax = fmaxf(kHeldTop, __uint_as_float(words[2]));         // (read behind the last barrier)
        xlow = words[3];
    }
    const bool xlost = xlow < (__float_as_uint(kTiny) << 1) - 1u;
    float doubtful = 0.f;
    if (xlost || wlost) {
#pragma unroll
        for (int s = 1; s < 64; s *= 2) wtop = max(wtop, (uint32_t)__shfl_xor((int)wtop, s));
        const float w = __uint_as_float(wtop), nred = (float)(p.C * taps);
        if constexpr (FLUSH) {
            doubtful = kDoubt * nred * (__uint_as_float(xtop >> 1) + w);
        } else {
            // (unscaled: what weights lose counts by the largest power that a chunk of the filter tiles is divided by)
            const float by_x = xlost ? w : 0.f, by_w = wlost ? xmax * fmaxf(w * 0x1p-23f, ldexpf(1.f, -kMostW)) : 0.f;
            doubtful = ldexpf(kDoubt * nred * (by_x + by_w), -xexp);
        }
    }

    // accumulator register r of a lane: filter row 8*(r/4) + 4*half + r%4 of the filter tile,
    // pixel column `col`
    float *dst = p.out + (size_t)n * p.F * OHW;
    uint32_t again[NT > 0 ? NT : 1], any = 0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        again[j] = 0;
        int oy, ox;
        if (pixel_of(tile0 + j, oy, ox)) {
            const int px = oy * p.OW + ox;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int f = f0 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                    const float v = FLUSH ? fmaf(sgn, acc[i][j][r], sum[i][j][r]) : acc[i][j][r];
                    if (f < p.F) {
                        if (!by_plain_sum) dst[(size_t)f * OHW + px] = v;
                        if (by_plain_sum || !(fabsf(v) >= doubtful && fabsf(v) <= 3.402823466e38f)) again[j] |= 1u << (16 * i + r);
                    }
                }
        }
        any |= again[j];
    }
    if constexpr (NT > 0) {
        if (!__any(any != 0)) return;
        plain_tiles<NT, FLUSH>(p, n, f0, [&](int j, int &oy, int &ox) { pixel_of(tile0 + j, oy, ox); },
                        [&](int i, int j, int r, float v) __attribute__((always_inline)) {
                            int oy, ox;
                            pixel_of(tile0 + j, oy, ox);
                            const int f = f0 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                            if ((again[j] >> (16 * i + r)) & 1u) dst[(size_t)f * OHW + oy * p.OW + ox] = v;
                        });
    }
}

// RING: of the form with pairs, 0 for the others
template <bool FLUSH, int GRAN, int RING>
__global__ __launch_bounds__(kThreads, 2) void conv_fp32_split_kernel(Fp32SplitParams p)
{
    int b = blockIdx.x;
    const int h = b % p.fgroups; b /= p.fgroups;
    const int g = b % p.groups;
    const int n = b / p.groups;
    const int OHW = p.OH * p.OW;
    int nt, t0 = 0, X0 = 0, Y0 = 0, oy0, oy1, ix0;
    if (p.tw == 0) {
        const int total = (OHW + 31) >> 5;
        t0 = g * p.tiles;
        const int t1 = min(total, t0 + p.tiles);
        nt = t1 - t0;
        oy0 = (t0 * 32) / p.OW;
        oy1 = (min(OHW, t1 * 32) - 1) / p.OW;
        ix0 = -p.pw;
    } else {
        const int gy = g / p.gx;
        X0 = (g - gy * p.gx) * p.tx * p.tw;
        Y0 = gy * p.ty * (32 / p.tw);
        const int rows_left = p.OH - Y0;                 // (tile rows below the image: none; columns beyond it stay)
        nt = p.tx * min(p.ty, (rows_left * p.tw + 31) / 32);
        oy0 = Y0;
        oy1 = min(p.OH, Y0 + p.ty * (32 / p.tw)) - 1;
        ix0 = X0 * p.sw - p.pw;
    }
    const int rows = (oy1 - oy0) * p.sh + p.kh;
    const int iy0 = oy0 * p.sh - p.ph;
    // wave -> (filter half, pixel group); the tiles are shared out evenly over the pixel groups
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wf = p.fwaves == 2 ? wave & 1 : 0, wp = p.fwaves == 2 ? wave >> 1 : wave;
    const int wps = 4 / p.fwaves;
    const int tile0 = wp * nt / wps;
    int my_nt = (wp + 1) * nt / wps - tile0;
    const int f0 = (h * p.fwaves + wf) * 64;
    if (f0 >= p.F) my_nt = 0;                             // no filters for this wave: staging only
    if constexpr (RING > 0) {
        const int fw0 = h * p.fwaves * 64;
        bool done;
        switch (my_nt) {
            case 0: done = pair_wave<0, GRAN, RING>(p, n, 0, fw0, t0, X0, Y0, oy0, iy0, ix0, rows, tile0); break;
            case 1: done = pair_wave<1, GRAN, RING>(p, n, f0, fw0, t0, X0, Y0, oy0, iy0, ix0, rows, tile0); break;
            default: done = pair_wave<2, GRAN, RING>(p, n, f0, fw0, t0, X0, Y0, oy0, iy0, ix0, rows, tile0); break;
        }
        if (done) return;
    }
    switch (my_nt) {
        case 0: split_wave<0, FLUSH, GRAN>(p, n, 0, t0, X0, Y0, oy0, iy0, ix0, rows, tile0); break;
        case 1: split_wave<1, FLUSH, GRAN>(p, n, f0, t0, X0, Y0, oy0, iy0, ix0, rows, tile0); break;
        default: split_wave<2, FLUSH, GRAN>(p, n, f0, t0, X0, Y0, oy0, iy0, ix0, rows, tile0); break;
    }
}

constexpr int word_bytes(bool flush) { return (flush ? 2 : 8) * (int)sizeof(uint32_t); }

struct Plan {
    bool ok, flush;
    int granules;
    int fwaves, tiles, tw, tx, ty, gx, groups, pitch, npos;
    size_t lds;
};

// How an image is cut into workgroups: 32 consecutive pixels per tile (no idle pixel slot but in an
// image's last tile; the whole width of every row under them is staged), or two-dimensional tiles of
// tw x 32 / tw pixels in blocks of tx x ty (only the block's own columns are staged: wide rows, large
// windows).  A workgroup's time is that of its busiest wave plus half a tile time of staging and
// epilogue, a tenth less where two workgroups fit a compute unit; a launch takes as many of those as
// its busiest compute unit has workgroups, or, over more than four rounds, as many as a compute unit has
// on average and half of one.  The cheapest that fits max_pos() positions is taken.
Plan search_plan(const Geom &g, int granules)
{
    Plan pl{};
    pl.granules = granules;
    const int taps = g.kh * g.kw;
    const long long OHW = (long long)g.OH * g.OW;
    if (taps > kMaxTaps || OHW > (1 << 24) || (long long)g.C * g.H * g.W >= (1LL << 29)) return pl;
    if ((long long)g.F * g.C * taps >= (1LL << 28)) return pl;      // (32-bit sizes; 2 GiB of split filters where C and F are whole tiles)
    // (the fp32 matrix kernel's chains are as long as this one's; what it does not take runs one thread
    //  per output otherwise)
    pl.flush = !conv_fp32_mfma_supports(g);
    pl.fwaves = g.F <= 64 ? 1 : 2;
    const int wps = 4 / pl.fwaves, most = wps * kWaveTiles;
    const long long maxpos = max_pos(granules);
    const long long fgroups = ceil_div(g.F, 64 * pl.fwaves);
    const int cus = kPlanUnits;
    double best = -1.0;
    // `last`: the tiles of the short workgroups, one in every `period`
    auto consider = [&](int tiles, int last, long long period, long long groups, long long rows, long long cols, int tw, int tx,
                        int ty, int gx) {
        const long long npos = rows * cols;
        if (npos > maxpos || groups > (1 << 24)) return;
        const size_t lds = 2 * (size_t)npos * pos_bytes(pl.flush) + word_bytes(pl.flush);
        const long long wgs = (long long)g.N * fgroups * groups;
        const double whole = ceil_div(tiles, wps) + 0.5, part = ceil_div(last, wps) + 0.5;
        const double mean = whole + (part - whole) / (double)period;
        const double time = wgs <= 4LL * cus ? (double)((wgs + cus - 1) / cus) * whole : (double)wgs / cus * mean + 0.5 * whole;
        const double cost = time * (lds <= kLdsShared ? 0.9 : 1.0) * (1.0 + 1e-3 * (double)npos / maxpos);
        if (best >= 0.0 && cost >= best) return;
        best = cost;
        pl.ok = true; pl.tiles = tiles; pl.tw = tw; pl.tx = tx; pl.ty = ty; pl.gx = gx; pl.groups = (int)groups;
        pl.pitch = (int)cols; pl.npos = (int)npos; pl.lds = lds;
    };
    const int total = (int)((OHW + 31) / 32);
    for (int T = std::min(most, total); T >= 1; --T) {
        const int orows = (int)std::min<long long>(g.OH, (32LL * T + g.OW - 2) / g.OW + 1);
        const int groups = ceil_div(total, T);
        consider(T, total - (groups - 1) * T, groups, groups, (long long)(orows - 1) * g.sh + g.kh, (long long)g.W + 2 * g.pw, 0, 1, 1, 1);
    }
    for (int tw = 32; tw >= 4; tw /= 2) {
        const int th = 32 / tw;
        if (tw > 4 && tw >= 2 * g.OW) continue;
        for (int tx = 1; tx <= std::min(most, ceil_div(g.OW, tw)); ++tx)
            for (int ty = 1; tx * ty <= most && ty <= ceil_div(g.OH, th); ++ty) {
                const int ow = std::min(tx * tw, g.OW), oh = std::min(ty * th, g.OH);
                const int gy = ceil_div(g.OH, ty * th), last = ceil_div(g.OH - (gy - 1) * ty * th, th);
                consider(tx * ty, tx * last, gy, (long long)ceil_div(g.OW, tx * tw) * gy,
                         (long long)(oh - 1) * g.sh + g.kh, (long long)(ow - 1) * g.sw + g.kw, tw, tx, ty, ceil_div(g.OW, tx * tw));
            }
    }
    return pl;
}

const Plan &make_plan(const Geom &g)
{
    static thread_local PlanMemo<Plan> memo;
    return memo.get(g, 0, [&] {
        const Plan pl = search_plan(g, kGranules);
        return pl.ok || pl.flush ? pl : search_plan(g, kMostGranules);
    });
}

template <bool FLUSH, int GRAN, int RING>
hipError_t launch_form(const Fp32SplitParams &p, unsigned blocks, size_t lds, hipStream_t st)
{
    if (lds > 64 * 1024) {
        // raise the kernel's dynamic-LDS limit once per device
        static std::atomic<unsigned long long> raised{0};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return hipGetLastError();
        const unsigned long long bit = 1ull << (dev & 63);
        if (!(raised.load() & bit)) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_fp32_split_kernel<FLUSH, GRAN, RING>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     2 * max_pos(GRAN) * pos_bytes(FLUSH) + word_bytes(FLUSH));
            if (e != hipSuccess) return e;
            raised.fetch_or(bit);
        }
    }
    conv_fp32_split_kernel<FLUSH, GRAN, RING><<<dim3(blocks), dim3(kThreads), lds, st>>>(p);
    return hipGetLastError();
}

// With three granules a thread whatever the positions, a launch loads and commits the last position again and again, and a
// chunk's head waited for all its loads where the powers of two came by vector loads.  Six products, us before and after both:
// 32 x 512 x 14 x 14 F=512 1x1 71 / 62, 36 x 224 x 19 x 19 F=64 3x3 58.6 / 55.0, 16 x 128 x 56 x 56 F=128 7x7 (short chains) 585 both.
template <bool FLUSH, int RING>
hipError_t launch_granules(int granules, const Fp32SplitParams &p, unsigned blocks, size_t lds, hipStream_t st)
{
    static_assert(kGranules == 3, "one line per number of granules");
    if (granules == 1) return launch_form<FLUSH, 1, RING>(p, blocks, lds, st);
    if constexpr (!FLUSH)                        // (with short chains 63 registers of it are spilled)
        if (granules == 2) return launch_form<FLUSH, 2, RING>(p, blocks, lds, st);
    return launch_form<FLUSH, 3, RING>(p, blocks, lds, st);
}

}  // namespace

namespace {
// Layers whose sums are long enough that pairs are no less exact than six products: 160 (tap, chunk of 16 channels) steps.  The
// errors are equal at 144 (3 x 3 on 256 channels 1.67e-7 both, 5 x 5 on 96 1.68e-7 against 1.63e-7); from there on 0.94 to 0.98 (3 x 3
// on 273 1.71e-7 against 1.81e-7, on 288 1.70e-7 against 1.77e-7, 5 x 5 on 97 1.75e-7 against 1.86e-7, on 112 1.72e-7 against 1.76e-7,
// 2 x 2 on 640 1.63e-7 against 1.68e-7); below, six products, at 1.1 to 1.3 times the time of pairs.
bool takes_pairs(const Geom &g, const Plan &pl)
{
    const long long taps = g.kh * g.kw, nchunks = ceil_div(g.C, kChan);
    return pl.ok && !pl.flush && pl.granules == kGranules && taps >= 4 && taps * nchunks >= 160 &&
           ceil_div(g.F, 32) * nchunks * taps * kPairOperandBytes < (1LL << 31);     // (32-bit offsets)
}

// The workspace: split filters, their words, their powers of two; of layers that take them the pairs, their powers and words.
struct Layout {
    size_t wstat, wexp, bytes, pairs, pexp, plow, pair_bytes;
};
Layout layout_of(const Geom &g, bool flush)
{
    const size_t nchunks = ceil_div(g.C, kChan), ftiles = ceil_div(g.F, 32);
    Layout l{};
    l.wstat = ftiles * nchunks * g.kh * g.kw * operand_bytes(flush);
    l.wexp = l.wstat + ftiles * nchunks * 2 * sizeof(uint32_t);
    l.bytes = l.wexp + (flush ? 0 : ftiles * nchunks * sizeof(int));
    l.pairs = (l.bytes + 255) / 256 * 256;
    l.pexp = l.pairs + ftiles * nchunks * g.kh * g.kw * kPairOperandBytes;
    l.plow = l.pexp + ftiles * nchunks * sizeof(int);
    l.pair_bytes = l.plow + ftiles * nchunks * 2 * sizeof(uint32_t);
    return l;
}
}  // namespace

size_t conv_fp32_split_workspace_bytes(const Geom &g)
{
    const Plan &pl = make_plan(g);
    return pl.ok ? layout_of(g, pl.flush).bytes : 0;
}

size_t conv_fp32_pairs_workspace_bytes(const Geom &g)
{
    const Plan &pl = make_plan(g);
    return takes_pairs(g, pl) ? layout_of(g, false).pair_bytes : 0;
}

hipError_t launch_conv_fp32_split(const float *I, const float *Wt, const Geom &g, float *out, void *workspace, size_t workspace_bytes,
                                  hipStream_t st)
{
    const Plan &pl = make_plan(g);
    if (!pl.ok) return hipErrorInvalidValue;
    const int taps = g.kh * g.kw;
    const Layout l = layout_of(g, pl.flush);
    unsigned char *const ws = static_cast<unsigned char *>(workspace);
    Fp32SplitParams p;
    p.I = I; p.Wt = Wt; p.Wx = ws; p.out = out;
    p.wstat = reinterpret_cast<const uint32_t *>(ws + l.wstat);
    p.wexp = reinterpret_cast<const int *>(ws + l.wexp);
    const bool pairs = takes_pairs(g, pl) && workspace_bytes >= l.pair_bytes;
    p.Wp = ws + l.pairs;
    p.pexp = reinterpret_cast<const int *>(ws + l.pexp);
    p.plow = reinterpret_cast<const uint32_t *>(ws + l.plow);
    p.N = g.N; p.C = g.C; p.H = g.H; p.W = g.W; p.F = g.F; p.kh = g.kh; p.kw = g.kw;
    p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw; p.OH = g.OH; p.OW = g.OW;
    p.nchunks = ceil_div(g.C, kChan); p.ftiles = ceil_div(g.F, 32);
    p.fwaves = pl.fwaves; p.fgroups = ceil_div(g.F, 64 * pl.fwaves); p.groups = pl.groups;
    p.tiles = pl.tiles; p.tw = pl.tw; p.tx = pl.tx; p.ty = pl.ty; p.gx = pl.gx;
    p.pitch = pl.pitch; p.npos = pl.npos;
    p.inv_pitch = reciprocal((unsigned long long)pl.pitch);
    const long long blocks = (long long)g.N * p.groups * p.fgroups;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t filter_lds = (size_t)32 * ((8 * taps) | 1) * sizeof(float);
    const auto split = pl.flush ? split_filters_kernel<true, false> : pairs ? split_filters_kernel<false, true> : split_filters_kernel<false, false>;
    split<<<dim3((unsigned)(p.ftiles * 2 * p.nchunks)), dim3(kThreads), filter_lds, st>>>(Wt, g.F, g.C, taps, p.nchunks, p.ftiles,
                                                                                          reciprocal(8ull * taps), ws, ws + l.pairs);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const unsigned b = (unsigned)blocks;
    const int granules = ceil_div(pl.npos, 128);
    if (pl.flush) return launch_granules<true, 0>(granules, p, b, pl.lds, st);
    if (!pairs) return granules > kGranules ? launch_form<false, kMostGranules, 0>(p, b, pl.lds, st) : launch_granules<false, 0>(granules, p, b, pl.lds, st);
    return taps % 3 == 0 ? launch_granules<false, 3>(granules, p, b, pl.lds, st) : launch_granules<false, 2>(granules, p, b, pl.lds, st);
}

}  // namespace xnor
