// HBM-streaming stages of the binary-convolution pipeline (Sec. III-A step list):
//   step 1a  sign-binarise + channel bit-pack          (Eq. 3 / Eq. 8)
//   step 2a  channel mean of |I| and its box filter K  (Eq. 10)
//            per-filter alpha = mean |W|               (Eq. 5)
// All three read fp32 once and write far less than they read, so each is laid out for coalesced
// 256-byte wavefront reads along the image's fastest axis with many loads in flight per lane.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "xnor_internal.hpp"

namespace xnor {

// Blocks go round the eight XCDs by their index, but neighbouring blocks share cache lines (a block's run of
// a channel plane starts and ends anywhere), and each XCD has an L2 of its own: XCD x takes the x-th eighth
// of the blocks.  A launch has 8 * ceil(blocks / 8) of them; a surplus one has nothing to do.  (Input pass:
// 128 x 512 x 28 x 28 39.5 -> 36.3 us, 100 x 512 x 27 x 29 40.4 -> 32.8, 128 x 384 x 13 x 13 12.6 -> 10.5.)
__device__ inline long long xcd_block(long long launched, long long blocks)
{
    const long long eighth = (blocks + 7) >> 3;
    return (launched & 7) * eighth + (launched >> 3);
}
static long long xcd_blocks(long long blocks) { return (blocks + 7) / 8 * 8; }

// ------------------------------------------------------------------------------------------------
// Step 1a.  One lane owns one pixel and builds WPT packed words from 32*WPT channel planes; the 64
// lanes of a wave read 64 consecutive pixels of one plane (256 contiguous bytes) per load.
// The paper sets bits one by one in a register per spatial tile (Alg. 1); packing along channels
// instead gives every bit of every word a use in the convolution.
// ------------------------------------------------------------------------------------------------
template <int WPT>
__global__ __launch_bounds__(256) void binarize_pack_kernel(const float *__restrict__ x,
                                                            long long NP, int C, int HW, int Cw, int groups, int full,
                                                            uint32_t *__restrict__ packed)
{
    // A pixel block's groups of words one after the other on the same XCD: its L2 puts their words together to whole
    // cache lines.  (With a group's blocks side by side instead, words of other XCDs between them, 49 x 396 x 32 x 32
    // took 20.9 us, 12.5 so, 85 x 326 x 23 x 23 16.4 / 11.3, 128 x 512 x 28 x 28 43.4 / 37.4.)
    // `full` < groups: the last group has few channels.  Its blocks come behind the others of their XCD, where they fill up
    // the launch's end (94 x 34 x 60 x 60: 10.4 us one after the other, 7.8 so; 22 x 161 x 46 x 46 5.5 / 5.1).
    const uint32_t blocks = (uint32_t)((NP + 255) / 256), eighth = (blocks + 7) >> 3;   // (blocks * groups below 2^31)
    uint32_t b = (uint32_t)xcd_block(blockIdx.x, (long long)blocks * groups), first = 0;
    bool behind = false;
    if (full < groups) {
        b = blockIdx.x >> 3;
        first = (blockIdx.x & 7) * eighth;
        behind = b >= eighth * (uint32_t)full;
    }
    const uint32_t q = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b / (uint32_t)full));   // (a quotient is a vector register otherwise)
    const uint32_t block = first + (behind ? b - eighth * (uint32_t)full : q);
    const int w0 = (int)(behind ? (uint32_t)full : b - q * (uint32_t)full) * WPT;
    const long long p = (long long)block * 256 + threadIdx.x;
    if (p >= NP) return;
    const long long n = p / HW;
    const int hw = (int)(p - n * HW);
    const float *src = x + (n * C) * (long long)HW + hw;

    uint32_t words[WPT];
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
        const int cbase = 32 * (w0 + k);
        uint32_t word = 0;
        if (cbase + 32 <= C) {
            float v[32];
#pragma unroll
            for (int j = 0; j < 32; ++j) v[j] = __builtin_nontemporal_load(src + (long long)(cbase + j) * HW);
#pragma unroll
            for (int j = 0; j < 32; ++j) word |= (v[j] >= 0.0f ? 1u : 0u) << j;
        } else {
            for (int j = 0; j < 32 && cbase + j < C; ++j)
                word |= (src[(long long)(cbase + j) * HW] >= 0.0f ? 1u : 0u) << j;
        }
        words[k] = word;
    }
    uint32_t *dst = packed + p * Cw + w0;
    if (WPT == 4 && (Cw & 3) == 0) {
        *reinterpret_cast<uint4 *>(dst) = make_uint4(words[0], words[1], words[2], words[3]);
    } else {
#pragma unroll
        for (int k = 0; k < WPT; ++k)
            if (w0 + k < Cw) dst[k] = words[k];
    }
}

hipError_t launch_binarize_pack(const float *x, int N, int C, int H, int W, uint32_t *packed,
                                hipStream_t st)
{
    const int HW = H * W, Cw = (C + 31) / 32;
    const long long NP = (long long)N * HW;
    const bool vec4 = (Cw % 4 == 0) && ((reinterpret_cast<uintptr_t>(packed) & 15) == 0);
    const int groups = vec4 ? Cw / 4 : Cw;                // of words: one per block and pixel
    const int full = !vec4 && groups > 1 && C % 32 != 0 && C % 32 <= 8 ? groups - 1 : groups;
    const long long blocks = full < groups ? xcd_blocks(ceil_div(NP, 256)) * groups : xcd_blocks((long long)ceil_div(NP, 256) * groups);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (vec4) binarize_pack_kernel<4><<<dim3((unsigned)blocks), 256, 0, st>>>(x, NP, C, HW, Cw, groups, full, packed);
    else binarize_pack_kernel<1><<<dim3((unsigned)blocks), 256, 0, st>>>(x, NP, C, HW, Cw, groups, full, packed);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Eq. 10, first half: A = (1/C) sum_c |I_c|.  A block is 64 pixels x S channel slices; each thread
// adds its slice in double, the slices are combined through LDS in a fixed order (deterministic,
// and the double accumulation keeps A within one rounding of the exact mean).
// The paper uses one thread per pixel over all channels; slicing the channels keeps enough loads
// in flight to stream HBM when N*H*W alone gives too few waves.
// ------------------------------------------------------------------------------------------------
constexpr int kMaxSlices = 16;

__global__ __launch_bounds__(64 * kMaxSlices) void channel_mean_abs_kernel(
    const float *__restrict__ I, long long NP, int C, int HW, int chunk, float *__restrict__ A)
{
    __shared__ double part[kMaxSlices][64];
    const int lane = threadIdx.x, s = threadIdx.y, S = blockDim.y;
    const long long p = xcd_block(blockIdx.x, (NP + 63) / 64) * 64 + lane;
    double acc = 0.0;
    if (p < NP) {
        const long long n = p / HW;
        const int hw = (int)(p - n * HW);
        const float *src = I + (n * C) * (long long)HW + hw;
        const int c0 = s * chunk;
        const int c1 = min(C, c0 + chunk);
        int c = c0;
        for (; c + 8 <= c1; c += 8) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = __builtin_nontemporal_load(src + (long long)(c + j) * HW);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc += (double)fabsf(v[j]);
        }
        for (; c < c1; ++c) acc += (double)fabsf(src[(long long)c * HW]);
    }
    part[s][lane] = acc;
    __syncthreads();
    if (s == 0 && p < NP) {
        double sum = part[0][lane];
        for (int k = 1; k < S; ++k) sum += part[k][lane];
        A[p] = (float)(sum / (double)C);
    }
}

hipError_t launch_channel_mean_abs(const float *I, int N, int C, int H, int W, float *A,
                                   hipStream_t st)
{
    const int HW = H * W;
    const long long NP = (long long)N * HW;
    int S = 1;
    while (S < kMaxSlices && C / (2 * S) >= 8) S *= 2;
    const int chunk = (C + S - 1) / S;
    channel_mean_abs_kernel<<<dim3((unsigned)xcd_blocks(ceil_div(NP, 64))), dim3(64, S), 0, st>>>(I, NP, C, HW, chunk, A);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Step 1a and the first half of Eq. 10 in ONE pass over the fp32 tensor: every element is read
// once, its sign goes into the packed word and its magnitude into the channel sum.  (The paper runs
// the two as separate kernels on two streams; on an HBM-bound pre-stage the second read is the cost.)
// Block = 64 (or 32) pixels x S slices; slice s owns packed words s, s+S, ...  The words are collected in
// LDS and written out as one contiguous run of words; the slices' partial |x| sums (double)
// are combined in a fixed order.
// ------------------------------------------------------------------------------------------------
// At most 16 waves (1024 threads) a block.
constexpr int kPackMeanWaves = 16;

// Pixels and waves of a block.  A slice's words come one after the other, each with the whole latency of its
// 32 loads, so a tensor that does not fill the chip's wave slots is bound by that chain: every word gets a
// slice of its own, up to 16 waves per compute unit, and a tensor of few pixels and many channels blocks of
// 32 pixels (a wave then takes two words at a time).  Above that the chains overlap with those of other
// blocks, and fewer, longer slices leave more blocks per unit to cover a block's last barrier and write-out
// (4 measured equal to 8 and faster than 16).  Input pass, 4 slices of 64 pixels -> this: 64 x 512 x 7 x 7
// 10.6 -> 6.5 us, 64 x 256 x 14 x 14 6.6 -> 5.4 us.
struct PackMeanShape { int px, waves; };
static size_t pack_mean_smem(const PackMeanShape &s, int Cwp)
{
    return (size_t)s.waves * 64 * sizeof(double) + (size_t)s.px * Cwp * sizeof(uint32_t);
}
static PackMeanShape pack_mean_shape(long long NP, int Cw)
{
    PackMeanShape s;
    s.px = NP <= 64 * 64 && Cw >= 8 ? 32 : 64;
    const int per_wave = 64 / s.px;
    const long long blocks = (NP + s.px - 1) / s.px;
    for (int rounds = 1;; ++rounds) {                     // words of a slice
        s.waves = ceil_div(ceil_div(Cw, rounds), per_wave);
        // (more than four waves only in the 64 KB of LDS that need no raised limit)
        if (s.waves <= 4 || (s.waves <= kPackMeanWaves && blocks * s.waves <= 256 * 16 && pack_mean_smem(s, Cw | 1) <= 64 * 1024))
            return s;
    }
}
// The same beside filter blocks of the same size, which give every tap a thread and read C * taps values: four
// waves for large windows, as far as there are words for them.  (160 channels, F = 64, 15 x 15 beside 64 x 29 x 29:
// 30.8 -> 27.0 us, 13 x 13 26.2 -> 22.7.)
static PackMeanShape pack_mean_shape_both(long long NP, int Cw, int taps)
{
    PackMeanShape s = pack_mean_shape(NP, Cw);
    if (taps > 64) s.waves = std::max(s.waves, Cw >= 4 ? 4 : Cw >= 2 ? 2 : 1);
    return s;
}

template <int PX>
__device__ __attribute__((always_inline)) void pack_and_mean_block(
    const float *__restrict__ x, long long NP, int C, int HW, int Cw, int Cwp,
    uint32_t *__restrict__ packed, float *__restrict__ A, long long block, double *pm_smem)
{
    // slice = wave * 64 / PX + (which part of the wave)
    const int tid = threadIdx.y * 64 + threadIdx.x, threads = 64 * blockDim.y;
    const int lane = tid & (PX - 1), s = tid / PX, S = threads / PX;
    double *part = pm_smem;                                              // [S][PX]
    uint32_t *words = reinterpret_cast<uint32_t *>(pm_smem + threads);   // [PX][Cwp], Cwp odd
    const long long p0 = block * PX;
    const long long p = p0 + lane;
    double acc = 0.0;
    if (p < NP) {
        const long long n = p / HW;
        const int hw = (int)(p - n * HW);
        const float *src = x + (n * C) * (long long)HW + hw;
        for (int w = s; w < Cw; w += S) {
            const int cbase = 32 * w;
            uint32_t word = 0;
            if (cbase + 32 <= C) {
                float v[32];
#pragma unroll
                for (int j = 0; j < 32; ++j) v[j] = __builtin_nontemporal_load(src + (long long)(cbase + j) * HW);
                // from the highest channel down, each bit shifted in at the bottom: one compare (0 <= x:
                // true for +0.0 and -0.0, false for NaN) and one add-with-carry (word + word + bit)
#pragma unroll
                for (int j = 31; j >= 0; --j) {
                    asm("v_cmp_le_f32 vcc, 0, %1\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(word) : "v"(v[j]) : "vcc");
                    acc += (double)fabsf(v[j]);
                }
            } else {
                for (int j = 0; j < 32 && cbase + j < C; ++j) {
                    const float v = src[(long long)(cbase + j) * HW];
                    word |= (v >= 0.0f ? 1u : 0u) << j;
                    acc += (double)fabsf(v);
                }
            }
            words[lane * Cwp + w] = word;
        }
    }
    part[tid] = acc;
    __syncthreads();
    if (s == 0 && p < NP) {
        double sum = part[lane];
        for (int k = 1; k < S; ++k) sum += part[k * PX + lane];
        A[p] = (float)(sum / (double)C);
    }
    const int npx = (int)min((long long)PX, NP - p0);
    const int nwords = npx * Cw;
    uint32_t *dst = packed + p0 * Cw;
    for (int i = tid; i < nwords; i += threads) {
        const int px = i / Cw, w = i - px * Cw;
        dst[i] = words[px * Cwp + w];
    }
}

template <int PX>
__global__ __launch_bounds__(64 * kPackMeanWaves) void pack_and_mean_kernel(
    const float *__restrict__ x, long long NP, int C, int HW, int Cw, int Cwp,
    uint32_t *__restrict__ packed, float *__restrict__ A)
{
    extern __shared__ double pm_smem[];
    const long long nb = (NP + PX - 1) / PX, block = xcd_block(blockIdx.x, nb);
    if (block < nb) pack_and_mean_block<PX>(x, NP, C, HW, Cw, Cwp, packed, A, block, pm_smem);
}

// The same pass with four consecutive pixels per lane (one 16-byte load per lane and channel, 1 KB
// contiguous per wave and load instruction): measured 6.7 TB/s for this access pattern against
// 5.5 TB/s with one pixel per lane.  Needs H*W to be a multiple of 4 (so that a lane's four pixels
// share an image) and 16-byte aligned x and A.  Block = 256 pixels x S slices.
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kPack4Slices = 8;
constexpr int kPack4Batch = 8;      // channels whose loads are in flight together

__device__ __attribute__((always_inline)) void pack_and_mean4_block(
    const float *__restrict__ x, long long NP, int C, int HW, int Cw, int Cwp,
    uint32_t *__restrict__ packed, float *__restrict__ A, long long block, int ppb, double *pm_smem)
{
    // `ppb`: pixels per block, a multiple of 4 up to 256 (lanes beyond it idle): the host picks it so
    // that the blocks share out evenly over the compute units
    const int lane = threadIdx.x, s = threadIdx.y, S = blockDim.y;
    double *part = pm_smem;                                               // [S][4][64]
    uint32_t *words = reinterpret_cast<uint32_t *>(pm_smem + S * 256);    // [4][64][Cwp], Cwp odd
    const long long p0 = block * ppb;
    const long long p = p0 + 4 * lane;
    const bool mine = 4 * lane < ppb && p < NP;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (mine) {
        const long long n = p / HW;
        const int hw = (int)(p - n * HW);
        const float *src = x + (n * C) * (long long)HW + hw;
        // batches of kPack4Batch channels; the next batch's loads are issued before the current
        // batch's values are used, so that a wave always has loads in flight
        auto fetch = [&](int w, int b, float4 (&v)[kPack4Batch]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < kPack4Batch; ++j) {
                const int c = 32 * w + b + j;
                if (w < Cw && c < C) {
                    const floatx4 t = __builtin_nontemporal_load(
                        reinterpret_cast<const floatx4 *>(src + (long long)c * HW));
                    v[j] = make_float4(t[0], t[1], t[2], t[3]);
                } else {
                    v[j] = make_float4(-1.f, -1.f, -1.f, -1.f);                     // tail channels: bit 0
                }
            }
        };
        float4 cur[kPack4Batch], nxt[kPack4Batch];
        // A word's channels are taken from the last batch down to the first and, within a batch, from
        // the last channel down: the word is built by shifting the next lower channel's bit in at the
        // bottom, which is one compare (0 <= x: true for +0.0 and -0.0, false for NaN) and one
        // add-with-carry (word + word + bit) per value instead of compare, select and shift-or.
        constexpr int kLastBatch = 32 - kPack4Batch;
        fetch(s, kLastBatch, cur);
        for (int w = s; w < Cw; w += S) {
            uint32_t word[4] = {0u, 0u, 0u, 0u};
            const int cbase = 32 * w;
            const bool whole = cbase + 32 <= C;               // (uniform) no tail channels in this word
#pragma unroll
            for (int b = kLastBatch; b >= 0; b -= kPack4Batch) {
                if (b > 0) fetch(w, b - kPack4Batch, nxt);
                else fetch(w + S, kLastBatch, nxt);
#pragma unroll
                for (int j = kPack4Batch - 1; j >= 0; --j) {
                    const float e[4] = {cur[j].x, cur[j].y, cur[j].z, cur[j].w};
                    if (whole) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            asm("v_cmp_le_f32 vcc, 0, %1\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc"
                                : "+v"(word[k]) : "v"(e[k]) : "vcc");
                            acc[k] += (double)fabsf(e[k]);
                        }
                    } else {
                        const bool live = cbase + b + j < C;  // (tail channels were fetched as -1: bit 0)
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            word[k] = (word[k] << 1) | (e[k] >= 0.0f ? 1u : 0u);
                            acc[k] += live ? (double)fabsf(e[k]) : 0.0;
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < kPack4Batch; ++j) cur[j] = nxt[j];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) words[(k * 64 + lane) * Cwp + w] = word[k];
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) part[(s * 4 + k) * 64 + lane] = acc[k];
    __syncthreads();
    // pixel 4*lane + k: slice k % S adds up the slices' sums (fixed order) when S >= 4
    for (int k = s; k < 4; k += S) {
        if (mine && p + k < NP) {
            double sum = part[k * 64 + lane];
            for (int t = 1; t < S; ++t) sum += part[(t * 4 + k) * 64 + lane];
            A[p + k] = (float)(sum / (double)C);
        }
    }
    const int npx = (int)min((long long)ppb, NP - p0);
    const int nwords = npx * Cw;
    uint32_t *dst = packed + p0 * Cw;
    for (int i = s * 64 + lane; i < nwords; i += 64 * S) {
        const int px = i / Cw, w = i - px * Cw;
        dst[i] = words[((px & 3) * 64 + (px >> 2)) * Cwp + w];
    }
}

__global__ __launch_bounds__(64 * kPack4Slices) void pack_and_mean4_kernel(
    const float *__restrict__ x, long long NP, int C, int HW, int Cw, int Cwp,
    uint32_t *__restrict__ packed, float *__restrict__ A, int ppb)
{
    extern __shared__ double pm_smem[];
    const long long nb = (NP + ppb - 1) / ppb, block = xcd_block(blockIdx.x, nb);
    if (block < nb) pack_and_mean4_block(x, NP, C, HW, Cw, Cwp, packed, A, block, ppb, pm_smem);
}

// Pixels per block of the four-pixel pass.  A compute unit pulls from HBM at a rate of its own
// (outstanding misses, not lanes, are what it runs out of: measured, a second block on the same unit
// halves the first one's rate), so a launch is as long as its busiest unit: the pixels are shared out
// as equal blocks over a multiple of the units instead of as 256-pixel blocks that leave the last
// round partly empty.
// `filter_blocks`: short blocks launched behind the input blocks in the same grid (the one-launch
// prepare): where the last round of 256-pixel blocks leaves enough units idle for them (a filter
// block takes about a fifth of an input block's time), that layout is the better one: the filter
// side then costs nothing (measured at 128 images of 28 x 28, 392 + 512 blocks: the step 2.4 us
// shorter than with 512 equal input blocks and the filter blocks after them).
static int pixels_per_block4(long long NP, int filter_blocks = 0)
{
    const int cus = compute_units();
    if (filter_blocks > 0) {
        const long long rem = ((NP + 255) / 256) % cus, idle = rem ? cus - rem : 0;
        if (idle > 0 && filter_blocks <= 5 * idle) return 256;
    }
    const long long quads = (NP + 3) / 4;
    for (long long k = 1;; ++k) {
        const long long per = (quads + cus * k - 1) / (cus * k);
        if (per <= 64) return (int)std::max<long long>(per, 16) * 4;   // (at least a quarter of the lanes busy)
    }
}

bool pack_and_mean_supports(int C) { return (C + 31) / 32 <= 512; }

hipError_t launch_pack_and_mean(const float *x, int N, int C, int H, int W, uint32_t *packed,
                                float *A, hipStream_t st)
{
    const int HW = H * W, Cw = (C + 31) / 32, Cwp = Cw | 1;
    const long long NP = (long long)N * HW;
    if (HW % 4 == 0 && ((uintptr_t)x & 15) == 0 && NP >= 256 * 256) {
        int S4 = 1;
        while (S4 < kPack4Slices && 2 * S4 <= Cw) S4 *= 2;
        const size_t smem4 = (size_t)S4 * 256 * sizeof(double) + (size_t)256 * Cwp * sizeof(uint32_t);
        if (smem4 <= 64 * 1024) {
            const int ppb = pixels_per_block4(NP);
            pack_and_mean4_kernel<<<dim3((unsigned)xcd_blocks(ceil_div(NP, ppb))), dim3(64, S4), smem4, st>>>(x, NP, C, HW, Cw,
                                                                                      Cwp, packed, A, ppb);
            return hipGetLastError();
        }
    }
    const PackMeanShape s = pack_mean_shape(NP, Cw);
    const dim3 grid((unsigned)xcd_blocks(ceil_div(NP, s.px))), block(64, s.waves);
    if (s.px == 32) pack_and_mean_kernel<32><<<grid, block, pack_mean_smem(s, Cwp), st>>>(x, NP, C, HW, Cw, Cwp, packed, A);
    else pack_and_mean_kernel<64><<<grid, block, pack_mean_smem(s, Cwp), st>>>(x, NP, C, HW, Cw, Cwp, packed, A);
    return hipGetLastError();
}

// Eq. 5 from per-tap channel means: alpha[f] = mean over the kh*kw taps of M[f][tap], where
// M = mean_c |Wt| is what pack_and_mean_kernel leaves in its A output when run on the filters.
__global__ __launch_bounds__(256) void alpha_from_tap_means_kernel(const float *__restrict__ M,
                                                                   int F, int taps,
                                                                   float *__restrict__ alpha)
{
    const int f = blockIdx.x * 256 + threadIdx.x;
    if (f >= F) return;
    double sum = 0.0;
    for (int t = 0; t < taps; ++t) sum += (double)M[(long long)f * taps + t];
    alpha[f] = (float)(sum / (double)taps);
}

hipError_t launch_alpha_from_tap_means(const float *M, int F, int taps, float *alpha, hipStream_t st)
{
    alpha_from_tap_means_kernel<<<ceil_div(F, 256), 256, 0, st>>>(M, F, taps, alpha);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Filters: step 1a (Eq. 3) and Eq. 5 in one pass, one workgroup per filter.  A filter's C*kh*kw
// floats are contiguous, so the workgroup reads them as one coalesced run into LDS (a chunk of CH
// channels at a time, CH a multiple of 32), then one thread per (tap, channel word) gathers its 32
// channel values from LDS (consecutive threads = consecutive taps = consecutive LDS words), builds
// the word and the |w| sum of its 32 channels.  Sums are combined in double in a fixed order:
// M[f][tap] = mean_c |Wt[f][c][tap]|, alpha[f] = mean over everything.
// ------------------------------------------------------------------------------------------------
constexpr int kFilterStageFloats = 8192;   // 32 KB of LDS for the staged chunk

__device__ __attribute__((always_inline)) void filter_pack_mean_block(
    const float *__restrict__ Wt, int C, int taps, int Cw, int CH, uint32_t *__restrict__ Wpk,
    float *__restrict__ M, float *__restrict__ alpha, int f, int tid, int nthr, double *fp_smem,
    uint4 *__restrict__ Wx = nullptr, ExpandLayout L = ExpandLayout{}, int F = 0)
{
    // With Wx the block also writes its filter's rows of the matrix-core kernel's expanded
    // workspace (what xnor_filter_expand would make of Wpk): the packed words are kept in LDS
    // ([taps][Cw] behind the staging area) and expanded once the filter is complete.
    const int WH = CH / 32;                                        // channel words per chunk
    double *part = fp_smem;                                         // [WH][taps]
    float *stage = reinterpret_cast<float *>(fp_smem + WH * taps);  // [CH][taps]
    uint32_t *kept = reinterpret_cast<uint32_t *>(stage + (size_t)CH * taps);   // [taps][Cw], only with Wx
    const float *src = Wt + (long long)f * C * taps;
    uint32_t *dst = Wpk + (long long)f * taps * Cw;
    double tap_total = 0.0;                                         // thread t < taps owns tap t
    for (int c0 = 0; c0 < C; c0 += CH) {
        const int nch = min(CH, C - c0);
        const int nfl = nch * taps;
        __syncthreads();                                            // previous chunk fully consumed
        for (int i = tid; i < nfl; i += nthr) stage[i] = src[(long long)c0 * taps + i];
        __syncthreads();
        const int nw = (nch + 31) / 32;
        for (int it = tid; it < nw * taps; it += nthr) {
            const int w = it / taps, tap = it - w * taps;
            const int nb = min(32, nch - 32 * w);
            uint32_t word = 0;
            double acc = 0.0;
            if (nb == 32) {
                // whole word: all 32 LDS reads in flight at once, four independent partial sums
                float v[32];
#pragma unroll
                for (int j = 0; j < 32; ++j) v[j] = stage[(32 * w + j) * taps + tap];
                double a4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int j = 0; j < 32; ++j) {
                    word |= (v[j] >= 0.0f ? 1u : 0u) << j;
                    a4[j & 3] += (double)fabsf(v[j]);
                }
                acc = (a4[0] + a4[1]) + (a4[2] + a4[3]);
            } else {
                for (int j = 0; j < nb; ++j) {
                    const float v = stage[(32 * w + j) * taps + tap];
                    word |= (v >= 0.0f ? 1u : 0u) << j;
                    acc += (double)fabsf(v);
                }
            }
            dst[tap * Cw + c0 / 32 + w] = word;
            if (Wx) kept[tap * Cw + c0 / 32 + w] = word;
            part[it] = acc;
        }
        __syncthreads();
        if (tid < taps)
            for (int w = 0; w < nw; ++w) tap_total += part[w * taps + tid];
    }
    __syncthreads();
    if (tid < taps) {
        M[(long long)f * taps + tid] = (float)(tap_total / (double)C);
        part[tid] = tap_total;
    }
    __syncthreads();
    if (tid == 0) {
        double sum = 0.0;
        for (int t = 0; t < taps; ++t) sum += part[t];
        alpha[f] = (float)(sum / ((double)C * (double)taps));
    }
    if (Wx) {
        // (the barriers above have made every kept word visible)
        const int tile = f >> 5, row = f & 31;
        uint4 *rows = Wx + (size_t)tile * L.tile_steps * 64;
        for (int e = tid; e < 2 * L.tile_steps; e += nthr) {
            const int step = e >> 1, kg = e & 1;
            rows[(size_t)step * 64 + row + 32 * kg] =
                expanded_entry(L, step, kg, taps, Cw, C, [&](int tap, int w) { return kept[tap * Cw + w]; });
        }
        // rows past the last filter are zeros: the rest of its tile and the tiles after it (the workspace holds whole
        // workgroup rows), shared out over all filters' blocks (one block's 64 threads took longer than all the
        // rest: 32 channels, F = 288 3x3 11.8 -> 4.3 us, 16 x 128 x 14 x 14 F = 300 5.0 -> 4.5)
        const int last = (F - 1) >> 5, last_row = (F - 1) & 31;
        const size_t first = ((size_t)last * L.tile_steps * 64), end = L.ws_bytes / sizeof(uint4);
        for (size_t i = first + (size_t)f * nthr + tid; i < end; i += (size_t)F * nthr) {
            const int lane = (int)(i & 63);
            if (i - first >= (size_t)L.tile_steps * 64 || (lane & 31) > last_row) Wx[i] = make_uint4(0, 0, 0, 0);
        }
    }
}

__global__ __launch_bounds__(256) void filter_pack_mean_kernel(
    const float *__restrict__ Wt, int C, int taps, int Cw, int CH, uint32_t *__restrict__ Wpk,
    float *__restrict__ M, float *__restrict__ alpha)
{
    extern __shared__ double fp_smem[];
    filter_pack_mean_block(Wt, C, taps, Cw, CH, Wpk, M, alpha, blockIdx.x, threadIdx.x, 256, fp_smem);
}

// Input side and filter side of a layer in ONE launch: the first blocks each pack up to 256 pixels
// of the input (pack_and_mean4_block; the pixels are shared out evenly over a multiple of the compute
// units, see pixels_per_block4), the last F blocks each prepare one filter (filter_pack_mean_block).
// The two sides do not depend on each other; the filter blocks, dispatched last, cost no launch of
// their own in front of the convolution.
__global__ __launch_bounds__(64 * kPack4Slices) void prepare_both_kernel(
    const float *__restrict__ x, long long NP, int C, int HW, int Cw, int Cwp,
    uint32_t *__restrict__ packed, float *__restrict__ A,
    const float *__restrict__ Wt, int F, int taps, int CH, uint32_t *__restrict__ Wpk,
    float *__restrict__ M, float *__restrict__ alpha, uint4 *__restrict__ Wx, ExpandLayout L, int ppb)
{
    extern __shared__ double both_smem[];
    const long long nb_in = (NP + ppb - 1) / ppb, first_filter = (nb_in + 7) / 8 * 8;
    if ((long long)blockIdx.x < first_filter) {
        const long long block = xcd_block(blockIdx.x, nb_in);
        if (block < nb_in) pack_and_mean4_block(x, NP, C, HW, Cw, Cwp, packed, A, block, ppb, both_smem);
    } else
        filter_pack_mean_block(Wt, C, taps, Cw, CH, Wpk, M, alpha, (int)(blockIdx.x - first_filter),
                               threadIdx.y * 64 + threadIdx.x, 64 * blockDim.y, both_smem, Wx, L, F);
}

// The same with the one-pixel-per-lane input pass (64 or 32 pixels per block): for inputs whose H*W is not
// a multiple of 4, that are not 16-byte aligned, or that are too small to fill the chip with
// 256-pixel blocks.  A filter's chain (read, pack, sums, expansion) is as long as the whole input side of
// such a layer and has to run beside it, so the filter blocks go first where that leaves the input room.
template <int PX>
__global__ __launch_bounds__(64 * kPackMeanWaves) void prepare_both1_kernel(
    const float *__restrict__ x, long long NP, int C, int HW, int Cw, int Cwp,
    uint32_t *__restrict__ packed, float *__restrict__ A,
    const float *__restrict__ Wt, int F, int taps, int CH, uint32_t *__restrict__ Wpk,
    float *__restrict__ M, float *__restrict__ alpha, uint4 *__restrict__ Wx, ExpandLayout L, bool filters_first)
{
    extern __shared__ double both_smem[];
    const long long nb_in = (NP + PX - 1) / PX, nb_launched = (nb_in + 7) / 8 * 8;
    const int f = filters_first ? (int)blockIdx.x : (int)(blockIdx.x - nb_launched);
    if (f < 0 || f >= F) {
        const long long block = xcd_block(filters_first ? blockIdx.x - F : blockIdx.x, nb_in);
        if (block < nb_in) pack_and_mean_block<PX>(x, NP, C, HW, Cw, Cwp, packed, A, block, both_smem);
    } else
        filter_pack_mean_block(Wt, C, taps, Cw, CH, Wpk, M, alpha, f,
                               threadIdx.y * 64 + threadIdx.x, 64 * blockDim.y, both_smem, Wx, L, F);
}

bool filter_pack_mean_supports(int taps) { return taps <= 256; }

hipError_t launch_filter_pack_mean(const float *Wt, int F, int C, int taps, uint32_t *Wpk, float *M,
                                   float *alpha, hipStream_t st)
{
    const int Cw = (C + 31) / 32;
    int CH = kFilterStageFloats / taps / 32 * 32;                   // >= 32 since taps <= 256
    CH = std::min(CH, Cw * 32);
    const int WH = CH / 32;
    const size_t smem = (size_t)WH * taps * sizeof(double) + (size_t)CH * taps * sizeof(float);
    filter_pack_mean_kernel<<<F, 256, smem, st>>>(Wt, C, taps, Cw, CH, Wpk, M, alpha);
    return hipGetLastError();
}

// One launch for both sides: with the four-pixel input pass where it applies with full-size blocks,
// else with the one-pixel pass; the caller falls back to separate launches where neither fits.
static bool four_pixel_pass(const float *x, int N, int C, int H, int W)
{
    const int HW = H * W, Cw = (C + 31) / 32;
    return HW % 4 == 0 && ((uintptr_t)x & 15) == 0 && (long long)N * HW >= 256 * 256 && Cw >= kPack4Slices;
}

static size_t filter_block_smem(int C, int taps, bool expand, int *CH_out)
{
    const int Cw = (C + 31) / 32;
    int CH = kFilterStageFloats / taps / 32 * 32;
    CH = std::min(CH, Cw * 32);
    *CH_out = CH;
    return (size_t)(CH / 32) * taps * sizeof(double) + (size_t)CH * taps * sizeof(float) +
           (expand ? (size_t)taps * Cw * sizeof(uint32_t) : 0);
}

// Which input pass a single launch for both sides can use: 4 (four pixels per lane), 1 (one pixel
// per lane) or 0 (neither fits: the caller launches the two sides separately).  Either pass shares
// its dynamic LDS (at most 64 KB) with the filter blocks' staging.
static int prepare_both_pass(const float *x, int N, int C, int H, int W, int taps, bool expand)
{
    const int Cw = (C + 31) / 32, Cwp = Cw | 1;
    const long long NP = (long long)N * H * W;
    if (Cw > 512 || taps > 256) return 0;
    int CH;
    const size_t smemf = filter_block_smem(C, taps, expand, &CH);
    if (smemf > 64 * 1024) return 0;
    if (four_pixel_pass(x, N, C, H, W)) {
        const size_t smem4 = (size_t)kPack4Slices * 256 * sizeof(double) + (size_t)256 * Cwp * sizeof(uint32_t);
        if (smem4 <= 64 * 1024) return 4;
    }
    // (the one-pixel pass: the filter block gives every tap a thread of its own)
    const PackMeanShape s = pack_mean_shape_both(NP, Cw, taps);
    if (64 * s.waves < taps) return 0;
    return pack_mean_smem(s, Cwp) <= 64 * 1024 ? 1 : 0;
}

bool prepare_both_supports(const float *x, int N, int C, int H, int W, int taps)
{
    // (with the filter expansion's LDS counted: the caller may ask for it)
    return prepare_both_pass(x, N, C, H, W, taps, true) != 0;
}

// `Wx` (may be null): the matrix-core kernel's filter workspace, filled as by launch_expand_filters.
bool prepare_both_can_expand(int C, int taps) { return (long long)taps * ((C + 31) / 32) <= 4096; }

hipError_t launch_prepare_both(const float *x, int N, int C, int H, int W, uint32_t *packed, float *A,
                               const float *Wt, int F, int taps, uint32_t *Wpk, float *M, float *alpha,
                               void *Wx, const ExpandLayout &L, hipStream_t st)
{
    const int HW = H * W, Cw = (C + 31) / 32, Cwp = Cw | 1;
    const long long NP = (long long)N * HW;
    int CH;
    const size_t smemf = filter_block_smem(C, taps, Wx != nullptr, &CH);
    const int pass = prepare_both_pass(x, N, C, H, W, taps, Wx != nullptr);
    if (pass == 4) {
        const size_t smem4 = (size_t)kPack4Slices * 256 * sizeof(double) + (size_t)256 * Cwp * sizeof(uint32_t);
        const size_t smem = std::max(smem4, smemf);
        const int ppb = pixels_per_block4(NP, F);
        const long long blocks = (long long)F + xcd_blocks(ceil_div(NP, ppb));
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        prepare_both_kernel<<<dim3((unsigned)blocks), dim3(64, kPack4Slices), smem, st>>>(
            x, NP, C, HW, Cw, Cwp, packed, A, Wt, F, taps, CH, Wpk, M, alpha, static_cast<uint4 *>(Wx), L, ppb);
        return hipGetLastError();
    }
    if (pass != 1) return hipErrorInvalidValue;   // (prepare_both_supports said no)
    const PackMeanShape s = pack_mean_shape_both(NP, Cw, taps);
    const size_t smem = std::max(pack_mean_smem(s, Cwp), smemf);
    const long long blocks = (long long)F + xcd_blocks(ceil_div(NP, s.px));
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // (in half of the chip's wave slots at most, and for inputs of up to 64 MB: 64 x 128 x 28 x 28 F=256 8.8 -> 7.7 us,
    //  128 x 96 x 27 x 27 F=256 5x5 12.0 -> 11.2; with F=384 blocks of 768 threads 11.9 -> 14.5, at 160 MB 35.1 -> 36.3)
    const bool filters_first = (long long)F * 64 * s.waves <= 256 * 1024 && NP * C * 4 <= (64LL << 20);
    auto launch = [&](auto kernel) {
        kernel<<<dim3((unsigned)blocks), dim3(64, s.waves), smem, st>>>(
            x, NP, C, HW, Cw, Cwp, packed, A, Wt, F, taps, CH, Wpk, M, alpha, static_cast<uint4 *>(Wx), L, filters_first);
    };
    if (s.px == 32) launch(prepare_both1_kernel<32>);
    else launch(prepare_both1_kernel<64>);
    return hipGetLastError();
}

// Eq. 10, second half: K = A * k with constant taps 1/(kh*kw), at the convolution's output
// positions; taps outside the image add nothing.  One thread per output pixel (A is C times smaller
// than I, so this pass is negligible).
__global__ __launch_bounds__(256) void box_filter_K_kernel(const float *__restrict__ A, Geom g,
                                                           long long total, float *__restrict__ K)
{
    const long long o = (long long)blockIdx.x * 256 + threadIdx.x;
    if (o >= total) return;
    const int ox = (int)(o % g.OW);
    const long long t = o / g.OW;
    const int oy = (int)(t % g.OH);
    const long long n = t / g.OH;
    const float *a = A + n * (long long)g.H * g.W;
    // no branches around the loads (out-of-image taps read the image's first value and add 0), so that the
    // unrolled loop has nine of them in flight: a chain of kh * kw load latencies otherwise
    double sum = 0.0;
    const int iy0 = oy * g.sh - g.ph, ix0 = ox * g.sw - g.pw;
    int ky = 0, kx = 0;
#pragma unroll 9
    for (int t2 = 0; t2 < g.kh * g.kw; ++t2) {
        const int iy = iy0 + ky, ix = ix0 + kx;
        const bool in = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
        const float v = a[in ? iy * g.W + ix : 0];
        sum += in ? (double)v : 0.0;
        if (++kx == g.kw) { kx = 0; ++ky; }
    }
    K[o] = (float)(sum / (double)(g.kh * g.kw));
}

hipError_t launch_box_filter_K(const float *A, const Geom &g, float *K, hipStream_t st)
{
    const long long total = (long long)g.N * g.OH * g.OW;
    box_filter_K_kernel<<<ceil_div(total, 256), 256, 0, st>>>(A, g, total, K);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Eq. 10 as a whole for small inputs, in one launch: a block forms A for the rows under a band of output rows (and for the band's own
// share of the image's rows, which it writes), keeps them in LDS and forms K from there.  The rows that bands share are read
// once for each of them, which at these sizes costs less than the second launch.  Sums in the order of channel_mean_abs_kernel and
// box_filter_K_kernel: the same bits.
// ------------------------------------------------------------------------------------------------
constexpr size_t kBandLds = 60 * 1024;
struct BandShape {
    bool ok;
    int S, G, chunk, rows, bands;      // channel slices, groups of 128 pixels side by side; channels of a slice; output rows of a band, bands
    size_t smem;
};
// The rows that band b forms A for: those under its windows, if there are any, and its own.
__host__ __device__ inline void band_rows(const Geom &g, const BandShape &s, int b, int *r0, int *r1)
{
    const int oy0 = b * s.rows, oy1 = oy0 + s.rows < g.OH ? oy0 + s.rows : g.OH;
    const int own0 = (int)((long long)b * g.H / s.bands), own1 = (int)((long long)(b + 1) * g.H / s.bands);
    const int top = oy0 * g.sh - g.ph, end = (oy1 - 1) * g.sh - g.ph + g.kh;
    const int w0 = top > 0 ? top : 0, w1 = end < g.H ? end : g.H;
    *r0 = w0 < w1 && w0 < own0 ? w0 : own0;
    *r1 = w0 < w1 && w1 > own1 ? w1 : own1;
}

__global__ __launch_bounds__(1024) void scale_K_band_kernel(const float *__restrict__ I, Geom g, BandShape s,
                                                            float *__restrict__ A, float *__restrict__ K)
{
    extern __shared__ double band_lds[];
    const int lane = threadIdx.x, slice = threadIdx.y, group = threadIdx.z, HW = g.H * g.W;
    double *const part = band_lds + group * s.S * 128;
    float *const a = reinterpret_cast<float *>(band_lds + s.G * s.S * 128);
    const int n = blockIdx.x / s.bands, b = blockIdx.x - n * s.bands;
    const int oy0 = b * s.rows, oy1 = min(g.OH, oy0 + s.rows);
    const int own0 = (int)((long long)b * g.H / s.bands), own1 = (int)((long long)(b + 1) * g.H / s.bands);
    int r0, r1;
    band_rows(g, s, b, &r0, &r1);
    const int pixels = (r1 - r0) * g.W;
    const float *const src = I + (size_t)n * g.C * HW + (size_t)r0 * g.W;
    const int c0 = slice * s.chunk, c1 = min(g.C, c0 + s.chunk);
    // two pixels of a thread at a time, their loads in flight together
    for (int base = 0; base < pixels; base += 128 * s.G) {
        const int q = base + 128 * group + lane;
        const float *const at[2] = {src + min(q, pixels - 1), src + min(q + 64, pixels - 1)};
        double acc[2] = {0.0, 0.0};
        auto sum_of = [&](auto count) __attribute__((always_inline)) {
            constexpr int N = decltype(count)::value;
            int c = c0;
            for (; c + 8 <= c1; c += 8) {
                float v[N][8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int u = 0; u < N; ++u) v[u][j] = at[u][(size_t)(c + j) * HW];
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int u = 0; u < N; ++u) acc[u] += (double)fabsf(v[u][j]);
            }
            for (; c < c1; ++c)
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] += (double)fabsf(at[u][(size_t)c * HW]);
        };
        if (base + 128 * group + 64 < pixels) sum_of(std::integral_constant<int, 2>{});
        else if (base + 128 * group < pixels) sum_of(std::integral_constant<int, 1>{});
#pragma unroll
        for (int u = 0; u < 2; ++u) part[slice * 128 + 64 * u + lane] = acc[u];
        __syncthreads();
        // (slice u sums the u-th pixels; of one slice that does both)
        for (int u = slice; u < 2; u += s.S) {
            const int p = q + 64 * u;
            if (p >= pixels) continue;
            double sum = part[64 * u + lane];
            for (int k = 1; k < s.S; ++k) sum += part[k * 128 + 64 * u + lane];
            const float mean = (float)(sum / (double)g.C);
            const int row = r0 + p / g.W;
            a[p] = mean;
            if (row >= own0 && row < own1) A[(size_t)n * HW + (size_t)r0 * g.W + p] = mean;
        }
        __syncthreads();
    }
    const int tid = (group * s.S + slice) * 64 + lane;
    for (int o = tid; o < (oy1 - oy0) * g.OW; o += 64 * s.S * s.G) {
        const int r = o / g.OW, ox = o - r * g.OW, oy = oy0 + r;
        const int iy0 = oy * g.sh - g.ph, ix0 = ox * g.sw - g.pw;
        double sum = 0.0;
        for (int ky = 0; ky < g.kh; ++ky)
            for (int kx = 0; kx < g.kw; ++kx) {
                const int iy = iy0 + ky, ix = ix0 + kx;
                const bool in = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
                const float v = a[in ? (iy - r0) * g.W + ix : 0];
                sum += in ? (double)v : 0.0;
            }
        K[((size_t)n * g.OH + oy) * g.OW + ox] = (float)(sum / (double)(g.kh * g.kw));
    }
}

// Inputs of less than 2^20 values in at most a band for each of 256 units, which fit LDS, read a row four times at most, and whose
// threads have two pixels of up to 16 channels or one of up to 48 (of any number if all bands together read up to 2.6e6 values), once; of
// one channel three times, where the bands fill half the units.  Past that a workgroup's loads take longer than the second launch:
// 1 x 1024 x 28 x 28 3 x 3, two pixels of 64, 7.6 us in two launches / 9.1 in one; 16 x 1023 x 8 x 8, one of 64, 7.9 / 9.0; 1 x 116 x 3 x 3000 3 x 3, on
// three units, 5.6 / 132; 1 x 512 x 1 x 2000 1 x 1, on one, 5.6 / 66.  Of 307 drawn inputs (1 to 64 images, 1 to 1024 channels, 1 x 4 to 300 x 3000,
// 1 x 1 to 7 x 7) it takes 262, at 0.39 to 1.01 of the time of two launches in a graph, 0.89 on average, 0.73 eager; one other would be 4 % faster.  us,
// eager; in a graph: 1 x 64 x 32 x 32 3 x 3 7.7 / 5.4; 4.6 / 4.1, 5 x 100 x 37 x 53 7.6 / 5.6; 5.5 / 5.3.
static BandShape band_shape(const Geom &g)
{
    BandShape s{};
    const long long values = (long long)g.N * g.C * g.H * g.W;
    if (values >= (1 << 20) || g.kh > 16) return s;
    s.S = 1;
    while (s.S < kMaxSlices && g.C / (2 * s.S) >= 8) s.S *= 2;      // (as in launch_channel_mean_abs)
    s.G = std::max(1, 16 / s.S);
    s.rows = std::max(1, ceil_div((long long)g.N * g.OH, 256));
    s.bands = ceil_div(g.OH, s.rows);
    s.chunk = ceil_div(g.C, s.S);
    const long long blocks = (long long)g.N * s.bands;
    if (blocks > 256) return s;
    long long read = 0, most = 0;
    for (int b = 0; b < s.bands; ++b) {
        int r0, r1;
        band_rows(g, s, b, &r0, &r1);
        most = std::max<long long>(most, r1 - r0);
        read += r1 - r0;
    }
    const long long pixels = most * g.W;
    if (read > 4LL * g.H + 8) return s;
    if (pixels > 128 * s.G) {
        if (g.C > 1 || blocks < 128 || pixels > 3 * 128 * s.G) return s;
    } else if (pixels > 64 ? s.chunk > 16 : s.chunk > 48 && g.N * read * g.W * g.C > (5 << 19)) {
        return s;
    }
    s.smem = (size_t)s.S * s.G * 128 * sizeof(double) + (size_t)pixels * sizeof(float);
    s.ok = s.smem <= kBandLds;
    return s;
}

hipError_t launch_scale_K(const float *I, const Geom &g, float *A, float *K, hipStream_t st)
{
    static thread_local PlanMemo<BandShape> memo;
    const BandShape &s = memo.get(g, 0, [&] { return band_shape(g); });
    if (s.ok) {
        scale_K_band_kernel<<<dim3((unsigned)(g.N * s.bands)), dim3(64, s.S, s.G), s.smem, st>>>(I, g, s, A, K);
        return hipGetLastError();
    }
    const hipError_t e = launch_channel_mean_abs(I, g.N, g.C, g.H, g.W, A, st);
    return e != hipSuccess ? e : launch_box_filter_K(A, g, K, st);
}

// ------------------------------------------------------------------------------------------------
// Eq. 5: alpha[f] = ||Wt[f]||_1 / n.  One block per filter, double partial sums, fixed-order tree.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void alpha_kernel(const float *__restrict__ Wt, long long n_red,
                                                    float *__restrict__ alpha)
{
    __shared__ double part[256];
    const float *w = Wt + (long long)blockIdx.x * n_red;
    double acc = 0.0;
    for (long long i = threadIdx.x; i < n_red; i += 256) acc += (double)fabsf(w[i]);
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int step = 128; step > 0; step >>= 1) {
        if ((int)threadIdx.x < step) part[threadIdx.x] += part[threadIdx.x + step];
        __syncthreads();
    }
    if (threadIdx.x == 0) alpha[blockIdx.x] = (float)(part[0] / (double)n_red);
}

hipError_t launch_alpha(const float *Wt, int F, long long n_red, float *alpha, hipStream_t st)
{
    alpha_kernel<<<F, 256, 0, st>>>(Wt, n_red, alpha);
    return hipGetLastError();
}

}  // namespace xnor
