// Matrix-core XNOR convolution for layers of little work: many small independent workgroups instead of
// persistent ones.  The arithmetic is that of conv_mfma.hip (+-1 as FP4, v_mfma_f32_32x32x64_f8f6f4, the
// filters expanded in operand order in the workspace, the input expanded while it is staged).
//
// A layer that gives a compute unit one or two items of the persistent kernel is as long as the chain of
// one item: set-up, expansion of the first channel chunk, three hand-overs of chunks between four waves,
// 128 x 256 outputs' worth of matrix instructions, stores.  Here a workgroup (4 waves) owns 128 (or 64)
// filters x 128 or fewer consecutive output pixels of the batch, and the input rows under them are
// expanded to FP4 in LDS once, over all channels: one barrier, then a loop of matrix instructions with
// nothing in it but its operands, then the stores.  Two or three workgroups share a compute unit, so that
// one's set-up and stores run under another's matrix instructions.
//   * wave tile: 32 * NF filters x 32 * NP pixels; WF waves along the filters, 4 / WF along the pixels (see
//     make_tplan for how they are chosen).
//   * The pixels of a tile are consecutive in (n, oy, ox), across rows and, for small images, across images
//     (every image under a tile then gets its own halo rows): few idle pixel slots at any image size.
//   * Filter operands come from the L2 a few steps ahead of their use (a ring of registers), pixel operands
//     from LDS (slot pitch an odd number of 16-byte units: conflict-free).
//   * Half of a small launch is a workgroup's way to its first matrix instruction, about 1200 instructions at one or two
//     waves a SIMD.  Scalar divisions by reciprocals, all first loads before the first wait and the padding's zeros
//     out of the lookup that expands the words took it from 7.8 to 6.2 k cycles for 64 x 128 x 28 x 28 F=256 3x3 stride 2
//     (with its input pass 17.1 -> 16.2 us), from 6.2 to 5.8 k for 64 x 256 x 14 x 14 F=256 3x3.
//   * Given the channel mean A instead of K, A is staged beside the input, one value per slot, and a lane
//     sums its own pixels' windows from LDS (the sum, order and rounding of box_filter_K_kernel).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "conv_mfma_common.hpp"

namespace xnor {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));

constexpr int kThreads = 256;
constexpr int kTabTail = 24;               // table entries read past the last step

struct TileParams {
    const uint32_t *Ipk;
    const uint4 *Wx;
    const float *K, *A, *alpha;
    float *out;
    int32_t *dot;
    uint32_t *Opk;      // chained form: packed signs [N][OH][OW][Cwn] and partial sums of |out| [pixel][parts]
    float *P;
    int Cwn, parts;
    int C, H, W, F, kh, kw, sh, sw, ph, pw, OH, OW, Cw, N;
    int npix;           // N * OH * OW
    int per_image;      // 0, or pixel tiles of an image
    int ptiles, wgs_per_xcd, fgroups;
    int Wp, RHfull;     // staged columns of a row, staged rows of a whole image
    int S2, T;          // steps (64 channels) of a tap, of all taps
    int tile_steps;     // ... and behind a filter tile in the workspace
    int pitch16;        // slot pitch in 16-byte units (odd)
    int write_through;      // stores go past the L2 (see launch_conv_mfma_tile)
    int tab16, al16, a16;   // start of the step table, alpha and the staged A in LDS (16-byte units)
    float iCHV, iWp, iRH, iOW, iOH, iS2, ikw;   // reciprocals for div_small
    uint32_t mGroups, mImage, mOW, mOH;         // ... and for div_scalar
};

// n / d for n < 2^20: (n + 0.5) / d is at least 0.5 / d away from a whole number and the rounding of the
// reciprocal and the product moves it by less (four full-rate instructions; the 32-bit multiplications
// of an exact integer division run at a quarter of the rate).
__device__ inline uint32_t div_small(uint32_t n, float inv) { return (uint32_t)(((float)n + 0.5f) * inv); }

// n / d and the rest for n < 2^32 in scalar registers: with m = floor(2^32 / d) the high half of n * m is the
// quotient or one less.  (The compiler's own division is a chain of 25 instructions through the vector unit: four of
// them, one behind the other, stood before a workgroup's first load.)
inline uint32_t scalar_reciprocal(long long d) { return d <= 1 ? 0xffffffffu : (uint32_t)((1LL << 32) / d); }
__device__ inline int div_scalar(uint32_t n, uint32_t d, uint32_t m, int &rest)
{
    uint32_t q = __umulhi(n, m), r = n - q * d;
    const bool more = r >= d;
    q += more ? 1u : 0u;
    rest = (int)(more ? r - d : r);
    return (int)q;
}

// Steps the filter operands are ahead of their use; one less of zeros lie behind a tile's last step, where the last
// loads of the loop end (step T + operand_ring - 2).
constexpr int operand_ring(int NF, int NP) { return NF * NP >= 4 ? 4 : 8; }

template <int NF, int NP>
struct Depth {                              // steps the operands are ahead of their use
    static constexpr int kA = operand_ring(NF, NP);
    static constexpr int kB = 4;
};

// FROM_A: the channel mean A is given and K is formed here, else K is given.
template <int NF, int NP, int WF, int VW, bool CHAIN, bool FROM_A>
__global__ __launch_bounds__(kThreads, NP >= 3 ? 2 : 3) void conv_mfma_tile_kernel(TileParams p)
{
    extern __shared__ uint4 lds[];
    constexpr int WP = 4 / WF, PT = WP * NP * 32, FT = WF * NF * 32;
    constexpr int RA = Depth<NF, NP>::kA, RB = Depth<NF, NP>::kB;
    static_assert(RA % RB == 0, "the loop is unrolled RA times");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wf = wave % WF, wp = wave / WF;
    const int l32 = lane & 31, kg = lane >> 5;
    const int OHW = p.OH * p.OW;

    // XCD x (workgroup id mod 8) takes the x-th eighth of the pixel tiles and their filter groups, a tile's
    // groups one after the other: they find its input in that XCD's L2.  (Eighths of the workgroups, not
    // of the tiles: with three filter groups of 169 tiles, 66 workgroups on an XCD's 32 compute units
    // instead of 64 meant a third round.)
    const int item = (blockIdx.x & (kXcds - 1)) * p.wgs_per_xcd + (blockIdx.x >> kXcdShift);
    int fgrp;
    const int ptile = div_scalar((uint32_t)item, (uint32_t)p.fgroups, p.mGroups, fgrp);
    if (ptile >= p.ptiles) return;           // padding of the last XCD's range (uniform over the workgroup)

    // (tiles of an image of their own, or of the whole batch where these would leave too many slots idle)
    int p0 = ptile * PT, p1 = min(p.npix, p0 + PT);
    if (p.per_image) {
        int k;
        const int n = div_scalar((uint32_t)ptile, (uint32_t)p.per_image, p.mImage, k);
        p0 = n * OHW + k * PT;
        p1 = min((n + 1) * OHW, p0 + PT);
    }
    int in_row, oy0, oy_last, unused;        // the first pixel's column and row, the last pixel's row
    const int R0 = div_scalar((uint32_t)p0, (uint32_t)p.OW, p.mOW, in_row);
    const int n_first = div_scalar((uint32_t)R0, (uint32_t)p.OH, p.mOH, oy0);
    const int rows = div_scalar((uint32_t)(in_row + p1 - p0 - 1), (uint32_t)p.OW, p.mOW, unused) + 1;
    const int r0 = (p.OH - 1 - oy0) * p.sh + p.kh;   // staged rows of the first image if the tile runs past it
    const int dn_last = div_scalar((uint32_t)(oy0 + rows - 1), (uint32_t)p.OH, p.mOH, oy_last);
    const int srows = dn_last == 0 ? (oy_last - oy0) * p.sh + p.kh
                                   : r0 + (dn_last - 1) * p.RHfull + oy_last * p.sh + p.kh;
    const int nslots = srows * p.Wp;

    // where staged slot `slot` lies in the input: pixel index from the first image, or -1 outside
    auto slot_pixel = [&](uint32_t slot) -> int {
        const uint32_t row = div_small(slot, p.iWp);
        const uint32_t ix = slot - __umul24(row, (uint32_t)p.Wp) - (uint32_t)p.pw;
        uint32_t dn = 0, iy = (uint32_t)(oy0 * p.sh - p.ph) + row;
        if (dn_last > 0) {                   // (uniform)
            const uint32_t t = row - (uint32_t)r0, sg = div_small(t, p.iRH);
            const bool past = (int)row >= r0;
            dn = past ? 1 + sg : 0u;
            iy = past ? t - __umul24(sg, (uint32_t)p.RHfull) - (uint32_t)p.ph : iy;
        }
        const bool in = iy < (uint32_t)p.H && ix < (uint32_t)p.W;
        const uint32_t px = __umul24(__umul24(dn, (uint32_t)p.H) + iy, (uint32_t)p.W) + ix;
        return in ? (int)px : -1;
    };
    typedef typename WordVec<VW>::type wvec;
    const int CHV = p.Cw / VW, items = nslots * CHV;
    const uint32_t *const src = p.Ipk + (long long)n_first * p.H * p.W * p.Cw;
    constexpr int UP = 4;                    // items per thread in flight
    wvec sv[UP];
    int dst[UP], at[UP];                     // LDS slot and word, pixel of an item
    auto fetch = [&](int first) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            if (first + u * kThreads >= items) break;                            // (uniform)
            const uint32_t it = (uint32_t)min(first + u * kThreads + tid, items - 1);   // (the last one again: no branch)
            const uint32_t slot = div_small(it, p.iCHV);
            const int w = (int)(it - __umul24(slot, (uint32_t)CHV)) * VW;
            const int px = slot_pixel(slot);
            at[u] = px;
            dst[u] = (int)(__umul24(slot, (uint32_t)p.pitch16) + (uint32_t)w);
            const uint32_t off = (__umul24((uint32_t)px, (uint32_t)p.Cw) + (uint32_t)w) * 4u;
            sv[u] = *reinterpret_cast<const wvec *>(reinterpret_cast<const char *>(src) + (px >= 0 ? off : 0u));
        }
    };
    auto put = [&](int first) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            if (first + u * kThreads >= items) break;                            // (uniform)
            uint32_t words[VW];
            if constexpr (VW == 1) words[0] = sv[u];
            if constexpr (VW == 4) { words[0] = sv[u].x; words[1] = sv[u].y; words[2] = sv[u].z; words[3] = sv[u].w; }
            const uint32_t mask = at[u] >= 0 ? 0x03030303u : 0u, zero = at[u] >= 0 ? 0u : kZeroBytes;
#pragma unroll
            for (int k = 0; k < VW; ++k) {
                lds[dst[u] + k] = expand_word_or_zero(words[k], mask, zero);   // (tail channels meet filter zeros)
            }
        }
    };
    fetch(0);
    // The channel mean of the slots, fetched beside the words (a load and its LDS write in one loop waited for
    // everything in flight, once per 256 slots).
    constexpr int UA = 4;
    static_assert(UA == UP, "items are slots where a slot is one item");
    float av[UA];
    int apx[UA];
    const float *const amean = p.A + (FROM_A ? (long long)n_first * p.H * p.W : 0);
    if constexpr (FROM_A) {
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            if (u * kThreads >= nslots) break;                                   // (uniform)
            apx[u] = CHV == 1 ? at[u] : slot_pixel((uint32_t)min(u * kThreads + tid, nslots - 1));
            av[u] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(amean) + (uint32_t)max(apx[u], 0) * 4u);
        }
    }
    // The XCD's workgroups of this filter group are about to walk the same filter operands at the same
    // pace, each line's first reader waiting for memory.  Each of them touches an eighth of the lines now.
    const int f0 = fgrp * FT;
    const char *const wx_lines = reinterpret_cast<const char *>(p.Wx + (long long)(f0 >> 5) * p.tile_steps * 64);
    const int nlines = FT / 32 * p.tile_steps * 8;          // of 128 bytes
    constexpr int kTouch = 4;
    int touched[kTouch];
#pragma unroll
    for (int k = 0; k < kTouch; ++k) {
        const int line = ((k * 8 + (ptile & 7)) * kThreads) + tid;
        touched[k] = *reinterpret_cast<const int *>(wx_lines + (uint32_t)min(line, nlines - 1) * 128u);
    }
    // alpha and A beside it
    float *const Al = reinterpret_cast<float *>(lds + p.al16);
    float *const As = reinterpret_cast<float *>(lds + p.a16);
    // byte offset of a step's pixel operands; past the last step: the last one's (read, not used).  (One entry in, so
    // that entry RB - 1, where the loop's reads of four begin, is 16-byte aligned)
    uint32_t *const Tab = reinterpret_cast<uint32_t *>(lds + p.tab16) + 1;
    static_assert(RB == 4, "see Tab");
    for (int s = tid; s < p.T + kTabTail - 1; s += kThreads) {
        const uint32_t st = (uint32_t)min(s, p.T - 1), tap = div_small(st, p.iS2), ky = div_small(tap, p.ikw);
        const uint32_t slot = __umul24(ky, (uint32_t)(p.Wp - p.kw)) + tap;
        Tab[s] = (__umul24(slot, (uint32_t)p.pitch16) + 2u * (st - __umul24(tap, (uint32_t)p.S2))) * 16u;
    }
    const float a_mine = tid < FT && f0 + tid < p.F ? p.alpha[f0 + tid] : 0.f;

    // this lane's pixels
    uint32_t bB[NP];                          // LDS byte address of tap (0,0), its half of the channels
    int slot0[NP];
    int opix[NP];                             // pixel within the image range, -1: none
    int odn[NP];
    float kv[NP];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)lds;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int q = (wp * NP + j) * 32 + l32;
        const bool has = p0 + q < p1;
        const int t = in_row + (has ? q : 0);
        const int Rl = (int)div_small((uint32_t)t, p.iOW), ox = t - Rl * p.OW;
        odn[j] = (int)div_small((uint32_t)(oy0 + Rl), p.iOH);
        const int oy = oy0 + Rl - odn[j] * p.OH;
        const int srow = odn[j] == 0 ? (oy - oy0) * p.sh : r0 + (odn[j] - 1) * p.RHfull + oy * p.sh;
        slot0[j] = srow * p.Wp + ox * p.sw;
        bB[j] = lds_base + (uint32_t)(slot0[j] * p.pitch16 + kg) * 16u;
        opix[j] = has ? oy * p.OW + ox : -1;
        kv[j] = !FROM_A && has ? p.K[p0 + q] : 0.f;
    }
    const char *wx[NF];                       // (scalar bases; the lane's part is one register)
    const uint32_t lane16 = (uint32_t)lane * 16u;
#pragma unroll
    for (int i = 0; i < NF; ++i) wx[i] = reinterpret_cast<const char *>(p.Wx + ((long long)((f0 >> 5) + wf * NF + i) * p.tile_steps) * 64);

    for (int it = 0;;) {
        put(it);
        it += UP * kThreads;
        if (it >= items) break;               // (uniform)
        fetch(it);
    }
    if constexpr (FROM_A) {
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            if (u * kThreads >= nslots) break;                                   // (uniform)
            As[min(u * kThreads + tid, nslots - 1)] = apx[u] >= 0 ? av[u] : 0.f; // (the last slot again: the same value)
        }
        for (int s = UA * kThreads + tid; s < nslots; s += kThreads) {
            const int px = slot_pixel((uint32_t)s);
            const float v = amean[max(px, 0)];
            As[s] = px >= 0 ? v : 0.f;
        }
    }
#pragma unroll
    for (int k = 0; k < kTouch; ++k) asm volatile("" : : "v"(touched[k]));    // (long since arrived)
    if (tid < FT) Al[tid] = a_mine;

    v4i a[RA][NF], b[RB][NP];
#pragma unroll
    for (int s = 0; s + 1 < RA; ++s)
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            a[s][i] = *reinterpret_cast<const v4i *>(wx[i] + (s * 1024 + lane16));
            __builtin_amdgcn_sched_barrier(0);    // (in this order: the loop waits for them one by one)
        }
    v16f acc[NF][NP];
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int j = 0; j < NP; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    __syncthreads();

    // The flat sequence of (tap, 64 channels) steps: whole turns of the operand ring, then what is left.  A
    // wave issues in order, so whatever stands between two matrix instructions beyond the 32 cycles of the
    // first delays the pipe (scalar arithmetic for the walk over taps and channels did: 283 cycles a step
    // instead of 128).  The steps' byte offsets therefore come from a table in LDS, four to a read, and each
    // load or read is laid behind a matrix instruction of its own; the fences keep the order.
    uint4 offs[RA / 4];                       // of the turn's pixel reads: steps t + RB - 1 ..
    const uint32_t *tab_at = Tab + (RB - 1);
    auto read_offs = [&](int q) __attribute__((always_inline)) {
        offs[q] = *reinterpret_cast<const uint4 *>(tab_at + 4 * q);
    };
    auto off_of = [&](int u) -> uint32_t {
        const uint4 o = offs[u >> 2];
        return (u & 3) == 0 ? o.x : (u & 3) == 1 ? o.y : (u & 3) == 2 ? o.z : o.w;
    };
    auto read_b = [&](v4i &to, int j, uint32_t off) __attribute__((always_inline)) {
        to = *(const __attribute__((address_space(3))) v4i *)(uintptr_t)(bB[j] + off);
    };
    auto load_a = [&](v4i &to, int i, int step) __attribute__((always_inline)) {
        to = *reinterpret_cast<const v4i *>(wx[i] + (step * 1024 + lane16));
    };
    auto product = [&](int i, int j, const v4i &x, const v4i &y) __attribute__((always_inline)) {
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
            __builtin_shufflevector(x, x, 0, 1, 2, 3, -1, -1, -1, -1),
            __builtin_shufflevector(y, y, 0, 1, 2, 3, -1, -1, -1, -1), acc[i][j], 4, 4, 0, 0, 0, 0);
    };
    // K of the lane's pixels, a tap per step (there are at least as many steps as taps): the sum, order
    // and rounding of box_filter_K_kernel
    double ksum[NP];
    float kval[NP];
    int ktap = 0, kslot = 0, kkx = 0;
    const int taps = p.kh * p.kw;
    auto k_read = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NP; ++j) kval[j] = As[slot0[j] + kslot];
        const bool wrap = kkx + 1 == p.kw;
        kslot += wrap ? p.Wp - p.kw + 1 : 1;
        kkx = wrap ? 0 : kkx + 1;
        kslot = ktap + 1 < taps ? kslot : 0;
    };
    auto k_add = [&](int j) __attribute__((always_inline)) { ksum[j] += ktap < taps ? (double)kval[j] : 0.0; };
    if constexpr (FROM_A) {
#pragma unroll
        for (int j = 0; j < NP; ++j) ksum[j] = 0.0;
        k_read();
    }
#pragma unroll
    for (int q = 0; q < RA / 4; ++q) read_offs(q);
#pragma unroll
    for (int s = 0; s + 1 < RB; ++s)
#pragma unroll
        for (int j = 0; j < NP; ++j) read_b(b[s][j], j, Tab[s]);
    int t = 0;
    auto turn = [&](auto with_k) __attribute__((always_inline)) {
        constexpr bool WITH_K = decltype(with_k)::value;
#pragma unroll
        for (int u = 0; u < RA; ++u) {
            // what this step issues, a piece behind each of its matrix instructions
            constexpr int M = NF * NP;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                product(m / NP, m % NP, a[u][m / NP], b[u % RB][m % NP]);
                if (m < NF) load_a(a[(u + RA - 1) % RA][m], m, u + RA - 1);
                if (m >= M - NP) read_b(b[(u + RB - 1) % RB][m - (M - NP)], m - (M - NP), off_of(u));
                if (WITH_K && m < NP) k_add(m);
                if (WITH_K && m == M - 1) { ++ktap; k_read(); }
                if (m == M - 1 && (u & 3) == 3) {                 // the offsets of the next turn's four steps
                    tab_at += 4;
                    offs[u >> 2] = *reinterpret_cast<const uint4 *>(tab_at + (RA - 4));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < NF; ++i) wx[i] += RA * 1024;
        t += RA;
    };
    if constexpr (FROM_A)
        while (t + RA <= p.T && ktap < taps) turn(std::integral_constant<bool, true>{});
    while (t + RA <= p.T) turn(std::integral_constant<bool, false>{});
#pragma unroll
    for (int u = 0; u + 1 < RA; ++u) {
        if (t + u >= p.T) break;
#pragma unroll
        for (int j = 0; j < NP; ++j) read_b(b[(u + RB - 1) % RB][j], j, off_of(u));
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < NP; ++j) product(i, j, a[u][i], b[u % RB][j]);
        if constexpr (FROM_A) {
#pragma unroll
            for (int j = 0; j < NP; ++j) k_add(j);
            ++ktap;
            k_read();
        }
    }
    if constexpr (FROM_A)
#pragma unroll
        for (int j = 0; j < NP; ++j) kv[j] = (float)(ksum[j] / (double)(p.kh * p.kw));
    // accumulator register r of a lane: filter row 8*(r/4) + 4*kg + r%4 of the wave's tile, pixel column l32
    if constexpr (CHAIN) {
        double total[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) total[j] = 0.0;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int ft = f0 + (wf * NF + i) * 32, nfilt = p.F - ft;     // (uniform) how many of the tile's 32 exist
            if (nfilt <= 0) break;
            float al[16];
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const float4 v = *reinterpret_cast<const float4 *>(&Al[(wf * NF + i) * 32 + 2 * r + 4 * kg]);
                al[r] = v.x; al[r + 1] = v.y; al[r + 2] = v.z; al[r + 3] = v.w;
            }
            auto filter_tile = [&](auto whole) __attribute__((always_inline)) {
                // (filters that exist only: past the last one alpha is 0, but an infinite K makes that NaN)
                constexpr bool WHOLE = decltype(whole)::value;
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    uint32_t word = 0;
                    double sum = 0.0;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = 8 * (r >> 2) + (r & 3);           // (+ 4 * kg)
                        const float o = acc[i][j][r] * (kv[j] * al[r]);
                        word |= (o >= 0.f ? 1u : 0u) << row;
                        sum += (double)(WHOLE || row + 4 * kg < nfilt ? fabsf(o) : 0.f);
                    }
                    word <<= 4 * kg;
                    word |= (uint32_t)__shfl_xor((int)word, 32);
                    if (!WHOLE) word &= (1u << nfilt) - 1u;
                    total[j] += sum;
                    if (kg == 0 && opix[j] >= 0)
                        p.Opk[(long long)(p0 + (wp * NP + j) * 32 + l32) * p.Cwn + (ft >> 5)] = word;
                }
            };
            if (nfilt >= 32) filter_tile(std::true_type{});
            else filter_tile(std::false_type{});
        }
        const int part = fgrp * WF + wf;
        if (f0 + wf * NF * 32 < p.F) {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const double sum = total[j] + __shfl_xor(total[j], 32);
                // (as the mean of the sums over 32 filters: a larger one would leave fp32's range sooner than they do)
                if (kg == 0 && opix[j] >= 0)
                    p.P[(long long)(p0 + (wp * NP + j) * 32 + l32) * p.parts + part] = (float)(sum * (1.0 / NF));
            }
        }
    } else {
        constexpr int kRaw = 0x00027000;      // (a plain buffer of dwords)
        constexpr int kWriteThrough = 16;     // a buffer store's sc1 bit (agent scope): past the L2 of the XCD
        uint32_t voff[NP];                    // byte offset from the first image's plane of filter row 0; no pixel: beyond the buffer
#pragma unroll
        for (int j = 0; j < NP; ++j)
            voff[j] = opix[j] < 0 ? 0xfffffff0u : (uint32_t)((odn[j] * p.F + 4 * kg) * OHW + opix[j]) * 4u;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int ft = f0 + (wf * NF + i) * 32, nfilt = p.F - ft;
            if (nfilt <= 0) break;
            float al[16];
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const float4 v = *reinterpret_cast<const float4 *>(&Al[(wf * NF + i) * 32 + 2 * r + 4 * kg]);
                al[r] = v.x; al[r + 1] = v.y; al[r + 2] = v.z; al[r + 3] = v.w;
            }
            const long long plane = ((long long)n_first * p.F + ft) * OHW;
            auto store_tile = [&](auto aux, auto value, void *base) __attribute__((always_inline)) {
                // (a scalar buffer per row of filters: no vector arithmetic for the addresses)
                const auto buf = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, kRaw);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 8 * (r >> 2) + (r & 3);
                    if (nfilt >= 32) {
#pragma unroll
                        for (int j = 0; j < NP; ++j)
                            __builtin_amdgcn_raw_buffer_store_b32(value(j, r), buf, (int)voff[j], row * OHW * 4, aux);
                    } else {
#pragma unroll
                        for (int j = 0; j < NP; ++j)
                            __builtin_amdgcn_raw_buffer_store_b32(value(j, r), buf, (int)(row + 4 * kg < nfilt ? voff[j] : 0xfffffff0u), row * OHW * 4, aux);
                    }
                }
            };
            auto store_both = [&](auto aux) __attribute__((always_inline)) {
                store_tile(aux, [&](int j, int r) { return __float_as_uint(acc[i][j][r] * (kv[j] * al[r])); }, p.out + plane);
                if (p.dot) store_tile(aux, [&](int j, int r) { return (uint32_t)(int)acc[i][j][r]; }, p.dot + plane);
            };
            if (p.write_through) store_both(std::integral_constant<int, kWriteThrough>{});
            else store_both(std::integral_constant<int, 0>{});
        }
    }
}

struct TPlan {
    bool ok;
    int NF, NP, WF, Wp, RHfull, S2, T, tile_steps, pitch16, slots_max, per_image;
    long long ptiles;
    size_t lds, lds_request, ws_bytes;
};

// most slots a tile of `pt` pixels can need: its rows with their halos, and those of the images it crosses
long long slots_of(const Geom &g, int pt, bool per_image, long long wp, long long rh)
{
    const long long total_rows = per_image ? g.OH : (long long)g.N * g.OH;
    const long long rows = std::min<long long>(total_rows, ((long long)pt + g.OW - 2) / g.OW + 1);
    if (per_image) return ((rows - 1) * g.sh + g.kh) * wp;
    long long most = 0;
    for (int oy0 = 0; oy0 < g.OH; ++oy0) {
        const long long last = oy0 + rows - 1, n_last = last / g.OH, oy_last = last % g.OH;
        const long long sr = n_last == 0 ? (oy_last - oy0) * g.sh + g.kh
                                         : (long long)(g.OH - 1 - oy0) * g.sh + g.kh + (n_last - 1) * rh + oy_last * g.sh + g.kh;
        most = std::max(most, sr);
    }
    return most * wp;
}

// Wave tiles: NF, NP, WF.  64 x 64 needs two LDS reads and two filter loads per four matrix instructions,
// which is about what the vector cache delivers (64 bytes a cycle); 64 x 96 is gentler on it, the smaller
// ones spread a small layer over more SIMDs; four waves along the filters halve the input under a workgroup
// (many channels).
constexpr int kShapes[][3] = {{2, 2, 2}, {2, 3, 2}, {2, 2, 4}, {2, 1, 2}, {1, 1, 2}, {2, 2, 1}, {2, 1, 1}, {1, 1, 1}};

// The hardware may put a third workgroup on one unit while another has one: where a unit is to have r = one or
// two, a launch asks for so much LDS that no more of it fit, and no more than that: what is left (half or a
// third) is for the kernels of other streams.  (Asking for all of it or for half keeps those off the unit; the same
// times to 0.1 us over 1 x 256 x 7 x 7 .. 64 x 256 x 14 x 14.)
constexpr size_t kLdsGranule = 1280;
constexpr size_t lds_to_ask_for(size_t lds, long long r)
{
    if (r > 2) return lds;
    const size_t no_more = kLdsMax / (r + 1) / kLdsGranule * kLdsGranule + kLdsGranule;
    return lds > no_more || lds > kLdsMax / r ? lds : no_more;
}
static_assert(lds_to_ask_for(1024, 1) > kLdsMax / 2 && lds_to_ask_for(1024, 1) + 64 * 1024 <= kLdsMax, "one and others'");
static_assert(3 * lds_to_ask_for(1024, 2) > kLdsMax && 2 * lds_to_ask_for(1024, 2) + 48 * 1024 <= kLdsMax, "two and others'");

// The shape with the smallest estimate of the launch's length in cycles: with r = the most workgroups a
// compute unit gets, r times (steps x what a step costs, matrix instructions or operand loads, and the
// stores), and once per batch of resident workgroups the set-up and the first loads (5000: stamps on 64 x
// 256 x 14 x 14: set-up 2.3 k, first words and their expansion 2.8 k, loop 6.4 k, stores 3.7 k).
TPlan search_tplan(const Geom &g)
{
    TPlan best{};
    const long long wp = (long long)(g.OW - 1) * g.sw + g.kw, rh = (long long)(g.OH - 1) * g.sh + g.kh;
    const long long npix = (long long)g.N * g.OH * g.OW, OHW = (long long)g.OH * g.OW;
    if (wp > 4096 || rh > 4096 || g.OW > 4096 || g.OH > 4096 || npix > (1LL << 30)) return best;   // (div_small's range)
    const int S2 = (g.Cw + 1) / 2;
    const long long T = (long long)g.kh * g.kw * S2;
    if (T > 8192) return best;
    const int cus = kPlanUnits;
    const int pitch16 = (2 * S2) | 1;
    double least = 0;
    for (const auto &s : kShapes) {
        const int NF = s[0], NP = s[1], WF = s[2];
        const int pt = 4 / WF * NP * 32, ft = WF * NF * 32;
        if (ft > 32 && ceil_div(g.F, ft / 2) < 2) continue;           // (half of the workgroup without filters)
        const long long per_image = ceil_div(OHW, pt);
        const bool own = per_image * pt * 20 <= OHW * 21;             // at most a twentieth of the slots idle
        const long long ptiles = own ? per_image * g.N : ceil_div(npix, pt);
        const long long slots = slots_of(g, pt, own, wp, rh);
        const size_t lds = (size_t)slots * pitch16 * 16 + (((size_t)T + kTabTail + 3) & ~(size_t)3) * 4 + (size_t)ft * 4 +
                           (((size_t)slots * 4 + 15) & ~(size_t)15);
        if (slots > (1 << 15) || lds > kLdsMax || slots * g.Cw >= (1 << 20)) continue;
        // 32-bit offsets: a tile's outputs from its first image's plane, its input words
        const long long images = (pt - 1) / OHW + 2;
        if ((images * g.F + 32) * OHW * 4 >= (1LL << 31) || images * g.H * g.W * g.Cw >= (1LL << 30) ||
            images * g.H * g.W >= (1LL << 24))
            continue;
        const long long fgroups = ceil_div(g.F, ft), wgs = ptiles * fgroups;
        if ((ptiles + 8) * fgroups > (1LL << 30)) continue;
        const long long r = ceil_div(ceil_div(wgs, kXcds), std::max(1, cus / kXcds));
        const int resident = (int)std::min<size_t>(NF * NP >= 6 ? 2 : 3, kLdsMax / lds);
        const double step = std::max(32.0 * NF * NP, 70.0 * NF);
        const double cost = (double)((r + resident - 1) / resident) * 5000.0 + (double)r * ((double)T * step + 900.0 * NF * NP);
        if (best.ok && cost >= least) continue;
        least = cost;
        best.ok = true;
        best.NF = NF; best.NP = NP; best.WF = WF; best.slots_max = (int)slots; best.per_image = own ? (int)per_image : 0;
        best.ptiles = ptiles; best.lds = lds;
        best.lds_request = lds_to_ask_for(lds, r);
    }
    best.Wp = (int)wp; best.RHfull = (int)rh; best.S2 = S2; best.T = (int)T; best.pitch16 = pitch16;
    if (best.ok) {
        best.tile_steps = (int)T + operand_ring(best.NF, best.NP) - 1;
        const int ft = best.WF * best.NF * 32;
        best.ws_bytes = (size_t)ceil_div(g.F, ft) * (ft / 32) * best.tile_steps * 64 * sizeof(uint4);
    }
    return best;
}

const TPlan &make_tplan(const Geom &g)
{
    static thread_local PlanMemo<TPlan> memo;
    return memo.get(g, 0, [&] { return search_tplan(g); });
}

template <int NF, int NP, int WF>
hipError_t launch_shape(const TileParams &p, bool vec4, unsigned grid, size_t lds, hipStream_t st)
{
    auto launch = [&](auto kernel, int slot) -> hipError_t {
        // raise the kernel's dynamic-LDS limit once per device and instance
        static std::atomic<unsigned long long> raised[8];
        if (lds > 64 * 1024) {
            int dev = 0;
            hipError_t err = hipGetDevice(&dev);
            if (err != hipSuccess) return err;
            const unsigned long long bit = 1ull << (dev & 63);
            if (!(raised[slot].load(std::memory_order_acquire) & bit)) {
                err = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax);
                if (err != hipSuccess) return err;
                raised[slot].fetch_or(bit, std::memory_order_release);
            }
        }
        kernel<<<dim3(grid), dim3(kThreads), lds, st>>>(p);
        return hipGetLastError();
    };
    if (p.A) {
        if (p.Opk) return vec4 ? launch(conv_mfma_tile_kernel<NF, NP, WF, 4, true, true>, 0) : launch(conv_mfma_tile_kernel<NF, NP, WF, 1, true, true>, 1);
        return vec4 ? launch(conv_mfma_tile_kernel<NF, NP, WF, 4, false, true>, 2) : launch(conv_mfma_tile_kernel<NF, NP, WF, 1, false, true>, 3);
    }
    if (p.Opk) return vec4 ? launch(conv_mfma_tile_kernel<NF, NP, WF, 4, true, false>, 4) : launch(conv_mfma_tile_kernel<NF, NP, WF, 1, true, false>, 5);
    return vec4 ? launch(conv_mfma_tile_kernel<NF, NP, WF, 4, false, false>, 6) : launch(conv_mfma_tile_kernel<NF, NP, WF, 1, false, false>, 7);
}

}  // namespace

bool conv_mfma_tile_supports(const Geom &g) { return make_tplan(g).ok; }

// Up to 18.5 k cycles of matrix instructions per SIMD; above that the set-up is a small part of the persistent
// kernel and its larger wave tiles (half the operand traffic per instruction) count for more.  Measured with
// K given / with A given, us per launch in a replayed graph, the faster of the persistent and the
// one-workgroup-per-band kernel -> this one:
//   1 x 64 x 32 x 32 F=64 3x3          7.6 / 8.3 -> 3.9 / 4.4     1 x 512 x 7 x 7 F=512 3x3     12.2 / 13.3 -> 5.8 / 6.5
//   5 x 100 x 37 x 53 F=75 3x3       10.1 / 11.4 -> 4.9 / 5.8     64 x 512 x 7 x 7 F=512 3x3    16.4 / 17.7 -> 9.8 / 10.2
//   64 x 128 x 28 x 28 F=256 3x3 s2  14.0 / 14.8 -> 8.3 / 9.4     64 x 256 x 28 x 28 F=512 1x1  26.0 / 26.8 -> 21.0 / 21.5
//   64 x 256 x 14 x 14 F=256 3x3     12.9 / 14.3 -> 9.3 / 10.1    16 x 64 x 112 x 112 F=64 3x3  22.8 / 24.6 -> 16.0 / 17.9
//   128 x 384 x 13 x 13 F=384 3x3    23.2 / 24.6 -> 19.2 / 19.2   16 x 128 x 56 x 56 F=128 5x5  17.0 / 19.7 -> 15.7 / 16.2
//   (19.2 k cycles) 16 x 128 x 56 x 56 F=128 7x7 22.6 / 26.0 against 23.1 / 24.3 here
//   (28 k) 32 x 512 x 28 x 28 F=512 3x3 31.8 / 33.2 against 35.0 / 35.3; (36 k) 128 x 96 x 27 x 27 F=256 5x5 40.9 against 41.0
bool conv_mfma_tile_preferred(const Geom &g)
{
    const TPlan &pl = make_tplan(g);
    if (!pl.ok) return false;
    const double per_simd = (double)g.N * g.OH * g.OW * (double)(ceil_div(g.F, 32) * 32) * pl.T * 32 / 1024 / (4.0 * kPlanUnits);
    return per_simd <= 18500.0;
}

ExpandLayout conv_mfma_tile_expand_layout(const Geom &g)
{
    const TPlan &pl = make_tplan(g);
    ExpandLayout L{};
    L.ok = pl.ok ? 1 : 0;
    L.CH = 2 * pl.S2; L.nchunks = 1; L.chunk_pad = pl.T; L.tile_steps = pl.tile_steps;
    L.Cw2 = 2 * pl.S2; L.ws_bytes = pl.ws_bytes;
    return L;
}

int conv_mfma_tile_sum_parts(const Geom &g)
{
    const TPlan &pl = make_tplan(g);
    return pl.ok ? ceil_div(g.F, 32 * pl.NF) : 0;
}

int conv_mfma_tile_sum_scale(const Geom &g) { return make_tplan(g).NF; }

hipError_t launch_conv_mfma_tile(const uint32_t *Ipk, const float *K, const float *A, const float *alpha,
                                 const Geom &g, float *out, int32_t *dot, uint32_t *Opk, float *P,
                                 const void *workspace, hipStream_t st)
{
    const TPlan &pl = make_tplan(g);
    if (!pl.ok) return hipErrorInvalidValue;
    TileParams p{};
    p.Ipk = Ipk; p.Wx = static_cast<const uint4 *>(workspace); p.K = K; p.A = A; p.alpha = alpha;
    p.out = out; p.dot = dot; p.Opk = Opk; p.P = P; p.Cwn = (g.F + 31) / 32; p.parts = ceil_div(g.F, 32 * pl.NF);
    p.C = g.C; p.H = g.H; p.W = g.W; p.F = g.F; p.kh = g.kh; p.kw = g.kw; p.sh = g.sh; p.sw = g.sw;
    p.ph = g.ph; p.pw = g.pw; p.OH = g.OH; p.OW = g.OW; p.Cw = g.Cw; p.N = g.N;
    p.npix = g.N * g.OH * g.OW;
    const int ft = pl.WF * pl.NF * 32;
    p.per_image = pl.per_image;
    p.ptiles = (int)pl.ptiles; p.fgroups = ceil_div(g.F, ft);
    p.wgs_per_xcd = ceil_div((long long)p.ptiles * p.fgroups, kXcds);
    p.Wp = pl.Wp; p.RHfull = pl.RHfull; p.S2 = pl.S2; p.T = pl.T; p.tile_steps = pl.tile_steps; p.pitch16 = pl.pitch16;
    // Where the planes of `out` and `dot` begin on 64-byte boundaries, their stores leave the L2 as they come (agent
    // scope): otherwise it is written back when the kernel ends, while nothing computes.  Planes that begin elsewhere share 64-byte
    // units with their neighbours, which are written twice then: while the kernel runs past 45 MB or so, and when the next one reads
    // them before.  Written back / through by time, 1x1 and 3x3, 64 to 256 channels and filters:
    //   MB of outputs                                       8     13     20     32     38     64    100    160
    //   64-byte boundaries, alone                         1.01                 1.14          1.11   1.08   1.05
    //     with a kernel that reads the outputs next       1.00   1.01   1.01   1.01   1.03   1.06
    //   16-byte boundaries, alone                         1.01                 1.06          1.00   0.96   0.90
    //     with a kernel that reads the outputs next       0.99   0.92   0.87   0.81   0.78
    // us per launch, written back -> through: 64 x 256 x 28 x 28 F=512 1x1 27.6 -> 22.3, 16 x 128 x 56 x 56 F=128 5x5 15.7 -> 14.0,
    // 64 x 128 x 28 x 28 F=128 3x3 10.6 -> 9.4.
    const uintptr_t at = reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(dot) | (uintptr_t)g.OH * g.OW * 4;
    p.write_through = (at & 63) == 0;
    p.tab16 = pl.slots_max * pl.pitch16;
    p.al16 = p.tab16 + (pl.T + kTabTail + 3) / 4;
    p.a16 = p.al16 + ft / 4;
    const bool vec4 = g.Cw % 4 == 0 && (reinterpret_cast<uintptr_t>(Ipk) & 15) == 0;
    p.iCHV = 1.0f / (float)(g.Cw / (vec4 ? 4 : 1));
    p.iWp = 1.0f / (float)pl.Wp;
    p.iRH = 1.0f / (float)pl.RHfull;
    p.mGroups = scalar_reciprocal(p.fgroups);
    p.mImage = scalar_reciprocal(p.per_image);
    p.mOW = scalar_reciprocal(g.OW);
    p.mOH = scalar_reciprocal(g.OH);
    p.iOW = 1.0f / (float)g.OW;
    p.iOH = 1.0f / (float)g.OH;
    p.iS2 = 1.0f / (float)pl.S2;
    p.ikw = 1.0f / (float)g.kw;
    const unsigned grid = (unsigned)(kXcds * p.wgs_per_xcd);
    switch (pl.NF * 100 + pl.NP * 10 + pl.WF) {
        case 222: return launch_shape<2, 2, 2>(p, vec4, grid, pl.lds_request, st);
        case 232: return launch_shape<2, 3, 2>(p, vec4, grid, pl.lds_request, st);
        case 224: return launch_shape<2, 2, 4>(p, vec4, grid, pl.lds_request, st);
        case 212: return launch_shape<2, 1, 2>(p, vec4, grid, pl.lds_request, st);
        case 112: return launch_shape<1, 1, 2>(p, vec4, grid, pl.lds_request, st);
        case 221: return launch_shape<2, 2, 1>(p, vec4, grid, pl.lds_request, st);
        case 211: return launch_shape<2, 1, 1>(p, vec4, grid, pl.lds_request, st);
        default: return launch_shape<1, 1, 1>(p, vec4, grid, pl.lds_request, st);
    }
}

}  // namespace xnor
