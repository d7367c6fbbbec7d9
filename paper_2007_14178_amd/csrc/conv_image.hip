// The whole forward pass in one kernel for images with one to four channels (first layers, and the
// workload the paper itself times: one channel, 3x3 filter, 256^2 ... 2048^2 pixels, Tables I-III).
//
// With so few channels a channel-packed word carries one to four useful bits, and per output there
// are only kh*kw*C binary MACs against 4 bytes read and 4*F bytes written: the layer is a stream
// through HBM, not arithmetic.  So nothing intermediate is written: steps 1a-1d, 2a-2b and 3 of
// Sec. III-A (Eq. 10, Eq. 11) run on registers between one read of the fp32 image and one write of
// the fp32 output.
//   * A lane owns one output column of a band of rows and slides down it (with a vertical stride an
//     output is due every sh-th input row).  For every input row it
//     loads the kw*C values under its window, forms their kw*C sign bits (bit = x >= 0) and the sum
//     of their magnitudes, and keeps the last kh of both: the spatially packed window of Sec. III-B
//     (kh*kw*C bits, rows side by side in as few 32-bit words as hold them) and the kh row sums
//     whose total is K * C*kh*kw.
//   * Per output and filter: popcount((window xor filter window) and mask); the mask holds the
//     in-image taps, so a padded tap adds nothing, and popcount(mask) = C * (#in-image taps).
//       dot = popcount(mask) - 2 * popcount(...),   out = float(dot) * K * alpha.
//     For rows whose window lies inside the image vertically the mask is a per-lane constant.
//   * Loads of the next rows are issued a few rows ahead of their use; neighbouring lanes read
//     overlapping addresses, which the vector cache serves.
// The paper's kernels (Alg. 1 and 2) also pack a spatial tile into one register, one channel and one
// 8x4 tile per thread, and run binarisation, K and the convolution as separate kernels on separate
// streams; here the row words live only in registers and the three are one pass.
#include <algorithm>

#include "xnor_internal.hpp"

namespace xnor {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr size_t kLdsBudget = 64 * 1024;

struct ImageParams {
    const float *I;
    const uint32_t *Wpk;
    const float *alpha;
    float *out;
    int32_t *dot;
    int N, H, W, F, OH, OW, ph, pw, sh, sw;
    int rows_per_band, bands, xtiles;
    int group, fgroups;  // filters per wave, ceil(F / group)
    long long waves;     // N * fgroups * bands * xtiles
    float kscale;        // 1 / (C * kh * kw)
};

template <int K, int C>
struct Cfg {
    static constexpr int kRowBits = K * C;                       // sign bits of one window row
    static constexpr int kRowsPerWord = 32 / kRowBits;
    static constexpr int kWords = (K + kRowsPerWord - 1) / kRowsPerWord;
    static constexpr int kAhead = kRowBits <= 3 ? 8 : kRowBits <= 7 ? 4 : kRowBits <= 12 ? 2 : 1;
    static constexpr uint32_t kChanMask = (1u << C) - 1u;
};

template <int K, int C, bool ONE_FILTER, bool UNIT_STRIDE>
__global__ __launch_bounds__(kThreads) void conv_image_kernel(ImageParams p)
{
    const int sh = UNIT_STRIDE ? 1 : p.sh, sw = UNIT_STRIDE ? 1 : p.sw;   // stride 1 is compiled in
    using G = Cfg<K, C>;
    constexpr int RB = G::kRowBits, NW = G::kWords, RPW = G::kRowsPerWord, D = G::kAhead;
    extern __shared__ uint32_t lds[];        // filter windows [F][NW], then alpha [F]
    uint32_t *wf = lds;
    float *al = reinterpret_cast<float *>(lds + (size_t)p.F * NW);

    // filter windows in the window's bit order: row r of the filter sits at bit (r % RPW) * RB of
    // word r / RPW, tap kx at kx * C inside the row, channel c at bit c of the tap
    auto filter_window = [&](int f, uint32_t (&w)[NW]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NW; ++i) w[i] = 0;
#pragma unroll
        for (int r = 0; r < K; ++r)
#pragma unroll
            for (int kx = 0; kx < K; ++kx)
                w[r / RPW] |= (p.Wpk[((size_t)f * K + r) * K + kx] & G::kChanMask)
                              << ((r % RPW) * RB + kx * C);
    };
    if (!ONE_FILTER) {
        for (int f = threadIdx.x; f < p.F; f += kThreads) {
            uint32_t w[NW];
            filter_window(f, w);
#pragma unroll
            for (int i = 0; i < NW; ++i) wf[(size_t)f * NW + i] = w[i];
            al[f] = p.alpha[f];
        }
        __syncthreads();
    }

    const int lane = threadIdx.x & 63;
    const long long gw = (long long)blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (gw >= p.waves) return;
    const int xt = __builtin_amdgcn_readfirstlane((int)(gw % p.xtiles));
    const long long t = gw / p.xtiles;
    const int band = __builtin_amdgcn_readfirstlane((int)(t % p.bands));
    const long long u = t / p.bands;
    const int f0 = __builtin_amdgcn_readfirstlane((int)(u % p.fgroups)) * p.group;
    const int f1 = min(p.F, f0 + p.group);
    const int n = __builtin_amdgcn_readfirstlane((int)(u / p.fgroups));
    const int x = xt * 64 + lane;
    if (x >= p.OW) return;

    // which of the window's columns lie inside the image: a per-lane constant
    bool cv[K];
    uint32_t row_mask = 0;
#pragma unroll
    for (int kx = 0; kx < K; ++kx) {
        const int xin = x * sw - p.pw + kx;
        cv[kx] = xin >= 0 && xin < p.W;
        row_mask |= cv[kx] ? (G::kChanMask << (kx * C)) : 0u;
    }
    uint32_t full_mask[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) full_mask[i] = 0;
#pragma unroll
    for (int r = 0; r < K; ++r) full_mask[r / RPW] |= row_mask << ((r % RPW) * RB);
    int full_valid = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) full_valid += __builtin_popcount(full_mask[i]);

    const int y0 = band * p.rows_per_band;
    const int y1 = min(p.OH, y0 + p.rows_per_band);
    const int nin = (y1 - y0 - 1) * sh + K;   // input rows this band walks through
    const int yb = y0 * sh - p.ph;            // the first of them (negative: above the image)
    const size_t HW = (size_t)p.H * p.W;
    const float *src = p.I + (size_t)n * C * HW + (x * sw - p.pw);   // only dereferenced where valid
    const size_t OHW = (size_t)p.OH * p.OW;

    float pre[D][RB];
    auto issue = [&](int slot, int i) __attribute__((always_inline)) {
        const int yin = yb + i;
        const bool rv = i < nin && yin >= 0 && yin < p.H;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int kx = 0; kx < K; ++kx)
                pre[slot][c * K + kx] =
                    (rv && cv[kx]) ? src[(size_t)c * HW + (size_t)yin * p.W + kx] : 0.f;
    };

    uint32_t rw[K];   // sign bits of the last K input rows
    float hs[K];      // sums of |I| over those rows' kw*C values
#pragma unroll
    for (int r = 0; r < K; ++r) { rw[r] = 0; hs[r] = 0.f; }

#pragma unroll
    for (int d = 0; d < D; ++d) issue(d, d);

    // a single filter stays in registers: its words come through wave-uniform loads that are in
    // flight together with the first image rows, and no workgroup barrier is needed
    uint32_t fw[NW];
    float a0 = 0.f;
    if (ONE_FILTER) {
        filter_window(0, fw);
        a0 = p.alpha[0];
    }

    int skip = 1;                           // input rows until the next output row is due
    for (int i0 = 0; i0 < nin; i0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int i = i0 + d;
            if (i >= nin) break;
            uint32_t bits = 0;
            float hsum = 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int kx = 0; kx < K; ++kx) {
                    const float v = pre[d][c * K + kx];
                    bits |= (v >= 0.f) ? (1u << (kx * C + c)) : 0u;
                    hsum += fabsf(v);
                }
            issue(d, i + D);
#pragma unroll
            for (int r = 0; r + 1 < K; ++r) { rw[r] = rw[r + 1]; hs[r] = hs[r + 1]; }
            rw[K - 1] = bits;
            hs[K - 1] = hsum;
            // an output row is complete when its last window row has arrived: every sh-th row
            if (i < K - 1) continue;
            if (--skip > 0) continue;
            skip = sh;

            const int y = y0 + (i - (K - 1)) / sh;
            uint32_t win[NW], m[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) win[w] = 0;
#pragma unroll
            for (int r = 0; r < K; ++r) win[r / RPW] |= rw[r] << ((r % RPW) * RB);
            int nvalid;
            const int ytop = y * sh - p.ph;
            if (ytop >= 0 && ytop + K - 1 < p.H) {
#pragma unroll
                for (int w = 0; w < NW; ++w) m[w] = full_mask[w];
                nvalid = full_valid;
            } else {
#pragma unroll
                for (int w = 0; w < NW; ++w) m[w] = 0;
#pragma unroll
                for (int r = 0; r < K; ++r) {
                    const bool rv = ytop + r >= 0 && ytop + r < p.H;
                    m[r / RPW] |= rv ? (row_mask << ((r % RPW) * RB)) : 0u;
                }
                nvalid = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) nvalid += __builtin_popcount(m[w]);
            }
            float ksum = hs[0];
#pragma unroll
            for (int r = 1; r < K; ++r) ksum += hs[r];
            const float kk = ksum * p.kscale;
            const size_t o = (size_t)n * p.F * OHW + (size_t)y * p.OW + x;
            if (ONE_FILTER) {
                int pop = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) pop += __builtin_popcount((win[w] ^ fw[w]) & m[w]);
                const int d1 = nvalid - 2 * pop;
                p.out[o] = (float)d1 * (kk * a0);
                if (p.dot) p.dot[o] = d1;
            } else {
                for (int f = f0; f < f1; ++f) {
                    int pop = 0;
#pragma unroll
                    for (int w = 0; w < NW; ++w)
                        pop += __builtin_popcount((win[w] ^ wf[(size_t)f * NW + w]) & m[w]);
                    const int d1 = nvalid - 2 * pop;
                    p.out[o + (size_t)f * OHW] = (float)d1 * (kk * al[f]);
                    if (p.dot) p.dot[o + (size_t)f * OHW] = d1;
                }
            }
        }
    }
}

// One channel, one filter, the paper's own workload, with "same" padding along x and 16-byte rows: a lane owns
// four neighbouring columns, which it loads and stores 16 bytes at a time.  The K - 1 columns on either side
// of its four are its neighbour lanes' (a wave shift of the registers) or, at the wave's ends, one more load that
// serves the first and the last lane.  Rows slide down as in conv_image_kernel: a window is K * K bits, a
// new row shifts in from the top.  Bound by memory (4 bytes read and 4 written per pixel): a quarter of the
// load instructions and of the address arithmetic of one column per lane.  Sums and roundings are those
// of conv_image_kernel: the same results bit for bit.
struct Row4Params {
    const float *I;
    const uint32_t *Wpk;
    const float *alpha;
    float *out;
    int32_t *dot;
    int H, W, OH, ph;
    int rows_per_band, bands, xtiles;
    long long waves;
    float kscale;
};

// lane l gets lane l - 1's (l + 1's) value; the wave's first (last) lane gets `end`
__device__ inline float from_left(float v, float end)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(end), __float_as_uint(v), 0x138, 0xf, 0xf, false));
}
__device__ inline float from_right(float v, float end)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(end), __float_as_uint(v), 0x130, 0xf, 0xf, false));
}

template <int K>
__global__ __launch_bounds__(kThreads) void conv_image_row4_kernel(Row4Params p)
{
    constexpr int R = K / 2, NV = 4 + 2 * R, D = 4;       // halo columns on a side, columns under a lane, rows ahead
    constexpr uint32_t kRow = (1u << K) - 1u;
    const int lane = threadIdx.x & 63;
    const long long gw = (long long)blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (gw >= p.waves) return;
    const int xt = __builtin_amdgcn_readfirstlane((int)(gw % p.xtiles));
    const long long t = gw / p.xtiles;
    const int band = __builtin_amdgcn_readfirstlane((int)(t % p.bands));
    const int n = __builtin_amdgcn_readfirstlane((int)(t / p.bands));
    const int x = xt * 256 + 4 * lane;
    const bool mine = x < p.W;
    // the extra column: the first lane's left ones, the last lane's right ones
    const int xe = lane == 0 ? x - 1 : x + 4, de = lane == 0 ? -1 : 1;
    const bool edge = lane == 0 || lane == 63;

    uint32_t wf = 0;                                      // the filter's window in the window's bit order
#pragma unroll
    for (int r = 0; r < K * K; ++r) wf |= (p.Wpk[r] & 1u) << r;
    const float a0 = p.alpha[0];
    uint32_t row_mask[4], full[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        row_mask[j] = 0;
#pragma unroll
        for (int kx = 0; kx < K; ++kx) row_mask[j] |= (unsigned)(x + j - R + kx) < (unsigned)p.W ? 1u << kx : 0u;
        full[j] = 0;
#pragma unroll
        for (int r = 0; r < K; ++r) full[j] |= row_mask[j] << (r * K);
    }

    const int y0 = band * p.rows_per_band, y1 = min(p.OH, y0 + p.rows_per_band);
    const int nin = y1 - y0 + K - 1, yb = y0 - p.ph;
    const float *img = p.I + (long long)n * p.H * p.W;
    float4 own[D];
    float ext[D][R];
    auto issue = [&](int slot, int i) __attribute__((always_inline)) {
        const int y = yb + i;
        const bool rv = i < nin && y >= 0 && y < p.H;     // (uniform)
        own[slot] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < R; ++k) ext[slot][k] = 0.f;
        if (!rv) return;
        const float *row = img + (long long)y * p.W;
        if (mine) own[slot] = *reinterpret_cast<const float4 *>(row + x);
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (edge && (unsigned)(xe + k * de) < (unsigned)p.W) ext[slot][k] = row[xe + k * de];
    };
#pragma unroll
    for (int d = 0; d < D; ++d) issue(d, d);

    uint32_t win[4] = {0, 0, 0, 0};
    float hs[K][4];
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) hs[r][j] = 0.f;
    for (int i0 = 0; i0 < nin; i0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int i = i0 + d;
            if (i >= nin) break;
            float v[NV];
            v[R] = own[d].x; v[R + 1] = own[d].y; v[R + 2] = own[d].z; v[R + 3] = own[d].w;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                v[R - 1 - k] = from_left(v[R + 3 - k], ext[d][k]);
                v[R + 4 + k] = from_right(v[R + k], ext[d][k]);
            }
            issue(d, i + D);
            uint32_t bits = 0;
#pragma unroll
            for (int k = 0; k < NV; ++k) bits |= v[k] >= 0.f ? 1u << k : 0u;
#pragma unroll
            for (int r = 0; r + 1 < K; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) hs[r][j] = hs[r + 1][j];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // (a column outside the image is 0 and adds nothing; its bit is masked)
                float s = 0.f;
#pragma unroll
                for (int kx = 0; kx < K; ++kx) s += fabsf(v[j + kx]);
                hs[K - 1][j] = s;
                win[j] = (win[j] >> K) | (((bits >> j) & kRow) << (K * (K - 1)));
            }
            if (i < K - 1) continue;
            const int y = y0 + i - (K - 1), top = y - p.ph;
            uint32_t rows_in = (1u << (K * K)) - 1u;      // (uniform) the window rows inside the image
            if (top < 0 || top + K > p.H) {
                rows_in = 0;
#pragma unroll
                for (int r = 0; r < K; ++r) rows_in |= top + r >= 0 && top + r < p.H ? kRow << (r * K) : 0u;
            }
            float o[4];
            int dd[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t m = full[j] & rows_in;
                float ksum = hs[0][j];
#pragma unroll
                for (int r = 1; r < K; ++r) ksum += hs[r][j];
                const float kk = ksum * p.kscale;
                dd[j] = __builtin_popcount(m) - 2 * __builtin_popcount((win[j] ^ wf) & m);
                o[j] = (float)dd[j] * (kk * a0);
            }
            if (mine) {
                const long long at = ((long long)n * p.OH + y) * p.W + x;
                *reinterpret_cast<float4 *>(p.out + at) = make_float4(o[0], o[1], o[2], o[3]);
                if (p.dot) *reinterpret_cast<int4 *>(p.dot + at) = make_int4(dd[0], dd[1], dd[2], dd[3]);
            }
        }
    }
}

// Several filters: a workgroup takes a tile of output pixels and all filters (or a group of them).
//   1. The input under the tile is read once, coalesced.  The 64 signs of a wave's 64 neighbouring
//      pixels of a channel are one compare (its result mask is the row's bit map), the sum of the
//      channels' magnitudes goes to LDS beside it; the filters' windows are packed in the same order.
//   2. The magnitudes are summed along the window rows.
//   3. A lane takes one or two output pixels.  A window row of a channel is K neighbouring bits of the bit
//      map (two words, one v_alignbit_b32); 32 / K such pieces share a word.  K (Eq. 10) is the sum of K
//      row sums.  Per filter and pixel: one v_bitop3_b32 ((window xor filter) and mask) and one
//      v_bcnt_u32_b32 per word, four instructions for dot and output, one store (64 neighbouring pixels).
// Both LDS arrays run along the rows first, so that the pieces and sums of a window are neighbours.
// Bound by the output stores and by that vector arithmetic: 17 instructions per output for 7 x 7 x 3.
template <int K, int C>
struct Tile {
    static constexpr int kPerWord = 32 / K;                              // pieces (K bits) in a word
    static constexpr int kPieces = K * C;
    static constexpr int kWords = (kPieces + kPerWord - 1) / kPerWord;
    static constexpr int kRecord = kWords < 4 ? 4 : 8;                   // a filter's words, then its alpha in the last one
    static constexpr uint32_t kBits = (1u << K) - 1u;
};
// (row, 64 columns) units a wave has in flight while staging: a tile's loads in one to three batches.  (Each holds a
// lane mask: with 15 or 16 of them the scalar registers spilled, 4 x 160 x 160 C=2 3x3 F=32 14.4 us, 11.9 with ten.)
constexpr int units_ahead(int C) { return C <= 3 ? 10 : 30 / C; }

struct TileParams {
    const float *I;
    const uint32_t *Wpk;
    const float *alpha;
    float *out;
    int32_t *dot;
    int N, H, W, F, OH, OW, ph, pw, sh, sw;
    int tw, th, gx, gy;      // output pixels of a tile, tiles of an image
    int group, fgroups;      // filters per workgroup
    int cols, chunks;        // staged columns, 64-column units of a row
    int map_rows, mag_rows;  // (row, channel) entries of a 32-column bit-map word, rows of a column of sums (odd)
    uint32_t inv_tw;         // ceil(2^32 / tw), 0 for 1
    float kscale;            // 1 / (C * K * K)
};

template <int K, int C, int kPixels, bool DOT>     // pixels per lane and pass; the dot products are wanted
__global__ __launch_bounds__(kThreads, 4) void conv_image_tile_kernel(TileParams p)
{
    using T = Tile<K, C>;
    constexpr int kUnits = units_ahead(C);
    extern __shared__ uint32_t lds[];
    uint32_t *const rec = lds;                                           // [group][kRecord]
    uint32_t *const map = rec + p.group * T::kRecord;                    // [2 * chunks + 1][rows][C]
    float *const mag = reinterpret_cast<float *>(map + (2 * p.chunks + 1) * p.map_rows);   // [cols][mag_rows]
    float *const row_sum = mag + p.cols * p.mag_rows;                    // [tw][mag_rows]

    int b = blockIdx.x;
    const int fg = b % p.fgroups; b /= p.fgroups;
    const int bx = b % p.gx; b /= p.gx;
    const int by = b % p.gy;
    const int n = b / p.gy;
    const int f0 = fg * p.group, nf = min(p.group, p.F - f0);
    const int X0 = bx * p.tw, Y0 = by * p.th;
    const int tw = min(p.tw, p.OW - X0), th = min(p.th, p.OH - Y0);
    const int rows = (th - 1) * p.sh + K;
    const int iy0 = Y0 * p.sh - p.ph, ix0 = X0 * p.sw - p.pw;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    // the input under the tile: the first batch of loads is on its way while the filters are packed
    const size_t HW = (size_t)p.H * p.W;
    const float *img = p.I + (size_t)n * C * HW;
    const int units = rows * p.chunks;
    float v[kUnits][C];
    bool in[kUnits];
    auto fetch = [&](int u0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kUnits; ++k) {
            const int u = min(u0 + k * kWaves, units - 1);               // (the last one again: loads without a branch)
            const int r = u / p.chunks, x = (u - r * p.chunks) * 64 + lane;
            const int iy = iy0 + r, ix = ix0 + x;
            in[k] = (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W && x < p.cols;
            const size_t at = in[k] ? (size_t)iy * p.W + ix : 0;
#pragma unroll
            for (int c = 0; c < C; ++c) v[k][c] = img[(size_t)c * HW + at];
        }
    };
    fetch(wave);
    for (int i = threadIdx.x; i < nf * T::kRecord; i += kThreads) rec[i] = 0;
    __syncthreads();
    // filter windows: piece r * C + c of a filter holds channel c of its row r
    for (int i = threadIdx.x; i < nf * K; i += kThreads) {
        const int f = i / K, r = i - f * K;
        uint32_t w[K];
#pragma unroll
        for (int kx = 0; kx < K; ++kx) w[kx] = p.Wpk[((size_t)(f0 + f) * K + r) * K + kx];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            uint32_t bits = 0;
#pragma unroll
            for (int kx = 0; kx < K; ++kx) bits |= ((w[kx] >> c) & 1u) << kx;
            const int piece = r * C + c;
            atomicOr(&rec[f * T::kRecord + piece / T::kPerWord], bits << ((piece % T::kPerWord) * K));
        }
        if (r == 0) rec[f * T::kRecord + T::kRecord - 1] = __float_as_uint(p.alpha[f0 + f]);
    }
    for (int u0 = wave; u0 < units; u0 += kWaves * kUnits) {
        if (u0 != wave) fetch(u0);
#pragma unroll
        for (int k = 0; k < kUnits; ++k) {
            const int u = u0 + k * kWaves;
            if (u >= units) break;
            const int r = u / p.chunks, ch = u - r * p.chunks, x = ch * 64 + lane;
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const unsigned long long signs = __ballot(in[k] && v[k][c] >= 0.f);
                if (lane < 2) map[(2 * ch + lane) * p.map_rows + r * C + c] = (uint32_t)(lane ? signs >> 32 : signs);
                s += fabsf(v[k][c]);
            }
            if (x < p.cols) mag[x * p.mag_rows + r] = in[k] ? s : 0.f;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < tw * rows; i += kThreads) {
        const int x = i / rows, r = i - x * rows;
        const float *src = mag + x * p.sw * p.mag_rows + r;
        float s = src[0];
#pragma unroll
        for (int kx = 1; kx < K; ++kx) s += src[kx * p.mag_rows];
        row_sum[x * p.mag_rows + r] = s;
    }
    __syncthreads();

    const int npx = tw * th;
    const size_t OHW = (size_t)p.OH * p.OW;
    const size_t plane0 = ((size_t)n * p.F + f0) * OHW;
    for (int q0 = threadIdx.x; q0 < npx; q0 += kThreads * kPixels) {
        uint32_t win[kPixels][T::kWords], m[kPixels][T::kWords];
        float kk[kPixels];
        int nvalid[kPixels];
        uint32_t at[kPixels];
#pragma unroll
        for (int k = 0; k < kPixels; ++k) {
            const int q = min(q0 + k * kThreads, npx - 1);
            // (a ragged tile has its own width: a division for the image's last tile column only)
            const int oy = tw == p.tw ? (p.inv_tw == 0 ? q : (int)__umulhi((uint32_t)q, p.inv_tw)) : q / tw;
            const int ox = q - oy * tw;
            const int x0 = ox * p.sw, y0 = oy * p.sh;
            at[k] = ((uint32_t)(Y0 + oy) * (uint32_t)p.OW + (uint32_t)(X0 + ox)) * 4u;   // (a plane is below 2 GiB)
            const int left = max(0, -(ix0 + x0)), right = max(0, ix0 + x0 + K - p.W);
            const uint32_t cols_in = left + right >= K ? 0u : (T::kBits << left) & (T::kBits >> right);
            const uint32_t sh = (uint32_t)x0 & 31u;
            const uint32_t *src = map + (x0 >> 5) * p.map_rows + y0 * C;
            const float *sums = row_sum + ox * p.mag_rows + y0;
            float total = sums[0];
#pragma unroll
            for (int r = 1; r < K; ++r) total += sums[r];
            kk[k] = total * p.kscale;
#pragma unroll
            for (int w = 0; w < T::kWords; ++w) win[k][w] = 0;
            constexpr int per = T::kPerWord;
#pragma unroll
            for (int i = 0; i < T::kPieces; ++i) {                        // piece i = row i / C, channel i % C
                const uint32_t bits = __builtin_amdgcn_alignbit(src[i + p.map_rows], src[i], sh) & T::kBits;
                win[k][i / per] |= bits << ((i % per) * K);
            }
            const int top = iy0 + y0;
            if (__all(top >= 0 && top + K <= p.H)) {                      // every word's pieces alike
                uint32_t all = 0;
#pragma unroll
                for (int i = 0; i < per; ++i) all |= cols_in << (i * K);
#pragma unroll
                for (int w = 0; w < T::kWords; ++w) {
                    const int live = min(per, T::kPieces - w * per) * K;  // (constant, at most 30 bits)
                    m[k][w] = all & ((1u << live) - 1u);
                }
                nvalid[k] = C * K * __builtin_popcount(cols_in);
            } else {
#pragma unroll
                for (int w = 0; w < T::kWords; ++w) m[k][w] = 0;
                nvalid[k] = 0;
#pragma unroll
                for (int i = 0; i < T::kPieces; ++i) {
                    const uint32_t piece = (unsigned)(top + i / C) < (unsigned)p.H ? cols_in : 0u;
                    m[k][i / per] |= piece << ((i % per) * K);
                    nvalid[k] += __builtin_popcount(piece);
                }
            }
        }
        // (a lane without a pixel of its own repeats the tile's last one: the same value to the same place)
        const float *out = p.out + plane0;
        const int32_t *dot = DOT ? p.dot + plane0 : nullptr;
        const int plane_bytes = (int)(OHW * 4);
        constexpr int kRaw = 0x00027000;                                  // (a plain buffer of dwords)
#pragma unroll 2
        for (int f = 0; f < nf; ++f) {
            uint32_t w[T::kRecord];
#pragma unroll
            for (int i = 0; i < T::kRecord; i += 4) {
                const uint4 x = *reinterpret_cast<const uint4 *>(&rec[f * T::kRecord + i]);
                w[i] = x.x; w[i + 1] = x.y; w[i + 2] = x.z; w[i + 3] = x.w;
            }
            const float al = __uint_as_float(w[T::kRecord - 1]);
            // stores as scalar plane + lane offset: no vector arithmetic for the address
            const auto to = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(out), 0, plane_bytes, kRaw);
#pragma unroll
            for (int k = 0; k < kPixels; ++k) {
                uint32_t pop = 0;
#pragma unroll
                for (int i = 0; i < T::kWords; ++i) pop += __builtin_popcount((win[k][i] ^ w[i]) & m[k][i]);
                const float d = fmaf(-2.f, (float)pop, (float)nvalid[k]);     // (small whole numbers: exact)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d * (kk[k] * al)), to, (int)at[k], 0, 0);
                if constexpr (DOT)
                    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)(int)d,
                        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(dot), 0, plane_bytes, kRaw), (int)at[k], 0, 0);
            }
            out += OHW;
            if constexpr (DOT) dot += OHW;
        }
    }
}

template <int K, int C>
hipError_t launch_kc(const ImageParams &p, dim3 grid, size_t lds, hipStream_t st)
{
    const bool unit = p.sh == 1 && p.sw == 1;
    if (p.F == 1 && unit)
        conv_image_kernel<K, C, true, true><<<grid, dim3(kThreads), lds, st>>>(p);
    else if (p.F == 1)
        conv_image_kernel<K, C, true, false><<<grid, dim3(kThreads), lds, st>>>(p);
    else if (unit)
        conv_image_kernel<K, C, false, true><<<grid, dim3(kThreads), lds, st>>>(p);
    else
        conv_image_kernel<K, C, false, false><<<grid, dim3(kThreads), lds, st>>>(p);
    return hipGetLastError();
}

template <int K>
hipError_t launch_k(int C, const ImageParams &p, dim3 grid, size_t lds, hipStream_t st)
{
    switch (C) {
        case 1: return launch_kc<K, 1>(p, grid, lds, st);
        case 2: return launch_kc<K, 2>(p, grid, lds, st);
        case 3: return launch_kc<K, 3>(p, grid, lds, st);
        default: return launch_kc<K, 4>(p, grid, lds, st);
    }
}

// Tiles of several filters' kernel: rows of a tile are the whole output rows where these are at most 256
// pixels, else equal parts of them; about 512 pixels a tile (two per lane), fewer where the launch would
// not give every compute unit four workgroups, and then the filters are shared out as well.
struct TilePlan { int tw, th, gx, gy, group; };
size_t tile_lds(const Geom &g, const TilePlan &pl, int record)
{
    const long long rows = (long long)(pl.th - 1) * g.sh + g.kh, cols = (long long)(pl.tw - 1) * g.sw + g.kw;
    return 4 * ((size_t)pl.group * record + (size_t)(2 * ceil_div(cols, 64) + 1) * rows * g.C + (size_t)(cols + pl.tw) * (rows | 1));
}

TilePlan tile_plan(const Geom &g)
{
    TilePlan pl;
    pl.group = std::min(g.F, 256);
    pl.gx = ceil_div(g.OW, 256);
    pl.tw = ceil_div(g.OW, pl.gx);
    pl.th = std::min(g.OH, std::max(1, 512 / pl.tw));
    // (large strides: what lies under the tile has to fit the LDS)
    while (tile_lds(g, pl, 8) > kLdsBudget) {
        if (pl.th > 1) pl.th = (pl.th + 1) / 2;
        else pl.tw = (pl.tw + 1) / 2;
    }
    pl.gx = ceil_div(g.OW, pl.tw);
    auto blocks = [&](int th) { return (long long)g.N * pl.gx * ceil_div(g.OH, th); };
    if (pl.th > 1 && blocks(pl.th) < 768) pl.th = std::max(1, std::min(pl.th, 256 / pl.tw));
    // (a launch that leaves units idle is as long as one workgroup: what it stages in one batch of loads)
    auto units = [&](int th) { return (long long)((th - 1) * g.sh + g.kh) * ceil_div((pl.tw - 1) * g.sw + g.kw, 64); };
    while (pl.th > 1 && blocks(pl.th) < 64 && units(pl.th) > kWaves * units_ahead(g.C)) pl.th = (pl.th + 1) / 2;
    pl.gy = ceil_div(g.OH, pl.th);
    while (pl.group > 16 && blocks(pl.th) * ceil_div(g.F, pl.group) < 768) pl.group = (pl.group + 1) / 2;
    return pl;
}

// Where the tiles are the faster form.  The sliding window (conv_image_kernel) reads kw * C values per
// lane and input row, several times over where filters are shared out or rows are skipped by a stride,
// but costs little per output; the tiles pay about 200 instructions per output pixel once and then 17
// or fewer per filter.  Measured, sliding window / tiles, 2 x C x 500 x 500 unless said otherwise:
// 16 x 3 x 227 x 227 F=64 7x7 stride 2 67 / 24 us; C=3 7x7 F=64 49 / 34 us, F=8 1.17x, F=4 0.94x; the same
// with stride 2 F=4 1.5x; C=3 3x3 F=16 1.28x, F=4 0.76x, stride 2 F=4 1.25x; C=1 3x3 F=16 0.97x, F=4 0.59x.
// On large images the sliding window has waves enough without sharing out its filters: 8 x 300 x 300 C=2 3x3 F=16 16.4 / 17.3,
// C=3 5x5 F=8 18.3 / 19.7, F=16 and C=3 7x7 1.0 to 1.1x; stride 2 C=3 3x3 F=2 8.8 / 10.3 (8 x 128 x 128: 1.24x).
bool tile_pays(const Geom &g)
{
    if (g.F < 2 || (long long)g.OH * g.OW >= (1LL << 29)) return false;    // (31-bit byte offsets in a plane)
    const int kc = g.kw * g.C;
    const long long pixels = (long long)g.N * g.OH * g.OW;
    if (g.sh >= 2 && g.sw >= 2 && kc >= 9) return g.F >= 8 || pixels < 150000;
    if (pixels >= 400000 && g.sh == 1 && g.sw == 1) return g.F >= 16 && kc >= 10;
    return (g.F >= 16 && kc >= 6) || (g.F >= 8 && kc >= 15);
}

template <int K, int C>
hipError_t launch_tile(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g, float *out, int32_t *dot,
                       const TilePlan &pl, hipStream_t st)
{
    TileParams p;
    p.I = I; p.Wpk = Wpk; p.alpha = alpha; p.out = out; p.dot = dot;
    p.N = g.N; p.H = g.H; p.W = g.W; p.F = g.F; p.OH = g.OH; p.OW = g.OW; p.ph = g.ph; p.pw = g.pw; p.sh = g.sh; p.sw = g.sw;
    p.tw = pl.tw; p.th = pl.th; p.gx = pl.gx; p.gy = pl.gy; p.group = pl.group; p.fgroups = ceil_div(g.F, pl.group);
    p.cols = (pl.tw - 1) * g.sw + K; p.chunks = ceil_div(p.cols, 64);
    const int rows = (pl.th - 1) * g.sh + K;
    p.map_rows = rows * C; p.mag_rows = rows | 1;
    p.inv_tw = pl.tw == 1 ? 0u : (uint32_t)(((1ULL << 32) + pl.tw - 1) / pl.tw);
    p.kscale = 1.0f / (float)(C * K * K);
    const long long blocks = (long long)g.N * pl.gx * pl.gy * p.fgroups;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = tile_lds(g, pl, Tile<K, C>::kRecord);
    const dim3 grid((unsigned)blocks);
    if (pl.tw * pl.th <= kThreads) {
        if (dot) conv_image_tile_kernel<K, C, 1, true><<<grid, dim3(kThreads), lds, st>>>(p);
        else conv_image_tile_kernel<K, C, 1, false><<<grid, dim3(kThreads), lds, st>>>(p);
    } else {
        if (dot) conv_image_tile_kernel<K, C, 2, true><<<grid, dim3(kThreads), lds, st>>>(p);
        else conv_image_tile_kernel<K, C, 2, false><<<grid, dim3(kThreads), lds, st>>>(p);
    }
    return hipGetLastError();
}

template <int K>
hipError_t launch_tile_k(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g, float *out, int32_t *dot,
                         const TilePlan &pl, hipStream_t st)
{
    switch (g.C) {
        case 1: return launch_tile<K, 1>(I, Wpk, alpha, g, out, dot, pl, st);
        case 2: return launch_tile<K, 2>(I, Wpk, alpha, g, out, dot, pl, st);
        case 3: return launch_tile<K, 3>(I, Wpk, alpha, g, out, dot, pl, st);
        default: return launch_tile<K, 4>(I, Wpk, alpha, g, out, dot, pl, st);
    }
}

int window_words(int k, int C) { return (k + 32 / (k * C) - 1) / (32 / (k * C)); }

}  // namespace

bool conv_image_supports(const Geom &g)
{
    if (g.C < 1 || g.C > 4) return false;
    if (g.kh != g.kw || (g.kh != 3 && g.kh != 5 && g.kh != 7)) return false;
    if ((size_t)g.F * (window_words(g.kh, g.C) + 1) * 4 > kLdsBudget) return false;
    return true;
}

hipError_t launch_conv_image(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g,
                             float *out, int32_t *dot, hipStream_t st)
{
    if (tile_pays(g)) {
        const TilePlan pl = tile_plan(g);
        switch (g.kh) {
            case 3: return launch_tile_k<3>(I, Wpk, alpha, g, out, dot, pl, st);
            case 5: return launch_tile_k<5>(I, Wpk, alpha, g, out, dot, pl, st);
            default: return launch_tile_k<7>(I, Wpk, alpha, g, out, dot, pl, st);
        }
    }
    // Four columns per lane from half a million pixels on; a smaller image is bound by latency and wants its rows
    // spread over more waves.  Measured, one column / four: 4096^2 33.2 / 24.7 us, 2048^2 13.3 / 9.4 (5 x 5: 16.9 /
    // 11.4), 1024^2 6.0 / 5.0, 4 x 300 x 500 5.2 / 4.7, 512^2 3.9 / 4.5, 256^2 3.9 / 4.4.
    const uintptr_t ptrs = reinterpret_cast<uintptr_t>(I) | reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(dot);
    if (g.F == 1 && g.C == 1 && g.sh == 1 && g.sw == 1 && (g.kw == 3 || g.kw == 5) && g.pw == g.kw / 2 && g.W % 4 == 0 &&
        (ptrs & 15) == 0 && (long long)g.N * g.OH * g.W >= (1 << 19)) {
        Row4Params p;
        p.I = I; p.Wpk = Wpk; p.alpha = alpha; p.out = out; p.dot = dot;
        p.H = g.H; p.W = g.W; p.OH = g.OH; p.ph = g.ph;
        p.xtiles = ceil_div(g.W, 256);
        // bands of 32 rows, halved until every SIMD has two waves, down to 4 (see the band heights below)
        int rows = 32;
        auto waves_with = [&](int r) { return (long long)g.N * p.xtiles * ceil_div(g.OH, r); };
        while (rows > 4 && waves_with(rows) < 256LL * 4 * 2) rows /= 2;
        p.rows_per_band = std::max(1, std::min(rows, g.OH));
        p.bands = ceil_div(g.OH, p.rows_per_band);
        p.waves = waves_with(p.rows_per_band);
        p.kscale = 1.0f / (float)(g.kh * g.kw);
        const long long blocks = (p.waves + kWaves - 1) / kWaves;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        if (g.kw == 3) conv_image_row4_kernel<3><<<dim3((unsigned)blocks), dim3(kThreads), 0, st>>>(p);
        else conv_image_row4_kernel<5><<<dim3((unsigned)blocks), dim3(kThreads), 0, st>>>(p);
        return hipGetLastError();
    }
    ImageParams p;
    p.I = I; p.Wpk = Wpk; p.alpha = alpha; p.out = out; p.dot = dot;
    p.N = g.N; p.H = g.H; p.W = g.W; p.F = g.F; p.OH = g.OH; p.OW = g.OW; p.ph = g.ph; p.pw = g.pw; p.sh = g.sh; p.sw = g.sw;
    p.xtiles = ceil_div(g.OW, 64);
    // Band height: tall bands re-read fewer halo rows, short ones give more waves.  Halve from 64
    // until the chip has about eight waves per SIMD; an image too small for that even with bands
    // of 8 rows is bound by the chain of load latencies down a band, so it gets bands of 4.
    // (Measured, one channel, 3x3: 4096^2 is fastest with 32 rows, 2048^2 with 16 or 8, 1024^2
    // with 8, 512^2 and below with 4.)
    auto waves_with = [&](int rows) { return (long long)g.N * p.xtiles * ceil_div(g.OH, rows); };
    int rows = 64;
    while (rows > 8 && waves_with(rows) < 256LL * 4 * 8) rows /= 2;
    if (waves_with(rows) < 256LL * 4 * 2) rows = 4;
    p.rows_per_band = std::max(1, std::min(rows, g.OH));
    p.bands = ceil_div(g.OH, p.rows_per_band);
    // With many filters and a small image the filters are shared out over waves as well (each
    // wave rebuilds the window, which costs little next to the work of its filters).
    p.group = g.F;
    while (p.group > 4 && waves_with(p.rows_per_band) * ceil_div(g.F, p.group) < 256LL * 4 * 4)
        p.group = (p.group + 1) / 2;
    p.fgroups = ceil_div(g.F, p.group);
    p.waves = waves_with(p.rows_per_band) * p.fgroups;
    p.kscale = 1.0f / (float)(g.C * g.kh * g.kw);
    const long long blocks = (p.waves + kWaves - 1) / kWaves;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = g.F == 1 ? 0 : (size_t)g.F * (window_words(g.kh, g.C) + 1) * 4;
    const dim3 grid((unsigned)blocks);
    switch (g.kh) {
        case 3: return launch_k<3>(g.C, p, grid, lds, st);
        case 5: return launch_k<5>(g.C, p, grid, lds, st);
        default: return launch_k<7>(g.C, p, grid, lds, st);
    }
}

}  // namespace xnor
