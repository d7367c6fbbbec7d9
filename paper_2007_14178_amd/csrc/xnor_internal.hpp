// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <atomic>
#include <stdint.h>
#include <string.h>

#include "xnor.h"
#include "fp4_expand.hpp"

namespace xnor {

// Derived geometry, computed once on the host after validation.
struct Geom {
    int N, C, H, W, F, kh, kw, sh, sw, ph, pw;
    int OH, OW, Cw;
};

// Compute units that plans and routes are made for.  A route fixes the layout of the expanded filters, which one
// call writes and another reads, perhaps from another thread: it is a function of the geometry alone, whatever
// the current device counts.  (Launch sizes go by compute_units().)
constexpr int kPlanUnits = 256;

// The last plans made on a thread, by geometry (and one more number: an operand's alignment), four to a set.  A plan
// is a function of these alone and costs the host several microseconds where it tries rows and shapes; a
// call asks for it two to five times.
template <class V, int SETS = 32>
struct PlanMemo {
    static constexpr int kWays = 4;
    struct Set {
        Geom g[kWays];
        int extra[kWays];
        V val[kWays];
        int used = 0, next = 0;
    };
    Set set[SETS];
    template <class Make>
    const V &get(const Geom &g, int extra, Make make)
    {
        const int *w = reinterpret_cast<const int *>(&g);
        uint32_t h = (uint32_t)extra;
        for (unsigned i = 0; i < sizeof g / sizeof(int); ++i) h = (h ^ (uint32_t)w[i]) * 0x9E3779B1u;
        Set &s = set[(h >> 20) % SETS];
        for (int i = 0; i < s.used; ++i)
            if (s.extra[i] == extra && memcmp(&s.g[i], &g, sizeof g) == 0) return s.val[i];
        const int at = s.next;
        s.val[at] = make();
        s.g[at] = g;
        s.extra[at] = extra;
        s.next = (at + 1) % kWays;
        s.used = s.used < kWays ? s.used + 1 : kWays;
        return s.val[at];
    }
};

// Compute units of the current device.
inline int compute_units()
{
    static std::atomic<int> cached[64];
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return kPlanUnits;
    }
    v = cached[dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) {
        (void)hipGetLastError();
        return kPlanUnits;
    }
    cached[dev].store(v, std::memory_order_relaxed);
    return v;
}

inline int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }

// n / d through one multiply-high with inv = ceil(2^32 / d), exact for n*d < 2^32; d = 1 has no
// such 32-bit reciprocal (2^32) and is flagged by inv = 0 (uniform: a scalar select).
inline uint32_t reciprocal(unsigned long long d) { return d == 1 ? 0u : (uint32_t)(((1ULL << 32) + d - 1) / d); }
__device__ inline uint32_t quot(uint32_t n, uint32_t inv) { return inv == 0 ? n : __umulhi(n, inv); }

// Launchers: enqueue on `st`, return the launch status.  Arguments are already validated.
hipError_t launch_binarize_pack(const float *x, int N, int C, int H, int W, uint32_t *packed,
                                hipStream_t st);
hipError_t launch_channel_mean_abs(const float *I, int N, int C, int H, int W, float *A,
                                   hipStream_t st);
hipError_t launch_scale_K(const float *I, const Geom &g, float *A, float *K, hipStream_t st);
bool pack_and_mean_supports(int C);
hipError_t launch_pack_and_mean(const float *x, int N, int C, int H, int W, uint32_t *packed,
                                float *A, hipStream_t st);
bool filter_pack_mean_supports(int taps);
hipError_t launch_filter_pack_mean(const float *Wt, int F, int C, int taps, uint32_t *Wpk, float *M,
                                   float *alpha, hipStream_t st);
bool prepare_both_supports(const float *x, int N, int C, int H, int W, int taps);
bool prepare_both_can_expand(int C, int taps);
hipError_t launch_prepare_both(const float *x, int N, int C, int H, int W, uint32_t *packed, float *A,
                               const float *Wt, int F, int taps, uint32_t *Wpk, float *M, float *alpha,
                               void *Wx, const ExpandLayout &L, hipStream_t st);
hipError_t launch_alpha_from_tap_means(const float *M, int F, int taps, float *alpha, hipStream_t st);
hipError_t launch_box_filter_K(const float *A, const Geom &g, float *K, hipStream_t st);
hipError_t launch_alpha(const float *Wt, int F, long long n_red, float *alpha, hipStream_t st);

hipError_t launch_conv_direct(const uint32_t *Ipk, const uint32_t *Wpk, const float *K,
                              const float *alpha, const Geom &g, float *out, int32_t *dot,
                              hipStream_t st);

bool conv_tiled_supports(const Geom &g);
hipError_t launch_conv_tiled(const uint32_t *Ipk, const uint32_t *Wpk, const float *K,
                             const float *alpha, const Geom &g, float *out, int32_t *dot,
                             hipStream_t st);

bool conv_image_supports(const Geom &g);
hipError_t launch_conv_image(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g,
                             float *out, int32_t *dot, hipStream_t st);

bool bwn_mfma_supports(const Geom &g);
bool bwn_split_supports(const Geom &g);
double bwn_split_cycles(const Geom &g);                  // about what the launch takes, if supported
bool bwn_split_plan(const Geom &g, int compute_units, int *tiles, int *row_segments, size_t *lds_bytes,
                    long long *workgroups);
hipError_t launch_bwn_split(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g,
                            float *out, hipStream_t st);
bool bwn_fp6_supports(const Geom &g);
double bwn_fp6_cycles(const Geom &g);
struct Fp6Shape {
    int filter_tiles, words, splits, tiles, stagers;
    size_t lds_bytes;
    long long workgroups;
};
bool bwn_fp6_plan(const Geom &g, int compute_units, Fp6Shape *out);
hipError_t launch_bwn_fp6(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g, float *out,
                          hipStream_t st);
bool conv_fp32_mfma_supports(const Geom &g);
hipError_t launch_conv_fp32_mfma(const float *I, const float *Wt, const Geom &g, float *out, hipStream_t st);
size_t conv_fp32_split_workspace_bytes(const Geom &g);   // 0 if the shape is not supported
size_t conv_fp32_pairs_workspace_bytes(const Geom &g);   // with which it works on pairs; 0 if it never does
hipError_t launch_conv_fp32_split(const float *I, const float *Wt, const Geom &g, float *out, void *workspace,
                                  size_t workspace_bytes, hipStream_t st);
hipError_t launch_conv_fp32_direct(const float *I, const float *Wt, const Geom &g, float *out, hipStream_t st);
hipError_t launch_bwn_mfma(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g,
                           float *out, hipStream_t st);
hipError_t launch_bwn_direct(const float *I, const uint32_t *Wpk, const float *alpha, const Geom &g,
                             float *out, hipStream_t st);

// The matrix-core convolution.  `algo`: XNOR_ALGO_MFMA for the kernel that the shape's rule picks, or one of the
// three by name, with its own workspace layout.
int conv_mfma_kernel_of(const Geom &g);                  // by name; XNOR_E_UNSUPPORTED if none takes the shape
size_t conv_mfma_workspace_bytes(const Geom &g, int algo = XNOR_ALGO_MFMA);         // 0 if the shape is not supported
size_t conv_mfma_chain_workspace_bytes(const Geom &g, int algo = XNOR_ALGO_MFMA);   // 0 if the shape is not supported
ExpandLayout conv_mfma_expand_layout(const Geom &g);
bool conv_mfma_bands_supports(const Geom &g);
hipError_t launch_expand_filters(const uint32_t *Wpk, const Geom &g, void *workspace, hipStream_t st,
                                 int algo = XNOR_ALGO_MFMA);
hipError_t launch_conv_mfma_expanded(const uint32_t *Ipk, const float *K, const float *A, const float *alpha,
                                     const Geom &g, float *out, int32_t *dot, const void *workspace,
                                     hipStream_t st, int algo);
hipError_t launch_conv_mfma_chain(const uint32_t *Ipk, const uint32_t *Wpk, const float *K, const float *A,
                                  const float *alpha, const Geom &g, uint32_t *Opk, float *A_next,
                                  void *workspace, hipStream_t st, int algo);
hipError_t launch_conv_mfma(const uint32_t *Ipk, const uint32_t *Wpk, const float *K, const float *alpha,
                            const Geom &g, float *out, int32_t *dot, void *workspace, hipStream_t st,
                            int algo = XNOR_ALGO_MFMA);

}  // namespace xnor
