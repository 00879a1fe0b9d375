// Device helpers shared by the rollout and adjoint kernels: counter-based
// Gaussian noise (Sec. 3.3 sampling) and wavefront segmented scans over the
// steps of one particle (the triangular sums of Sec. 3.1, Eq. 7).
#pragma once

#include "storm_internal.h"

namespace storm {
namespace {

// a b as one instruction (written as two halves, or as a 64-bit product of two
// words, it compiles to two: v_mul_lo_u32 and v_mul_hi_u32).
__device__ __forceinline__ uint64_t wide_mul(uint32_t a, uint32_t b)
{
    uint64_t r;
    asm("v_mad_u64_u32 %0, vcc, %1, %2, 0" : "=v"(r) : "s"(a), "v"(b) : "vcc");
    return r;
}

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64-bit
// products with the Weyl key schedule.
__device__ __forceinline__ void philox4x32_10(uint32_t &c0, uint32_t &c1, uint32_t &c2, uint32_t &c3, uint32_t k0,
                                              uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        // (one 64-bit product each)
        const uint64_t p0 = wide_mul(0xD2511F53u, c0), p1 = wide_mul(0xCD9E8D57u, c2);
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        const uint32_t n0 = hi1 ^ c1 ^ k0;
        const uint32_t n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Box-Muller on 24-bit uniforms u1 in (0, 1], u2 in [0, 1).
__device__ __forceinline__ void box_muller(uint32_t x0, uint32_t x1, float &zc, float &zs)
{
    const float u1 = (float)((x0 >> 8) + 1u) * 0x1.0p-24f;
    const float u2 = (float)(x1 >> 8) * 0x1.0p-24f;
    const float r = sqrtf(-2.0f * logf(u1));
    float s, c;
    sincospif(2.0f * u2, &s, &c);
    zc = r * c;
    zs = r * s;
}

// Lane move through DPP: lane l receives x from the lane that `kCtrl` names
// (row shifts, row broadcasts); lanes whose source is outside the row, or
// in a row that kRowMask leaves out, receive 0.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ float dpp_or_zero(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, kRowMask, 0xf, true));
}

// Inclusive prefix sum over the lanes of one particle (lanes p*H .. p*H+H-1;
// h = step index of this lane), without LDS traffic: a Kogge-Stone scan
// inside each 16-lane row (DPP row shifts by 1, 2, 4, 8, each term taken
// only from the lane's own segment and row), then the two row broadcasts
// that carry the sums of rows 0 and 2 into rows 1 and 3, and of rows 0-1
// into rows 2-3, each taken only by lanes whose particle began before the
// source lane.  Segments of the padding lanes past the last particle are
// scanned the same way.
// (Several scans step by step together: one alone is a serial chain.)
template <int kCtrl, int kRowMask, int n>
__device__ __forceinline__ void scan_step(float (&x)[n], bool take)
{
    float y[n];
#pragma unroll
    for (int k = 0; k < n; ++k) y[k] = dpp_or_zero<kCtrl, kRowMask>(x[k]);
#pragma unroll
    for (int k = 0; k < n; ++k) x[k] += take ? y[k] : 0.0f;
}
template <int n>
__device__ __forceinline__ void segmented_scans(float (&x)[n], int lane, int h)
{
    const int in_row = lane & 15;
    const int reach = h < in_row ? h : in_row;  // lanes back to the row or segment start
    scan_step<0x111, 0xf>(x, reach >= 1);  // row_shr:1
    scan_step<0x112, 0xf>(x, reach >= 2);  // row_shr:2
    scan_step<0x114, 0xf>(x, reach >= 4);  // row_shr:4
    scan_step<0x118, 0xf>(x, reach >= 8);  // row_shr:8
    scan_step<0x142, 0xa>(x, h > in_row);  // row_bcast:15 -> rows 1, 3
    scan_step<0x143, 0xc>(x, lane >= 32 && h > lane - 32);  // row_bcast:31 -> rows 2, 3
}
__device__ __forceinline__ float segmented_scan(float x, int h, int H)
{
    (void)H;
    float a[1] = {x};
    segmented_scans(a, (int)(threadIdx.x & (kLanes - 1)), h);
    return a[0];
}

__device__ __forceinline__ float hinge_box(float x, float lo, float hi)
{
    return fmaxf(lo - x, 0.0f) + fmaxf(x - hi, 0.0f);
}

// Inclusive suffix sum over the lanes of one particle (the transpose of
// segmented_scan, used by the reverse pass; `left` = H - 1 - h, the steps after
// this lane's): the same scan towards lower lanes, the rows' sums carried by
// scalar reads of the rows' first lanes, the last row's first.
template <int n>
__device__ __forceinline__ void segmented_suffix_scans(float (&x)[n], int lane, int left)
{
    const int in_row = 15 - (lane & 15);
    const int reach = left < in_row ? left : in_row;  // lanes on to the row or segment end
    scan_step<0x101, 0xf>(x, reach >= 1);  // row_shl:1
    scan_step<0x102, 0xf>(x, reach >= 2);  // row_shl:2
    scan_step<0x104, 0xf>(x, reach >= 4);  // row_shl:4
    scan_step<0x108, 0xf>(x, reach >= 8);  // row_shl:8
#pragma unroll
    for (int row = 2; row >= 0; --row) {
        const bool take = (lane >> 4) == row && left > in_row;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const float y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[k]), 16 * (row + 1)));
            x[k] += take ? y : 0.0f;
        }
    }
}

// Comb-filtered noise of one joint at step h (Sec. 3.3), from that joint's
// row of standard noise over the tile's lanes: the filter's recursion in
// step order written as its convolution, sum over k <= h of g_k e_{h-k},
// with the response g in the tables; e_{h-k} is the lane k below, in the
// same particle.
__device__ __forceinline__ float comb_noise(const float *row, int lane, int h, int H, global_ptr<const float> tab)
{
    // eight terms per batch, every read of a batch in flight at once (the
    // response is zero past H, and within the table's kMaxH entries)
    float acc = 0.0f;
    for (int k0 = 0; k0 < H; k0 += 8) {
        float g[8], e[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            g[m] = tab[kTabComb + k0 + m];
            e[m] = row[max(lane - k0 - m, 0)];
        }
#pragma unroll
        for (int m = 0; m < 8; ++m) acc = fmaf(g[m], k0 + m <= h ? e[m] : 0.0f, acc);
    }
    return acc;
}

// Standard noise of joints 4k + 2 half and 4k + 2 half + 1 for one (particle,
// step) point: from the override, the Halton table, or the Box-Muller
// transform of one half of Philox call k.  Prob: anything with N, H,
// n_halton and halton.
template <class Prob>
__device__ __forceinline__ void standard_noise2(Prob &P, uint32_t seed_lo, uint32_t seed_hi,
                                                const float *__restrict__ noise, int k, int half, int i, int h,
                                                uint32_t counter, float e[2])
{
    const int j0 = 4 * k + 2 * half;
    if (noise != nullptr) {
#pragma unroll
        for (int m = 0; m < 2; ++m) e[m] = j0 + m < kDof ? noise[((size_t)(j0 + m) * P.N + i) * P.H + h] : 0.0f;
    } else if (i < P.n_halton) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
            e[m] = j0 + m < kDof ? as_global(P.halton)[((size_t)(j0 + m) * P.n_halton + i) * P.H + h] : 0.0f;
    } else {
        uint32_t c0 = (uint32_t)i, c1 = (uint32_t)h, c2 = (uint32_t)k, c3 = counter;
        philox4x32_10(c0, c1, c2, c3, seed_lo, seed_hi);
        if (half == 0)
            box_muller(c0, c1, e[0], e[1]);
        else
            box_muller(c2, c3, e[0], e[1]);
    }
}

// Standard noise of joints 4k..4k+3 (k = 0 or 1): the same values as
// standard_noise2's of both halves.
template <class Prob>
__device__ __forceinline__ void standard_noise4(Prob &P, uint32_t seed_lo, uint32_t seed_hi, const float *__restrict__ noise, int k, int i, int h,
                                                uint32_t counter, float e[4])
{
    const int j0 = 4 * k;
    if (noise != nullptr) {
#pragma unroll
        for (int m = 0; m < 4; ++m) e[m] = j0 + m < kDof ? noise[((size_t)(j0 + m) * P.N + i) * P.H + h] : 0.0f;
    } else if (i < P.n_halton) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            e[m] = j0 + m < kDof ? as_global(P.halton)[((size_t)(j0 + m) * P.n_halton + i) * P.H + h] : 0.0f;
    } else {
        uint32_t c0 = (uint32_t)i, c1 = (uint32_t)h, c2 = (uint32_t)k, c3 = counter;
        philox4x32_10(c0, c1, c2, c3, seed_lo, seed_hi);
        box_muller(c0, c1, e[0], e[1]);
        box_muller(c2, c3, e[2], e[3]);
    }
}

}  // namespace
}  // namespace storm
