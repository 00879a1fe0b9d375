// Device helpers of the learned self-collision network (Sec. 3.2, Eq. 13,
// the jointNERF form) on the matrix cores: MFMA operand types, the LDS row
// layout of the activations and the fragment loads / activation stores of a
// 16 x 16 tile.
//
// Precision.  The weights are FP16 values (the context rejects weights that
// FP16 cannot hold exactly), and every activation a that feeds a matrix
// product is carried as two FP16 values, hi = fp16(a) and lo = fp16(a - hi),
// kept side by side in its LDS row.  A product is W hi + W lo, two FP16 MFMAs
// into one FP32 accumulator; each FP16 x FP16 product is exact in FP32, so
// the result matches an FP32 evaluation of the layer up to the lo rounding
// (about 2^-22 relative to a) and the FP32 accumulation order.
#pragma once

#include "storm_internal.h"

namespace storm {

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

// LDS row strides: the first two hidden layers' rows hold [hi (width) | lo
// (width) | pad] in halves, the last hidden layer's FP32 values; padded so
// that the 16 rows of an operand tile fall in different banks.
constexpr int kNetA1 = 2 * kNetH1 + 8;
constexpr int kNetA2 = 2 * kNetH2 + 8;
constexpr int kNetA3 = kNetH3 + 4;

// MFMA operands, lane l (both layouts checked on the device).  The weights are
// the A operand and the activations the B operand, so that a lane's four
// results are neighbouring units of one row, which the next layer's LDS rows
// take in one 8-byte write (as the B operand, the weights left neighbouring
// rows of one unit: four 2-byte writes).
//   v_mfma_f32_16x16x16_f16 (layer 1, k = 16)
//     A (16 x 16, units x k): A[l % 16][4 (l / 16) + j], j < 4
//     B (16 x 16, k x rows):  B[4 (l / 16) + j][l % 16]
//   v_mfma_f32_16x16x32_f16 (layers 2 and 3, twice the k per instruction)
//     A (16 x 32):            A[l % 16][8 (l / 16) + j], j < 8
//     B (32 x 16):            B[8 (l / 16) + j][l % 16]
//   D (16 x 16), both:        D[4 (l / 16) + j][l % 16], units x rows
__device__ __forceinline__ half4_t net_load_a(const _Float16 *s, int stride, int m, int ks, int lane)
{
    return *reinterpret_cast<const half4_t *>(s + (16 * m + (lane & 15)) * stride + 16 * ks + 4 * (lane >> 4));
}

__device__ __forceinline__ half8_t net_load_a8(const _Float16 *s, int stride, int m, int ks, int lane)
{
    return *reinterpret_cast<const half8_t *>(s + (16 * m + (lane & 15)) * stride + 32 * ks + 8 * (lane >> 4));
}

// The FP16 pair (hi, lo) of a: hi = fp16(a), lo = fp16(a - hi).
__device__ __forceinline__ void split_half(float a, _Float16 &hi, _Float16 &lo)
{
    hi = (_Float16)a;
    lo = (_Float16)(a - (float)hi);
}

// The biases of this lane's four units of block n.
__device__ __forceinline__ float4_t net_bias(const float *bias, int n, int lane)
{
    return *(global_ptr<const float4_t>)(bias + 16 * n + 4 * (lane >> 4));
}

// D tile (row block m, unit block n) + bias, ReLU, stored as the (hi, lo)
// pairs of the next layer's input rows (lo `width` halves after hi).
__device__ __forceinline__ void net_store_relu_h(_Float16 *s, int stride, int width, int m, int n, int lane,
                                                 float4_t d, float4_t bias)
{
    half4_t hi, lo;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        _Float16 h, l;
        split_half(fmaxf(d[j] + bias[j], 0.0f), h, l);
        hi[j] = h;
        lo[j] = l;
    }
    _Float16 *r = s + (16 * m + (lane & 15)) * stride + 16 * n + 4 * (lane >> 4);
    *reinterpret_cast<half4_t *>(r) = hi;
    *reinterpret_cast<half4_t *>(r + width) = lo;
}

// Same, FP32 rows (the last hidden layer, read by the output dot product).
__device__ __forceinline__ void net_store_relu_f(float *s, int stride, int m, int n, int lane, float4_t d,
                                                 float4_t bias)
{
    float4_t v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = fmaxf(d[j] + bias[j], 0.0f);
    *reinterpret_cast<float4_t *>(s + (16 * m + (lane & 15)) * stride + 16 * n + 4 * (lane >> 4)) = v;
}

// Unit blocks n0 .. n0 + kN - 1 of row blocks m0 .. m0 + kM - 1 of a layer of
// kSteps k-steps of 32 over the previous layer's outputs in LDS (rows of
// `stride` halves, lo `width` after hi), each taken as hi and as lo; b holds
// the weights by block, then step.
template <int kM, int kN, int kSteps>
__device__ __forceinline__ void net_layer(const _Float16 *s, int stride, int width, const half8_t (&b)[kN][kSteps],
                                          int m0, int lane, float4_t (&d)[kM][kN])
{
#pragma unroll
    for (int m = 0; m < kM; ++m)
#pragma unroll
        for (int n = 0; n < kN; ++n) d[m][n] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < kSteps; ++k)
#pragma unroll
        for (int m = 0; m < kM; ++m)
        {
            const half8_t hi = net_load_a8(s, stride, m0 + m, k, lane), lo = net_load_a8(s + width, stride, m0 + m, k, lane);
#pragma unroll
            for (int n = 0; n < kN; ++n) {
                d[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b[n][k], hi, d[m][n], 0, 0, 0);
                d[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b[n][k], lo, d[m][n], 0, 0, 0);
            }
        }
}

// Output layer for row `lane`: d = b4 + w4 . a3[lane] (w4 in LDS).
__device__ __forceinline__ float net_output(const float *s_a3, const float *s_w4, float b4, int lane)
{
    float dist = b4;
    const float *a3 = s_a3 + lane * kNetA3;
#pragma unroll
    for (int k = 0; k < kNetH3; k += 4) {
        const float4 v = *reinterpret_cast<const float4 *>(a3 + k);
        const float4 w = *reinterpret_cast<const float4 *>(s_w4 + k);
        dist = fmaf(w.x, v.x, dist);
        dist = fmaf(w.y, v.y, dist);
        dist = fmaf(w.z, v.z, dist);
        dist = fmaf(w.w, v.w, dist);
    }
    return dist;
}

}  // namespace storm
