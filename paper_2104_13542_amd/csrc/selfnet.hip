// Learned self-collision term (Sec. 3.2, Eq. 13, the jointNERF form) on the
// matrix cores.  The network maps the encoding [sin q, cos q] through ReLU
// layers of 256, 128 and 64 units to one output d, the predicted closest
// distance between the links (positive when they penetrate); the term is
// max(0, d).
//
// One workgroup (8 waves) per 64-lane tile of the rollout (the same
// (particle, step) rows): the three hidden layers are 64-row GEMMs on
// v_mfma_f32_16x16x16_f16 (layer 1) and v_mfma_f32_16x16x32_f16 (FP16
// weights, activations as FP16 (hi, lo) pairs, FP32 accumulation), with
// the activations staged in LDS between layers and the weights read as
// pre-packed per-lane fragments (one coalesced 512-byte load per wave and
// fragment).  The output layer is a 64-term dot product per row on the
// vector units; the term then joins the running cost (weight a_coll, as the
// sphere model's) and, through a segmented scan over the steps, the horizon
// cost C_i that the rollout kernel wrote.
//
// One workgroup per CU (104 KB of LDS) and one or two rounds at the usual sizes:
// bound by latency and by LDS traffic.  A wave takes 32 units of 32 rows of
// layer 2, so that the activations are read four times (eight with 16 units of
// all rows), a lane's results go to LDS in one write (four), and what the last
// phase reads of memory is loaded at the start.  At 500 x 30 8.9 -> 7.6 us, the
// control call with the network 22.9 -> 21.6 us.
#include "sampling.h"
#include "selfnet.h"
#include "storm_internal.h"

namespace storm {

namespace {

constexpr int kNetWaves = 8;
constexpr int kNetThreads = kNetWaves * kLanes;
constexpr int kIn = 16;      // 14 inputs padded to one k-step
constexpr int kX = 2 * kIn;  // LDS row stride of the encoding in halves: hi (16), lo (16)
// LDS: encoding, first and second hidden layers; the last hidden layer's
// FP32 rows reuse the first layer's space (dead once layer 2 has run)
constexpr int kOffA1 = 64 * kX * 2;
constexpr int kOffA2 = kOffA1 + 64 * kNetA1 * 2;
constexpr int kNetLds = kOffA2 + 64 * kNetA2 * 2;
static_assert(64 * kNetA3 * 4 <= 64 * kNetA1 * 2, "last hidden layer fits in the first layer's space");

// kDebug: with the per-step outputs, which are read from the argument segment
// (the other arguments are preloaded into SGPRs).
template <bool kDebug>
__global__ __launch_bounds__(kNetThreads) void selfnet_kernel(const PlainDev *dev, int32_t N, int32_t H,
                                                              const float *__restrict__ qbuf,
                                                              const _Float16 *__restrict__ frag,
                                                              const float *__restrict__ bias, float *C_out,
                                                              float *c_out, float *terms_out)
{
    ProblemRef P = uniform_ptr(dev)->P;
    // what the last phase reads of the problem, issued first and waited for
    // behind the weight loads
    float a_coll = P.a_coll;
    const float *tables = P.tables;
    float *C_sum = P.C;
    __builtin_amdgcn_sched_barrier(0);
    __shared__ __attribute__((aligned(16))) float s_w4[kNetH3];
    __shared__ __attribute__((aligned(16))) unsigned char s_lds[kNetLds];
    _Float16 *s_x = reinterpret_cast<_Float16 *>(s_lds);
    _Float16 *s_a1 = reinterpret_cast<_Float16 *>(s_lds + kOffA1);
    _Float16 *s_a2 = reinterpret_cast<_Float16 *>(s_lds + kOffA2);
    float *s_a3 = reinterpret_cast<float *>(s_lds + kOffA1);

    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x;
    const int ppt = kLanes / H;

    // row `lane` of the tile; wave j < 7 encodes joint j of every row.  Its
    // position is loaded first, so that waiting for it does not wait for the
    // weight loads behind it (an invalid row reads particle 0 and is ignored).
    const int pl = (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)H));  // lane / H (exact, as in kernel R)
    const int h = lane - pl * H;
    const int i = tile * ppt + pl;
    const bool valid = pl < ppt && i < N;
    const int jq = wave < kDof ? wave : 0;
    const float qv = qbuf[((size_t)jq * N + (valid ? i : 0)) * H + h];
    __builtin_amdgcn_sched_barrier(0);  // keep that load ahead of the weight loads

    // every weight fragment this wave uses, loaded up front (104 VGPRs)
    // (in the order of use, each layer's biases with its fragments)
    const half4_t *F1 = reinterpret_cast<const half4_t *>(frag + kNetFrag1);
    const half8_t *F2 = reinterpret_cast<const half8_t *>(frag + kNetFrag2);
    const half8_t *F3 = reinterpret_cast<const half8_t *>(frag + kNetFrag3);
    half4_t b1[2];
    half8_t b2[2][8], b3[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) b1[t] = F1[(2 * wave + t) * kLanes + lane];
    const float4_t bias1[2] = {net_bias(bias + kNetBias1, 2 * wave, lane), net_bias(bias + kNetBias1, 2 * wave + 1, lane)};
    __builtin_amdgcn_sched_barrier(0);
    const int n2 = 2 * (wave >> 1), m2 = 2 * (wave & 1);  // layer 2: 32 units of 32 rows
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int n = 0; n < 2; ++n) b2[n][s] = F2[((n2 + n) * 8 + s) * kLanes + lane];
    const float4_t bias2[2] = {net_bias(bias + kNetBias2, n2, lane), net_bias(bias + kNetBias2, n2 + 1, lane)};
    __builtin_amdgcn_sched_barrier(0);
    const int n3 = 2 * (wave & 1), m3 = wave >> 1;  // layer 3: 32 units of 16 rows
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int n = 0; n < 2; ++n) b3[n][s] = F3[((n3 + n) * 4 + s) * kLanes + lane];
    const float4_t bias3[2] = {net_bias(bias + kNetBias3, n3, lane), net_bias(bias + kNetBias3, n3 + 1, lane)};

    // What the last phase needs, so that no memory round trip stands in it:
    // the output weights (to LDS before the last barrier), and on wave 0 the
    // horizon weight and the cost that the rollout wrote (every point of a
    // particle reads its particle's).
    asm volatile("" : "+s"(a_coll), "+s"(tables), "+s"(C_sum));
    const float w4 = bias[kNetW4 + lane], b4 = vector_load_f32(bias + kNetBias4);
    const float hw = as_global(tables)[kTabHw + h], C_rollout = as_global(C_sum)[valid ? i : 0];

    // encoding [sin q, cos q, 0, 0] of the 64 rows, as (hi, lo) pairs (by
    // every wave: a branch here would take the load of q with it, behind the
    // weights)
    {
        float sn, cs;
        sincosf(valid ? qv : 0.0f, &sn, &cs);
        const bool joint = wave < kDof;
        _Float16 *r = s_x + lane * kX;
        const int a = joint ? wave : 14, b = joint ? kDof + wave : 15;
        split_half(joint ? sn : 0.0f, r[a], r[kIn + a]);
        split_half(joint ? cs : 0.0f, r[b], r[kIn + b]);
    }
    __syncthreads();

    // layer 1: 64 x 16 by 16 x 256 for hi and for lo; wave w: columns
    // 32 w .. 32 w + 31
    {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const half4_t ahi = net_load_a(s_x, kX, m, 0, lane);
            const half4_t alo = net_load_a(s_x + kIn, kX, m, 0, lane);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float4_t d = {0.0f, 0.0f, 0.0f, 0.0f};
                d = __builtin_amdgcn_mfma_f32_16x16x16f16(b1[t], ahi, d, 0, 0, 0);
                d = __builtin_amdgcn_mfma_f32_16x16x16f16(b1[t], alo, d, 0, 0, 0);
                net_store_relu_h(s_a1, kNetA1, kNetH1, m, 2 * wave + t, lane, d, bias1[t]);
            }
        }
    }
    __syncthreads();

    // layer 2: 64 x 256 by 256 x 128; a wave: 32 units of 32 rows
    {
        float4_t d[2][2];
        net_layer(s_a1, kNetA1, kNetH1, b2, m2, lane, d);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n) net_store_relu_h(s_a2, kNetA2, kNetH2, m2 + m, n2 + n, lane, d[m][n], bias2[n]);
    }
    __syncthreads();

    // layer 3: 64 x 128 by 128 x 64; a wave: 32 units of 16 rows; its FP32
    // output rows go where layer 1's were
    {
        float4_t d[1][2];
        net_layer(s_a2, kNetA2, kNetH2, b3, m3, lane, d);
#pragma unroll
        for (int n = 0; n < 2; ++n) net_store_relu_f(s_a3, kNetA3, m3, n3 + n, lane, d[0][n], bias3[n]);
    }
    if (wave == kNetWaves - 1) s_w4[lane] = w4;
    __syncthreads();

    // output layer, cost term and horizon cost (wave 0, lane = row)
    if (wave == 0) {
        const float dist = net_output(s_a3, s_w4, b4, lane);
        const float term = fmaxf(dist, 0.0f);  // Eq. 13
        const float dc = a_coll * term;
        const float added = segmented_scan(hw * dc, h, H);
        if (valid) {
            if (kDebug && terms_out) terms_out[((size_t)6 * N + i) * H + h] = term;
            if (kDebug && c_out) c_out[(size_t)i * H + h] += dc;
            if (h == H - 1) {
                const float sum = C_rollout + added;
                as_global(C_sum)[i] = sum;
                if (C_out) C_out[i] = sum;
            }
        }
    }
}

}  // namespace

hipError_t launch_selfnet(const ProblemDev &P, const PlainDev *dev, const StepOut &out, hipStream_t stream)
{
    auto kernel = out.c != nullptr || out.terms != nullptr ? selfnet_kernel<true> : selfnet_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)P.n_tiles), dim3(kNetThreads), 0, stream, dev, P.N, P.H, P.qbuf,
                       P.net_frag, P.net_bias, out.C, out.c, out.terms);
    return hipGetLastError();
}

bool selfnet_weights_fp16(const float *prm)
{
    const float *W1 = prm, *W2 = W1 + kNetH1 * kNetIn + kNetH1, *W3 = W2 + kNetH2 * kNetH1 + kNetH2;
    auto exact = [](const float *W, int n) {
        for (int k = 0; k < n; ++k)
            if ((float)(_Float16)W[k] != W[k]) return false;
        return true;
    };
    return exact(W1, kNetH1 * kNetIn) && exact(W2, kNetH2 * kNetH1) && exact(W3, kNetH3 * kNetH2);
}

// Pack the network's parameters (weights [out][in], FP32 holding FP16
// values) into the per-lane FP16 fragments the kernel loads, and the biases
// and output weights (FP32).
void pack_selfnet(const float *prm, std::vector<_Float16> &frag, std::vector<float> &bias)
{
    const float *W1 = prm, *b1 = W1 + kNetH1 * kNetIn;
    const float *W2 = b1 + kNetH1, *b2 = W2 + kNetH2 * kNetH1;
    const float *W3 = b2 + kNetH2, *b3 = W3 + kNetH3 * kNetH2;
    const float *w4 = b3 + kNetH3, *b4 = w4 + kNetH3;
    frag.assign((size_t)kNetFragHalves, (_Float16)0.0f);
    // fragment (column block t, k-step s) of B = W^T with `per` halves per
    // lane (k-steps of 4 per): lane l, element j is
    // W[16 t + l % 16][4 per s + per (l / 16) + j]
    auto put = [&](int base, const float *W, int n_in, int n_tiles, int n_steps, int per) {
        for (int t = 0; t < n_tiles; ++t)
            for (int s = 0; s < n_steps; ++s)
                for (int l = 0; l < kLanes; ++l)
                    for (int j = 0; j < per; ++j) {
                        const int o = 16 * t + (l & 15), k = 4 * per * s + per * (l >> 4) + j;
                        frag[(size_t)base + (((size_t)t * n_steps + s) * kLanes + l) * per + j] =
                            (_Float16)(k < n_in ? W[o * n_in + k] : 0.0f);
                    }
    };
    put(kNetFrag1, W1, kNetIn, kNetH1 / 16, 1, 4);
    put(kNetFrag2, W2, kNetH1, kNetH2 / 16, kNetH1 / 32, 8);
    put(kNetFrag3, W3, kNetH2, kNetH3 / 16, kNetH2 / 32, 8);
    bias.assign((size_t)kNetBiasSize, 0.0f);
    for (int k = 0; k < kNetH1; ++k) bias[kNetBias1 + k] = b1[k];
    for (int k = 0; k < kNetH2; ++k) bias[kNetBias2 + k] = b2[k];
    for (int k = 0; k < kNetH3; ++k) bias[kNetBias3 + k] = b3[k];
    for (int k = 0; k < kNetH3; ++k) bias[kNetW4 + k] = w4[k];
    bias[kNetBias4] = b4[0];
}

}  // namespace storm
