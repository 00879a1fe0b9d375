// Batched forward kinematics and manipulability (Sec. 3.1, Eq. 8; Eq. 12):
// one lane per joint configuration.  Configurations come as columns [7][n] or
// as rows [n][7]; rows go through LDS, so that memory is read in whole lines
// (transposing them in a pass of its own took 7 us of 22 at n = 262144; the
// kernel, bound by VALU issue, 10 us).
#include "kinematics.h"

namespace storm {
namespace {

constexpr int kFkThreads = 256;

template <bool kRows>
__global__ __launch_bounds__(kFkThreads) void fk_kernel(RobotDev R, const float *__restrict__ q, int n,
                                                        float *__restrict__ pose, float *__restrict__ manip)
{
    const int t = blockIdx.x * kFkThreads + threadIdx.x;
    float qj[kDof];
    if (kRows) {
        __shared__ float s_q[kFkThreads * kDof];
        const size_t base = (size_t)blockIdx.x * kFkThreads * kDof, end = (size_t)n * kDof;
#pragma unroll
        for (int k = 0; k < kDof; ++k) {
            const size_t e = base + k * kFkThreads + threadIdx.x;
            qj[k] = e < end ? q[e] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < kDof; ++k) s_q[k * kFkThreads + threadIdx.x] = qj[k];
        __syncthreads();
        // (a stride of 7 words: no bank conflicts)
#pragma unroll
        for (int j = 0; j < kDof; ++j) qj[j] = s_q[threadIdx.x * kDof + j];
    } else {
#pragma unroll
        for (int j = 0; j < kDof; ++j) qj[j] = t < n ? q[(size_t)j * n + t] : 0.0f;
    }
    if (t >= n) return;
    float r[9] = {1.0f, 0.0f, 0.0f, 0.0f, 1.0f, 0.0f, 0.0f, 0.0f, 1.0f};
    float p[3] = {0.0f, 0.0f, 0.0f};
    float z[kDof][3], o[kDof][3];
#pragma unroll
    for (int f = 0; f < kFrames; ++f) {
        float st = 0.0f, ct = 1.0f;
        if (f < kDof) sincosf(qj[f], &st, &ct);
        dh_step(r, p, R.ca[f], R.sa[f], R.a[f], R.d[f], ct, st);
        if (f < kDof) {
            z[f][0] = r[2];
            z[f][1] = r[5];
            z[f][2] = r[8];
            o[f][0] = p[0];
            o[f][1] = p[1];
            o[f][2] = p[2];
        }
    }
#pragma unroll
    for (int c = 0; c < 9; ++c) pose[(size_t)c * n + t] = r[c];
#pragma unroll
    for (int c = 0; c < 3; ++c) pose[(size_t)(9 + c) * n + t] = p[c];
    if (manip) manip[t] = manipulability(z, o, p);
}

}  // namespace

hipError_t launch_fk(const RobotDev &R, const float *q, bool rows, int n, float *pose, float *manip,
                     hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(rows ? fk_kernel<true> : fk_kernel<false>, dim3((unsigned)((n + kFkThreads - 1) / kFkThreads)),
                       dim3(kFkThreads), 0, stream, R, q, n, pose, manip);
    return hipGetLastError();
}

}  // namespace storm
