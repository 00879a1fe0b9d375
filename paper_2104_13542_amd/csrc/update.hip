// Kernel U: exponentiated-cost policy update of STORM (Sec. 3, Eq. 4-6),
// followed by the next command and the warm-start shift of Alg. 1.
//
//   w_i     = exp(-(C_i - min C) / beta) / sum_k exp(-(C_k - min C) / beta)
//   mu'     = mu + alpha_mu sum_i w_i d_i,          d_i = u_i - mu
//   sigma2' = (1 - alpha_sigma) sigma2
//             + alpha_sigma mean_h sum_i w_i (u_ih - mu'_h)^2   (per joint)
//
// Three forms.  Up to 32 R particles (R = 1024 / H rows) and 2048, one
// 1024-thread workgroup per (problem, joint): a joint's new mean and variance
// depend only on the weights and on that joint's controls, so the seven joints
// need no synchronisation with each other; every workgroup recomputes min C and
// the weights of all particles (N exponentials).  The joint's H columns are
// read by rows of threads, row r taking particles r, r + R, ...; every thread
// loads its up to 32 controls at the start, together with the costs, so the
// only global-memory latency on the path is the first one.  Bound by latency:
// two exchanges, a division and the tail's chain behind the first loads
// (4.2 us at 500 x 30).  Past those sizes, the controls of the particles that
// have a weight, gathered by one workgroup per joint (update_all) or, of more
// points, by one per chain of sums (update_chain and update_join), both below.
//
// The variance about the new mean comes from the moments about the old one,
// sum w (d - delta)^2 = S2/S0 - 2 delta S1/S0 + delta^2, in one pass.  Wave
// reductions use DPP lane moves; every sum has a fixed order, so results are
// bitwise reproducible; there is no floating-point atomic and no
// synchronisation between workgroups.
#include "storm_internal.h"

namespace storm {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kLanes;
constexpr int kRows = 8192;   // most rows times controls per thread (weights staged in LDS)
constexpr int kRegU = 32;     // most controls per thread held in registers

// Full-wave reductions through DPP lane moves (quad permutes, half-row and
// row mirrors, then the row broadcasts that carry each row's result into the
// next); lane 63, which every step feeds, holds the result, read back into
// an SGPR.  The order of the operations is fixed.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_move(int x)
{
    return __builtin_amdgcn_mov_dpp(x, kCtrl, kRowMask, 0xf, false);
}

__device__ __forceinline__ float wave_sum(float x)
{
    x += __int_as_float(dpp_move<0xb1, 0xf>(__float_as_int(x)));
    x += __int_as_float(dpp_move<0x4e, 0xf>(__float_as_int(x)));
    x += __int_as_float(dpp_move<0x141, 0xf>(__float_as_int(x)));
    x += __int_as_float(dpp_move<0x140, 0xf>(__float_as_int(x)));
    x += __int_as_float(dpp_move<0x142, 0xa>(__float_as_int(x)));
    x += __int_as_float(dpp_move<0x143, 0xc>(__float_as_int(x)));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// IEEE bits mapped so that signed-integer order is float order (negative
// values have their magnitude bits flipped); the map is its own inverse.
__device__ __forceinline__ int ordered(int b) { return b ^ (int)((uint32_t)(b >> 31) >> 1); }

__device__ __forceinline__ float wave_min(float x)
{
    int b = ordered(__float_as_int(x));
    b = min(b, dpp_move<0xb1, 0xf>(b));
    b = min(b, dpp_move<0x4e, 0xf>(b));
    b = min(b, dpp_move<0x141, 0xf>(b));
    b = min(b, dpp_move<0x140, 0xf>(b));
    b = min(b, dpp_move<0x142, 0xa>(b));
    b = min(b, dpp_move<0x143, 0xc>(b));
    return __int_as_float(ordered(__builtin_amdgcn_readlane(b, 63)));
}

// x moved into VGPRs at this point (a wave-uniform value the compiler
// would otherwise keep, or reload, as a scalar).
template <typename T>
__device__ __forceinline__ T in_vgpr(T x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// The same for a pointer, kept a global-memory pointer so that accesses
// through it stay global (not flat) instructions.
template <typename T>
__device__ __forceinline__ global_ptr<T> global_in_vgpr(T *p)
{
    global_ptr<T> g = (global_ptr<T>)p;
    asm volatile("" : "+v"(g));
    return g;
}

// Minimum of v over the workgroup (all threads get it).
__device__ __forceinline__ float block_min(float v, float *s_wave, int lane, int wave)
{
    v = wave_min(v);
    if (lane == 0) s_wave[wave] = v;
    __syncthreads();
    float m = s_wave[0];
    for (int k = 1; k < kWaves; ++k) m = fminf(m, s_wave[k]);
    __syncthreads();
    return m;
}

// Workgroup LDS of the update, declared once per kernel.
struct UpdateLds {
    float buf[kRows];  // weights
    float red[2 * kThreads];
    float wave[kWaves];
    float wsum[kWaves];
    int count[kWaves];
    float mold[kMaxH];
};

// Controls per thread for N particles over `rows` rows: the smallest of 8, 16
// and 32 that holds them (0: the larger form).
__host__ __device__ inline int update_slots(int N, int H)
{
    const int rows = kThreads / H;
    if (N > 2 * kThreads) return 0;
    for (int k = 8; k <= kRegU; k *= 2)
        if (N <= k * rows && k * rows <= kRows) return k;
    return 0;
}

// The fields of a problem that the first loads depend on.
struct UpdateFirst {
    const float *C, *u;
    int32_t N, H;
};

// What an update reads of its problem's descriptor, in one go: a scalar load
// wherever a field is used would put one memory round trip after another.
struct UpdateProblem {
    float beta, alpha_mu, alpha_sigma, sigma2_min;
    const float *tables;
    float *mean, *sigma2;
    uint32_t *step, *status;
};
__device__ __forceinline__ UpdateProblem fetch_problem(ProblemRef P)
{
    return UpdateProblem{P.beta, P.alpha_mu, P.alpha_sigma, P.sigma2_min, P.tables, P.mean, P.sigma2, P.step, P.status};
}
// (here they have to be there)
__device__ __forceinline__ void wait_problem(UpdateProblem &Q)
{
    asm volatile("" : "+s"(Q.beta), "+s"(Q.alpha_mu), "+s"(Q.alpha_sigma), "+s"(Q.sigma2_min), "+s"(Q.tables),
                 "+s"(Q.mean), "+s"(Q.sigma2), "+s"(Q.step), "+s"(Q.status));
}

// What the tail of an update reads besides the moments.
struct TailArgs {
    float sig_old, sig_init, a_mu, a_sigma, s2_min;
    uint32_t step0;
    int shift;
    global_ptr<float> mean, sigma2, cmd, mean_out, sigma2_out;
    global_ptr<uint32_t> step, status;
};

// Fetched with the kernel's first loads, since each would add a memory round
// trip to the tail: the old variances and the noise counter through vector
// loads (waited for only where they are used); the scalars go into VGPRs,
// because the kernel runs at its SGPR limit and the compiler would otherwise
// reload each there, one scalar-memory round trip after another.
__device__ __forceinline__ TailArgs fetch_tail(const UpdateProblem &P, float *mean_out, float *sigma2_out, float *cmd,
                                               int shift, const bool cov, int j, int t, int H)
{
    TailArgs T;
    T.sig_old = cov ? (t < H ? vector_load_f32(P.sigma2 + t * kDof + j) : 0.0f) : vector_load_f32(P.sigma2 + j);
    T.sig_init = cov && shift ? vector_load_f32(P.tables + kTabSig0 + j) : 0.0f;
    T.step0 = vector_load_u32(P.step);
    T.mean = global_in_vgpr(P.mean);
    T.sigma2 = global_in_vgpr(P.sigma2);
    T.cmd = global_in_vgpr(cmd);
    T.mean_out = global_in_vgpr(mean_out);
    T.sigma2_out = global_in_vgpr(sigma2_out);
    T.step = global_in_vgpr(P.step);
    T.status = global_in_vgpr(P.status);
    T.shift = in_vgpr(shift);
    T.a_mu = in_vgpr(P.alpha_mu);
    T.a_sigma = in_vgpr(P.alpha_sigma);
    T.s2_min = in_vgpr(P.sigma2_min);
    return T;
}

// The end of joint j's update on one wave: lane h holds the weighted sums S1
// and S2 of step h about the old mean muo; S0 is the sum of the weights.
// Forms the new mean and the variance about it, then one wave sum gives the
// variance over the horizon.
__device__ __forceinline__ void update_tail(const TailArgs &T, const int j, const int H, const int lane, float s1,
                                            float s2, float S0, float muo, bool ok, int any_nonfinite, const bool cov)
{
    const float inv_S0 = 1.0f / S0;
    const float m1 = s1 * inv_S0, m2 = s2 * inv_S0;
    const float delta = T.a_mu * m1;
    const float mu_new = ok ? muo + delta : muo;
    const float var = lane < H ? fmaxf(fmaf(delta, delta - 2.0f * m1, m2), 0.0f) : 0.0f;  // about mu'
    const float acc = wave_sum(var);
    // the new mean of step h + 1 (the shifted warm start), 0 past the end
    const float mu_next = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mu_new), 0x130, 0xf, 0xf,
                                                                     true));  // wave_shl:1
    if (lane == 0) {
        if (j == 0) {
            // the increment here, not at the load (where it would wait for
            // every load in flight), and before the other stores (whose
            // completion a wait for the load would otherwise include)
            uint32_t next = T.step0;
            asm volatile("" : "+v"(next));
            *T.step = next + 1u;
            if (!ok)
                __hip_atomic_fetch_or(T.status, any_nonfinite ? STORM_FLAG_NONFINITE_COST : STORM_FLAG_ZERO_WEIGHT,
                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (!cov) {
            float s2n = T.sig_old;
            if (ok) s2n = fmaxf(fmaf(T.a_sigma, acc / (float)H - T.sig_old, T.sig_old), T.s2_min);
            T.sigma2[j] = s2n;
            if (T.sigma2_out) T.sigma2_out[j] = s2n;
        }
        T.cmd[j] = mu_new;
    }
    if (lane < H) {
        if (T.mean_out) T.mean_out[lane * kDof + j] = mu_new;
        T.mean[lane * kDof + j] = T.shift ? (lane + 1 < H ? mu_next : 0.0f) : mu_new;
    }
    if (cov) {
        // Eq. 5 per step: lane h updates sigma^2[h][j] from the variance at
        // step h; the shift moves it one step, sigma_init^2 appended
        const float old = T.sig_old;  // sigma^2[lane][j] (0 past H)
        const float s2n = ok ? fmaxf(fmaf(T.a_sigma, var - old, old), T.s2_min) : old;
        const float s2_next = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s2n), 0x130, 0xf, 0xf,
                                                                         true));  // wave_shl:1
        if (lane < H) {
            if (T.sigma2_out) T.sigma2_out[lane * kDof + j] = s2n;
            T.sigma2[lane * kDof + j] = T.shift ? (lane + 1 < H ? s2_next : T.sig_init) : s2n;
        }
    }
}

// `cov` is P.cov_step, passed apart so that the plain kernel can fix it at
// compile time; kSlots the controls per thread (update_slots).
template <int kSlots>
__device__ __forceinline__ void update_joint(ProblemRef descriptor, const UpdateFirst &first, const int j,
                                             float *__restrict__ mean_out, float *__restrict__ sigma2_out,
                                             float *__restrict__ cmd, int shift, const bool cov, UpdateLds &L)
{
    // issued before the arithmetic of the addresses below: the descriptor,
    // and this thread's first two costs
    const int t = threadIdx.x;
    const int N = first.N, H = first.H;
    const global_ptr<const float> C = as_global(first.C);
    UpdateProblem P = fetch_problem(descriptor);
    float c0 = C[min(t, N - 1)], c1 = C[min(t + kThreads, N - 1)];
    __builtin_amdgcn_sched_barrier(0);
    float *s_buf = L.buf;
    float *s_red = L.red;
    float *s_wave = L.wave;
    float *s_wsum = L.wsum;
    int *s_count = L.count;
    float *s_mold = L.mold;

    const int lane = t & (kLanes - 1), wave = __builtin_amdgcn_readfirstlane(t / kLanes);

    // thread (r, h): step h of particles r, r + rows, ...
    const int rows = kThreads / H;
    const int r = t / H, h = t - r * H;
    const bool in_rows = r < rows;
    // Every control load, in flight at once, through a buffer resource bounded
    // by the joint's N H values: slots past the last particle read 0 and cost no
    // address arithmetic (the load returns the raw 32 bits).
    float uu[kSlots];
    {
        const __amdgpu_buffer_rsrc_t ub = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(first.u + (size_t)j * N * H), (short)0, N * H * (int)sizeof(float), 0x00020000);
        const int stride = rows * H * (int)sizeof(float);
#pragma unroll
        for (int k = 0; k < kSlots; ++k)
            uu[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ub, t * 4 + k * stride, 0, 0));
    }
    wait_problem(P);
    const float nib = -1.0f / P.beta;
    const float mu = as_global(P.mean)[h * kDof + j];
    const TailArgs T = fetch_tail(P, mean_out, sigma2_out, cmd, shift, cov, j, t, H);

    float S0 = 0.0f, x1 = 0.0f, x2 = 0.0f;
    int any_nonfinite = 0;
    bool ok = false;
    // min C and the non-finite flag in one exchange, then the weights
    // and their sum in a second (separate LDS slots: no third barrier)
    if (t >= N) c0 = INFINITY;
    if (t + kThreads >= N) c1 = INFINITY;
    const bool bad = (t < N && !isfinite(c0)) || (t + kThreads < N && !isfinite(c1));
    const uint64_t bad_lanes = __builtin_amdgcn_ballot_w64(bad);
    const float wmin = wave_min(fminf(c0, c1));
    if (lane == 0) {
        s_wave[wave] = wmin;
        s_count[wave] = bad_lanes != 0;
    }
    __syncthreads();
    float cmin = s_wave[0];
    any_nonfinite = s_count[0];
    for (int k = 1; k < kWaves; ++k) {
        cmin = fminf(cmin, s_wave[k]);
        any_nonfinite |= s_count[k];
    }
    const float w0 = t < N ? expf((c0 - cmin) * nib) : 0.0f;
    const float w1 = t + kThreads < N ? expf((c1 - cmin) * nib) : 0.0f;
    s_buf[t] = w0;
    s_buf[t + kThreads] = w1;
    for (int i = 2 * kThreads + t; i < kSlots * rows; i += kThreads) s_buf[i] = 0.0f;  // slots past N
    const float sw = wave_sum(w0 + w1);
    if (lane == 0) s_wsum[wave] = sw;
    __syncthreads();
    for (int k = 0; k < kWaves; ++k) S0 += s_wsum[k];
    ok = !any_nonfinite && S0 > 0.0f && isfinite(S0);
    // straight-line over the 32 slots (weight 0 and control 0 past the
    // last particle) so that every LDS read is in flight before the first use
    float a1[4] = {0.0f, 0.0f, 0.0f, 0.0f}, a2[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (in_rows && ok) {
#pragma unroll
        for (int k = 0; k < kSlots; ++k) {
            const float d = uu[k] - mu;
            const float wd = s_buf[r + k * rows] * d;
            a1[k & 3] += wd;
            a2[k & 3] = fmaf(wd, d, a2[k & 3]);
        }
    }
    x1 = (a1[0] + a1[1]) + (a1[2] + a1[3]);
    x2 = (a2[0] + a2[1]) + (a2[2] + a2[3]);

    // Wave 0 finishes alone: lane h adds the rows of step h in order (S1, S2)
    // and update_tail does the rest; no further workgroup barrier.
    s_red[t] = x1;
    s_red[kThreads + t] = x2;
    if (r == 0) s_mold[h] = mu;  // stored late: an early store would wait for every load in flight
    __syncthreads();
    if (wave == 0) {
        float s1 = 0.0f, s2 = 0.0f, muo = 0.0f;
        if (lane < H) {
            for (int k = 0; k < rows; ++k) {
                s1 += s_red[k * H + lane];
                s2 += s_red[kThreads + k * H + lane];
            }
            muo = s_mold[lane];
        }
        update_tail(T, j, H, lane, s1, s2, S0, muo, ok, any_nonfinite, cov);
    }
}

// All arguments fit the 14 dwords that are preloaded into SGPRs; the rest of
// the problem comes from its descriptor in device memory.  kCov: one variance
// per (step, joint) instead of one per joint.
template <bool kCov, int kSlots>
__global__ __launch_bounds__(kThreads) void update_kernel(const PlainDev *dev, const float *C, const float *u,
                                                          float *__restrict__ mean_out,
                                                          float *__restrict__ sigma2_out, float *__restrict__ cmd,
                                                          int32_t N, int16_t H, int16_t shift)
{
    __shared__ UpdateLds L;
    ProblemRef P = uniform_ptr(dev)->P;
    const UpdateFirst first{C, u, N, H};
    update_joint<kSlots>(P, first, blockIdx.x, mean_out, sigma2_out, cmd, shift, kCov, L);
}

// The larger forms: the same update for more particles.  A thread (row r, step
// h) sums its particles in eight accumulators, number m taking every eighth of
// them: eight chains.  Two ways to gather the particles:
//   list   (at most 4096 weights not exactly zero, beta small against the spread
//          of C): only those, from a list compacted in ascending order;
//   dense  otherwise: all, weights staged in LDS by chunks.
// update_all: one workgroup per joint sums all eight.  It pulls the N H controls
// of the joint through one CU, eight loads in flight per thread, and that time is
// its bound.  update_chain: a workgroup per (joint, m) sums one chain, each in the
// order that one workgroup would, and update_join adds the eight and takes the
// tail, to the same bits; each workgroup finds min C and the weights it needs
// itself (three passes over C, from L2).  The update alone, one kernel and two,
// us: 600 x 64 8.0 and 10.5, 1500 x 30 8.9 and 11.2, 2500 x 30 10.5 and 11.4, 4096
// x 30 13.4 and 12.2, 2048 x 64 12.7 and 10.8, 8000 x 6 15.2 and 16.4, 65536 x 30
// (by one workgroup per joint 90-180) 67: the line lies at 90000 points.  A batch
// has workgroups enough and takes update_all as far as its registers hold the
// costs (64 problems of 2048 x 64 42 us, of 4096 x 64 102).
constexpr int kChains = 8;    // accumulators of a thread
constexpr int kList = 4096;   // capacity of the list
constexpr int kChunk = 8192;  // weights staged at a time
// floats of a joint's partial sums, S1 and S2 of [chain][2][thread]; after all
// joints', the sum of the weights and whether a cost is not finite
constexpr int kJointPart = kChains * 2 * kThreads;
constexpr int kOnce = 8 * kThreads;  // costs that a workgroup holds in registers
constexpr int kUpdateParts = kDof * kChains + 1;  // workgroups: chains, and one for the weights' sum

// Whether one workgroup per joint takes a single problem past the register form.
inline bool update_once(int N, int H) { return N <= kOnce && N * H <= 90000; }

// Whether the weight exp(x) is not zero in FP32: below -104 it is (half the
// least denormal is exp(-103.97)), above -103 it is not.
constexpr float kNoWeight = -104.0f;
__device__ __forceinline__ bool has_weight(float x)
{
    if (x < kNoWeight) return false;
    return x > -103.0f || expf(x) > 0.0f;
}

// Part c of a problem: chain c % 8 of joint c / 8, or, last, the weights' sum.
__device__ __forceinline__ void update_chain(const float *__restrict__ C_in, const float *__restrict__ u_in,
                                             const float *__restrict__ mean_in, float *__restrict__ part_in,
                                             const int N, const int H, const float nib, const int c)
{
    __shared__ float s_w[kChunk];  // the list's weights, or a chunk's
    __shared__ int s_idx[kList];
    __shared__ float s_wave[kWaves];
    __shared__ int s_count[kWaves];
    const global_ptr<const float> C = as_global(C_in), mean = as_global(mean_in);
    const int t = threadIdx.x, lane = t & (kLanes - 1), wave = __builtin_amdgcn_readfirstlane(t / kLanes);
    const int rows = kThreads / H, r = t / H, h = t - r * H;
    const bool in_rows = r < rows;
    const int j = min(c / kChains, kDof - 1), m = c % kChains;
    const global_ptr<const float> U = as_global(u_in) + (size_t)j * N * H + h;
    const float mu = mean[h * kDof + j];

    // Min C.  A run of the particles per wave, eight costs per lane in flight
    // (an index past the end reads the last cost, and is left out below); a run
    // of at most eight per lane stays in registers for the passes that follow.
    const int run = (N + kThreads - 1) / kThreads * kLanes, i0 = wave * run, i1 = min(N, i0 + run);
    const bool once = run <= 8 * kLanes;
    float cv[8];
    auto fetch = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 8; ++k) cv[k] = C[min(i + k * kLanes, N - 1)];
    };
    float cmin = INFINITY;
    int nonfinite = 0;
    for (int i = i0 + lane; i < i0 + run; i += 8 * kLanes) {
        fetch(i);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            nonfinite |= !isfinite(cv[k]);
            cmin = fminf(cmin, cv[k]);
        }
    }
    nonfinite = __syncthreads_or(nonfinite);
    cmin = block_min(cmin, s_wave, lane, wave);

    if (c == kDof * kChains) {
        // the sum of the weights (per thread in stride order, per wave, waves
        // in order)
        float sw = 0.0f;
        for (int i = t; i < N; i += 8 * kThreads) {
            float x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = C[min(i + k * kThreads, N - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                x[k] = (x[k] - cmin) * nib;
                if (i + k * kThreads < N && !(x[k] < kNoWeight)) sw += expf(x[k]);
            }
        }
        sw = wave_sum(sw);
        if (lane == 0) s_wave[wave] = sw;
        __syncthreads();
        float S0 = 0.0f;
        for (int k = 0; k < kWaves; ++k) S0 += s_wave[k];
        const global_ptr<float> out = as_global(part_in) + (size_t)kDof * kJointPart;
        if (t == 0) {
            out[0] = S0;
            out[1] = nonfinite ? 1.0f : 0.0f;
        }
        return;
    }

    // the number of nonzero weights, in all and before this wave's
    int count = 0;
    for (int i = i0 + lane; i < i0 + run; i += 8 * kLanes) {
        if (!once) fetch(i);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            count += __builtin_popcountll(
                __builtin_amdgcn_ballot_w64(i + k * kLanes < i1 && has_weight((cv[k] - cmin) * nib)));
    }
    if (lane == 0) s_count[wave] = count;
    __syncthreads();
    int M = 0, at = 0;
    for (int k = 0; k < kWaves; ++k) {
        at += k < wave ? s_count[k] : 0;
        M += s_count[k];
    }

    // the chain: particles r + m rows, + 8 rows, ... while all eight chains have
    // one; the first takes the others that remain
    float a1 = 0.0f, a2 = 0.0f;
    if (M <= kList) {
        for (int i = i0 + lane; i < i0 + run; i += 8 * kLanes) {
            if (!once) fetch(i);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float x = (cv[k] - cmin) * nib;
                const bool nz = i + k * kLanes < i1 && has_weight(x);
                const uint64_t bal = __builtin_amdgcn_ballot_w64(nz);
                if (bal == 0) continue;
                if (nz) {
                    const int pos = at + __builtin_popcountll(bal & ((1ull << lane) - 1ull));
                    s_idx[pos] = i + k * kLanes;
                    s_w[pos] = expf(x);
                }
                at += __builtin_popcountll(bal);
            }
        }
        __syncthreads();
        if (in_rows) {
            int k = r;
#pragma unroll 4
            for (; k + (kChains - 1) * rows < M; k += kChains * rows) {
                const float d = U[(size_t)s_idx[k + m * rows] * H] - mu;
                const float wd = s_w[k + m * rows] * d;
                a1 += wd;
                a2 = fmaf(wd, d, a2);
            }
            for (; m == 0 && k < M; k += rows) {
                const float d = U[(size_t)s_idx[k] * H] - mu;
                const float wd = s_w[k] * d;
                a1 += wd;
                a2 = fmaf(wd, d, a2);
            }
        }
    } else {
        for (int c0 = 0; c0 < N; c0 += kChunk) {
            const int nc = min(kChunk, N - c0);
            __syncthreads();
            for (int k = t; k < nc; k += kThreads) s_w[k] = expf((C[c0 + k] - cmin) * nib);
            __syncthreads();
            if (!in_rows) continue;
            int k = r;
#pragma unroll 8
            for (; k + (kChains - 1) * rows < nc; k += kChains * rows) {
                const float d = U[(size_t)(c0 + k + m * rows) * H] - mu;
                const float wd = s_w[k + m * rows] * d;
                a1 += wd;
                a2 = fmaf(wd, d, a2);
            }
            for (; m == 0 && k < nc; k += rows) {
                const float d = U[(size_t)(c0 + k) * H] - mu;
                const float wd = s_w[k] * d;
                a1 += wd;
                a2 = fmaf(wd, d, a2);
            }
        }
    }
    const global_ptr<float> part = as_global(part_in) + (size_t)j * kJointPart;
    part[(2 * m) * kThreads + t] = a1;
    part[(2 * m + 1) * kThreads + t] = a2;
}

__global__ __launch_bounds__(kThreads) void update_chain_kernel(const float *__restrict__ C,
                                                                const float *__restrict__ u,
                                                                const float *__restrict__ mean,
                                                                float *__restrict__ part, int32_t N, int32_t H,
                                                                float nib)
{
    update_chain(C, u, mean, part, N, H, nib, blockIdx.x);
}

// Workgroup k of a batch takes part items[k] = (problem, part).
__global__ __launch_bounds__(kThreads) void update_chain_batch_kernel(const ProblemDev *__restrict__ probs,
                                                                      const int2 *__restrict__ items)
{
    const STORM_CONST_AS int32_t *it = uniform_ptr(reinterpret_cast<const int32_t *>(items));
    const int p = it[2 * blockIdx.x], c = it[2 * blockIdx.x + 1];
    ProblemRef P = uniform_ptr(probs)[p];
    update_chain(P.C, P.u, P.mean, P.upd_part, P.N, P.H, -1.0f / P.beta, c);
}

// The rows' sums, then the tail, on wave 0.
__device__ __forceinline__ void sum_rows(const TailArgs &T, const int j, const int H, float x1, float x2, float S0,
                                         const float *s_mold, const bool bad, const bool cov, float *s_red)
{
    const int t = threadIdx.x, lane = t & (kLanes - 1), rows = kThreads / H;
    s_red[t] = x1;
    s_red[kThreads + t] = x2;
    __syncthreads();
    if (t >= kLanes) return;
    float s1 = 0.0f, s2 = 0.0f;
    if (lane < H)
        for (int k = 0; k < rows; ++k) {
            s1 += s_red[k * H + lane];
            s2 += s_red[kThreads + k * H + lane];
        }
    const bool ok = !bad && S0 > 0.0f && isfinite(S0);
    update_tail(T, j, H, lane, s1, s2, S0, lane < H ? s_mold[lane] : 0.0f, ok, bad, cov);
}

// Joint j's update from its chains.
__device__ __forceinline__ void update_join(ProblemRef descriptor, const float *__restrict__ part_in, const int j,
                                            float *__restrict__ mean_out, float *__restrict__ sigma2_out,
                                            float *__restrict__ cmd, const int H, const int shift, const bool cov,
                                            UpdateLds &L)
{
    float *s_red = L.red;
    const global_ptr<const float> part = as_global(part_in) + (size_t)j * kJointPart;
    UpdateProblem P = fetch_problem(descriptor);
    const int t = threadIdx.x;
    float a[2 * kChains];
#pragma unroll
    for (int k = 0; k < 2 * kChains; ++k) a[k] = part[k * kThreads + t];
    const global_ptr<const float> sum = as_global(part_in) + (size_t)kDof * kJointPart;
    const float S0 = sum[0], bad = sum[1];
    wait_problem(P);
    const float mu = as_global(P.mean)[min(t, H - 1) * kDof + j];
    const TailArgs T = fetch_tail(P, mean_out, sigma2_out, cmd, shift, cov, j, t, H);
    float x1 = 0.0f, x2 = 0.0f;
#pragma unroll
    for (int m = 0; m < kChains; ++m) {
        x1 += a[2 * m];
        x2 += a[2 * m + 1];
    }
    if (t < H) L.mold[t] = mu;
    sum_rows(T, j, H, x1, x2, S0, L.mold, bad != 0.0f, cov, s_red);
}

// Joint j's update by one workgroup: its eight chains, with every cost read once
// (thread t holds those of particles t, t + 1024, ...) and the controls at byte
// offsets from the joint's first (with 64-bit addresses the loads in flight cost
// twice the registers: 600 x 64 9.0 us, 64 x 2048 x 64 46).
__device__ __forceinline__ void update_all(ProblemRef descriptor, const float *__restrict__ C_in,
                                           const float *__restrict__ u_in, const int N, const int H, const int j,
                                           float *__restrict__ mean_out, float *__restrict__ sigma2_out,
                                           float *__restrict__ cmd, const int shift, const bool cov, UpdateLds &L)
{
    static_assert(kOnce <= kRows && 2 * kList <= kRows, "the weights, or the list, fit in the weights' space");
    constexpr int kMost = kOnce / kThreads;  // costs of a thread
    __shared__ int s_nonzero[kMost][kWaves];
    UpdateProblem P = fetch_problem(descriptor);
    const global_ptr<const float> C = as_global(C_in);
    const int t = threadIdx.x, lane = t & (kLanes - 1), wave = __builtin_amdgcn_readfirstlane(t / kLanes);
    const int rows = kThreads / H, r = t / H, h = t - r * H;
    const int n_each = (N + kThreads - 1) / kThreads;
    float w[kMost];
#pragma unroll
    for (int k = 0; k < kMost; ++k)
        if (k < n_each) w[k] = C[min(t + k * kThreads, N - 1)];
    wait_problem(P);
    const float nib = -1.0f / P.beta;
    const float mu = as_global(P.mean)[h * kDof + j];
    const TailArgs T = fetch_tail(P, mean_out, sigma2_out, cmd, shift, cov, j, t, H);

    // min C and whether a cost is not finite
    float least = INFINITY;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kMost; ++k) {
        if (k >= n_each) break;
        bad |= !isfinite(w[k]);
        least = fminf(least, w[k]);
    }
    const uint64_t bad_lanes = __builtin_amdgcn_ballot_w64(bad);
    least = wave_min(least);
    if (lane == 0) {
        L.wave[wave] = least;
        L.count[wave] = bad_lanes != 0;
    }
    __syncthreads();
    float cmin = L.wave[0];
    int any_nonfinite = L.count[0];
    for (int k = 1; k < kWaves; ++k) {
        cmin = fminf(cmin, L.wave[k]);
        any_nonfinite |= L.count[k];
    }

    // the weights, their sum (per thread, per wave, waves in order), and how
    // many are not zero
    float sw = 0.0f;
#pragma unroll
    for (int k = 0; k < kMost; ++k) {
        if (k >= n_each) break;
        w[k] = t + k * kThreads < N ? expf((w[k] - cmin) * nib) : 0.0f;
        sw += w[k];
        const uint64_t nonzero = __builtin_amdgcn_ballot_w64(w[k] > 0.0f);
        if (lane == 0) s_nonzero[k][wave] = __builtin_popcountll(nonzero);
    }
    sw = wave_sum(sw);
    if (lane == 0) L.wsum[wave] = sw;
    __syncthreads();
    float S0 = 0.0f;
    for (int k = 0; k < kWaves; ++k) S0 += L.wsum[k];
    // the particles in ascending order, as the chains take them: the list, or,
    // where it overflows, all
    int *s_at = reinterpret_cast<int *>(L.buf + kList);
    int M = 0;
#pragma unroll
    for (int k = 0; k < kMost; ++k) {
        if (k >= n_each) break;
        int at = 0;
        for (int v = 0; v < kWaves; ++v) {
            if (v == wave) at = M;
            M += s_nonzero[k][v];
        }
        const uint64_t nonzero = __builtin_amdgcn_ballot_w64(w[k] > 0.0f);
        at += __builtin_popcountll(nonzero & ((1ull << lane) - 1ull));
        if (w[k] > 0.0f && at < kList) {
            L.buf[at] = w[k];
            s_at[at] = 4 * H * (t + k * kThreads);  // (of its controls in bytes)
        }
    }
    const bool list = M <= kList;
    __syncthreads();
    if (!list) {
#pragma unroll
        for (int k = 0; k < kMost; ++k)
            if (t + k * kThreads < N) L.buf[t + k * kThreads] = w[k];
        __syncthreads();
    }
    const __amdgpu_buffer_rsrc_t U = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(u_in + (size_t)j * N * H), (short)0, N * H * (int)sizeof(float), 0x00020000);
    float a1[kChains], a2[kChains];
#pragma unroll
    for (int m = 0; m < kChains; ++m) a1[m] = a2[m] = 0.0f;
    auto gather = [&](int n, auto offset) __attribute__((always_inline)) {
        int k = r;
#pragma unroll 1
        for (; k + (kChains - 1) * rows < n; k += kChains * rows) {
            float d[kChains];
#pragma unroll
            for (int m = 0; m < kChains; ++m)
                d[m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(U, offset(k + m * rows), 0, 0)) - mu;
#pragma unroll
            for (int m = 0; m < kChains; ++m) {
                const float wd = L.buf[k + m * rows] * d[m];
                a1[m] += wd;
                a2[m] = fmaf(wd, d[m], a2[m]);
            }
        }
        for (; k < n; k += rows) {
            const float d = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(U, offset(k), 0, 0)) - mu;
            const float wd = L.buf[k] * d;
            a1[0] += wd;
            a2[0] = fmaf(wd, d, a2[0]);
        }
    };
    if (r < rows) {
        if (list)
            gather(M, [&](int k) { return s_at[k] + 4 * h; });
        else
            gather(N, [&](int k) { return 4 * (k * H + h); });
    }
    float x1 = 0.0f, x2 = 0.0f;
#pragma unroll
    for (int m = 0; m < kChains; ++m) {
        x1 += a1[m];
        x2 += a2[m];
    }
    if (r == 0) L.mold[h] = mu;
    sum_rows(T, j, H, x1, x2, S0, L.mold, any_nonfinite != 0, cov, L.red);
}

template <bool kCov>
__global__ __launch_bounds__(kThreads) void update_all_kernel(const PlainDev *dev, const float *__restrict__ C,
                                                              const float *__restrict__ u,
                                                              float *__restrict__ mean_out,
                                                              float *__restrict__ sigma2_out, float *__restrict__ cmd,
                                                              int32_t N, int16_t H, int16_t shift)
{
    __shared__ UpdateLds L;
    update_all(uniform_ptr(dev)->P, C, u, N, H, blockIdx.x, mean_out, sigma2_out, cmd, shift, kCov, L);
}

template <bool kCov>
__global__ __launch_bounds__(kThreads) void update_join_kernel(const PlainDev *dev, const float *__restrict__ part,
                                                               float *__restrict__ mean_out,
                                                               float *__restrict__ sigma2_out,
                                                               float *__restrict__ cmd, int16_t H, int16_t shift)
{
    __shared__ UpdateLds L;
    update_join(uniform_ptr(dev)->P, part, blockIdx.x, mean_out, sigma2_out, cmd, H, shift, kCov, L);
}

// Workgroup (p, j) of a batch; commands go to cmd[p][7].  (The larger problems'
// chains are there.)  At most 96 VGPRs, so that the next workgroup of a CU starts
// beside the last wavefront of the one before (1024 problems of 256 x 30 111 -> 88
// us).
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5))) void update_batch_kernel(const ProblemDev *__restrict__ probs,
                                                                float *__restrict__ cmd, int shift)
{
    __shared__ UpdateLds L;
    const int p = blockIdx.x / kDof, j = blockIdx.x - p * kDof;
    ProblemRef P = uniform_ptr(probs)[p];
    const UpdateFirst first{P.C, P.u, P.N, P.H};
    const int slots = update_slots(P.N, P.H);
    float *c = cmd + (size_t)p * kDof;
    if (slots == 8)
        update_joint<8>(P, first, j, nullptr, nullptr, c, shift, P.cov_step != 0u, L);
    else if (slots == 16)
        update_joint<16>(P, first, j, nullptr, nullptr, c, shift, P.cov_step != 0u, L);
    else if (slots == 32)
        update_joint<32>(P, first, j, nullptr, nullptr, c, shift, P.cov_step != 0u, L);
    else if (P.N <= kOnce)
        update_all(P, P.C, P.u, P.N, P.H, j, nullptr, nullptr, c, shift, P.cov_step != 0u, L);
    else
        update_join(P, P.upd_part, j, nullptr, nullptr, c, P.H, shift, P.cov_step != 0u, L);
}

}  // namespace

hipError_t launch_update_batch(const ProblemDev *probs, int n_problems, const int2 *part_items, int n_part_items,
                               float *cmd, int shift, hipStream_t stream)
{
    if (n_part_items > 0) {
        hipLaunchKernelGGL(update_chain_batch_kernel, dim3((unsigned)n_part_items), dim3(kThreads), 0, stream, probs,
                           part_items);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(update_batch_kernel, dim3((unsigned)(n_problems * kDof)), dim3(kThreads), 0, stream, probs,
                       cmd, shift);
    return hipGetLastError();
}

hipError_t launch_update(const ProblemDev &P, const PlainDev *dev, float *mean_out, float *sigma2_out, float *cmd, int shift,
                         hipStream_t stream)
{
    const int slots = update_slots(P.N, P.H);
    if (slots == 0 && update_once(P.N, P.H)) {
        auto kernel = P.cov_step ? update_all_kernel<true> : update_all_kernel<false>;
        hipLaunchKernelGGL(kernel, dim3(kDof), dim3(kThreads), 0, stream, dev, P.C, P.u, mean_out, sigma2_out, cmd,
                           P.N, (int16_t)P.H, (int16_t)shift);
        return hipGetLastError();
    }
    if (slots == 0) {
        hipLaunchKernelGGL(update_chain_kernel, dim3(kUpdateParts), dim3(kThreads), 0, stream, P.C, P.u, P.mean,
                           P.upd_part, P.N, P.H, -1.0f / P.beta);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        auto join = P.cov_step ? update_join_kernel<true> : update_join_kernel<false>;
        hipLaunchKernelGGL(join, dim3(kDof), dim3(kThreads), 0, stream, dev, P.upd_part, mean_out, sigma2_out, cmd,
                           (int16_t)P.H, (int16_t)shift);
        return hipGetLastError();
    }
    auto kernel = P.cov_step ? (slots == 8    ? update_kernel<true, 8>
                                : slots == 16 ? update_kernel<true, 16>
                                              : update_kernel<true, 32>)
                             : (slots == 8    ? update_kernel<false, 8>
                                : slots == 16 ? update_kernel<false, 16>
                                              : update_kernel<false, 32>);
    hipLaunchKernelGGL(kernel, dim3(kDof), dim3(kThreads), 0, stream, dev, P.C, P.u, mean_out, sigma2_out, cmd,
                       P.N, (int16_t)P.H, (int16_t)shift);
    return hipGetLastError();
}

int update_batch_parts(int N, int H) { return update_slots(N, H) != 0 || N <= kOnce ? 0 : kUpdateParts; }

size_t update_part_floats(int N, int H)
{
    return update_slots(N, H) != 0 || update_once(N, H) ? 0 : (size_t)kDof * kJointPart + 4;
}

}  // namespace storm
