// Kernel A: reverse-mode gradient of the expected horizon cost
//   J(mu) = (1/N) sum_i C_i(mu + sigma * eps_i),  eps held fixed,
// with respect to the mean control sequence mu [H][7] (not in the paper: the
// differentiable form).  Differentiated terms: pose (Eq. 9), joint and
// velocity limits (Eq. 11 form) and stop (Eq. 10); hinge and norm kinks take
// subgradient 0.  States are recomputed from mu and the noise, never stored.
//
// One wavefront per 64-lane tile (ppt particles x H steps; a lane is one point
// and holds all seven joints): the noise, the controls and the integrator (as
// kernel R); limit costs and their gradients; forward kinematics, keeping each
// joint's axis z_k and origin o_k; pose cost and dC/dq through the Jacobian
// columns, dp/dq_k = z_k x (p - o_k) and dR/dq_k = [z_k]x R; then the
// integrator backwards, two segmented suffix sums:
//   dC/dv_k = gv_k + dt_k sum_{h>=k} gq_h,  dC/du_m = dt_m sum_{k>=m} dC/dv_k.
// Nothing is exchanged between wavefronts until the tiles are done, so there is
// no barrier in the loop and the only idle issue slots are latencies that the
// other wavefronts of the SIMD cover (four: 128 VGPRs); bound by VALU issue.
// The same work split over eight wavefronts by joint and row (1.65 ms for 64
// problems of 4096 x 64, with six barriers a tile, against 0.82) is the shorter
// path where a launch has few tiles: it is kept for those (kSplitTiles), with the
// same bits.
// A second kernel adds the partials per (joint, step) in a fixed order and,
// when refining, takes an Adam step (Kingma and Ba, 2015) on mu.
#include "kinematics.h"
#include "sampling.h"

// The same point costs the same bits in either form below: no product is
// fused into a sum but where fmaf says so.
#pragma clang fp contract(off)

namespace storm {
namespace {

constexpr int kSplitWaves = 8;
constexpr int kRedThreads = 1024;

// What a chunk's start reads of the problem, fetched in one go.
struct AdjFirst {
    int32_t n_halton, n_null, ppt, n_tiles, n_chunks;
    uint32_t seed_lo, seed_hi, grad_mask, comb, cov_step;
    const float *tables, *halton;
    float *sigma2;
    uint32_t *step;
    int32_t N, H;
};
// (issued; wait_for: here they have to be there)
__device__ __forceinline__ AdjFirst load_first(ProblemRef P, int32_t N, int32_t H)
{
    return AdjFirst{P.n_halton, P.n_null, P.ppt,    P.n_tiles, P.n_chunks, P.seed_lo, P.seed_hi, P.grad_mask,
                    P.comb,     P.cov_step, P.tables, P.halton, P.sigma2,  P.step,    N,         H};
}
__device__ __forceinline__ void wait_for(AdjFirst &F)
{
    asm volatile("" : "+s"(F.n_halton), "+s"(F.n_null), "+s"(F.ppt), "+s"(F.n_tiles), "+s"(F.n_chunks),
                 "+s"(F.seed_lo), "+s"(F.seed_hi), "+s"(F.grad_mask), "+s"(F.comb), "+s"(F.cov_step), "+s"(F.tables),
                 "+s"(F.halton), "+s"(F.sigma2), "+s"(F.step));
}

// This lane's number, counted anew at each use (threadIdx, or a count that the
// compiler may keep, would take up a register throughout).
__device__ __forceinline__ int lane_id()
{
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// n consecutive scalars in one go: a load wherever one is used would put one
// round trip after another.
template <int n>
__device__ __forceinline__ void load_scalars(const STORM_CONST_AS float *p, float (&x)[n])
{
#pragma unroll
    for (int k = 0; k < n; ++k) x[k] = p[k];
}
template <int n>
__device__ __forceinline__ void wait_for(float (&x)[n])
{
    static_assert(n % 4 == 0, "four per statement");
#pragma unroll
    for (int k = 0; k < n; k += 4) asm volatile("" : "+s"(x[k]), "+s"(x[k + 1]), "+s"(x[k + 2]), "+s"(x[k + 3]));
}
template <int n>
__device__ __forceinline__ void fetch_scalars(const STORM_CONST_AS float *p, float (&x)[n])
{
    load_scalars(p, x);
    wait_for(x);
}

// The weights and scales of the differentiated terms.
struct AdjWeights {
    float a_joint, a_vel, a_stop, w_pos, w_rot, alpha_pos[3], alpha_rot[3];
};
__device__ __forceinline__ AdjWeights load_weights(ProblemRef P)
{
    return AdjWeights{P.a_joint, P.a_vel, P.a_stop, P.w_pos, P.w_rot, {P.alpha_pos[0], P.alpha_pos[1], P.alpha_pos[2]},
                      {P.alpha_rot[0], P.alpha_rot[1], P.alpha_rot[2]}};
}
__device__ __forceinline__ void wait_for(AdjWeights &w)
{
    asm volatile("" : "+s"(w.a_joint), "+s"(w.a_vel), "+s"(w.a_stop), "+s"(w.w_pos), "+s"(w.w_rot),
                 "+s"(w.alpha_pos[0]), "+s"(w.alpha_pos[1]), "+s"(w.alpha_pos[2]), "+s"(w.alpha_rot[0]),
                 "+s"(w.alpha_rot[1]), "+s"(w.alpha_rot[2]));
}

// Limit and stop costs of a point from the squared norms of its violations:
// the cost, and what the violations are scaled by in its gradients.
struct AdjLimits {
    float cost, kj, kv, ks;
};
__device__ __forceinline__ AdjLimits limit_terms(const AdjWeights &w, uint32_t mask, float nj, float nv, float ns)
{
    nj = (mask & STORM_COST_JOINT) ? fast_sqrt(nj) : 0.0f;
    nv = (mask & STORM_COST_VEL) ? fast_sqrt(nv) : 0.0f;
    ns = (mask & STORM_COST_STOP) ? fast_sqrt(ns) : 0.0f;
    return AdjLimits{fmaf(w.a_joint, nj, fmaf(w.a_vel, nv, w.a_stop * ns)), nj > 0.0f ? w.a_joint / nj : 0.0f,
                     nv > 0.0f ? w.a_vel / nv : 0.0f, ns > 0.0f ? w.a_stop / ns : 0.0f};
}

// Pose cost of a point with flange (Re, pe), added to `cost`, and its gradient
// with respect to the flange's motion: gp to its position, gr to its rotation.
__device__ __forceinline__ void pose_gradient(const AdjWeights &w, const float (&goal)[12], const float Re[9],
                                              const float pe[3], float gp[3], float gr[3], float &cost)
{
    // position: e = diag(a2) R_g^T (p - p_g), gradient g_p = w_pos R_g diag(a2) e / |e|
    float ep[3], pos2 = 0.0f;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        ep[r] = w.alpha_pos[r] * fmaf(goal[0 * 3 + r], pe[0] - goal[9],
                                      fmaf(goal[1 * 3 + r], pe[1] - goal[10], goal[2 * 3 + r] * (pe[2] - goal[11])));
        pos2 = fmaf(ep[r], ep[r], pos2);
    }
    const float pos = fast_sqrt(pos2);
    const float kp = pos > 0.0f ? w.w_pos / pos : 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        gp[a] = kp * fmaf(goal[a * 3 + 0], w.alpha_pos[0] * ep[0],
                          fmaf(goal[a * 3 + 1], w.alpha_pos[1] * ep[1], goal[a * 3 + 2] * w.alpha_pos[2] * ep[2]));
    // rotation: M = diag(a1)(I - R_g^T R), gradient G = -w_rot R_g diag(a1) M / |M|_F
    float M[9], rot2 = 0.0f;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float m = fmaf(goal[0 * 3 + r], Re[0 * 3 + c],
                                 fmaf(goal[1 * 3 + r], Re[1 * 3 + c], goal[2 * 3 + r] * Re[2 * 3 + c]));
            M[r * 3 + c] = w.alpha_rot[r] * ((r == c ? 1.0f : 0.0f) - m);
            rot2 = fmaf(M[r * 3 + c], M[r * 3 + c], rot2);
        }
    const float rot = fast_sqrt(rot2);
    const float kr = rot > 0.0f ? -w.w_rot / rot : 0.0f;
    float G[9];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            G[a * 3 + c] = kr * fmaf(goal[a * 3 + 0], w.alpha_rot[0] * M[0 * 3 + c],
                                     fmaf(goal[a * 3 + 1], w.alpha_rot[1] * M[1 * 3 + c],
                                          goal[a * 3 + 2] * w.alpha_rot[2] * M[2 * 3 + c]));
    // <G, [z]x R> = z . w with A = R G^T, w = (A12 - A21, A20 - A02, A01 - A10)
    auto A = [&](int a, int b) __attribute__((always_inline)) {
        return fmaf(Re[a * 3 + 0], G[b * 3 + 0], fmaf(Re[a * 3 + 1], G[b * 3 + 1], Re[a * 3 + 2] * G[b * 3 + 2]));
    };
    gr[0] = A(1, 2) - A(2, 1);
    gr[1] = A(2, 0) - A(0, 2);
    gr[2] = A(0, 1) - A(1, 0);
    cost = fmaf(w.w_pos, pos, fmaf(w.w_rot, rot, cost));
}

// The same gradient with respect to the joint of axis z and origin o.
__device__ __forceinline__ float pose_joint(const float pe[3], const float z[3], const float o[3], const float gp[3],
                                            const float gr[3])
{
    const float r0 = pe[0] - o[0], r1 = pe[1] - o[1], r2 = pe[2] - o[2];
    // (p - o) x g_p
    const float c0 = fmaf(r1, gp[2], -(r2 * gp[1]));
    const float c1 = fmaf(r2, gp[0], -(r0 * gp[2]));
    const float c2 = fmaf(r0, gp[1], -(r1 * gp[0]));
    return fmaf(z[0], c0 + gr[0], fmaf(z[1], c1 + gr[1], z[2] * (c2 + gr[2])));
}

// One tile on one wavefront: acc gains dC/du of this lane's point, cacc its
// weighted cost.  row: [8][64] floats of LDS of this wavefront's own.
__device__ __forceinline__ void adjoint_tile(ProblemRef P, RobotRef R, AdjFirst F, const int tile,
                                             const uint32_t counter, const STORM_CONST_AS float *x0,
                                             const STORM_CONST_AS float *goal_in, const float *mean,
                                             const float *__restrict__ noise, float *row, float acc[kDof],
                                             float &cacc)
{
    // What follows from the lane and the seed is formed, and the step's inputs
    // are read, in each tile: kept over the loop they would spill.
    const int lane = lane_id();
    asm volatile("" : "+s"(F.seed_lo), "+s"(F.seed_hi), "+s"(F.H), "+s"(F.grad_mask));
    const int N = F.N, H = F.H;
    const int pl = (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)H));  // lane / H (exact, as in kernel R)
    const int h = lane - pl * H;
    const int i = tile * F.ppt + pl;
    const bool valid = pl < F.ppt && i < N;
    const bool live = valid && i < N - F.n_null;
    const uint32_t mask = F.grad_mask;
    const STORM_CONST_AS float *tab = uniform_ptr(F.tables);
    const float dt = as_global(F.tables)[kTabDt + h], hw = as_global(F.tables)[kTabHw + h],
                vs = as_global(F.tables)[kTabVstop + h];
    float mu[kDof], sigma2[kDof];
    {
        const global_ptr<const float> m = as_global(mean) + h * kDof,
                                      s = as_global(F.sigma2) + (F.cov_step ? h * kDof : 0);
#pragma unroll
        for (int j = 0; j < kDof; ++j) {
            mu[j] = m[j];
            sigma2[j] = s[j];
        }
    }

    // noise
    float e[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) e[m] = 0.0f;
    if (live) {
        standard_noise4(F, F.seed_lo, F.seed_hi, noise, 0, i, h, counter, e);
        standard_noise4(F, F.seed_lo, F.seed_hi, noise, 1, i, h, counter, e + 4);
    }
    if (F.comb && noise == nullptr) {
        // the comb filter on the sampled Gaussian particles' noise, as in kernel R
        const bool comb = live && i >= F.n_halton;
#pragma unroll
        for (int j = 0; j < kDof; ++j) row[j * kLanes + lane] = e[j];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < kDof; ++j) {
            const float f = comb_noise(row + j * kLanes, lane, h, H, as_global(F.tables));
            if (comb) e[j] = f;
        }
        __builtin_amdgcn_wave_barrier();
    }

    // controls and the integrator; limit costs and their gradients (signed
    // violations: negative below the band, positive above)
    float gq[kDof], gv[kDof], sq[kDof], cq[kDof], cost = 0.0f;
    AdjWeights w;
    {
        // (all scans of a kind together: a joint's alone is a serial chain)
        float vj[kDof], qj[kDof], es[kDof], x[16], lim[4 * 8];
        fetch_scalars<12>(x0, reinterpret_cast<float (&)[12]>(x));
        x[12] = x0[12];
        x[13] = x0[13];
        asm volatile("" : "+s"(x[12]), "+s"(x[13]));
        fetch_scalars(tab + kTabJlo, lim);
        float nj = 0.0f, nv = 0.0f, ns = 0.0f;
#pragma unroll
        for (int j = 0; j < kDof; ++j)
            vj[j] = dt * (live ? fmaf(sqrtf(sigma2[j]), e[j], mu[j]) : 0.0f);
        segmented_scans(vj, lane, h);
#pragma unroll
        for (int j = 0; j < kDof; ++j) {
            vj[j] += x[kDof + j];
            qj[j] = dt * vj[j];
        }
        segmented_scans(qj, lane, h);
#pragma unroll
        for (int j = 0; j < kDof; ++j) {
            const float v = vj[j], q = x[j] + qj[j];
            sincosf(q, &sq[j], &cq[j]);
            gq[j] = fminf(q - lim[j], 0.0f) + fmaxf(q - lim[8 + j], 0.0f);
            gv[j] = fminf(v - lim[16 + j], 0.0f) + fmaxf(v - lim[24 + j], 0.0f);
            const float a = fmaxf(fabsf(v) - vs, 0.0f);
            nj = fmaf(gq[j], gq[j], nj);
            nv = fmaf(gv[j], gv[j], nv);
            ns = fmaf(a, a, ns);
            es[j] = v > 0.0f ? a : -a;
        }
        w = load_weights(P);
        wait_for(w);
        const AdjLimits lt = limit_terms(w, mask, nj, nv, ns);
#pragma unroll
        for (int j = 0; j < kDof; ++j) {
            gq[j] = lt.kj * gq[j];
            gv[j] = fmaf(lt.kv, gv[j], lt.ks * es[j]);
        }
        cost = lt.cost;
    }

    // pose cost and its gradient
    if (mask & STORM_COST_POSE) {
        float Re[9] = {1.0f, 0.0f, 0.0f, 0.0f, 1.0f, 0.0f, 0.0f, 0.0f, 1.0f}, pe[3] = {0.0f, 0.0f, 0.0f};
        float z[kDof][3], o[kDof][3], dh[4 * kFrames];
        fetch_scalars(R.ca, dh);
#pragma unroll
        for (int f = 0; f < kFrames; ++f) {
            dh_step(Re, pe, dh[f], dh[kFrames + f], dh[2 * kFrames + f], dh[3 * kFrames + f], f < kDof ? cq[f < kDof ? f : 0] : 1.0f,
                    f < kDof ? sq[f < kDof ? f : 0] : 0.0f);
            if (f < kDof)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    z[f][c] = Re[3 * c + 2];
                    o[f][c] = pe[c];
                }
        }
        float goal[12];
        fetch_scalars(goal_in, goal);
        float gp[3], gr[3];
        pose_gradient(w, goal, Re, pe, gp, gr, cost);
#pragma unroll
        for (int k = 0; k < kDof; ++k) gq[k] += pose_joint(pe, z[k], o[k], gp, gr);
    }
    cacc += valid ? hw * cost : 0.0f;

    // the integrator backwards
    const int left = H - 1 - h;
#pragma unroll
    for (int j = 0; j < kDof; ++j) gq[j] *= hw;
    segmented_suffix_scans(gq, lane, left);
#pragma unroll
    for (int j = 0; j < kDof; ++j) gq[j] = fmaf(dt, gq[j], hw * gv[j]);
    segmented_suffix_scans(gq, lane, left);
#pragma unroll
    for (int j = 0; j < kDof; ++j) acc[j] += live ? dt * gq[j] : 0.0f;
}

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, kLanes);
    return x;
}

// The partials of chunk c from its runs' sums in LDS (rows of seven joints,
// then the cost, by lane), over particles, then runs.  t of `threads` threads.
template <int runs>
__device__ __forceinline__ void write_partial(float *__restrict__ part, const int c, const float *rows, const int ppt,
                                              const int H, const int t, const int threads)
{
    for (int k = t; k < kDof * H; k += threads) {
        const int j = k / H, hh = k - j * H;
        float s = 0.0f;
        for (int p = 0; p < ppt; ++p) {
            float v[runs];
#pragma unroll
            for (int w = 0; w < runs; ++w) v[w] = rows[(w * 8 + j) * kLanes + p * H + hh];
#pragma unroll
            for (int w = 0; w < runs; ++w) s += v[w];
        }
        as_global(part)[kAdjChunks + ((size_t)c * kDof + j) * kMaxH + hh] = s;
    }
    if (t < kLanes) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < runs; ++w) s += rows[(w * 8 + kDof) * kLanes + t];
        s = wave_sum(s);
        if (t == 0) as_global(part)[c] = s;
    }
}

// A workgroup of W wavefronts, a tile per wavefront at a time.  The order of
// every sum is the problem's alone, not W's nor the batch's: up to kSplitTiles
// tiles a partial is one tile's (here wavefront w of workgroup c takes tile
// c W + w); past that, chunk c of a problem covers T / n tiles, the first T % n
// chunks one more, in runs of every kRuns-th tile (adjoint_runs), a wavefront
// taking one run after another.
template <int W>
__device__ __forceinline__ void adjoint_chunk(ProblemRef P, RobotRef R, const int N, const int H, const int c,
                                              const float *__restrict__ x0, const float *__restrict__ goal,
                                              const float *__restrict__ mean, const float *__restrict__ noise,
                                              float *__restrict__ part)
{
    __shared__ float s_buf[kAdjRuns][8 * kLanes];  // the wavefronts' rows, then the runs' sums
    AdjFirst F = load_first(P, N, H);
    wait_for(F);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t counter = *uniform_ptr(F.step + 2);
    const bool single = F.n_tiles <= kSplitTiles;
    const int runs = single ? W : adjoint_runs(F.n_tiles);
    const int base = F.n_tiles / F.n_chunks, more = F.n_tiles - base * F.n_chunks;
    const int t0 = single ? c * W : c * base + min(c, more);
    const int t1 = single ? min(t0 + W, F.n_tiles) : t0 + base + (c < more ? 1 : 0);
    for (int run = wave; run < runs; run += W) {
        float acc[kDof] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f}, cacc = 0.0f;
        for (int tile = t0 + run; tile < t1; tile += runs) {
            // (scalars read in each tile, not kept over the loop)
            const STORM_CONST_AS ProblemDev *p = &P;
            const STORM_CONST_AS RobotDev *r = &R;
            const STORM_CONST_AS float *x = uniform_ptr(x0), *g = uniform_ptr(goal);
            asm volatile("" : "+s"(p), "+s"(r), "+s"(x), "+s"(g));
            adjoint_tile(*p, *r, F, tile, counter, x, g, mean, noise, s_buf[run], acc, cacc);
        }
        const int lane = lane_id();
#pragma unroll
        for (int j = 0; j < kDof; ++j) s_buf[run][j * kLanes + lane] = acc[j];
        s_buf[run][kDof * kLanes + lane] = cacc;
    }
    __syncthreads();
    const int lane = lane_id();
    if (single) {
        if (t0 + wave >= t1) return;
        write_partial<1>(part, t0 + wave, s_buf[wave], F.ppt, H, lane, kLanes);
        return;
    }
    if (runs == kAdjRuns)
        write_partial<kAdjRuns>(part, c, s_buf[0], F.ppt, H, wave * kLanes + lane, W * kLanes);
    else
        write_partial<kAdjWaves>(part, c, s_buf[0], F.ppt, H, wave * kLanes + lane, W * kLanes);
}

// One tile split over a workgroup of eight wavefronts, into the partials of
// chunk `tile`; bound by latency:
//   A   waves 0-3: noise; waves 0-6, one joint each: controls, the integrator,
//       sin/cos of q, violations of the limits
//   B   waves 0-2: forward kinematics to LDS, one frame row each; wave 3: limit
//       costs and what the violations are scaled by
//   C   wave 0: pose cost, its gradient by the flange's motion; horizon cost
//   D   waves 0-6: dC/dq of the joint, the integrator backwards
//   E   per (joint, step) sum over the tile's particles
// Every load is issued at the start, and a joint's share of the gradient is
// formed by its own wave (a step and three refinements of 64 x 16 43.5 -> 38.4 us,
// of 1024 x 30 48.2 -> 44.7, with the partials' sum below).
__device__ __forceinline__ void adjoint_split(ProblemRef P, RobotRef R, const int N, const int H, const int tile,
                                              const float *__restrict__ x0, const float *__restrict__ goal_in,
                                              const float *__restrict__ mean, const float *__restrict__ noise,
                                              float *__restrict__ part)
{
    __shared__ float s_eps[8][kLanes];
    __shared__ float s_sc[2 * kDof][kLanes];  // sin q_j, cos q_j
    __shared__ float s_ej[kDof][kLanes], s_ev[kDof][kLanes], s_es[kDof][kLanes];  // signed violations
    __shared__ float s_fr[kFrames * 12][kLanes];
    __shared__ float s_k[4][kLanes];   // the violations' scales, the weighted limit costs
    __shared__ float s_g[6][kLanes];   // the pose cost's gradient by the flange's motion
    __shared__ float s_gu[kDof][kLanes];  // d C / d u
    __shared__ float s_Cp[kLanes];        // horizon cost per particle of the tile

    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    AdjFirst F = load_first(P, N, H);
    AdjWeights w = load_weights(P);
    float dh[4 * kFrames], goal[12];
    load_scalars(R.ca, dh);
    load_scalars(uniform_ptr(goal_in), goal);
    __builtin_amdgcn_sched_barrier(0);  // (all of them before the first is waited for)
    wait_for(F);
    const int pl = (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)H));  // lane / H (exact, as in kernel R)
    const int h = lane - pl * H;
    const int i = tile * F.ppt + pl;
    const bool valid = pl < F.ppt && i < N;
    const bool live = valid && i < N - F.n_null;
    const uint32_t mask = F.grad_mask;
    const global_ptr<const float> tab = as_global(F.tables);
    const int j = min(wave, kDof - 1);  // (this wave's joint)
    const float dt = tab[kTabDt + h], hw = tab[kTabHw + h], vs = tab[kTabVstop + h];
    const float mu = as_global(mean)[h * kDof + j],
                sigma2 = as_global(F.sigma2)[F.cov_step ? h * kDof + j : j];
    const float q0 = vector_load_f32(x0 + j), v0 = vector_load_f32(x0 + kDof + j);
    const float jlo = tab[kTabJlo + j], jhi = tab[kTabJhi + j], vlo = tab[kTabVlo + j], vhi = tab[kTabVhi + j];

    wait_for(w);
    wait_for(dh);
    wait_for(goal);

    // ---- A: noise, controls, integrator ---------------------------------------
    if (wave < 4) {
        const int k = wave & 1, half = wave >> 1;
        float e[2] = {0.0f, 0.0f};
        const uint32_t counter = *uniform_ptr(F.step + 2);
        if (live) standard_noise2(F, F.seed_lo, F.seed_hi, noise, k, half, i, h, counter, e);
        s_eps[4 * k + 2 * half][lane] = e[0];
        s_eps[4 * k + 2 * half + 1][lane] = e[1];
    }
    __syncthreads();
    if (wave < kDof) {
        float e = s_eps[j][lane];
        // the comb filter on the sampled Gaussian particles' noise, as in kernel R
        const bool comb = F.comb && noise == nullptr && live && i >= F.n_halton;
        if (__builtin_amdgcn_ballot_w64(comb) != 0) {
            const float f = comb_noise(&s_eps[j][0], lane, h, H, tab);
            if (comb) e = f;
        }
        const float u = live ? fmaf(sqrtf(sigma2), e, mu) : 0.0f;
        const float v = v0 + segmented_scan(dt * u, h, H);
        const float q = q0 + segmented_scan(dt * v, h, H);
        // signed violations: negative below the band, positive above
        s_ej[j][lane] = fminf(q - jlo, 0.0f) + fmaxf(q - jhi, 0.0f);
        s_ev[j][lane] = fminf(v - vlo, 0.0f) + fmaxf(v - vhi, 0.0f);
        const float a = fmaxf(fabsf(v) - vs, 0.0f);
        s_es[j][lane] = v > 0.0f ? a : -a;
        float sq, cq;
        sincosf(q, &sq, &cq);
        s_sc[2 * j][lane] = sq;
        s_sc[2 * j + 1][lane] = cq;
    }
    __syncthreads();

    // ---- B: kinematics, one frame row per wave | limit costs ------------------
    if (wave < 3) {
        const int row = wave;
        float r[3] = {row == 0 ? 1.0f : 0.0f, row == 1 ? 1.0f : 0.0f, row == 2 ? 1.0f : 0.0f};
        float p = 0.0f;
#pragma unroll
        for (int f = 0; f < kFrames; ++f) {
            float st = 0.0f, ct = 1.0f;
            if (f < kDof) {
                st = s_sc[2 * f][lane];
                ct = s_sc[2 * f + 1][lane];
            }
            dh_step_row(r, p, dh[f], dh[kFrames + f], dh[2 * kFrames + f], dh[3 * kFrames + f], ct, st);
#pragma unroll
            for (int c = 0; c < 3; ++c) s_fr[f * 12 + row * 3 + c][lane] = r[c];
            s_fr[f * 12 + 9 + row][lane] = p;
        }
    } else if (wave == 3) {
        float nj = 0.0f, nv = 0.0f, ns = 0.0f;
#pragma unroll
        for (int k = 0; k < kDof; ++k) {
            const float ej = s_ej[k][lane], ev = s_ev[k][lane], es = s_es[k][lane];
            nj = fmaf(ej, ej, nj);
            nv = fmaf(ev, ev, nv);
            ns = fmaf(es, es, ns);
        }
        const AdjLimits lt = limit_terms(w, mask, nj, nv, ns);
        s_k[0][lane] = lt.kj;
        s_k[1][lane] = lt.kv;
        s_k[2][lane] = lt.ks;
        s_k[3][lane] = lt.cost;
    }
    __syncthreads();

    // ---- C: pose cost and its gradient; horizon cost ------------------------
    if (wave == 0) {
        float cost = s_k[3][lane];
        if (mask & STORM_COST_POSE) {
            float Re[9], pe[3], gp[3], gr[3];
#pragma unroll
            for (int c = 0; c < 9; ++c) Re[c] = s_fr[7 * 12 + c][lane];
#pragma unroll
            for (int c = 0; c < 3; ++c) pe[c] = s_fr[7 * 12 + 9 + c][lane];
            pose_gradient(w, goal, Re, pe, gp, gr, cost);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                s_g[c][lane] = gp[c];
                s_g[3 + c][lane] = gr[c];
            }
        }
        const float Ci = segmented_scan(hw * cost, h, H);
        if (h == H - 1) s_Cp[pl] = valid ? Ci : 0.0f;
    }
    __syncthreads();
    if (threadIdx.x == 7 * kLanes) {
        float cacc = 0.0f;
        for (int p = 0; p < F.ppt; ++p) cacc += s_Cp[p];
        as_global(part)[tile] = cacc;
    }

    // ---- D: dC/dq, then the integrator backwards --------------------------------
    if (wave < kDof) {
        float g[1] = {s_k[0][lane] * s_ej[j][lane]};
        if (mask & STORM_COST_POSE) {
            float pe[3], z[3], o[3], gp[3], gr[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                pe[c] = s_fr[7 * 12 + 9 + c][lane];
                z[c] = s_fr[j * 12 + 3 * c + 2][lane];
                o[c] = s_fr[j * 12 + 9 + c][lane];
                gp[c] = s_g[c][lane];
                gr[c] = s_g[3 + c][lane];
            }
            g[0] += pose_joint(pe, z, o, gp, gr);
        }
        g[0] *= hw;
        const float gv = fmaf(s_k[1][lane], s_ev[j][lane], s_k[2][lane] * s_es[j][lane]);
        const int left = H - 1 - h;
        segmented_suffix_scans(g, lane, left);
        g[0] = fmaf(dt, g[0], hw * gv);
        segmented_suffix_scans(g, lane, left);
        s_gu[j][lane] = live ? dt * g[0] : 0.0f;
    }
    __syncthreads();

    // ---- E: the tile's partial of dJ/dmu (sum over the tile's particles) -----
    if ((int)threadIdx.x < kDof * H) {
        const int jj = threadIdx.x / H, hh = threadIdx.x - jj * H;
        float acc = 0.0f;
        for (int p = 0; p < F.ppt; ++p) acc += s_gu[jj][p * H + hh];
        as_global(part)[kAdjChunks + ((size_t)tile * kDof + jj) * kMaxH + hh] = acc;
    }
}

// All arguments fit the 14 dwords that are preloaded into SGPRs; the rest of
// the problem comes from its descriptor in device memory.
template <int W>
__global__ __launch_bounds__(W *kLanes) __attribute__((amdgpu_waves_per_eu(4))) void adjoint_kernel(
    const PlainDev *dev, const float *__restrict__ mean, const float *__restrict__ x0, const float *__restrict__ goal,
    const float *__restrict__ noise, float *__restrict__ part, int32_t N, int32_t H)
{
    const STORM_CONST_AS PlainDev &D = *uniform_ptr(dev);
    adjoint_chunk<W>(D.P, D.R, N, H, blockIdx.x, x0, goal, mean, noise, part);
}

__global__ __launch_bounds__(kSplitWaves *kLanes) void adjoint_split_kernel(
    const PlainDev *dev, const float *__restrict__ mean, const float *__restrict__ x0, const float *__restrict__ goal,
    const float *__restrict__ noise, float *__restrict__ part, int32_t N, int32_t H)
{
    const STORM_CONST_AS PlainDev &D = *uniform_ptr(dev);
    adjoint_split(D.P, D.R, N, H, blockIdx.x, x0, goal, mean, noise, part);
}

// Batched forms: workgroup k takes chunk items[k] = (problem, chunk).
__global__ __launch_bounds__(kAdjWaves *kLanes) __attribute__((amdgpu_waves_per_eu(4))) void adjoint_batch_kernel(
    const ProblemDev *__restrict__ probs, const int2 *__restrict__ items, const RobotDev *robot,
    const float *__restrict__ x0s, const float *__restrict__ goals)
{
    const STORM_CONST_AS int32_t *it = uniform_ptr(reinterpret_cast<const int32_t *>(items));
    const int p = it[2 * blockIdx.x], c = it[2 * blockIdx.x + 1];
    ProblemRef P = uniform_ptr(probs)[p];
    adjoint_chunk<kAdjWaves>(P, *uniform_ptr(robot), P.N, P.H, c, x0s + (size_t)p * 3 * kDof, goals + (size_t)p * 12,
                             P.mean, nullptr, P.grad_part);
}

__global__ __launch_bounds__(kSplitWaves *kLanes) void adjoint_split_batch_kernel(
    const ProblemDev *__restrict__ probs, const int2 *__restrict__ items, const RobotDev *robot,
    const float *__restrict__ x0s, const float *__restrict__ goals)
{
    const STORM_CONST_AS int32_t *it = uniform_ptr(reinterpret_cast<const int32_t *>(items));
    const int p = it[2 * blockIdx.x], c = it[2 * blockIdx.x + 1];
    ProblemRef P = uniform_ptr(probs)[p];
    adjoint_split(P, *uniform_ptr(robot), P.N, P.H, c, x0s + (size_t)p * 3 * kDof, goals + (size_t)p * 12, P.mean,
                  nullptr, P.grad_part);
}

// One Adam step with gradient g on the stored mean mu, element t, with the
// moments m0 and v0 before it; returns the new mean.  b1_it, b2_it: b1^it, b2^it.
__device__ __forceinline__ float adam_step(float *adam_m, float *adam_v, int t, float g, float m0, float v0, float mu,
                                           float lr, float b1, float b2, float b1_it, float b2_it, float eps)
{
    const float m = fmaf(b1, m0, (1.0f - b1) * g);
    const float v = fmaf(b2, v0, (1.0f - b2) * g * g);
    as_global(adam_m)[t] = m;
    as_global(adam_v)[t] = v;
    const float mh = m / (1.0f - b1_it);
    const float vh = v / (1.0f - b2_it);
    return mu - lr * mh / (sqrtf(vh) + eps);
}

// cmd = mu_0, then the warm-start shift of the stored mean (and of a
// per-step variance, sigma_init^2 appended) if requested.
__device__ __forceinline__ void command(ProblemRef P, float *__restrict__ cmd, int shift)
{
    __shared__ float s_mu[kDof * kMaxH];
    __shared__ float s_s2[kDof * kMaxH];
    const int t = threadIdx.x;
    const int n = P.H * kDof;
    for (int k = t; k < n; k += blockDim.x) {
        s_mu[k] = as_global(P.mean)[k];
        if (P.cov_step) s_s2[k] = as_global(P.sigma2)[k];
    }
    __syncthreads();
    if (t < kDof) cmd[t] = s_mu[t];
    if (shift)
        for (int k = t; k < n; k += blockDim.x) {
            as_global(P.mean)[k] = k + kDof < n ? s_mu[k + kDof] : 0.0f;
            if (P.cov_step) as_global(P.sigma2)[k] = k + kDof < n ? s_s2[k + kDof] : as_global(P.tables)[kTabSig0 + k % kDof];
        }
}

// Gradient of joint j: the chunk partials of (h, j) summed in a fixed order
// (thread (r, h) over chunks r, r + rows, ..., every load in flight at once,
// then wave 0 over the rows), divided by N; joint 0 also sums the chunk
// costs into J.  With it > 0, lane h of wave 0 then takes the Adam step on
// mu[h][j]; with cmd, it writes the command mu[0][j] and the warm-start
// shift of the joint (the next step's value through a DPP wave shift), with
// a per-step variance shifted alike.
// (Bound by latency: everything it reads is loaded at the start.)
struct GradFields {
    int32_t N, H, n_chunks;
    uint32_t cov_step;
    const float *tables;
    float *mean, *sigma2, *grad, *adam_m, *adam_v;
};
// The sum over chunks r, r + rows, ... of a thread's partial, the first `kAt`
// of them in flight at once; past the last chunk the resource reads 0.
template <int kAt>
__device__ __forceinline__ float sum_chunks(__amdgpu_buffer_rsrc_t src, int first, int stride)
{
    float v[kAt], acc = 0.0f;
#pragma unroll
    for (int i = 0; i < kAt; ++i)
        v[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(src, first + i * stride, 0, 0));
#pragma unroll
    for (int i = 0; i < kAt; ++i) acc += v[i];
    return acc;
}
__device__ __forceinline__ void grad_step(ProblemRef P, int j, const float *__restrict__ part,
                                          float *__restrict__ grad_out,
                                          float *__restrict__ J_out, int it, float lr, float *__restrict__ cmd,
                                          int shift)
{
    constexpr int kMaxPerThread = (kAdjChunks * kMaxH + kRedThreads - 1) / kRedThreads;
    static_assert(kMaxPerThread <= 32, "chunks of a thread at the longest horizon");
    __shared__ float s_red[kRedThreads];
    __shared__ float s_wave[kRedThreads / kLanes];
    const int t = threadIdx.x;
    const int lane = t & (kLanes - 1), wave = __builtin_amdgcn_readfirstlane(t / kLanes);
    GradFields F{P.N, P.H, P.n_chunks, P.cov_step, P.tables, P.mean, P.sigma2, P.grad, P.adam_m, P.adam_v};
    asm volatile("" : "+s"(F.N), "+s"(F.H), "+s"(F.n_chunks), "+s"(F.cov_step), "+s"(F.tables), "+s"(F.mean),
                 "+s"(F.sigma2), "+s"(F.grad), "+s"(F.adam_m), "+s"(F.adam_v));
    const int H = F.H, T = F.n_chunks;
    const int rows = kRedThreads / H;
    const int r = t / H, h = t - r * H;
    // what the end of wave 0 reads (element e = (step `lane`, joint j))
    const int e = min(lane, H - 1) * kDof + j;
    float m0 = 0.0f, v0 = 0.0f, mu = 0.0f, s2 = 0.0f, sig0 = 0.0f, b1_it = 0.0f, b2_it = 0.0f;
    const bool shift_cov = cmd != nullptr && shift && F.cov_step;
    if (wave == 0) {
        if (it > 1) {  // (the moments restart with the first step)
            m0 = as_global(F.adam_m)[e];
            v0 = as_global(F.adam_v)[e];
        }
        if (it > 0 || cmd) mu = as_global(F.mean)[e];
        if (shift_cov) {
            s2 = as_global(F.sigma2)[e];
            sig0 = as_global(F.tables)[kTabSig0 + j];
        }
    }
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(part + kAdjChunks), (short)0, T * kDof * kMaxH * (int)sizeof(float), 0x00020000);
    const int first = ((r * kDof + j) * kMaxH + h) * (int)sizeof(float), stride = rows * kDof * kMaxH * (int)sizeof(float);
    const int need = (T + rows - 1) / rows;
    const float acc = need <= 8    ? sum_chunks<8>(src, first, stride)
                      : need <= 16 ? sum_chunks<16>(src, first, stride)
                                   : sum_chunks<32>(src, first, stride);
    s_red[t] = r < rows ? acc : 0.0f;
    if (j == 0 && J_out) {
        float cs = 0.0f;
        for (int k = t; k < T; k += kRedThreads) cs += as_global(part)[k];
        cs = wave_sum(cs);
        if (lane == 0) s_wave[wave] = cs;
    }
    if (wave == 0 && it > 0) {
        b1_it = powf(0.9f, (float)it);
        b2_it = powf(0.999f, (float)it);
    }
    __syncthreads();
    if (wave != 0) return;
    const float invN = 1.0f / (float)F.N;
    if (j == 0 && lane == 0 && J_out) {
        float J = 0.0f;
        for (int k = 0; k < kRedThreads / kLanes; ++k) J += s_wave[k];
        *J_out = J * invN;
    }
    if (lane < H) {
        float p4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        int k = 0;
        for (; k + 3 < rows; k += 4)
#pragma unroll
            for (int m = 0; m < 4; ++m) p4[m] += s_red[(k + m) * H + lane];
#pragma unroll
        for (int m = 0; m < 3; ++m)
            if (k + m < rows) p4[m] += s_red[(k + m) * H + lane];
        const float g = ((p4[0] + p4[1]) + (p4[2] + p4[3])) * invN;
        as_global(F.grad)[e] = g;
        if (grad_out) grad_out[e] = g;
        if (it > 0) mu = adam_step(F.adam_m, F.adam_v, e, g, m0, v0, mu, lr, 0.9f, 0.999f, b1_it, b2_it, 1e-8f);
    } else {
        mu = 0.0f;
    }
    if (cmd) {
        const float mu_next = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mu), 0x130, 0xf, 0xf,
                                                                         true));  // wave_shl:1
        if (lane == 0) cmd[j] = mu;
        if (shift) mu = lane + 1 < H ? mu_next : 0.0f;
        if (shift_cov) {
            // a per-step variance moves forward too, sigma_init^2 appended
            const float s2_next = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s2), 0x130, 0xf, 0xf,
                                                                             true));  // wave_shl:1
            if (lane < H) as_global(F.sigma2)[e] = lane + 1 < H ? s2_next : sig0;
        }
    }
    if ((it > 0 || cmd) && lane < H) as_global(F.mean)[e] = mu;
}

// All arguments fit the 14 dwords that are preloaded into SGPRs.
__global__ __launch_bounds__(kRedThreads) void grad_step_kernel(const PlainDev *dev,
                                                                const float *__restrict__ part,
                                                                float *__restrict__ grad_out,
                                                                float *__restrict__ J_out, float *__restrict__ cmd,
                                                                int it, float lr, int shift)
{
    grad_step(uniform_ptr(dev)->P, blockIdx.x, part, grad_out, J_out, it, lr, cmd, shift);
}

__global__ void command_kernel(const PlainDev *dev, float *__restrict__ cmd, int shift)
{
    command(uniform_ptr(dev)->P, cmd, shift);
}

// Batched forms: workgroup p * 7 + j serves joint j of problem p.
__global__ __launch_bounds__(kRedThreads) void grad_step_batch_kernel(const ProblemDev *__restrict__ probs, int it,
                                                                      float lr, float *__restrict__ cmd, int shift)
{
    const int p = blockIdx.x / kDof, j = blockIdx.x - p * kDof;
    ProblemRef P = uniform_ptr(probs)[p];
    grad_step(P, j, P.grad_part, nullptr, nullptr, it, lr, cmd ? cmd + (size_t)p * kDof : nullptr, shift);
}

__global__ void command_batch_kernel(const ProblemDev *__restrict__ probs, float *__restrict__ cmd, int shift)
{
    ProblemRef P = uniform_ptr(probs)[blockIdx.x];
    command(P, cmd + (size_t)blockIdx.x * kDof, shift);
}

}  // namespace

hipError_t launch_grad(const ProblemDev &P, const PlainDev *dev, float *part, const float *x0, const float *goal,
                       const float *mean, const float *noise, float *grad_out, float *J_out, int it, float lr,
                       float *cmd, int shift, hipStream_t stream)
{
    const bool wide = adjoint_runs(P.n_tiles) > kAdjWaves;
    auto kernel = P.n_tiles <= kSplitTiles ? adjoint_split_kernel
                  : wide                   ? adjoint_kernel<2 * kAdjWaves>
                                           : adjoint_kernel<kAdjWaves>;
    const int waves = P.n_tiles <= kSplitTiles ? kSplitWaves : wide ? 2 * kAdjWaves : kAdjWaves;
    hipLaunchKernelGGL(kernel, dim3((unsigned)P.n_chunks), dim3((unsigned)(waves * kLanes)), 0, stream, dev, mean, x0,
                       goal, noise, part, P.N, P.H);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(grad_step_kernel, dim3(kDof), dim3(kRedThreads), 0, stream, dev, part, grad_out, J_out, cmd,
                       it, lr, shift);
    return hipGetLastError();
}

hipError_t launch_command(const PlainDev *dev, float *cmd, int shift, hipStream_t stream)
{
    hipLaunchKernelGGL(command_kernel, dim3(1), dim3(256), 0, stream, dev, cmd, shift);
    return hipGetLastError();
}

hipError_t launch_refine_batch(const ProblemDev *probs, int n_problems, const int2 *items, int n_items, bool split,
                               const RobotDev *robot, const float *x0s, const float *goals, int iterations,
                               float lr, float *cmd, int shift, hipStream_t stream)
{
    hipError_t e = hipSuccess;
    for (int it = 1; e == hipSuccess && it <= iterations; ++it) {
        hipLaunchKernelGGL(split ? adjoint_split_batch_kernel : adjoint_batch_kernel, dim3((unsigned)n_items),
                           dim3((unsigned)((split ? kSplitWaves : kAdjWaves) * kLanes)), 0, stream, probs, items, robot,
                           x0s, goals);
        e = hipGetLastError();
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(grad_step_batch_kernel, dim3((unsigned)(n_problems * kDof)), dim3(kRedThreads), 0, stream,
                           probs, it, lr, it == iterations ? cmd : nullptr, shift);
        e = hipGetLastError();
    }
    if (e == hipSuccess && iterations == 0) {
        hipLaunchKernelGGL(command_batch_kernel, dim3((unsigned)n_problems), dim3(256), 0, stream, probs, cmd, shift);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace storm
