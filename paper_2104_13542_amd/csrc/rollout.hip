// Kernel R: sample -> integrate -> kinematics -> running cost -> horizon cost
// for one MPC problem (STORM, Sec. 3.1-3.3, Eq. 2 and 7-15).
//
// Work decomposition.  A tile is one 64-lane point set holding
// ppt = floor(64 / H) whole particles, lane = particle_in_tile * H + step.
// One workgroup of W wavefronts owns one tile; the waves split the work of
// the tile's 64 (particle, step) points and exchange data through LDS:
//   A0  waves 0-3  standard noise: one Philox4x32-10 call gives four normals
//                  (joints 4k..4k+3), each wave the Box-Muller pair of one
//                  half of a call; or the Halton table; or the override
//   A1  waves 0-6  one joint each: u = mu + sigma eps, then the two
//                  segmented prefix sums of the triple integrator (Eq. 7) as
//                  wavefront DPP scans over the particle's lanes, the joint's
//                  sine and cosine, and its squared joint, velocity and stop
//                  hinges (Eq. 10-11)
//   B   waves 0-2  forward kinematics (Eq. 8), one row of the eight frames
//                  per wave, to LDS
//       wave W-1   the hinge norms over the joints (Eq. 10-11)
//   C   waves 0..W-3  world centres of the body spheres and the capsules
//                  that hold them, to LDS
//       wave W-2   manipulability (Eq. 12)
//       wave W-1   pose (Eq. 9)
//   D1  all waves  obstacles near each body, by capsules
//   D2  all waves  environment (spheres x obstacles) split over waves, then
//                  self-collision (sphere pairs) as items taken from a queue,
//                  each behind a broad-phase test
//   E   wave 4     weighted running cost (Eq. 15), horizon sum (Eq. 2) as a
//                  segmented DPP scan
// Obstacle, sphere and pair records are indexed by wave-uniform loop
// counters, so they are fetched with scalar loads into SGPRs; every per-point
// LDS array is [row][lane] (conflict-free), and rows whose lifetimes do not
// overlap share space (about 80 KB per workgroup with 52 spheres, so that the
// batched form holds two workgroups per CU).  Reductions run in a fixed
// order: results are bitwise reproducible.
#include <algorithm>

#include "kinematics.h"
#include "sampling.h"

namespace storm {
namespace {

// Rows of the sphere-centre block, which also holds the noise, sine/cosine
// and hinge rows of phases A0-B (8 + 14 + 21) before the centres exist.
__host__ __device__ constexpr int rollout_cen_rows(int S) { return 3 * S > 43 ? 3 * S : 43; }
static_assert(2 * 16 <= 96, "the collision partials of 16 waves fit over the frame rows");

// Value of lane kLane of the caller's 16-lane row.
template <int kLane>
__device__ __forceinline__ float row_lane(float x)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x150 + kLane, 0xf, 0xf, false));  // row_newbcast
}

// Maximum of a non-negative float over the caller's 16-lane row, in every
// lane: IEEE bit patterns of non-negative floats order like unsigned
// integers, so it runs on the bits through DPP lane moves.
__device__ __forceinline__ float row_max_nonneg(float x)
{
    uint32_t b = __float_as_uint(x);
    b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0xb1, 0xf, 0xf, false));   // quad_perm [1, 0, 3, 2]
    b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0x4e, 0xf, 0xf, false));   // quad_perm [2, 3, 0, 1]
    b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0x141, 0xf, 0xf, false));  // row_half_mirror
    b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0x140, 0xf, 0xf, false));  // row_mirror
    return __uint_as_float(b);
}

// Whether the capsule (segment a.xyz + t b.xyz, t in [0, 1], radius `reach`
// already holding the obstacle's; b.w = 1 / |b.xyz|^2) meets the point o.
// The margin of the culling radii covers the rounding of t, which moves the
// nearest point by far less.
__device__ __forceinline__ bool capsule_hits(const float4 a, const float4 b, float reach, float ox, float oy, float oz)
{
    const float dx = ox - a.x, dy = oy - a.y, dz = oz - a.z;
    const float t = fminf(fmaxf(fmaf(dx, b.x, fmaf(dy, b.y, dz * b.z)) * b.w, 0.0f), 1.0f);
    const float ex = fmaf(-t, b.x, dx), ey = fmaf(-t, b.y, dy), ez = fmaf(-t, b.z, dz);
    return fmaf(ex, ex, fmaf(ey, ey, ez * ez)) < reach * fabsf(reach);
}

// The fields of a problem that the first loads of a tile depend on.
struct TileFirst {
    uint32_t *step;
    const float *mean, *halton;
    int32_t N, H, n_halton, n_null;
};

// LDS copy of the goal (R row-major, p) and the cost weights, by index.
constexpr int kParArot = 12, kParApos = 15, kParW = 18, kParKm = 25, kParCount = 26;

// The ball-on-tray term (appendix on dynamic object balancing), by the pose
// wave: every lane forms the flange frame of the current state q0 and moves
// the ball's world state into it (its z velocity dropped); lane (particle,
// h) takes the in-plane gravity in the flange frame of its rolled-out state
// and the two segmented scans of Eq. 7's scheme give the ball's velocity
// and position; the term is the distance from the tray centre.
__device__ __forceinline__ void ball_term(ProblemRef P, RobotRef R, const float *__restrict__ x0,
                                          const float *s_fr, float *s_terms, const int pos, const int h,
                                          const int H, global_ptr<const float> tab)
{
    float r0[9] = {1.0f, 0.0f, 0.0f, 0.0f, 1.0f, 0.0f, 0.0f, 0.0f, 1.0f}, p0[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int f = 0; f < kFrames; ++f) {
        float st = 0.0f, ct = 1.0f;
        if (f < kDof) sincosf(x0[f], &st, &ct);
        dh_step(r0, p0, R.ca[f], R.sa[f], R.a[f], R.d[f], ct, st);
    }
    const float bw[3] = {as_global(P.ball)[0] - p0[0], as_global(P.ball)[1] - p0[1], as_global(P.ball)[2] - p0[2]};
    float xb[2], vb[2], ab[2];
    const float *E = s_fr + 7 * 12 * kLanes + pos;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        xb[c] = fmaf(r0[c], bw[0], fmaf(r0[3 + c], bw[1], r0[6 + c] * bw[2]));
        vb[c] = fmaf(r0[c], as_global(P.ball)[3], fmaf(r0[3 + c], as_global(P.ball)[4], r0[6 + c] * as_global(P.ball)[5]));
        ab[c] = fmaf(E[c * kLanes], P.ball_g[0], fmaf(E[(3 + c) * kLanes], P.ball_g[1],
                                                      E[(6 + c) * kLanes] * P.ball_g[2]));
    }
    const float dt_h = tab[kTabDt + h];
    float d2 = 0.0f;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float v = vb[c] + segmented_scan(dt_h * ab[c], h, H);
        const float x = xb[c] + segmented_scan(dt_h * v, h, H);
        const float e = x - P.ball_c[c];
        d2 = fmaf(e, e, d2);
    }
    s_terms[8 * kLanes + pos] = fast_sqrt(d2);
}

// Where a workgroup's next tile comes from.  The last wave draws it while it
// has nothing else to do in the current tile, so that neither the atomic's
// nor the item's memory round trip stands between two tiles; the others read
// it from LDS after the tile's last barrier.
struct NoQueue {  // the plain form: one tile per workgroup
    static constexpr int parity = 0;
    __device__ __forceinline__ void draw() {}
    __device__ __forceinline__ void fetch() {}
    __device__ __forceinline__ void store() {}
};
struct TileQueue {
    uint32_t *next;
    const int2 *items;
    int n_items, n_groups;
    int (*s_item)[2];  // LDS [2][2]: problem (negative: none left), tile, by parity
    int parity = 0;    // of the current tile
    int item = 0, p = -1, tile = 0;

    // the items after the first one of each workgroup, in queue order
    __device__ __forceinline__ void draw() { item = n_groups + (int)atomicAdd(next, 1u); }
    __device__ __forceinline__ void fetch()
    {
        p = -1;
        if (item < n_items) {
            const global_ptr<const int32_t> it = as_global(reinterpret_cast<const int32_t *>(items)) + 2 * item;
            p = it[0];
            tile = it[1];
        } else if (item == n_items + n_groups - 1) {
            atomicExch(next, 0u);  // the last draw of the launch
        }
    }
    __device__ __forceinline__ void store()
    {
        s_item[parity ^ 1][0] = p;
        s_item[parity ^ 1][1] = tile;
    }
};

// One 64-lane tile of one problem, executed by the W waves of the calling
// workgroup; smem is the workgroup's dynamic LDS (rollout_lds_bytes).
// kTask: the task-space form, which adds the flange velocity and
// acceleration outputs (Eq. 8), the ball-on-tray term and the joint
// positions the learned self-collision network reads.
// The fields of the descriptors are scalar loads where they are used (held as
// copies they overflowed the SGPRs into lanes of VGPRs, 180 lane moves per
// wave and tile).
template <int W, bool kTask, class Queue>
__device__ __forceinline__ void rollout_tile(Queue &queue, ProblemRef P, RobotRef R, const TileFirst &first, const int tile,
                                             const float *__restrict__ x0, const float *__restrict__ goal,
                                             const float *__restrict__ noise, const StepOut &out, float *smem)
{
    // LDS rows of 64 floats, overlaid where their lifetimes do not meet
    // (rollout_lds_bytes), so that two workgroups of the batched form fit on
    // one CU:
    //   frames [96]              B - C,  then the collision partials [2W]  D2 - E
    //   terms [kTerms]           B - E
    //   centres [3S]             C - D2;  before them noise [8] A0 - A1,
    //                            sin/cos [14] and hinges [21] A1 - B
    //   velocities, accelerations [14]  A1 - C (task-space form only)
    // then the capsules of the spheres [S][4 rows][8] (C - D2) and the
    // culling records of the obstacles (A0 - D2).
    const int S = R.n_spheres;
    float *s_fr = smem;                        // [8 frames][12][64]: R row-major, p
    float *s_penv = s_fr;                      // [W][64] (over the frames, after phase C)
    float *s_pself = s_penv + W * kLanes;      // [W][64]
    float *s_terms = s_fr + 96 * kLanes;       // [kTerms][64]
    float *s_cen = s_terms + kTerms * kLanes;  // [S][3][64]
    float *s_eps = s_cen;                      // [8][64] (before the centres)
    float *s_sc = s_eps + 8 * kLanes;          // [7][2][64]: sin q_j, cos q_j
    float *s_lim = s_sc + 14 * kLanes;         // [3][7][64]: squared joint, velocity, stop hinges per joint
    float *s_v = s_cen + rollout_cen_rows(S) * kLanes;  // [7][64] (task-space form only)
    float *s_acc = s_v + kDof * kLanes;                  // [7][64]
    float4 *s_cap = reinterpret_cast<float4 *>(s_v + (kTask ? 2 * kDof * kLanes : 0));  // [S][4][2]
    float4 *s_bound = s_cap + 8 * S;                     // [obstacles]

    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = first.N, H = first.H, ppt = P.ppt;
    // the particle and step of this lane (lane / H by a reciprocal: exact, as
    // the quotients of lane + 1/2 stay 1/128 away from the integers)
    const int pl = (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)H));
    const int h = lane - pl * H;
    const int i = tile * ppt + pl;
    const bool valid = pl < ppt && i < N;
    // From the joint angles on, the points of the tile lie in LDS by step,
    // then particle, so that the 16 lanes of a row are neighbours in time:
    // `pos` is where this lane's point goes; positions past the last point
    // repeat it (`src`, from phase B on).
    const int n_pts = ppt * H;
    const int pos = pl < ppt ? h * ppt + pl : lane;
    const int src = min(lane, n_pts - 1);
    const bool live = valid && i < N - first.n_null;  // sampled (non-null) particle
    const uint32_t mask = P.cost_mask;
    const global_ptr<const float> tab = as_global(P.tables);

    // Per-joint inputs of phase A1, loaded up front so that their latency
    // overlaps the noise generation.
    const int jw = wave < kDof ? wave : 0;
    // (vector loads throughout, so that the first barrier waits for none of
    // them: the state and the policy come fresh from the previous kernels)
    const float mu_j = live ? as_global(first.mean)[h * kDof + jw] : 0.0f;
    const float sig_j = sqrtf(P.cov_step ? as_global(P.sigma2)[h * kDof + jw] : vector_load_f32(P.sigma2 + jw));
    const float dt_h = tab[kTabDt + h];
    const float vs_h = tab[kTabVstop + h];
    const float q0_j = vector_load_f32(x0 + jw), v0_j = vector_load_f32(x0 + kDof + jw);
    // the obstacles' culling records for phase D, one per thread of the waves
    // that draw no noise
    const int nobs = (mask & STORM_COST_ENV) && S > 0 ? P.n_sph_obs + P.n_box_obs : 0;
    const int ob_t = (int)threadIdx.x - 4 * kLanes;
    static_assert((W - 4) * kLanes >= STORM_MAX_OBSTACLES, "one culling record per thread");
    if (ob_t >= 0 && ob_t < nobs) s_bound[ob_t] = load_float4(as_global(P.obs_bound) + ob_t);
    // the goal and the cost weights that phases C and E read, staged in
    // LDS by the last wave while the noise is drawn (read where they are
    // used, as scalar loads, they would add a memory round trip to those
    // serial phases)
    __shared__ float s_par2[2][kParCount];  // (by parity: the costs of a tile are summed during the next one's noise)
    float *s_par = s_par2[queue.parity];
    __shared__ int s_self_next;  // head of the self-collision item queue (phase D2)
    __shared__ int s_near_n[kFrames];  // obstacles near each body (phase D1)
    __shared__ uint8_t s_near[kFrames * STORM_MAX_OBSTACLES];
    if (wave == W - 1 && lane == kParCount) s_self_next = 0;
    if (wave == W - 2 && lane < kFrames) s_near_n[lane] = 0;
    // ---- A0: standard noise ------------------------------------------------
    // waves 0-3, one per SIMD: wave w makes the normal pair w / 2 of Philox
    // call w % 2, i.e. joints 4 (w % 2) + 2 (w / 2) and the next (the
    // Philox call is repeated by the two waves that share it; its Box-Muller
    // half is not)
    if (wave < 4) {
        const int k = wave & 1, half = wave >> 1;
        const int j0 = 4 * k + 2 * half;
        float e[2] = {0.0f, 0.0f};
        const uint32_t counter = *as_global(first.step);
        if (live) standard_noise2(first, P.seed_lo, P.seed_hi, noise, k, half, i, h, counter, e);
        s_eps[j0 * kLanes + lane] = e[0];
        s_eps[(j0 + 1) * kLanes + lane] = e[1];
        if (tile == 0 && threadIdx.x == 0) *as_global(P.last_step) = counter;
    } else if (wave == W - 1 && lane < kParCount) {
        const float g = goal[lane < 12 ? lane : 0], w = tab[kTabPar + (lane < 12 ? 0 : lane - 12)];
        s_par[lane] = lane < 12 ? g : w;
    }
    __syncthreads();

    // ---- A1: controls and the triple integrator (Eq. 7) ---------------------
    if (wave < kDof) {
        const int j = wave;
        float e = s_eps[j * kLanes + lane];
        // the comb filter on the sampled Gaussian particles' noise (Sec. 3.3)
        const bool comb = P.comb && noise == nullptr && live && i >= first.n_halton;
        if (__builtin_amdgcn_ballot_w64(comb) != 0) {
            const float f = comb_noise(s_eps + j * kLanes, lane, h, H, tab);
            if (comb) e = f;
        }
        float u = 0.0f;
        if (live) u = fmaf(sig_j, e, mu_j);
        const float v = v0_j + segmented_scan(dt_h * u, h, H);
        const float q = q0_j + segmented_scan(dt_h * v, h, H);
        if (kTask) s_v[j * kLanes + pos] = v;
        // this joint's squared joint, velocity and stop hinges (Eq. 10-11),
        // summed over the joints in phase C
        const float hj = hinge_box(q, tab[kTabJlo + j], tab[kTabJhi + j]);
        const float hv = hinge_box(v, tab[kTabVlo + j], tab[kTabVhi + j]);
        const float hs = fmaxf(fabsf(v) - vs_h, 0.0f);
        s_lim[(0 * kDof + j) * kLanes + pos] = hj * hj;
        s_lim[(1 * kDof + j) * kLanes + pos] = hv * hv;
        s_lim[(2 * kDof + j) * kLanes + pos] = hs * hs;
        float sq, cq;
        sincosf(q, &sq, &cq);
        s_sc[(2 * j) * kLanes + pos] = sq;
        s_sc[(2 * j + 1) * kLanes + pos] = cq;
        if (kTask) s_acc[j * kLanes + pos] = u;
        if (valid) {
            const size_t o = ((size_t)j * N + i) * H + h;
            as_global(P.u)[o] = u;
            if (kTask && P.qbuf != nullptr) as_global(P.qbuf)[o] = q;
            if (out.u) out.u[o] = u;
            if (out.q) out.q[o] = q;
            if (out.v) out.v[o] = v;
            if (out.a) out.a[o] = u;
        }
    } else if (wave == W - 1 && lane == 0) {
        queue.draw();
    }
    __syncthreads();

    // ---- B: forward kinematics, one row of the frames per wave ----------------
    if (wave < 3) {
        const int row = wave;
        float r[3] = {row == 0 ? 1.0f : 0.0f, row == 1 ? 1.0f : 0.0f, row == 2 ? 1.0f : 0.0f};
        float p = 0.0f;
#pragma unroll
        for (int f = 0; f < kFrames; ++f) {
            float st = 0.0f, ct = 1.0f;
            if (f < kDof) {
                st = s_sc[(2 * f) * kLanes + src];
                ct = s_sc[(2 * f + 1) * kLanes + src];
            }
            dh_step_row(r, p, R.ca[f], R.sa[f], R.a[f], R.d[f], ct, st);
#pragma unroll
            for (int c = 0; c < 3; ++c) s_fr[(f * 12 + row * 3 + c) * kLanes + lane] = r[c];
            s_fr[(f * 12 + 9 + row) * kLanes + lane] = p;
        }
    } else if (wave == W - 1) {
        // Eq. 10-11: norms over the joints of the hinges formed in phase A1
        // (here, so that the hinge rows are free for the centres of phase C)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            float acc = 0.0f;
#pragma unroll
            for (int j = 0; j < kDof; ++j) acc += s_lim[(k * kDof + j) * kLanes + lane];
            s_terms[(2 + k) * kLanes + lane] = fast_sqrt(acc);
        }
        if (lane == 0) queue.fetch();
    }
    __syncthreads();

    // ---- C: world centres of the body spheres | pose | manipulability --------
    // The last two waves evaluate the pose (Eq. 9) and manipulability
    // (Eq. 12) terms from the frames while the others place the spheres, so
    // that the collision phase is spread evenly over all waves.
    constexpr int WC = W - kPoseWaves;
    if (wave < WC) {
        if (mask & (STORM_COST_SELF | STORM_COST_ENV)) {
            // a contiguous run of spheres per wave (sorted by body): the
            // frame of a body is read from LDS once per run
            const int s0 = wave * S / WC, s1 = (wave + 1) * S / WC;
            const STORM_CONST_AS int32_t *body = uniform_ptr(R.sph_body);
            int fb = -1;
            float F[12];
            // where in its row's span of steps this lane lies, in [0, 1]
            const float step = floorf(((float)src + 0.5f) * __builtin_amdgcn_rcpf((float)ppt));
            const float step0 = row_lane<0>(step);
            const float tau =
                fminf((step - step0) * __builtin_amdgcn_rcpf(fmaxf(row_lane<15>(step) - step0, 1.0f)), 1.0f);
            for (int s = s0; s < s1; ++s) {
                const STORM_CONST_AS float *sl = uniform_ptr(reinterpret_cast<const float *>(R.sph_local)) + 4 * s;
                const int b = body[s];
                if (b != fb) {
#pragma unroll
                    for (int c = 0; c < 12; ++c) F[c] = s_fr[(b * 12 + c) * kLanes + lane];
                    fb = b;
                }
                float cc[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    cc[c] = fmaf(F[c * 3 + 0], sl[0], fmaf(F[c * 3 + 1], sl[1], fmaf(F[c * 3 + 2], sl[2], F[9 + c])));
                    s_cen[(s * 3 + c) * kLanes + lane] = cc[c];
                }
                if (nobs == 0) continue;
                // The capsule of each row of 16 points, which phase D tests
                // against the obstacles: the chord from the row's first
                // centre a to its last, and as radius the largest distance
                // of a centre to the chord's point at its own time (any
                // point of the chord serves), plus r_s.  A row with a
                // centre that is not finite gets a ball that meets
                // everything.
                const float ax = row_lane<0>(cc[0]), ay = row_lane<0>(cc[1]), az = row_lane<0>(cc[2]);
                const float dx = cc[0] - ax, dy = cc[1] - ay, dz = cc[2] - az;
                const float bx = row_lane<15>(dx), by = row_lane<15>(dy), bz = row_lane<15>(dz);
                const float ex = fmaf(-tau, bx, dx), ey = fmaf(-tau, by, dy), ez = fmaf(-tau, bz, dz);
                const float rad =
                    fast_sqrt(row_max_nonneg(fminf(fmaf(ex, ex, fmaf(ey, ey, ez * ez)), 1.0e30f)));
                const float len2 = fmaf(bx, bx, fmaf(by, by, bz * bz));
                if ((lane & 15) == 0) {
                    const bool cull = rad < 1.0e6f;
                    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    float4 *cap = s_cap + (s * 4 + (lane >> 4)) * 2;
                    cap[0] = cull ? make_float4(ax, ay, az, rad + sl[3]) : make_float4(0.0f, 0.0f, 0.0f, 1.0e15f);
                    cap[1] = cull ? make_float4(bx, by, bz, __builtin_amdgcn_rcpf(fmaxf(len2, 1.0e-20f))) : zero;
                }
            }
        }
    } else if (wave == W - 1) {
        if (mask & STORM_COST_POSE) {
            // Eq. 9: rotation error |diag(alpha_rot)(I - R_g^T R)|_F and position
            // error |diag(alpha_pos) R_g^T (p - p_g)|.
            const float *E = s_fr + 7 * 12 * kLanes + lane;
            float Re[9], pe[3];
#pragma unroll
            for (int c = 0; c < 9; ++c) Re[c] = E[c * kLanes];
#pragma unroll
            for (int c = 0; c < 3; ++c) pe[c] = E[(9 + c) * kLanes];
            float rot2 = 0.0f, pos2 = 0.0f;
#pragma unroll
            for (int r = 0; r < 3; ++r) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float m = fmaf(s_par[0 * 3 + r], Re[0 * 3 + c],
                                         fmaf(s_par[1 * 3 + r], Re[1 * 3 + c], s_par[2 * 3 + r] * Re[2 * 3 + c]));
                    const float e = s_par[kParArot + r] * ((r == c ? 1.0f : 0.0f) - m);
                    rot2 = fmaf(e, e, rot2);
                }
                const float l = fmaf(s_par[0 * 3 + r], pe[0] - s_par[9],
                                     fmaf(s_par[1 * 3 + r], pe[1] - s_par[10], s_par[2 * 3 + r] * (pe[2] - s_par[11])));
                const float e = s_par[kParApos + r] * l;
                pos2 = fmaf(e, e, pos2);
            }
            s_terms[0 * kLanes + lane] = fast_sqrt(pos2);
            s_terms[1 * kLanes + lane] = fast_sqrt(rot2);
        }
        if (kTask && (mask & STORM_COST_BALL)) ball_term(P, R, x0, s_fr, s_terms, pos, h, H, tab);
    } else {
        const bool task_out = kTask && (out.xd != nullptr || out.xdd != nullptr);
        if ((mask & STORM_COST_MANIP) || task_out) {
            float z[kDof][3], o[kDof][3], pe[3];
#pragma unroll
            for (int k = 0; k < kDof; ++k) {
                const float *F = s_fr + k * 12 * kLanes + lane;
                z[k][0] = F[2 * kLanes];
                z[k][1] = F[5 * kLanes];
                z[k][2] = F[8 * kLanes];
                o[k][0] = F[9 * kLanes];
                o[k][1] = F[10 * kLanes];
                o[k][2] = F[11 * kLanes];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) pe[c] = s_fr[(7 * 12 + 9 + c) * kLanes + lane];
            if (mask & STORM_COST_MANIP) s_terms[5 * kLanes + lane] = manipulability(z, o, pe);
            if (task_out) {
                float qd[kDof], qdd[kDof], xd[6], xdd[6];
#pragma unroll
                for (int k = 0; k < kDof; ++k) {
                    qd[k] = s_v[k * kLanes + lane];
                    qdd[k] = s_acc[k * kLanes + lane];
                }
                task_space(s_fr + lane, kLanes, qd, qdd, xd, xdd);
                // the point at position `lane`
                const int hp = lane / ppt, ip = tile * ppt + (lane - hp * ppt);
                if (lane < n_pts && ip < N)
#pragma unroll
                    for (int c = 0; c < 6; ++c) {
                        const size_t at = ((size_t)c * N + ip) * H + hp;
                        if (out.xd) out.xd[at] = xd[c];
                        if (out.xdd) out.xdd[at] = xdd[c];
                    }
            }
        }
    }
    __syncthreads();

    if (wave == W - 1 && lane == 0) queue.store();

    // ---- D1: obstacles near each body ------------------------------------------
    // The environment term is bound by VALU issue, so what counts is how many
    // exact tests (20 instructions each) survive the cull.  Rows of 16 points
    // ordered by step sweep short, nearly straight pieces, which a capsule
    // holds tightly: on 4096 x 64 with 100 obstacles (one particle per wave)
    // 171 of 5200 sphere-obstacle pairs stay, against 131 that truly come
    // within a lane's reach; one ball per wave refined into eight kept 267-374
    // and tested every sphere against every obstacle first.  Issued VALU per
    // tile 24.6k -> 15.5k there, 12.9k -> 10.1k in the 256-problem batch;
    // the control step of 64 x 4096 x 64 20.7 -> 16.0 ms.
    // Both collision terms cull at the level of the whole wave and take exact
    // distances (and their square roots) only where some lane of the wave may
    // touch; a culled record touches at no lane, so the terms equal the
    // brute-force ones.  First, bodies against obstacles: a lane holds one
    // row's capsule of one body (that of the body's anchor sphere, widened to
    // hold all of the body's spheres) and each half of the wave takes another
    // obstacle; the waves share the obstacles.
    if (nobs > 0) {
        const int body = lane & 7, row = (lane >> 3) & 3, half = lane >> 5;
        const float anchor = as_global(R.body_bound)[2 * body], widen = as_global(R.body_bound)[2 * body + 1];
        const float4 *cap = s_cap + (__float_as_int(anchor) * 4 + row) * 2;
        const float4 a = cap[0], b = cap[1];
        const float reach = a.w + widen;
        for (int o0 = 2 * wave; o0 < nobs; o0 += 2 * W) {
            const int o = o0 + half;
            const float4 ob = o < nobs ? s_bound[o] : make_float4(3.0e38f, 3.0e38f, 3.0e38f, 0.0f);
            uint64_t near = __builtin_amdgcn_ballot_w64(capsule_hits(a, b, reach + ob.w, ob.x, ob.y, ob.z));
            if (near == 0) continue;
            near |= near >> 16;  // the four rows of a body
            near |= near >> 8;
            if (row == 0 && ((near >> lane) & 1ull)) {
                const int k = atomicAdd(&s_near_n[body], 1);
                s_near[body * STORM_MAX_OBSTACLES + k] = (uint8_t)o;
            }
        }
    }
    __syncthreads();

    // ---- D2: collision terms --------------------------------------------------
    // Environment (spheres round robin over the waves), then self-collision
    // (items from a queue).
    float env = 0.0f, selfpen = 0.0f;
    if (nobs > 0) {
        const STORM_CONST_AS float *sob = uniform_ptr(reinterpret_cast<const float *>(P.sph_obs));
        const STORM_CONST_AS float *box = uniform_ptr(P.box_obs);
        const STORM_CONST_AS float *sloc = uniform_ptr(reinterpret_cast<const float *>(R.sph_local));
        const STORM_CONST_AS int32_t *sbody = uniform_ptr(R.sph_body);
        const int nso = P.n_sph_obs;
        for (int s = wave; s < S; s += W) {
            const int b = sbody[s];
            const int n_near = __builtin_amdgcn_readfirstlane(s_near_n[b]);
            if (n_near == 0) continue;
            const float x = s_cen[(s * 3 + 0) * kLanes + lane];
            const float y = s_cen[(s * 3 + 1) * kLanes + lane];
            const float z = s_cen[(s * 3 + 2) * kLanes + lane];
            const float rs = sloc[4 * s + 3];
            const float rs2 = rs * rs;
            const float4 *cap = s_cap + (s * 4 + (lane >> 4)) * 2;
            const float4 ca = cap[0], cb = cap[1];
            float best = 0.0f;
            for (int k0 = 0; k0 < n_near; k0 += 16) {
                // the sphere's four capsules against 16 of its body's
                // obstacles at a time
                const int k = k0 + (lane & 15);
                const int ob_l = s_near[b * STORM_MAX_OBSTACLES + min(k, n_near - 1)];
                const float4 ob = s_bound[ob_l];
                uint64_t hits =
                    __builtin_amdgcn_ballot_w64(k < n_near && capsule_hits(ca, cb, ca.w + ob.w, ob.x, ob.y, ob.z));
                hits |= hits >> 32;  // the four rows
                uint32_t cand = (uint32_t)(hits | hits >> 16) & 0xffffu;
                // Narrow phase over the candidates (the maximum does not
                // depend on their order).
                while (cand != 0) {
                    const int o = __builtin_amdgcn_readlane(ob_l, __builtin_ctz(cand));
                    cand &= cand - 1;
                    if (o < nso) {
                        // the direct squared distance (no cancellation) against
                        // the squared contact distance, from the obstacle's own
                        // 16-byte record; where a lane touches, the penetration
                        // (r_s + r_o) - |x - c| at every lane (at or below zero
                        // where a lane does not touch)
                        const STORM_CONST_AS float *so = sob + 4 * o;
                        const float dx = x - so[0], dy = y - so[1], dz = z - so[2];
                        const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                        const float rc = rs + so[3];
                        if (__builtin_amdgcn_ballot_w64(d2 < rc * rc) != 0) best = fmaxf(best, rc - fast_sqrt(d2));
                    } else {
                        const STORM_CONST_AS float *bb = box + (size_t)(o - nso) * 16;
                        const float lx = fmaf(bb[0], x, fmaf(bb[1], y, fmaf(bb[2], z, bb[9])));
                        const float ly = fmaf(bb[3], x, fmaf(bb[4], y, fmaf(bb[5], z, bb[10])));
                        const float lz = fmaf(bb[6], x, fmaf(bb[7], y, fmaf(bb[8], z, bb[11])));
                        // excess per axis, clamped to [0, 1 m]: one instruction
                        // with the clamp modifier; body spheres are below 1 m, so
                        // clamping cannot turn a miss into a hit and leaves every
                        // axis of a hit exact
                        const float ox = fminf(fmaxf(fabsf(lx) - bb[12], 0.0f), 1.0f);
                        const float oy = fminf(fmaxf(fabsf(ly) - bb[13], 0.0f), 1.0f);
                        const float oz = fminf(fmaxf(fabsf(lz) - bb[14], 0.0f), 1.0f);
                        const float out2 = fmaf(ox, ox, fmaf(oy, oy, oz * oz));
                        const bool hit = out2 < rs2;
                        if (__builtin_amdgcn_ballot_w64(hit) != 0) {
                            const float qin =
                                fminf(fmaxf(fabsf(lx) - bb[12], fmaxf(fabsf(ly) - bb[13], fabsf(lz) - bb[14])), 0.0f);
                            const float pen = rs - (fast_sqrt(out2) + qin);
                            if (hit) best = fmaxf(best, pen);
                        }
                    }
                }
            }
            env += best;
        }
    }
    if (mask & STORM_COST_SELF) {
        // Pairs by groups of up to four spheres t of one body, held in
        // registers as (-2 c_t, |c_t|^2), against their partners s streamed
        // from LDS, two partners per round.  Per pair, the expanded form
        // a = |c_t|^2 - 2 c_s.c_t (three FMAs) less the pair's threshold;
        // the group's minimum plus |c_s|^2 is negative at a lane where some
        // pair may touch: one compare per partner and one branch per round,
        // no per-pair lane masks.  Only a partner, and then a pair, that some
        // lane passes gets the exact penetration (r_s + r_t) - |c_s - c_t|,
        // at every lane: a lane whose pair fails the expanded test is apart
        // by more than the contact distance plus the rounding, so its
        // penetration is negative and leaves the maximum unchanged.  Unused
        // slots of a short group repeat its last sphere against a threshold
        // of -1e30, and the round after the last partner of an odd count
        // repeats that partner.
        //
        // Work comes as items (one group against the spheres of one partner
        // body) from a queue in LDS, so that waves done early with the
        // environment term take more.  Broad phase per item: one sphere of
        // each side (the anchors) with the radius about it that holds all of
        // that side's spheres; where the anchors are farther apart than the
        // two radii at every lane, no pair of the item touches and the item
        // is skipped (its penetrations are all negative: the maximum is the
        // same).
        const STORM_CONST_AS int32_t *items = uniform_ptr(R.self_items);
        const STORM_CONST_AS float *thr = uniform_ptr(R.self_thr);
        const int n_items = R.n_self_items;
        for (;;) {
            int g = 0;
            if (lane == 0) g = atomicAdd(&s_self_next, 1);
            g = __builtin_amdgcn_readfirstlane(g);
            if (g >= n_items) break;
            const STORM_CONST_AS int32_t *it = items + 8 * g;
            const int code = it[0], grp = it[1], s_begin = it[2], s_end = it[3], at = it[4], as = it[5];
            const float reach2 = __int_as_float(it[6]);
            const float ax = s_cen[(at * 3 + 0) * kLanes + lane] - s_cen[(as * 3 + 0) * kLanes + lane];
            const float ay = s_cen[(at * 3 + 1) * kLanes + lane] - s_cen[(as * 3 + 1) * kLanes + lane];
            const float az = s_cen[(at * 3 + 2) * kLanes + lane] - s_cen[(as * 3 + 2) * kLanes + lane];
            if (__builtin_amdgcn_ballot_w64(fmaf(ax, ax, fmaf(ay, ay, az * az)) < reach2) == 0) continue;
            const int t_first = code & 255, count = code >> 8;
            float mx[4], my[4], mz[4], nt[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int t = t_first + (k < count ? k : count - 1);
                mx[k] = -2.0f * s_cen[(t * 3 + 0) * kLanes + lane];
                my[k] = -2.0f * s_cen[(t * 3 + 1) * kLanes + lane];
                mz[k] = -2.0f * s_cen[(t * 3 + 2) * kLanes + lane];
                nt[k] = 0.25f * fmaf(mx[k], mx[k], fmaf(my[k], my[k], mz[k] * mz[k]));
            }
            const STORM_CONST_AS float *tg = thr + (size_t)grp * S * 8;
            // one round: partners s0 and s1 (s1 == s0 for the last of an odd
            // count), whose records start at tp and tp + dt
            auto round = [&](const int s0, const int s1, const STORM_CONST_AS float *tp, const int dt)
                              __attribute__((always_inline)) {
                const int ps[2] = {s0, s1};
                float cx[2], cy[2], cz[2], ns[2], m[2], d[2][4];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int s = ps[u];
                    cx[u] = s_cen[(s * 3 + 0) * kLanes + lane];
                    cy[u] = s_cen[(s * 3 + 1) * kLanes + lane];
                    cz[u] = s_cen[(s * 3 + 2) * kLanes + lane];
                    ns[u] = fmaf(cx[u], cx[u], fmaf(cy[u], cy[u], cz[u] * cz[u]));
                    const STORM_CONST_AS float *th = tp + u * dt;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        d[u][k] = fmaf(cx[u], mx[k], fmaf(cy[u], my[k], fmaf(cz[u], mz[k], nt[k]))) - th[k];
                    m[u] = fminf(fminf(d[u][0], d[u][1]), fminf(d[u][2], d[u][3])) + ns[u];
                }
                // the contact distances come with the thresholds (one scalar
                // load per round), not in the rare branch
                float rc[2][4];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int k = 0; k < 4; ++k) rc[u][k] = tp[u * dt + 4 + k];
                asm volatile("" : : "s"(rc[0][0]), "s"(rc[0][1]), "s"(rc[0][2]), "s"(rc[0][3]), "s"(rc[1][0]),
                             "s"(rc[1][1]), "s"(rc[1][2]), "s"(rc[1][3]));
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(fminf(m[0], m[1]) < 0.0f) != 0, 0)) {
                    // the partners, then the pairs, that some lane passes
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        if (__builtin_amdgcn_ballot_w64(m[u] < 0.0f) == 0) continue;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            if (k >= count || __builtin_amdgcn_ballot_w64(d[u][k] + ns[u] < 0.0f) == 0) continue;
                            const float dx = fmaf(0.5f, mx[k], cx[u]), dy = fmaf(0.5f, my[k], cy[u]),
                                        dz = fmaf(0.5f, mz[k], cz[u]);
                            const float pen = rc[u][k] - fast_sqrt(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
                            selfpen = fmaxf(selfpen, pen);
                        }
                    }
                }
            };
            int sp = s_begin;
            const STORM_CONST_AS float *tp = tg + 8 * s_begin;
            for (; sp + 1 < s_end; sp += 2, tp += 16) round(sp, sp + 1, tp, 8);
            if (sp < s_end) round(sp, sp, tp, 0);
        }
    }
    s_penv[wave * kLanes + lane] = env;
    s_pself[wave * kLanes + lane] = selfpen;

    __syncthreads();

    // ---- E: running cost (Eq. 15) and horizon cost (Eq. 2) ------------------
    // (by a wave that draws no noise: in the batched form the others are already
    // at the next tile's)
    if (wave == 4) {
        float t[kTerms];
#pragma unroll
        for (int k = 0; k < kTerms; ++k) t[k] = 0.0f;
        if (mask & STORM_COST_POSE) {
            t[0] = s_terms[0 * kLanes + pos];
            t[1] = s_terms[1 * kLanes + pos];
        }
        if (mask & STORM_COST_JOINT) t[2] = s_terms[2 * kLanes + pos];
        if (mask & STORM_COST_VEL) t[3] = s_terms[3 * kLanes + pos];
        if (mask & STORM_COST_STOP) t[4] = s_terms[4 * kLanes + pos];
        if (mask & STORM_COST_MANIP) {
            const float m = s_terms[5 * kLanes + pos];
            t[5] = m < s_par[kParKm] ? 1.0f - m : 0.0f;
        }
        if (mask & STORM_COST_SELF)
            for (int w = 0; w < W; ++w) t[6] = fmaxf(t[6], s_pself[w * kLanes + pos]);
        if (mask & STORM_COST_ENV)
            for (int w = 0; w < W; ++w) t[7] += s_penv[w * kLanes + pos];
        const float *wc = s_par + kParW;  // w_pos, w_rot, a_joint, a_vel, a_stop, a_manip, a_coll
        float c = wc[0] * t[0];
        c = fmaf(wc[1], t[1], c);
        c = fmaf(wc[2], t[2], c);
        c = fmaf(wc[3], t[3], c);
        c = fmaf(wc[4], t[4], c);
        c = fmaf(wc[5], t[5], c);
        c = fmaf(wc[6], t[6] + t[7], c);
        if (kTask && (mask & STORM_COST_BALL)) {
            t[8] = s_terms[8 * kLanes + pos];
            c = fmaf(P.w_ball, t[8], c);
        }
        if (valid) {
            if (out.c) out.c[(size_t)i * H + h] = c;
            if (out.terms)
#pragma unroll
                for (int k = 0; k < kTerms; ++k) out.terms[((size_t)k * N + i) * H + h] = t[k];
        }
        // horizon cost (Eq. 2): segmented inclusive scan of the weighted
        // running costs; the particle's last lane holds its total
        const float C_i = segmented_scan(tab[kTabHw + h] * c, h, H);
        if (valid && h == H - 1) {
            as_global(P.C)[i] = C_i;
            if (out.C) out.C[i] = C_i;
        }
    }
}

// Every argument of the usual call fits the 14 dwords that are preloaded into
// SGPRs at wave launch, so that no load of the kernel arguments (host memory)
// stands before the work; what else a tile needs it reads from the descriptor
// in device memory.  The fields that most first loads depend on come along.
// kDebug: with the noise override and the optional outputs, which are read
// from the argument segment.
template <int W, bool kTask, bool kDebug>
__global__ __launch_bounds__(W * kLanes) void rollout_kernel(const PlainDev *dev, int32_t N, int32_t H,
                                                             const float *__restrict__ x0,
                                                             const float *__restrict__ goal, const float *mean,
                                                             uint32_t *step, float *C_out,
                                                             const float *__restrict__ noise, StepOut out)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];  // (holds 16-byte records)
    StepOut o{};
    if (kDebug) o = out;
    o.C = C_out;
    const STORM_CONST_AS PlainDev &D = *uniform_ptr(dev);
    const TileFirst first{step, mean, D.P.halton, N, H, D.P.n_halton, D.P.n_null};
    NoQueue none;
    rollout_tile<W, kTask>(none, D.P, D.R, first, blockIdx.x, x0, goal, kDebug ? noise : nullptr, o, smem);
}

// Persistent form for many problems: each workgroup takes (problem, tile)
// items in the order of `items` (the scheduler puts the most expensive tiles
// first), the first by its index and the others from an integer work queue,
// until the queue is empty.  Every workgroup draws exactly one index past the
// end; the one that draws the last of those resets the counter for the next
// launch.  A tile's last phase, on one wave, runs beside the next tile's
// first, and the next item is drawn during the current one: no barrier and no
// memory round trip of its own stands between two tiles.  256 problems 2.35
// -> 2.19 ms, 64 x 4096 x 64 with refinement 16.36 -> 16.00 ms.
template <int W>
__global__ __launch_bounds__(W * kLanes) void rollout_batch_kernel(const ProblemDev *__restrict__ probs,
                                                                   const int2 *__restrict__ items, int n_items,
                                                                   uint32_t *next, const RobotDev *robot,
                                                                   const float *__restrict__ x0s,
                                                                   const float *__restrict__ goals)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];  // (holds 16-byte records)
    __shared__ int s_item[2][2];
    if ((int)blockIdx.x >= n_items) return;
    TileQueue queue{next, items, n_items, min((int)gridDim.x, n_items), s_item};
    const STORM_CONST_AS int32_t *it = uniform_ptr(reinterpret_cast<const int32_t *>(items)) + 2 * blockIdx.x;
    int p = it[0], tile = it[1];
    while (p >= 0) {
        const STORM_CONST_AS RobotDev *R = uniform_ptr(robot);
        asm volatile("" : "+s"(R));  // fields read in each tile, not kept over the loop
        ProblemRef P = uniform_ptr(probs)[p];
        const TileFirst first{P.step, P.mean, P.halton, P.N, P.H, P.n_halton, P.n_null};
        rollout_tile<W, false>(queue, P, *R, first, tile, x0s + (size_t)p * 3 * kDof, goals + (size_t)p * 12, nullptr,
                               StepOut{}, smem);
        queue.parity ^= 1;
        p = __builtin_amdgcn_readfirstlane(s_item[queue.parity][0]);
        tile = __builtin_amdgcn_readfirstlane(s_item[queue.parity][1]);
    }
}

// The rows, the capsules of S spheres and the culling records of n_obs
// obstacles (the 2 W collision partials sit over the 96 frame rows).
size_t rollout_lds_bytes(int S, int n_obs, bool task = false)
{
    return (size_t)(96 + kTerms + rollout_cen_rows(S) + (task ? 2 * kDof : 0)) * kLanes * sizeof(float) +
           (size_t)(8 * S + n_obs) * sizeof(float4);
}

}  // namespace

hipError_t set_rollout_lds_limit()
{
    const int plain = (int)rollout_lds_bytes(STORM_MAX_SPHERES, STORM_MAX_OBSTACLES);
    const int task = (int)rollout_lds_bytes(STORM_MAX_SPHERES, STORM_MAX_OBSTACLES, true);
    const void *fns[10] = {reinterpret_cast<const void *>(&rollout_kernel<16, false, false>),
                           reinterpret_cast<const void *>(&rollout_kernel<8, false, false>),
                           reinterpret_cast<const void *>(&rollout_kernel<16, false, true>),
                           reinterpret_cast<const void *>(&rollout_kernel<8, false, true>),
                           reinterpret_cast<const void *>(&rollout_batch_kernel<16>),
                           reinterpret_cast<const void *>(&rollout_batch_kernel<8>),
                           reinterpret_cast<const void *>(&rollout_kernel<16, true, false>),
                           reinterpret_cast<const void *>(&rollout_kernel<8, true, false>),
                           reinterpret_cast<const void *>(&rollout_kernel<16, true, true>),
                           reinterpret_cast<const void *>(&rollout_kernel<8, true, true>)};
    for (int k = 0; k < 10; ++k) {
        const hipError_t e =
            hipFuncSetAttribute(fns[k], hipFuncAttributeMaxDynamicSharedMemorySize, k < 6 ? plain : task);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_rollout_batch(const ProblemDev *probs, const int2 *items, int n_items, uint32_t *next,
                                const RobotDev *robot, int n_spheres, int max_obs, const float *x0s,
                                const float *goals, int waves, int grid, hipStream_t stream)
{
    const size_t lds = rollout_lds_bytes(n_spheres, max_obs);
    if (waves == 16) {
        hipLaunchKernelGGL(rollout_batch_kernel<16>, dim3((unsigned)grid), dim3(16 * kLanes), lds, stream, probs,
                           items, n_items, next, robot, x0s, goals);
    } else if (waves == 8) {
        hipLaunchKernelGGL(rollout_batch_kernel<8>, dim3((unsigned)grid), dim3(8 * kLanes), lds, stream, probs,
                           items, n_items, next, robot, x0s, goals);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_rollout(const ProblemDev &P, int n_spheres, const PlainDev *dev, const float *x0, const float *goal,
                          const float *noise, const StepOut &out, int waves, hipStream_t stream)
{
    // the task-space form only where it is asked for: the ball term, the
    // network's joint positions, or the flange velocity and acceleration
    const bool task = (P.cost_mask & STORM_COST_BALL) || P.selfnet || out.xd != nullptr || out.xdd != nullptr;
    const bool debug = noise != nullptr || out.u != nullptr || out.q != nullptr || out.v != nullptr ||
                       out.a != nullptr || out.c != nullptr || out.terms != nullptr || out.xd != nullptr ||
                       out.xdd != nullptr;
    const size_t lds = rollout_lds_bytes(n_spheres, P.n_sph_obs + P.n_box_obs, task);
    const dim3 grid((unsigned)P.n_tiles);
    if (waves != 16 && waves != 8) return hipErrorInvalidValue;
    auto kernel = waves == 16 ? (task ? (debug ? rollout_kernel<16, true, true> : rollout_kernel<16, true, false>)
                                      : (debug ? rollout_kernel<16, false, true> : rollout_kernel<16, false, false>))
                              : (task ? (debug ? rollout_kernel<8, true, true> : rollout_kernel<8, true, false>)
                                      : (debug ? rollout_kernel<8, false, true> : rollout_kernel<8, false, false>));
    hipLaunchKernelGGL(kernel, grid, dim3(waves * kLanes), lds, stream, dev, P.N, P.H, x0, goal, P.mean, P.step,
                       out.C, noise, out);
    return hipGetLastError();
}

}  // namespace storm
