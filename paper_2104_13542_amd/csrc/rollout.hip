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
//   C   waves 0..W-3  world centres of the body spheres, and the capsules
//                  that hold the anchor spheres, to LDS
//       wave W-2   manipulability (Eq. 12)
//       wave W-1   pose (Eq. 9)
//   D1  all waves  obstacles near each body and near pairs of sphere runs,
//                  by capsules
//   D2  all waves  environment (spheres x obstacles) split over waves, then
//                  self-collision (sphere pairs) as items taken from a queue
//   E   wave 4     weighted running cost (Eq. 15), horizon sum (Eq. 2) as a
//                  segmented DPP scan
// From the joint angles on, the points of a tile lie by step, then particle, so
// that a row of 16 lanes is a short piece of time: the capsules of phase C bound
// a sphere over such a row.  Obstacle and sphere records are staged in LDS (A0),
// every per-point LDS array is [row][lane] (conflict-free), and rows whose
// lifetimes do not overlap share space (at most 80 KB per workgroup with 52
// spheres and any scene, so that the looping and batched forms hold two
// workgroups per CU; rollout_boxes).
// Reductions run in a fixed order: results are bitwise reproducible.
//
// Three forms: a 16-wave workgroup per tile up to one tile per CU (bound by the
// latency of its phases), 8-wave workgroups that loop over the tiles of one
// larger problem, and the same over the tiles of a batch (both bound by VALU
// issue).  Against sphere balls, sixteen waves for every plain tile and a barrier
// between a batch's, over four scenes: 500 x 30 control call 17.5-19.5 -> 13.9-14.3
// us, 4096 x 64 236-269 -> 130-151, 65536 x 30 step 1530-1810 -> 755-815, a batch of
// 256 problems 2520-2630 -> 1820-1900.
#include <algorithm>

#include "kinematics.h"
#include "sampling.h"

namespace storm {
namespace {

// Rows of the sphere-centre block, which also holds the noise, sine/cosine
// and hinge rows of phases A0-B (8 + 14 + 21) before the centres exist.
__host__ __device__ constexpr int rollout_cen_rows(int S) { return 3 * S > 43 ? 3 * S : 43; }

// LDS of a tile apart from the cuboids' records: the rows, n_cap capsules, the
// balls of n_obs obstacles, and the lists of phase D1 (of n_items self-collision
// items, and of the obstacles near each body).
__host__ __device__ constexpr int rollout_base_bytes(int S, int n_cap, int n_obs, int n_items, bool task)
{
    return (96 + kTerms + rollout_cen_rows(S) + (task ? 2 * kDof : 0)) * kLanes * 4 + 8 * n_cap * 16 +
           n_obs * (16 + kFrames) + n_items * 8;
}

// The dense form (kDense), for scenes past the LDS of two 8-wave workgroups on a
// CU (160 KB, kStaticLds of each workgroup's static): capsules by their rank in
// cap_mask, and the records of the cuboids past the first rollout_boxes loaded in
// phase D1, over the frames, which are dead by then.  A form of its own, since
// both cost 1% where all fits, and such records read from memory instead 4%
// (65536 x 30 with 50 obstacles 760, 770 and 783 us).  64 problems of 512 x 30
// with 60 spheres and 60 cuboids, one workgroup per CU and two: 747 and 441 us;
// a control call of 4096 x 64 with them, by a 16-wave workgroup per tile: 139 and
// 109.
constexpr int kStaticLds = 1360;
constexpr int kTwoGroupsLds = 80 * 1024 - kStaticLds;
__host__ __device__ constexpr int rollout_boxes(int base_bytes, int n_box)
{
    const int room = (kTwoGroupsLds - base_bytes) / 64;
    return base_bytes > kTwoGroupsLds || room > n_box ? n_box : room;
}
constexpr int kLateRow = 32;
static_assert(kLateRow >= 3 * 8 && kLateRow * kLanes * 4 + STORM_MAX_OBSTACLES * 64 <= 96 * kLanes * 4,
              "the partials of 8 waves, then the cuboids' records, fit over the frame rows");

// Value of lane kLane of the caller's 16-lane row.
template <int kLane>
__device__ __forceinline__ float row_lane(float x)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x150 + kLane, 0xf, 0xf, true));  // row_newbcast
}

// Maximum of a non-negative float over the caller's 16-lane row, in every
// lane: IEEE bit patterns of non-negative floats order like unsigned
// integers, so it runs on the bits through DPP lane moves.
__device__ __forceinline__ float row_max_nonneg(float x)
{
    uint32_t b = __float_as_uint(x);
    b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0xb1, 0xf, 0xf, true));   // quad_perm [1, 0, 3, 2]
    b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0x4e, 0xf, 0xf, true));   // quad_perm [2, 3, 0, 1]
    b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0x141, 0xf, 0xf, true));  // row_half_mirror
    b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0x140, 0xf, 0xf, true));  // row_mirror
    return __uint_as_float(b);
}

// What every culling radius is widened by (m): it dwarfs the FP32 rounding of
// any distance that a cull or an exact test forms, so that no contact which an
// exact test would report is ever culled.
constexpr float kCullMargin = 1.0e-4f;

// The capsule that holds a sphere's centres cc over the caller's row of 16
// points, in every lane: the chord from the row's first centre a (a.xyz) to its
// last (a + b.xyz), and as radius (a.w) the largest distance of a centre to the
// chord's point at its own time (tau in [0, 1]; any point of the chord serves)
// plus r_s and a margin; b.w is 1 / |b|^2.  Where a row holds a centre that is
// not finite, a ball that meets everything.
__device__ __forceinline__ void row_capsule(const float cc[3], float tau, float rs, float4 &a, float4 &b)
{
    const float ax = row_lane<0>(cc[0]), ay = row_lane<0>(cc[1]), az = row_lane<0>(cc[2]);
    const float dx = cc[0] - ax, dy = cc[1] - ay, dz = cc[2] - az;
    const float bx = row_lane<15>(dx), by = row_lane<15>(dy), bz = row_lane<15>(dz);
    const float ex = fmaf(-tau, bx, dx), ey = fmaf(-tau, by, dy), ez = fmaf(-tau, bz, dz);
    const float rad = fast_sqrt(row_max_nonneg(fminf(fmaf(ex, ex, fmaf(ey, ey, ez * ez)), 1.0e30f)));
    a = make_float4(ax, ay, az, rad + (rs + kCullMargin));
    b = make_float4(bx, by, bz, __builtin_amdgcn_rcpf(fmaxf(fmaf(bx, bx, fmaf(by, by, bz * bz)), 1.0e-20f)));
    if (__builtin_amdgcn_ballot_w64(!(rad < 1.0e6f)) != 0) {
        const bool bad = !(rad < 1.0e6f);
        const float zero = fminf(fabsf(rad), 0.0f);  // (formed here, rarely)
        a = make_float4(bad ? zero : a.x, bad ? zero : a.y, bad ? zero : a.z, bad ? 1.0e15f : a.w);
        b = make_float4(bad ? zero : b.x, bad ? zero : b.y, bad ? zero : b.z, bad ? zero : b.w);
    }
}

// Whether the capsule (segment a.xyz + t b.xyz, t in [0, 1], radius `reach`
// already holding the obstacle's; b.w = 1 / |b.xyz|^2) meets the point o.
__device__ __forceinline__ bool capsule_hits(const float4 a, const float4 b, float reach, float ox, float oy, float oz)
{
    const float dx = ox - a.x, dy = oy - a.y, dz = oz - a.z;
    const float t = fminf(fmaxf(fmaf(dx, b.x, fmaf(dy, b.y, dz * b.z)) * b.w, 0.0f), 1.0f);
    const float ex = fmaf(-t, b.x, dx), ey = fmaf(-t, b.y, dy), ez = fmaf(-t, b.z, dz);
    return fmaf(ex, ex, fmaf(ey, ey, ez * ez)) < reach * fabsf(reach);
}

// What the start of a tile reads of the problem and the robot, fetched in one
// go: a scalar load wherever a field is used would put one memory round trip
// after another before the first work.
struct TileFirst {
    uint32_t *step;
    const float *mean;
    int32_t N, H, n_halton, n_null, n_sph_obs, n_box_obs, ppt, n_spheres, n_self_items;
    uint32_t cost_mask, seed_lo, seed_hi, comb, cov_step;
    const float *tables, *halton;
    const float4 *obs_bound;
    const float *box_obs;
    float *sigma2;
    const float4 *sph_local;
    const int32_t *sph_body;
    const float *body_bound;
    const int32_t *self_items;
    uint64_t cap_mask;
};
// (step, mean, N and H: known to the plain kernel from its arguments)
__device__ __forceinline__ TileFirst fetch_first(ProblemRef P, RobotRef R, uint32_t *step, const float *mean,
                                                 int32_t N, int32_t H)
{
    TileFirst F{step,         mean,          N,           H,           P.n_halton,  P.n_null,     P.n_sph_obs,
                P.n_box_obs,  P.ppt,         R.n_spheres, R.n_self_items, P.cost_mask, P.seed_lo, P.seed_hi,
                P.comb,       P.cov_step,    P.tables,    P.halton,    P.obs_bound, P.box_obs,    P.sigma2,
                R.sph_local,  R.sph_body,    R.body_bound, R.self_items, R.cap_mask};
    asm volatile("" : "+s"(F.n_halton), "+s"(F.n_null), "+s"(F.n_sph_obs), "+s"(F.n_box_obs), "+s"(F.ppt),
                 "+s"(F.n_spheres), "+s"(F.n_self_items), "+s"(F.cost_mask), "+s"(F.seed_lo), "+s"(F.seed_hi),
                 "+s"(F.comb), "+s"(F.cov_step), "+s"(F.tables), "+s"(F.halton), "+s"(F.obs_bound), "+s"(F.box_obs),
                 "+s"(F.sigma2), "+s"(F.sph_local), "+s"(F.sph_body), "+s"(F.body_bound), "+s"(F.self_items), "+s"(F.cap_mask));
    return F;
}

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
struct TileStride {  // the plain form with many tiles: every gridDim-th
    int parity = 0;
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

// Whether two capsules of the same row of points may meet: the difference of
// their axes runs from a1 - a2 along b1 - b2 (both at the same time at every
// point of the row), and the spheres come within `reach` of each other at no
// point where that segment stays farther from the origin.
__device__ __forceinline__ bool capsules_meet(const float4 a1, const float4 b1, const float4 a2, const float4 b2,
                                              float reach)
{
    const float dx = a1.x - a2.x, dy = a1.y - a2.y, dz = a1.z - a2.z;
    const float bx = b1.x - b2.x, by = b1.y - b2.y, bz = b1.z - b2.z;
    const float len2 = fmaf(bx, bx, fmaf(by, by, bz * bz));
    const float dot = fmaf(dx, bx, fmaf(dy, by, dz * bz));
    const float t = fminf(fmaxf(-dot * __builtin_amdgcn_rcpf(fmaxf(len2, 1.0e-20f)), 0.0f), 1.0f);
    const float ex = fmaf(t, bx, dx), ey = fmaf(t, by, dy), ez = fmaf(t, bz, dz);
    return fmaf(ex, ex, fmaf(ey, ey, ez * ez)) < reach * reach;
}

// One 64-lane tile of one problem, executed by the W waves of the calling
// workgroup; smem is the workgroup's dynamic LDS (rollout_lds).
// kSums: the environment term's partial sums, over spheres s, s + kSums, ...
// (W, or 2 W: the bits of a workgroup of twice the waves).
// kDense: with the scene packed (rollout_boxes).
// kTask: the task-space form, which adds the flange velocity and
// acceleration outputs (Eq. 8), the ball-on-tray term and the joint
// positions the learned self-collision network reads.
// The fields of the descriptors are scalar loads where they are used (held as
// copies they overflowed the SGPRs into lanes of VGPRs, 180 lane moves per
// wave and tile).
template <int W, bool kTask, int kSums, bool kDense, class Queue>
__device__ __forceinline__ void rollout_tile(Queue &queue, ProblemRef P, RobotRef R, const TileFirst &first, const int tile,
                                             const float *__restrict__ x0, const float *__restrict__ goal,
                                             const float *__restrict__ noise, const StepOut &out, float *smem)
{
    // LDS rows of 64 floats, overlaid where their lifetimes do not meet
    // (rollout_lds), so that two workgroups of the batched form fit on
    // one CU:
    //   frames [96]              B - C,  then the collision partials [2W]  D2 - E
    //   terms [kTerms]           B - E
    //   centres [3S]             C - D2;  before them noise [8] A0 - A1,
    //                            sin/cos [14] and hinges [21] A1 - B
    //   velocities, accelerations [14]  A1 - C (task-space form only)
    // then the capsules of the spheres [S][4 rows][8] (C - D2; kDense: of the
    // anchors, by rank), the records of the obstacles (A0 - D2) and the lists of
    // phase D1 (D1 - D2).  kDense: the other cuboids' records lie over the frames
    // from row kLateRow on (D1 - D2).
    const int S = first.n_spheres;
    float *s_fr = smem;                        // [8 frames][12][64]: R row-major, p
    float *s_penv = s_fr;                      // [kSums][64] (over the frames, after phase C)
    float *s_pself = s_penv + kSums * kLanes;  // [W][64]
    float *s_terms = s_fr + 96 * kLanes;       // [kTerms][64]
    float *s_cen = s_terms + kTerms * kLanes;  // [S][3][64]
    float *s_eps = s_cen;                      // [8][64] (before the centres)
    float *s_sc = s_eps + 8 * kLanes;          // [7][2][64]: sin q_j, cos q_j
    float *s_lim = s_sc + 14 * kLanes;         // [3][7][64]: squared joint, velocity, stop hinges per joint
    float *s_v = s_cen + rollout_cen_rows(S) * kLanes;  // [7][64] (task-space form only)
    float *s_acc = s_v + kDof * kLanes;                  // [7][64]
    float4 *s_cap = reinterpret_cast<float4 *>(s_v + (kTask ? 2 * kDof * kLanes : 0));  // [S, or anchors][4][2]
    const int n_cap = kDense ? __builtin_popcountll(first.cap_mask) : S;
    auto cap_index = [&](int s) __attribute__((always_inline)) {  // of an anchor
        return kDense ? __builtin_popcountll(first.cap_mask & ((1ull << s) - 1ull)) : s;
    };
    const uint32_t mask = first.cost_mask;
    const int nobs = (mask & STORM_COST_ENV) && S > 0 ? first.n_sph_obs + first.n_box_obs : 0;
    const int n_items = (mask & STORM_COST_SELF) ? first.n_self_items : 0;
    float4 *s_bound = s_cap + 8 * n_cap;         // [obstacles] centre, radius (of a cuboid: to its corners)
    float4 *s_box = s_bound + nobs;              // [n_box][4] records of the first cuboids
    const int n_box = nobs == 0 ? 0
                      : kDense  ? rollout_boxes(rollout_base_bytes(S, n_cap, nobs, n_items, kTask), first.n_box_obs)
                                : first.n_box_obs;
    int2 *s_self = reinterpret_cast<int2 *>(s_box + 4 * n_box);  // [items] those that stay: runs and anchors, and the
                                                                 // runs' joint reach
    uint8_t *s_near = reinterpret_cast<uint8_t *>(s_self + n_items);  // [8][obstacles] obstacles near each body
    const float4 *s_late = reinterpret_cast<float4 *>(s_fr + kLateRow * kLanes) - 4 * n_box;  // [cuboids][4] from n_box on

    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = first.N, H = first.H, ppt = first.ppt;
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
    const global_ptr<const float> tab = as_global(first.tables);

    // Per-joint inputs of phase A1, loaded up front so that their latency
    // overlaps the noise generation (vector loads throughout, so that the
    // first barrier waits for none of them: the state and the policy come
    // fresh from the previous kernels).
    float mu_j = 0.0f, sig2_j = 0.0f, dt_h = 0.0f, vs_h = 0.0f, q0_j = 0.0f, v0_j = 0.0f;
    if (wave < kDof) {
        if (live) mu_j = as_global(first.mean)[h * kDof + wave];
        sig2_j = first.cov_step ? as_global(first.sigma2)[h * kDof + wave] : vector_load_f32(first.sigma2 + wave);
        dt_h = tab[kTabDt + h];
        vs_h = tab[kTabVstop + h];
        q0_j = vector_load_f32(x0 + wave);
        v0_j = vector_load_f32(x0 + kDof + wave);
    }
    // The records that the waves that draw no noise stage in LDS, the first of
    // each thread: obstacles (their balls, then the cuboids), body spheres with
    // their frames.  Loads from here on are unconditional, at an index that
    // exists, and all in flight before the first is waited for.
    const int n_obs_rec = nobs + 4 * n_box;
    const int n_rec = n_obs_rec + ((mask & (STORM_COST_SELF | STORM_COST_ENV)) ? S : 0);
    const global_ptr<const float4> g_bound = as_global(first.obs_bound), g_sph = as_global(first.sph_local),
                                   g_box = as_global(reinterpret_cast<const float4 *>(first.box_obs));
    auto record = [=](int k) __attribute__((always_inline)) {
        global_ptr<const float4> r = g_sph + max(min(k - n_obs_rec, S - 1), 0);
        if (k < n_obs_rec) r = g_box + (k - nobs);
        if (k < nobs) r = g_bound + k;
        return r;
    };
    const int k_first = (int)threadIdx.x - 4 * kLanes;
    float4 rec = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    int rec_frame = 0;
    if (wave >= 4) {
        rec = load_float4(record(k_first));
        rec_frame = as_global(first.sph_body)[max(min(k_first - n_obs_rec, S - 1), 0)];
    }
    // phase D1's bound of the body that this lane tests, and its first
    // self-collision item (last wave first)
    const int body8 = lane & (kFrames - 1);
    const float anchor = as_global(first.body_bound)[2 * body8], widen = as_global(first.body_bound)[2 * body8 + 1];
    const int g_first = 16 * (W - 1 - wave) + (lane & 15);
    const float4 item_bits = load_float4(as_global(reinterpret_cast<const float4 *>(first.self_items)) +
                                         max(min(g_first, n_items - 1), 0));
    int item[4] = {__float_as_int(item_bits.x), __float_as_int(item_bits.y), __float_as_int(item_bits.z),
                   __float_as_int(item_bits.w)};
    // the goal and the cost weights that phases C and E read, staged by the
    // last wave
    __shared__ float s_par2[2][kParCount];  // (by parity: the costs of a tile are summed during the next one's noise)
    float *s_par = s_par2[queue.parity];
    __shared__ int s_self_n, s_self_next;  // self-collision items that stay (phase D1), and the queue's head (D2)
    __shared__ float4 s_sph[STORM_MAX_SPHERES];  // body-frame centre, radius
    __shared__ uint8_t s_body[STORM_MAX_SPHERES];  // frame
    __shared__ int s_near_n[kFrames];  // obstacles near each body (phase D1)
    if (wave == W - 1 && lane == kParCount) s_self_n = s_self_next = 0;
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
        if (live) standard_noise2(first, first.seed_lo, first.seed_hi, noise, k, half, i, h, counter, e);
        s_eps[j0 * kLanes + lane] = e[0];
        s_eps[(j0 + 1) * kLanes + lane] = e[1];
        // (the counter block: step, status, last step)
        if (tile == 0 && threadIdx.x == 0) as_global(first.step)[2] = counter;
    } else {
        float g = 0.0f, w = 0.0f;
        if (wave == W - 1) {
            g = goal[lane < 12 ? lane : 0];
            w = tab[kTabPar + (lane < 12 ? 0 : min(lane - 12, kParCount - 13))];
        }
        for (int k = k_first; k < n_rec; k += (W - 4) * kLanes) {
            if (k != k_first) {
                rec = load_float4(record(k));
                rec_frame = as_global(first.sph_body)[max(min(k - n_obs_rec, S - 1), 0)];
            }
            if (k < n_obs_rec) {
                s_bound[k] = rec;
            } else {
                s_sph[k - n_obs_rec] = rec;
                s_body[k - n_obs_rec] = (uint8_t)rec_frame;
            }
        }
        if (wave == W - 1 && lane < kParCount) s_par[lane] = lane < 12 ? g : w;
    }
    __syncthreads();

    // ---- A1: controls and the triple integrator (Eq. 7) ---------------------
    if (wave < kDof) {
        const int j = wave;
        float e = s_eps[j * kLanes + lane];
        // the comb filter on the sampled Gaussian particles' noise (Sec. 3.3)
        const bool comb = first.comb && noise == nullptr && live && i >= first.n_halton;
        if (__builtin_amdgcn_ballot_w64(comb) != 0) {
            const float f = comb_noise(s_eps + j * kLanes, lane, h, H, tab);
            if (comb) e = f;
        }
        float u = 0.0f;
        if (live) u = fmaf(sqrtf(sig2_j), e, mu_j);
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
    // where in its row's span of steps this lane lies, in [0, 1]
    const float step_l = floorf(((float)src + 0.5f) * __builtin_amdgcn_rcpf((float)ppt));
    const float step0 = row_lane<0>(step_l);
    const float tau =
        fminf((step_l - step0) * __builtin_amdgcn_rcpf(fmaxf(row_lane<15>(step_l) - step0, 1.0f)), 1.0f);
    if (wave < WC) {
        const int s0 = wave * S / WC, s1 = (wave + 1) * S / WC;
        if ((mask & (STORM_COST_SELF | STORM_COST_ENV)) && s0 < s1) {
            // a contiguous run of spheres per wave (sorted by body): the
            // frame of a body is read from LDS once per run
            // (the next sphere's record is read one ahead)
            float F[12];
            int fb = __builtin_amdgcn_readfirstlane((int)s_body[s0]);
            int rank = kDense ? cap_index(s0) : 0;
            float4 next = s_sph[s0];
#pragma unroll
            for (int c = 0; c < 12; ++c) F[c] = s_fr[(fb * 12 + c) * kLanes + lane];
            for (int s = s0; s < s1; ++s) {
                const float4 loc = next;
                const int after = min(s + 1, s1 - 1), b_next = s_body[after];
                next = s_sph[after];
                float cc[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    cc[c] = fmaf(F[c * 3 + 0], loc.x, fmaf(F[c * 3 + 1], loc.y, fmaf(F[c * 3 + 2], loc.z, F[9 + c])));
                    s_cen[(s * 3 + c) * kLanes + lane] = cc[c];
                }
                // The capsules of the anchors, which phase D1 tests.  The
                // others (about 30 of 52) are formed in D2, only where an
                // obstacle is near their body: this phase is bound by issue
                // (batch of 256 1937 -> 1840 us, 65536 x 30 748 -> 717 us,
                // 4096 x 64 127 -> 123 us, 64 x 4096 x 64 12.84 -> 12.55 ms).
                if (first.cap_mask >> s & 1) {
                    float4 a, b;
                    row_capsule(cc, tau, loc.w, a, b);
                    float4 *cap = s_cap + ((kDense ? rank++ : s) * 4 + (lane >> 4)) * 2;
                    if ((lane & 15) == 0) {
                        cap[0] = a;
                        cap[1] = b;
                    }
                }
                const int b = __builtin_amdgcn_readfirstlane(b_next);
                if (b != fb) {
#pragma unroll
                    for (int c = 0; c < 12; ++c) F[c] = s_fr[(b * 12 + c) * kLanes + lane];
                    fb = b;
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

    // the cuboids' records that had no room before (D2 reads them)
    if (kDense && nobs > 0) {
        float4 *late = reinterpret_cast<float4 *>(s_fr + kLateRow * kLanes);
        for (int k = threadIdx.x; k < 4 * (first.n_box_obs - n_box); k += W * kLanes)
            late[k] = load_float4(g_box + 4 * n_box + k);
    }

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
    if (2 * wave < nobs) {
        const int body = body8, row = (lane >> 3) & 3, half = lane >> 5;
        const float4 *cap = s_cap + (cap_index(__float_as_int(anchor)) * 4 + row) * 2;
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
                s_near[body * nobs + k] = (uint8_t)o;
            }
        }
    }
    // Self-collision items (pairs of runs of up to four spheres of a body) by
    // the capsules of the runs' anchor spheres, widened to hold the runs: a
    // lane tests one row of one item.
    if (mask & STORM_COST_SELF) {
        const global_ptr<const int32_t> items = as_global(first.self_items);
        const int row = lane >> 4;
        // (16 items a wave, from the last wave down: the obstacles of the
        // loop above start at the first)
        for (int g0 = 16 * (W - 1 - wave); g0 < n_items; g0 += 16 * W) {
            const int g = g0 + (lane & 15);
            if (g != g_first && g < n_items)
#pragma unroll
                for (int k = 0; k < 4; ++k) item[k] = items[4 * g + k];
            const int anchors = item[1];
            const float4 *ct = s_cap + (cap_index(anchors & 63) * 4 + row) * 2,
                         *cs = s_cap + (cap_index(anchors >> 6) * 4 + row) * 2;
            uint64_t meet = __builtin_amdgcn_ballot_w64(
                g < n_items &&
                capsules_meet(ct[0], ct[1], cs[0], cs[1], (ct[0].w + cs[0].w) + __int_as_float(item[3])));
            if (meet == 0) continue;
            meet |= meet >> 32;  // the four rows
            meet |= meet >> 16;
            if (row == 0 && ((meet >> lane) & 1ull)) {
                const int k = atomicAdd(&s_self_n, 1);
                s_self[k] = make_int2(item[0] | anchors << 16, item[2]);
            }
        }
    }
    __syncthreads();

    // ---- D2: collision terms --------------------------------------------------
    // Environment (spheres round robin over the waves), then self-collision
    // (items from a queue).
    float env[kSums / W], selfpen = 0.0f;
#pragma unroll
    for (int m = 0; m < kSums / W; ++m) env[m] = 0.0f;
    if (nobs > 0) {
        const int nso = first.n_sph_obs;
        // lane k holds the body of this wave's k-th sphere and how many
        // obstacles are near it
        const int s_mine = wave + lane * W;
        const int body_l = s_mine < S ? (int)s_body[s_mine] : 0;
        const int near_l = s_mine < S ? s_near_n[body_l] : 0;
        for (uint64_t left = __builtin_amdgcn_ballot_w64(near_l > 0); left != 0; left &= left - 1) {
            const int k_s = (int)__builtin_ctzll(left), s = wave + k_s * W;
            const int n_near = __builtin_amdgcn_readlane(near_l, k_s);
            const uint8_t *near = s_near + __builtin_amdgcn_readlane(body_l, k_s) * nobs;
            const float x = s_cen[(s * 3 + 0) * kLanes + lane];
            const float y = s_cen[(s * 3 + 1) * kLanes + lane];
            const float z = s_cen[(s * 3 + 2) * kLanes + lane];
            const float rs = s_sph[s].w;
            float4 ca, cb;
            if (first.cap_mask >> s & 1) {
                const float4 *cap = s_cap + (cap_index(s) * 4 + (lane >> 4)) * 2;
                ca = cap[0];
                cb = cap[1];
            } else {
                const float cc[3] = {x, y, z};
                row_capsule(cc, tau, rs, ca, cb);
            }
            float best = 0.0f;
            for (int k0 = 0; k0 < n_near; k0 += 16) {
                // the sphere's four capsules against 16 of its body's
                // obstacles at a time
                const int k = k0 + (lane & 15);
                const int ob_l = near[min(k, n_near - 1)];
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
                        // the squared contact distance; where a lane touches,
                        // the penetration (r_s + r_o) - |x - c| at every lane
                        // (at or below zero where a lane does not touch)
                        const float4 so = s_bound[o];
                        const float dx = x - so.x, dy = y - so.y, dz = z - so.z;
                        const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                        const float rc = rs + so.w;
                        if (__builtin_amdgcn_ballot_w64(d2 < rc * rc) != 0) best = fmaxf(best, rc - fast_sqrt(d2));
                    } else {
                        const float4 *bb = (!kDense || o - nso < n_box ? s_box : s_late) + (o - nso) * 4;
                        const float4 b0 = bb[0], b1 = bb[1], b2 = bb[2], b3 = bb[3];
                        const float lx = fmaf(b0.x, x, fmaf(b0.y, y, fmaf(b0.z, z, b2.y)));
                        const float ly = fmaf(b0.w, x, fmaf(b1.x, y, fmaf(b1.y, z, b2.z)));
                        const float lz = fmaf(b1.z, x, fmaf(b1.w, y, fmaf(b2.x, z, b2.w)));
                        // excess per axis, clamped to [0, 1 m]: one instruction
                        // with the clamp modifier; body spheres are below 1 m, so
                        // clamping cannot turn a miss into a hit and leaves every
                        // axis of a hit exact
                        const float ox = fminf(fmaxf(fabsf(lx) - b3.x, 0.0f), 1.0f);
                        const float oy = fminf(fmaxf(fabsf(ly) - b3.y, 0.0f), 1.0f);
                        const float oz = fminf(fmaxf(fabsf(lz) - b3.z, 0.0f), 1.0f);
                        const float out2 = fmaf(ox, ox, fmaf(oy, oy, oz * oz));
                        const bool hit = out2 < rs * rs;
                        if (__builtin_amdgcn_ballot_w64(hit) != 0) {
                            const float qin =
                                fminf(fmaxf(fabsf(lx) - b3.x, fmaxf(fabsf(ly) - b3.y, fabsf(lz) - b3.z)), 0.0f);
                            const float pen = rs - (fast_sqrt(out2) + qin);
                            if (hit) best = fmaxf(best, pen);
                        }
                    }
                }
            }
            if (W == kSums || (k_s & 1) == 0)
                env[0] += best;
            else
                env[kSums / W - 1] += best;
        }
    }
    if (mask & STORM_COST_SELF) {
        // The items that stayed, from a queue in LDS (their order does not
        // matter to a maximum), so that waves done early with the
        // environment take more; the next one is drawn ahead.  An item whose
        // runs' balls (about their anchors) meet at some point gets the
        // squared distances of all its pairs; where the least of them is
        // within the largest contact distance at some point, the
        // penetrations (r_s + r_t) - |c_s - c_t| of all, at every point
        // (negative where the spheres are apart).  Short runs repeat their
        // last sphere.  Everything of an item is in flight at once: the
        // plain form has about one item per wave here, and its time is the
        // chain of LDS round trips.
        const int n_near_items = __builtin_amdgcn_readfirstlane(s_self_n);
        auto draw = [&]() __attribute__((always_inline)) {
            // (an address the compiler takes for divergent: it would sum a
            // uniform one's additions over the wave first, and wait there)
            __attribute__((address_space(3))) int *head = (__attribute__((address_space(3))) int *)&s_self_next;
            asm volatile("" : "+v"(head));
            int g = 0;
            if (lane == 0) g = __hip_atomic_fetch_add(head, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            return g;
        };
        int drawn = draw();
        for (;;) {
            const int g = __builtin_amdgcn_readfirstlane(drawn);
            if (g >= n_near_items) break;
            drawn = draw();
            const int2 rec = s_self[g];
            const int code = __builtin_amdgcn_readfirstlane(rec.x);
            const float *at = s_cen + (code >> 16 & 63) * 3 * kLanes + lane;
            const float *as = s_cen + (code >> 22) * 3 * kLanes + lane;
            const float ax = at[0] - as[0], ay = at[kLanes] - as[kLanes], az = at[2 * kLanes] - as[2 * kLanes];
            const float reach = __int_as_float(rec.y);
            if (__builtin_amdgcn_ballot_w64(fmaf(ax, ax, fmaf(ay, ay, az * az)) < reach * reach) == 0) continue;
            const int t_first = code & 63, t_last = code >> 6 & 3, s_first = code >> 8 & 63, s_last = code >> 14 & 3;
            float ct[4][3], cs[4][3], rt[4], rs[4], d2[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int t = t_first + min(k, t_last), u = s_first + min(k, s_last);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    ct[k][c] = s_cen[(t * 3 + c) * kLanes + lane];
                    cs[k][c] = s_cen[(u * 3 + c) * kLanes + lane];
                }
                rt[k] = s_sph[t].w;
                rs[k] = s_sph[u].w;
            }
            float least = 3.0e38f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float dx = cs[u][0] - ct[k][0], dy = cs[u][1] - ct[k][1], dz = cs[u][2] - ct[k][2];
                    d2[k][u] = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                    least = fminf(least, d2[k][u]);
                }
            const float r_max = fmaxf(fmaxf(rt[0], rt[1]), fmaxf(rt[2], rt[3])) +
                                fmaxf(fmaxf(rs[0], rs[1]), fmaxf(rs[2], rs[3]));
            // (an equal or smaller penetration than 0 changes nothing, so the
            // rounding of either side's square does not matter)
            if (__builtin_amdgcn_ballot_w64(least < r_max * r_max * 1.000001f) == 0) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int u = 0; u < 4; ++u) selfpen = fmaxf(selfpen, (rs[u] + rt[k]) - fast_sqrt(d2[k][u]));
        }
    }
    static_assert(kSums == W || kSums == 2 * W, "one or two sums a wave");
#pragma unroll
    for (int m = 0; m < kSums / W; ++m) s_penv[(wave + m * W) * kLanes + lane] = env[m];
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
            for (int w = 0; w < kSums; ++w) t[7] += s_penv[w * kLanes + pos];
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
    const TileFirst first = fetch_first(D.P, D.R, step, mean, N, H);
    NoQueue none;
    rollout_tile<W, kTask, W, false>(none, D.P, D.R, first, blockIdx.x, x0, goal, kDebug ? noise : nullptr, o, smem);
}

// Persistent form for one problem with more tiles than compute units: two
// workgroups of 8 waves share a CU, so that one's barriers and serial phases
// are covered by the other, and each takes every gridDim-th tile, the last
// phase of a tile beside the first of the next.  (No queue: tiles of one
// problem differ little, and a counter would be one more state that two
// streams could share.)  Same bits as one tile per workgroup.
template <int W, bool kDense>
__global__ __launch_bounds__(W * kLanes) __attribute__((amdgpu_waves_per_eu(4))) void rollout_loop_kernel(
    const PlainDev *dev, const float *__restrict__ x0, const float *__restrict__ goal, float *C_out, int32_t n_tiles)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];  // (holds 16-byte records)
    StepOut o{};
    o.C = C_out;
    TileStride stride;
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const STORM_CONST_AS PlainDev *D = uniform_ptr(dev);
        asm volatile("" : "+s"(D));  // fields read in each tile, not kept over the loop
        const TileFirst first = fetch_first(D->P, D->R, D->P.step, D->P.mean, D->P.N, D->P.H);
        rollout_tile<W, false, 2 * W, kDense>(stride, D->P, D->R, first, tile, x0, goal, nullptr, o, smem);
        stride.parity ^= 1;
    }
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
// (Four waves per SIMD: two workgroups of 8 waves share a CU.)
template <int W, bool kDense>
__global__ __launch_bounds__(W * kLanes) __attribute__((amdgpu_waves_per_eu(4))) void rollout_batch_kernel(const ProblemDev *__restrict__ probs,
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
        const TileFirst first = fetch_first(P, *R, P.step, P.mean, P.N, P.H);
        rollout_tile<W, false, W, kDense>(queue, P, *R, first, tile, x0s + (size_t)p * 3 * kDof, goals + (size_t)p * 12, nullptr,
                               StepOut{}, smem);
        queue.parity ^= 1;
        p = __builtin_amdgcn_readfirstlane(s_item[queue.parity][0]);
        tile = __builtin_amdgcn_readfirstlane(s_item[queue.parity][1]);
    }
}

// What a problem's tiles need in workgroups of `waves` waves.
RolloutLds rollout_lds(const ProblemDev &P, const RobotDev &R, int waves, bool task)
{
    const bool env = (P.cost_mask & STORM_COST_ENV) && R.n_spheres > 0;
    const int n_obs = env ? P.n_sph_obs + P.n_box_obs : 0, n_box = env ? P.n_box_obs : 0;
    const int n_items = P.cost_mask & STORM_COST_SELF ? R.n_self_items : 0;
    const int all = rollout_base_bytes(R.n_spheres, R.n_spheres, n_obs, n_items, task) + 64 * n_box;
    const int base = rollout_base_bytes(R.n_spheres, __builtin_popcountll(R.cap_mask), n_obs, n_items, task);
    if (waves > 8 || all <= kTwoGroupsLds || base > kTwoGroupsLds) return RolloutLds{(size_t)all, false};
    return RolloutLds{(size_t)(base + 64 * rollout_boxes(base, n_box)), true};
}

}  // namespace

hipError_t set_rollout_lds_limit()
{
    constexpr int boxes = 64 * STORM_MAX_OBSTACLES;
    const int items = kMaxSelfItems;
    const int plain = rollout_base_bytes(STORM_MAX_SPHERES, STORM_MAX_SPHERES, STORM_MAX_OBSTACLES, items, false) + boxes;
    const int task = rollout_base_bytes(STORM_MAX_SPHERES, STORM_MAX_SPHERES, STORM_MAX_OBSTACLES, items, true) + boxes;
    const void *fns[] = {reinterpret_cast<const void *>(&rollout_kernel<16, false, false>),
                         reinterpret_cast<const void *>(&rollout_kernel<16, false, true>),
                         reinterpret_cast<const void *>(&rollout_loop_kernel<8, false>),
                         reinterpret_cast<const void *>(&rollout_loop_kernel<8, true>),
                         reinterpret_cast<const void *>(&rollout_batch_kernel<16, false>),
                         reinterpret_cast<const void *>(&rollout_batch_kernel<8, false>),
                         reinterpret_cast<const void *>(&rollout_batch_kernel<8, true>),
                         reinterpret_cast<const void *>(&rollout_kernel<16, true, false>),
                         reinterpret_cast<const void *>(&rollout_kernel<16, true, true>)};
    for (int k = 0; k < 9; ++k) {
        const hipError_t e =
            hipFuncSetAttribute(fns[k], hipFuncAttributeMaxDynamicSharedMemorySize, k < 7 ? plain : task);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

RolloutLds rollout_batch_lds(const ProblemDev &P, const RobotDev &R, int waves) { return rollout_lds(P, R, waves, false); }

hipError_t launch_rollout_batch(const ProblemDev *probs, const int2 *items, int n_items, uint32_t *next,
                                const RobotDev *robot, const RolloutLds &lds, const float *x0s, const float *goals, int waves,
                                int grid, hipStream_t stream)
{
    if (waves == 16) {
        hipLaunchKernelGGL((rollout_batch_kernel<16, false>), dim3((unsigned)grid), dim3(16 * kLanes), lds.bytes, stream, probs,
                           items, n_items, next, robot, x0s, goals);
    } else if (waves == 8) {
        hipLaunchKernelGGL((lds.dense ? rollout_batch_kernel<8, true> : rollout_batch_kernel<8, false>),
                           dim3((unsigned)grid), dim3(8 * kLanes), lds.bytes, stream, probs, items, n_items, next, robot, x0s, goals);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// From one tile more than there are compute units, and where two workgroups'
// LDS (with their static part) fits a CU, the looping form; up to that, a tile
// has a CU to itself and 16 waves are the shorter path.  Control calls, a
// 16-wave workgroup per tile and looping: 200 x 64 (a tile each) 12.5 and 13.8
// us, 257 x 64 17.8 and 15.8, 512 x 64 19.5 and 16.7, 640 x 64 28.5 and 25.5,
// 2048 x 64 54.9 and 45.0, 65536 x 30 644 and 501.
constexpr int kLoopGroups = 512, kLoopTiles = 257;

hipError_t launch_rollout(const ProblemDev &P, const RobotDev &R, const PlainDev *dev, const float *x0, const float *goal,
                          const float *noise, const StepOut &out, hipStream_t stream)
{
    // the task-space form only where it is asked for: the ball term, the
    // network's joint positions, or the flange velocity and acceleration
    const bool task = (P.cost_mask & STORM_COST_BALL) || P.selfnet || out.xd != nullptr || out.xdd != nullptr;
    const bool debug = noise != nullptr || out.u != nullptr || out.q != nullptr || out.v != nullptr ||
                       out.a != nullptr || out.c != nullptr || out.terms != nullptr || out.xd != nullptr ||
                       out.xdd != nullptr;
    const RolloutLds loop = rollout_lds(P, R, 8, false);
    if (!task && !debug && P.n_tiles >= kLoopTiles && loop.bytes <= kTwoGroupsLds) {
        hipLaunchKernelGGL((loop.dense ? rollout_loop_kernel<8, true> : rollout_loop_kernel<8, false>), dim3(kLoopGroups),
                           dim3(8 * kLanes), loop.bytes, stream, dev, x0, goal, out.C, P.n_tiles);
        return hipGetLastError();
    }
    const size_t lds = rollout_lds(P, R, 16, task).bytes;
    auto kernel = task ? (debug ? rollout_kernel<16, true, true> : rollout_kernel<16, true, false>)
                       : (debug ? rollout_kernel<16, false, true> : rollout_kernel<16, false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)P.n_tiles), dim3(16 * kLanes), lds, stream, dev, P.N, P.H, x0, goal,
                       P.mean, P.step, out.C, noise, out);
    return hipGetLastError();
}

}  // namespace storm
