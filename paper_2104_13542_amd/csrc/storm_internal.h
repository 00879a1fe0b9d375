// Internal definitions of the HIP library: device-side problem descriptors,
// table offsets and the kernel launchers shared by the translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "storm.h"

namespace storm {

constexpr int kDof = STORM_DOF;
constexpr int kFrames = STORM_NFRAMES;
constexpr int kTerms = STORM_NTERMS;
constexpr int kLanes = 64;  // CDNA wavefront width
// waves at the end of a rollout workgroup that evaluate the pose and
// manipulability terms while the others place the body spheres
constexpr int kPoseWaves = 2;
constexpr int kMaxH = STORM_MAX_HORIZON;
constexpr int kMaxSelfItems = 276;  // pairs of at most 24 groups of one body's spheres each
constexpr int kAdjChunks = 512;  // adjoint workgroups (tile chunks) per problem, at most
constexpr int kAdjWaves = 4;     // wavefronts of an adjoint workgroup, one tile each at a time

// Up to this many tiles, the most that have a partial each, the adjoint splits
// each tile over a workgroup: the latency of a tile is then all there is.  One
// gradient, split and a tile per wavefront, us: 513 tiles of 30 steps 9.7 and
// 11.0, 640 11.0 and 11.0, 768 11.1 and 11.0 (of 16 steps 10.3 and 11.3, of 64
// 11.7 and 11.1), and past three workgroups per CU 900 13.4 and 11.0, 1024 13.5
// and 11.0 (512, split, 9.2).
constexpr int kSplitTiles = 512;

// The adjoint's partials: per tile up to kSplitTiles; then per chunk, a tile per
// wavefront while there are chunks; and past that in twice the runs, so that a
// plain launch of twice the wavefronts fills the chip (four per SIMD).
constexpr int adjoint_chunks(int n_tiles)
{
    const int n = n_tiles <= kSplitTiles ? n_tiles : (n_tiles + kAdjWaves - 1) / kAdjWaves;
    return n < kAdjChunks ? n : kAdjChunks;
}
constexpr int kAdjRuns = 2 * kAdjWaves;
__host__ __device__ constexpr int adjoint_runs(int n_tiles)
{
    return n_tiles > kAdjWaves * kAdjChunks ? kAdjRuns : kAdjWaves;
}

// Offsets (in floats) inside the per-problem table block built at init.
constexpr int kTabDt = 0;           // dt[H]
constexpr int kTabVstop = 64;       // stop-cost velocity limit per step [H]
constexpr int kTabHw = 128;         // horizon weight gamma^h (terminal scaled) [H]
constexpr int kTabJlo = 192;        // band-shrunk joint position limits [7]
constexpr int kTabJhi = 200;
constexpr int kTabVlo = 208;        // band-shrunk joint velocity limits [7]
constexpr int kTabVhi = 216;
constexpr int kTabComb = 224;        // comb filter response g_k (e'_h = sum_k g_k e_{h-k}) [H]
constexpr int kTabSig0 = 288;        // sigma_init^2 [7], appended by a per-step covariance shift
constexpr int kTabPar = 295;         // cost weights in the order of the rollout's LDS copy [14]
constexpr int kTabSize = 309;

// Learned self-collision network (Eq. 13): layer widths, the packed FP16
// weight fragments (offsets in halves: per column block, k-step and lane, 4
// halves per lane for layer 1's k-steps of 16, 8 for layers 2 and 3's
// k-steps of 32) and the FP32 block of biases and output weights.
constexpr int kNetIn = 14, kNetH1 = 256, kNetH2 = 128, kNetH3 = 64;
constexpr int kNetFrag1 = 0;                                        // 16 column blocks x 1 k-step x 4
constexpr int kNetFrag2 = kNetFrag1 + (kNetH1 / 16) * 1 * 64 * 4;   // 8 x 8 x 8
constexpr int kNetFrag3 = kNetFrag2 + (kNetH2 / 16) * 8 * 64 * 8;   // 4 x 4 x 8
constexpr int kNetFragHalves = kNetFrag3 + (kNetH3 / 16) * 4 * 64 * 8;
constexpr int kNetBias1 = 0, kNetBias2 = 256, kNetBias3 = 384, kNetW4 = 448, kNetBias4 = 512;
constexpr int kNetBiasSize = 516;
static_assert(kNetH1 * kNetIn + kNetH1 + kNetH2 * kNetH1 + kNetH2 + kNetH3 * kNetH2 + 2 * kNetH3 + 1 ==
                  STORM_SELF_MLP_SIZE,
              "network parameter count");


// Per-problem description read by the kernels.  All pointers are device
// memory.  The first three groups are scalar-cache lines of 64 bytes, each
// holding what is read together: the sizes and switches and the pointers of a
// rollout's start, and with the second line what an update reads.
struct alignas(64) ProblemDev {
    int32_t N, H, n_halton, n_null;
    int32_t n_sph_obs, n_box_obs, ppt, n_tiles;  // ppt = particles per 64-lane tile
    uint32_t cost_mask, seed_lo, seed_hi, grad_mask;  // grad_mask: terms of the differentiable form
    uint32_t comb;      // the Gaussian particles' noise is comb-filtered (response in the tables)
    uint32_t cov_step;  // sigma2 is [H][7] (Eq. 5 per step) instead of [7]
    uint32_t selfnet;   // the self-collision term comes from the learned network (its own kernel)
    int32_t n_chunks;   // the adjoint's workgroups, each a run of tiles (adjoint_chunks)

    const float *tables;    // [kTabSize]
    const float *halton;    // [7][n_halton][H] smoothed Halton standard noise
    const float4 *obs_bound;  // [n_sph_obs + n_box_obs] centre, radius (of a cuboid: to its corners)
    const float *box_obs;   // [n_box_obs][16]: M = R^T (9, row-major), t = -R^T c (3), half extents (3), pad
    float *mean;            // [H][7]
    float *sigma2;          // [7], or [H][7] with cov_step
    float *u;               // [7][N][H] controls of the last step
    float *C;               // [N] horizon costs of the last step

    uint32_t *step;         // sampling step counter (Philox counter word 3); [1] and [2]: status, last_step
    uint32_t *status;       // asynchronous status flags
    uint32_t *last_step;    // counter value the last rollout sampled with (reused by the adjoint)
    float beta, alpha_mu, alpha_sigma, sigma2_min;
    float *ball;            // [8]: ball position, velocity (world frame) at the current state, pad
    float *qbuf;            // [7][N][H] joint positions of the last step (stand-alone network pass)
    float *upd_part;        // partial sums of the update (many particles)

    float k_m, w_pos, w_rot, a_stop;
    float a_joint, a_vel, a_manip, a_coll;
    float alpha_pos[3], alpha_rot[3];
    float w_ball, ball_g[3], ball_c[2];  // ball term: weight, gravity (world), tray centre (flange x, y)
    float *grad_part;       // adjoint partials per tile chunk: horizon-cost sums [kAdjChunks], gradients [chunks][7][kMaxH]
    float *grad;            // [H][7] gradient of the expected horizon cost
    float *adam_m, *adam_v; // [H][7] Adam moments of the refinement
    const _Float16 *net_frag;  // packed network weights (pack_selfnet)
    const float *net_bias;
};
static_assert(offsetof(ProblemDev, tables) == 64 && offsetof(ProblemDev, step) == 128 &&
                  offsetof(ProblemDev, k_m) == 192,
              "groups of 64 bytes");

// Robot constants (wave-uniform; in device memory for the rollouts and the adjoint,
// by value for the FK kernel).
struct alignas(64) RobotDev {
    int32_t n_spheres, n_self_items, pad0[2];
    const float4 *sph_local;  // [S] body-frame centre (x, y, z), radius
    const int32_t *sph_body;  // [S] frame index 0..7 the sphere is attached to
    const float *body_bound;  // [8][2] per frame: anchor sphere (int bits), what its radius lacks to hold the body's spheres
    const int32_t *self_items;  // [n_self_items][4] self-collision work items (self_pairs)
    uint64_t cap_mask;  // spheres that anchor a body or a run of self_items (their capsules are kept in LDS)
    int32_t pad1[2];
    float ca[kFrames], sa[kFrames], a[kFrames], d[kFrames];  // DH: cos/sin alpha_{k-1}, a_{k-1}, d_k
};

// What the plain kernels read of one problem, in device memory.  Kernel
// arguments lie in host memory, which a wave reads over PCIe; a descriptor in
// device memory behind one preloaded pointer is nearer (traced rollout at
// N=64, H=16: 5.5 -> 4.7 us; at N=1024, H=30 without collisions 9.0 -> 8.5 us,
// its adjoint 8.5 -> 8.0 us).
struct PlainDev {
    ProblemDev P;
    RobotDev R;
};

// Wave-uniform reads through the constant address space: the backend turns
// them into scalar loads whose results feed VALU instructions as SGPR operands.
#define STORM_CONST_AS __attribute__((address_space(4)))
using ProblemRef = const STORM_CONST_AS ProblemDev &;
using RobotRef = const STORM_CONST_AS RobotDev &;
template <typename T>
__device__ __forceinline__ const STORM_CONST_AS T *uniform_ptr(const T *p)
{
    return (const STORM_CONST_AS T *)(p);
}

// Pointers known to point to global memory: one that a kernel reads from a
// descriptor in memory is otherwise accessed with flat instructions, which
// count as LDS traffic too, so that LDS waits wait for them.
template <typename T>
using global_ptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ global_ptr<T> as_global(T *p)
{
    return (global_ptr<T>)p;
}

// A 16-byte record of global memory.
__device__ __forceinline__ float4 load_float4(global_ptr<const float4> p)
{
    typedef float vec4 __attribute__((ext_vector_type(4)));
    const vec4 v = *(global_ptr<const vec4>)p;
    return make_float4(v.x, v.y, v.z, v.w);
}

// A 32-bit word read by a vector (buffer) load even where its address is
// wave-uniform: workgroup barriers wait for outstanding scalar and LDS
// traffic only, so a value needed after a barrier, fetched this way early,
// does not hold the barrier up for its memory latency.
__device__ __forceinline__ uint32_t vector_load_u32(const void *p)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, 4, 0x00020000);
    return __builtin_amdgcn_raw_buffer_load_b32(r, 0, 0, 0);
}
__device__ __forceinline__ float vector_load_f32(const float *p) { return __uint_as_float(vector_load_u32(p)); }

// Hardware square root (v_sqrt_f32, 1 ulp) for norms and distances.
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// Optional per-step outputs.
struct StepOut {
    float *u, *q, *v, *a, *c, *terms, *C;
    float *xd, *xdd;  // [6][N][H] flange velocity and acceleration (Eq. 8)
};

// Launchers (defined in the .hip translation units).
hipError_t launch_init_tables(const ProblemDev &P, const float *d_dt_raw, const float *d_lim_raw, float acc_stop,
                              float gamma, float w_term, float k_jl, float k_vl, const float *d_sigma_init,
                              const float comb[3], int n_knots, const float *d_obs_raw, int n_obs,
                              float *d_box_obs,
                              float4 *d_obs_bound, const float *d_sph_raw, int n_spheres, float4 *d_sph_local,
                              int32_t *d_sph_body, hipStream_t stream);
// Plain launches take the host's copy of the problem for the launch shape and
// the device's (PlainDev) for the kernel.
hipError_t launch_rollout(const ProblemDev &P, const RobotDev &R, const PlainDev *dev, const float *x0, const float *goal,
                          const float *noise, const StepOut &out, hipStream_t stream);
// Raise the dynamic-LDS limit of the rollout kernels to what the largest
// sphere model needs (idempotent).
hipError_t set_rollout_lds_limit();
// Whether the learned self-collision network's weight matrices (W1, W2, W3
// of storm_robot.self_mlp) hold FP16 values only, as its kernel requires.
bool selfnet_weights_fp16(const float *prm);
// The work of storm_rollout_init; a context of a batch (`batched`) lacks the
// buffers that only plain launches use.
int32_t init_context(storm_ctx *out, const storm_params *params, const storm_robot *robot, const storm_scene *scene,
                     void *stream, bool batched);
// Workgroups of a problem's update in a batch before the join (0: none), and the
// floats of its partial sums (ProblemDev::upd_part; 0 where one workgroup per
// joint takes a single problem).
int update_batch_parts(int N, int H);
size_t update_part_floats(int N, int H);
hipError_t launch_update(const ProblemDev &P, const PlainDev *dev, float *mean_out, float *sigma2_out, float *cmd, int shift,
                         hipStream_t stream);
// Learned self-collision term: after the rollout, adds a_coll max(0, d) to
// every running cost and its horizon sum to C (weights packed by pack_selfnet
// from the parameter layout of storm_robot.self_mlp).
hipError_t launch_selfnet(const ProblemDev &P, const PlainDev *dev, const StepOut &out, hipStream_t stream);
void pack_selfnet(const float *prm, std::vector<_Float16> &frag, std::vector<float> &bias);
// Many problems: persistent rollout over a (problem, tile) work queue, and one
// update workgroup per problem and joint, behind the larger problems' chains
// (descriptors in device memory).
struct RolloutLds {
    size_t bytes;  // dynamic LDS
    bool dense;    // in the form that packs a scene to leave room for a second workgroup
};
hipError_t launch_rollout_batch(const ProblemDev *probs, const int2 *items, int n_items, uint32_t *next,
                                const RobotDev *robot, const RolloutLds &lds, const float *x0s, const float *goals,
                                int waves, int grid, hipStream_t stream);
// What a problem's tiles need in a batch in workgroups of `waves` waves.
RolloutLds rollout_batch_lds(const ProblemDev &P, const RobotDev &R, int waves);
hipError_t launch_update_batch(const ProblemDev *probs, int n_problems, const int2 *part_items, int n_part_items,
                               float *cmd, int shift, hipStream_t stream);
// Differentiable form: adjoint + fixed-order reduction (grad, J) per joint;
// with it > 0 the same launch takes Adam step `it` on the stored mean, and
// with cmd it also writes the command and the shift of the refined mean.
// launch_command writes them for a refinement of zero steps.
// The partials go to `part` (layout of ProblemDev::grad_part).
hipError_t launch_grad(const ProblemDev &P, const PlainDev *dev, float *part, const float *x0, const float *goal,
                       const float *mean, const float *noise, float *grad_out, float *J_out, int it, float lr,
                       float *cmd, int shift, hipStream_t stream);
hipError_t launch_command(const PlainDev *dev, float *cmd, int shift, hipStream_t stream);
// Batched refinement: `iterations` Adam steps on the gradient of every
// problem (adjoint over the (problem, chunk) items, then reduce + Adam per
// (problem, joint)), the last also writing the commands cmd [P][7] and the
// shift.
hipError_t launch_refine_batch(const ProblemDev *probs, int n_problems, const int2 *items, int n_items, bool split,
                               const RobotDev *robot, const float *x0s, const float *goals, int iterations,
                               float lr, float *cmd, int shift, hipStream_t stream);
hipError_t launch_fk(const RobotDev &R, const float *q, bool rows, int n, float *pose, float *manip, hipStream_t stream);

// Self-collision work items of the robot: pairs of groups (runs of up to four
// spheres of one body) on bodies at least two apart, four integers each.
void self_pairs(const storm_robot *robot, std::vector<int> &items);
// The sphere of [lo, hi) about whose centre (in the body's frame) the ball
// that holds all of them is smallest, and that ball's radius.
int anchor_sphere(const float *spheres, int lo, int hi, double &radius);
// Two floats per frame, the bodies' bounds of RobotDev::body_bound.
std::vector<float> body_bounds(const storm_robot *robot);

}  // namespace storm

// One plain-form problem (the storm_ctx handle of the C ABI).
struct storm_ctx_s {
    int device = 0;
    int32_t error = STORM_OK;  // sticky device error
    bool pending = false;      // a step waits for its update
    storm_params params{};
    storm::ProblemDev P{};
    storm::RobotDev R{};
    storm::PlainDev *dev = nullptr;  // P and R in device memory
    _Float16 *net_frag = nullptr;  // learned self-collision weights (packed), when self_model = 1
    float *net_bias = nullptr;
    float *scratch = nullptr;    // this device's static scratch (storm_rollout_grad_noalloc)
    std::vector<void *> allocs;  // every device allocation of this context
};

// An instantiated graph of one control step (plain or batched).
struct storm_graph_s {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int32_t *error = nullptr;  // sticky error word of the owning context or batch
};
