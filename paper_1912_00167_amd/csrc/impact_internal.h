// Internal declarations shared by the host code and the HIP kernels of libimpact.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "impact.h"

namespace impact {

// Tiling of the loss kernels: a workgroup of 256 threads owns NB consecutive trajectories
// and sweeps time backwards in chunks.  P lanes share one (t, b) step (each takes 1/P of the
// actions / action dimensions), so a wavefront covers 64 / (NB * P) consecutive time rows of
// the tile and a chunk is NWAVES times that.  The scan buffers are sized for P = 1.
constexpr int NB = 8;
constexpr int NTHREADS = 256;
constexpr int NWAVES = NTHREADS / 64;
constexpr int TC_MAX = NTHREADS / NB;       // time steps per chunk when P = 1
constexpr int T_PRELOAD = 128;              // longest trajectory whose rewards and flags a single-wavefront tile keeps in LDS
constexpr int PARTIAL_STRIDE = 8;           // floats per workgroup in the partial-sum workspace

struct LossArgs {
    int T, B, A;
    // learner side, always time-major fp32
    const void *learner;      // [T][B][W], fp32 or (learner_bf16) bf16
    const float *values;      // [T][B]
    const float *bootstrap;   // [B]
    // buffer-resident side: time-major [T][B][..] or slot-major [slot][T][..]
    const void *worker;
    const void *target;
    const void *actions;
    int act_bytes;            // categorical: the action index is an int32 (4) or one byte (1)
    const void *rewards;
    const uint8_t *dones;
    // cached log pi_worker(a), log pi_target(a): [T][B][2] or the buffer's plane [slot][T][2], or null.
    // Where given, `worker` is null, and `target` may be (then the KL coefficient is zero).
    const double *logp;
    int learner_bf16;
    int batch_major;          // learner, values and every per-step output are [B][T][..] instead of [T][B][..] (generic kernels only)
    const int32_t *slots;     // device [B]; slot-major only
    int num_slots;
    int slot_first;           // >= 0: trajectory b lies in slot (slot_first + b) mod num_slots and `slots` is not read
    // slot-major only: bytes from one slot's trajectory to the next in the distribution planes and in
    // the action plane (multiples of 16; rewards and flags lie T elements apart)
    size_t stride_dist, stride_act, stride_lp;
    // hyper-parameters, pre-digested on the host
    float gamma, lambda, rho_bar, c_bar;
    float rho_clip;           // target-worker clipping rho; may be +inf
    double log_rho_clip;      // its logarithm (+inf with it)
    int ratio_worker;         // surrogate ratio pi_theta / pi_worker instead (Section 4.1, R_2)
    double clip_lo, clip_hi;  // 1 - eps, 1 + eps (-inf / +inf when eps = +inf)
    float vf_coeff, ent_coeff, kl_coeff;
    double inv_M;             // 1 / (T * B)
    // outputs
    float *grad_dist;         // [T][B][W]
    float *grad_values;       // [T][B]
    float *vs;                // [T][B] or null
    float *adv;               // [T][B] or null
    float4 *step_out;         // [T][B] records {dL/dV, vs, adv, 0} in place of the three tensors above, or null
    float *partials;          // [num_partials][PARTIAL_STRIDE]
    mutable int num_partials; // sets of partial sums the launch leaves (one per workgroup); set by the launcher
    // Long trajectories of a small batch are cut into num_segs time segments of seg_chunks chunks each,
    // one workgroup per (tile, segment).  The scan is affine in its carry, acc_t = A_t + P_t * carry, so a
    // first launch (phase 1) only finds every segment's A and P at its first step (seg_agg[seg][b][2]) and a
    // second launch (phase 2) starts each segment from the carry that the later segments' pairs compose to.
    // num_segs = 1, phase = 0: the whole trajectory in one workgroup.
    int num_segs, seg_chunks, phase;
    double *seg_agg;
    // completion counter for the in-kernel final reduction (zero between launches), or null: then the
    // caller launches the reduction; loss5 is only written by the kernel in the first case
    unsigned *done_count;
    float *loss5;
    float *fractions;         // [2] {clipped, truncated} shares of the steps, or null
    mutable bool dpp;         // the order in which the partial sums' last sum combines (see reduce_tiles); set by the launcher
};

struct ReduceArgs {
    const float *partials;
    int num_tiles;
    double inv_M;
    float vf_coeff, ent_coeff, kl_coeff;
    float *loss5;
    float *fractions;
    bool dpp;                 // see reduce_tiles
};

__host__ __device__ inline int num_tiles(int B) { return (B + NB - 1) / NB; }

// Time segments (see LossArgs): at most SEG_MAX per trajectory, and only for batches of at most
// SEG_MAX_TILES tiles, which bounds the workspace the pairs and the per-segment partial sums need.
constexpr int SEG_MAX = 64, SEG_MAX_TILES = 128;

// Launchers (defined in the .hip files).  `slot_major` selects the fused-gather addressing.
// Return false when no specialised kernel exists for (A, alignment): the caller then uses the generic one.
// They set a.num_segs: the partial sums to reduce are num_tiles * num_segs.
bool launch_loss_cat_static(int dtype, bool slot_major, LossArgs &a, hipStream_t s);
bool launch_loss_gauss_static(int dtype, bool slot_major, LossArgs &a, hipStream_t s);
// ... on cached log-probabilities (a.logp; with the KL term if a.target is there)
bool launch_loss_cat_cached(int dtype, bool slot_major, LossArgs &a, hipStream_t s);
// ... for one-byte action indices (a.act_bytes == 1), all three forms
bool launch_loss_cat_u8(int dtype, bool slot_major, LossArgs &a, hipStream_t s);
bool launch_loss_gauss_cached(int dtype, bool slot_major, LossArgs &a, hipStream_t s);
// ... for any shape: the register-resident kernels below, or loss_generic where they do not reach
void launch_loss_generic(int dist, int dtype, bool slot_major, const LossArgs &a, hipStream_t s);

// Shape of a launch of the register-resident kernels (loss_lanes.h): 2^p_log2 lanes per step, 2^nb_log2 trajectories
// per workgroup, `rows` time steps per chunk, nchunk chunks; in the scan, 2^l_log2 lanes per trajectory with per_lane rows
// each (per_lane_pad: up to a multiple of the scan's block); t_fastest: neighbouring lanes take neighbouring time steps
// (else neighbouring trajectories).  rows_magic, per_lane_magic: i / rows = (i * rows_magic) >> 20 and
// i / per_lane = (i * per_lane_magic) >> 16 for 0 <= i < 1024.  Strides: bytes between time steps
// (_t) and between trajectories or slots (_b) of the buffer-side tensors; elements, in steps, of the learner's.
constexpr int LANES_MAX_THREADS = 1024, LANES_MAX_NB = 64, LANES_MAX_ELEMS = 512;
struct LanesShape {
    int p_log2, nb_log2, rows, nchunk, l_log2, t_fastest, per_lane, per_lane_pad, rows_magic, per_lane_magic, waves;
    unsigned dist_b, dist_t, act_b, act_t, lp_b, lp_t, rew_b, rew_t, done_b, done_t, ln_b, ln_t;
};
// False where there is no such kernel (more than LANES_MAX_ELEMS actions).
bool launch_loss_lanes(int dist, int dtype, bool slot_major, const LossArgs &a, hipStream_t s);
// Whether they are the faster choice where a specialised kernel exists too.
bool lanes_suit(int dist, int A, int T, int B, int chunk_rows);
// One kernel of the family, by the element type of the buffer's floats: R elements per lane (1..6 or 8).
struct LanesLaunch { unsigned blocks, threads, lds_bytes; int R; };
void launch_lanes_cat_f32(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s);
void launch_lanes_cat_bf16(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s);
void launch_lanes_gauss_f32(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s);
void launch_lanes_gauss_bf16(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s);
void launch_reduce(const ReduceArgs &r, hipStream_t s);
// A completion counter (zero between launches) for a loss call on this stream that has no buffer handle, or null
// (stream_counters.hip): with one, the kernel's last workgroup sums the loss terms and no second launch follows.
unsigned *done_counter_of_stream(hipStream_t s);
void launch_zero_words(unsigned *p, int n, hipStream_t s);

// Buffer data movement.  A "run" is cnt consecutive slots starting at slot0 that take
// trajectories i0 .. i0+cnt-1 of time-major sources with n trajectories.  One launch moves all fields of a run.
struct PlaneTask {
    const void *src;     // time-major [T][n][Wd]
    void *dst;           // slot-major plane [N][T][Wd], slots slot_stride bytes apart; log-probabilities: [N][T][2]
    size_t slot_stride;
    int Wd;              // elements per record; log-probabilities: of the distribution
    int kind;            // InsertKind
    int which;           // log-probabilities: column of the plane
    int rows;            // time steps per tile; the tiles of a task are numbered along the trajectories first
    int end;             // first workgroup after this task's
};
enum InsertKind { INSERT_FLOATS, INSERT_I32, INSERT_U8, INSERT_LOGP };
constexpr int INSERT_TASKS = 8;
// For the log-probabilities: the actions, which count as the ring stores them.
struct LogpArgs {
    const void *actions;         // time-major, about to be stored, or the ring's plane
    size_t stride_act;           // bytes between slots of the plane; 0: time-major
    int dist, A, act_bytes;      // act_bytes: categorical, of an index
};
struct PlaneCopyArgs {
    int T, n, i0, slot0, cnt;
    int num;
    PlaneTask task[INSERT_TASKS];
    LogpArgs logp;
    void add(int kind, const void *src, void *dst, size_t slot_stride, int Wd, int which = 0)
    {
        task[num++] = PlaneTask{src, dst, slot_stride, Wd, kind, which, 0, 0};
    }
};
enum PlaneKind { PLANE_F32, PLANE_BF16 };                  // what the ring stores the float fields as
void launch_insert_plane(PlaneKind kind, const PlaneCopyArgs &a, hipStream_t s);

// ... and out of it: all fields of B slots in one launch.
struct GatherTask {
    const void *src;     // slot-major plane [N][T][Wd], slots slot_stride bytes apart
    void *dst;           // time-major [T][B][Wd]
    size_t slot_stride;
    int Wd;
    int elem_bytes;      // 1, 2 or 4
    int word_bytes;      // records: the largest of 4, 2, 1 that divides a record
    int rows;            // records: time steps per tile; -1: scalars, by tile; 0: element by element
    int end;             // first workgroup after this task's
};
constexpr int GATHER_TASKS = 6;
struct GatherArgs {
    const int32_t *slots;
    int T, B, num_slots;
    int num;
    GatherTask task[GATHER_TASKS];
};
void launch_gather_plane(const GatherArgs &a, hipStream_t s);

}  // namespace impact
