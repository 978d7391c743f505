// Launch shapes of the register-resident loss kernels.
#include "loss_device.h"

namespace impact {

static int log2_of(int x)
{
    int l = 0;
    while ((1 << l) < x) ++l;
    return l;
}

namespace {
struct Split { int R, blocks; };
}

// How a batch is split over lanes, workgroups and chunks.
static Split split(int A, int T, int B, LanesShape &g)
{
    // Lanes per step: as few as hold the record (6 elements each, 8 where records are long), since what a step needs once
    // (logarithms, ratio, surrogate) is computed by all its lanes: T = 61, B = 2047, A = 7 takes 16 us with 2 lanes per
    // step, 20 with 4, 28 with 8.
    int P = 1;
    while ((A + P - 1) / P > (A > 48 ? 8 : 6)) P <<= 1;
    // Trajectories per workgroup: few enough for a workgroup on (nearly) every compute unit, at most 8, which make the
    // row segments of the time-major tensors 8 records long.  (Above 1024 trajectories not fewer: the workspace holds a
    // set of partial sums per 8.)  T = 50, B = 512, A = 18: 2 trajectories 14.0 us, 1 or 4: 16.2, 8: 21.
    int nb = 1;
    while (nb < 8 && (B > 1024 || B >= 2 * nb * 192)) nb <<= 1;
    const int blocks = (B + nb - 1) / nb;
    // With the chip hardly filled more lanes shorten the chains (T = 50, B = 10, A = 18: 10.3 us; 16 lanes instead of 8: 12.1).
    while (P < 64 && blocks <= 320 && (A + P - 1) / P > 1 && (long long)T * nb * P * 2 <= 512) P <<= 1;
    // Threads: a whole trajectory as one chunk where that takes at most 1024; long ones in chunks of 1024 threads with
    // a workgroup per compute unit, of fewer threads with several (Gaussian T = 64, B = 8192, A = 13: 256 threads
    // 75 us, 512 79, 1024 92).
    int threads = LANES_MAX_THREADS;
    while (threads > 256 && (long long)blocks * threads > 256 * 1024) threads >>= 1;
    if (threads < P * nb) threads = P * nb;
    g.p_log2 = log2_of(P);
    g.nb_log2 = log2_of(nb);
    g.rows = min(threads / P / nb, T);
    // The scan: a lane per 4 rows or more, within one wavefront.
    g.l_log2 = 0;
    while (g.l_log2 < 6 - g.nb_log2 && (4 << g.l_log2) < g.rows) ++g.l_log2;
    if (g.rows < T) {                            // several chunks: no lane of the scan partly filled
        while (g.l_log2 > 0 && (g.rows >> g.l_log2) < 4) --g.l_log2;
        g.rows = g.rows >> g.l_log2 << g.l_log2;
    }
    g.nchunk = (T + g.rows - 1) / g.rows;
    g.per_lane = (g.rows + (1 << g.l_log2) - 1) >> g.l_log2;
    g.per_lane_pad = (g.per_lane + 3) & ~3;
    return Split{(A + P - 1) / P, blocks};
}

// The pipeline walks a tile's chunks (chunk_rows time steps each) one after the other, a chain of latencies for every
// chunk, which only a batch that fills the chip hides; these kernels take a whole trajectory, or a large part, at once.
// Both measured over T = 20 .. 1024, B = 4 .. 4096 and every specialised record: with at most 1024 trajectories these are
// 1.0 to 2.6 times as fast (A = 18, T = 50: B = 10 10.3 us against 19.6, B = 512 15.0 against 20.5, B = 1024 18.6 against
// 21.5), with more the pipeline is (B = 2048: 27.6 against 23.3), but for
//   - trajectories of a single chunk (A = 4, T = 20, B = 512: 10.6 us against 8.5), unless few and Gaussian (D = 6, T = 20,
//     B = 64: 8.2 against 10.2);
//   - long ones on a few compute units, whose share of the memory rate they would wait for, where the pipeline cuts the
//     time axis into segments that run side by side (with inputs from memory, Gaussian D = 6, T = 1024, B = 32, 220 KB per
//     workgroup: 33 us against 24; A = 18, T = 1024, B = 64, inputs in the cache: 40 against 31, T = 300: 23 against 31).
bool lanes_suit(int dist, int A, int T, int B, int chunk_rows)
{
    if (B > SEG_MAX_TILES * NB) return false;
    if (T <= chunk_rows && (dist == IMPACT_CATEGORICAL || B > 192)) return false;
    LanesShape g;
    const Split sp = split(A, T, B, g);
    const int W = dist == IMPACT_CATEGORICAL ? A : 2 * A;
    return sp.blocks >= 192 || (g.nchunk <= 2 && ((long long)T << g.nb_log2) * W <= 6400);     // (16 bytes each: 100 KB)
}

bool launch_loss_lanes(int dist, int dtype, bool slot_major, const LossArgs &a, hipStream_t s)
{
    if (a.A > LANES_MAX_ELEMS) return false;
    const bool cat = dist == IMPACT_CATEGORICAL;
    const size_t W = cat ? a.A : 2 * (size_t)a.A, es = dtype == IMPACT_F32 ? 4 : 2, T = a.T, B = a.B;
    const size_t act = cat ? (size_t)a.act_bytes : a.A * es;
    // strides are 32-bit numbers in the kernels
    constexpr size_t LIMIT = (size_t)1 << 32;
    if (B * W * 4 >= LIMIT || B * 16 >= LIMIT || T * 16 >= LIMIT) return false;
    if (slot_major && (a.stride_dist >= LIMIT || a.stride_act >= LIMIT)) return false;
    LanesShape g;
    if (slot_major) {
        g.dist_b = a.stride_dist; g.dist_t = W * es; g.act_b = a.stride_act; g.act_t = act;
        g.lp_b = a.stride_lp; g.lp_t = 16; g.rew_b = T * es; g.rew_t = es; g.done_b = T; g.done_t = 1;
    } else {
        g.dist_b = W * es; g.dist_t = B * W * es; g.act_b = act; g.act_t = B * act;
        g.lp_b = 16; g.lp_t = B * 16; g.rew_b = es; g.rew_t = B * es; g.done_b = 1; g.done_t = B;
    }
    g.ln_t = a.batch_major ? 1 : B;
    g.ln_b = a.batch_major ? T : 1;
    g.t_fastest = slot_major && a.batch_major;     // every tensor is laid out trajectory by trajectory

    const Split sp = split(a.A, a.T, a.B, g);
    g.rows_magic = ((1 << 20) + g.rows - 1) / g.rows;
    g.per_lane_magic = ((1 << 16) + g.per_lane - 1) / g.per_lane;
    g.waves = (((g.rows << g.nb_log2) << g.p_log2) + 63) / 64;

    LanesLaunch l;
    l.blocks = (unsigned)sp.blocks;
    l.threads = (unsigned)g.waves * 64;
    l.lds_bytes = (unsigned)((g.nchunk > 1 ? 4 : 2) * 64 * g.per_lane_pad * sizeof(double));
    l.R = sp.R == 7 ? 8 : sp.R;
    a.num_partials = sp.blocks;
    a.dpp = true;
    if (cat) {
        if (dtype == IMPACT_F32) launch_lanes_cat_f32(l, a, g, s);
        else launch_lanes_cat_bf16(l, a, g, s);
    } else {
        if (dtype == IMPACT_F32) launch_lanes_gauss_f32(l, a, g, s);
        else launch_lanes_gauss_bf16(l, a, g, s);
    }
    return true;
}

}  // namespace impact
