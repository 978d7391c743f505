// Loss kernels for any number of actions (up to LANES_MAX_ELEMS), any layout and any batch size: a step's record
// is split over the registers of P neighbouring lanes, R consecutive elements each.
//
// A workgroup owns `nb` neighbouring trajectories and walks time backwards in chunks of `rows` time steps; every
// (t, b) of a chunk has its own P lanes, so a chunk is one round of loads, one scan and one round of stores.  Nothing
// is staged through LDS: lane p of a step loads elements p R .. p R + R - 1 straight into registers, as one or two
// wide loads (4-byte alignment is enough for them), and neighbouring lanes continue each other's addresses.  The
// distributions stay in registers from the loads to the gradients, so each is read once.
//
// All arithmetic is fp64, with exponentials of relative error 5e-14.
//
// What bounds it: instruction issue (at T = 61, B = 2047, A = 7 about 700 instructions per wavefront and chunk, 16 us
// against 3 us of memory traffic), and for small batches the length of the chains: arguments, loads, sums, scan, final
// sum.  The kernel that read every value from memory in several passes, with the library's exp, took 34 us there, and
// 62 us at T = 100, B = 1000, D = 8 on batch-major bf16 tensors (now 17).
#pragma once
#include "loss_device.h"

namespace impact {

// ---- exponential and logarithm ----------------------------------------------------------------------------

constexpr int LANES_TABLE = 64;                    // 2^(j/64), j = 0..63

// 2^(j/64) by the Taylor series of e^r about the middle of the range, |r| < 0.35 (r^14/14! < 5e-18).  (As constants in
// memory they would cost every workgroup a miss of 2000 cycles; the library's exp2 takes twice the instructions.)
__device__ __forceinline__ double table_entry(int j)
{
    const double r = (double)(j - 32) * (0.693147180559945309417 / 64.0);
    double p = 1.0 / 6227020800.0;
    constexpr double F[13] = {1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0, 1.0 / 5040.0,
                              1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5, 1.0, 1.0};
#pragma unroll
    for (int i = 0; i < 13; ++i) p = __builtin_fma(p, r, F[i]);
    return p * 1.41421356237309504880;
}

// e^x, relative error 5e-14: exp64's reduction with one more term of the Taylor polynomial (r^5/120 < 4e-14).  Any
// argument: below the fp64 range 0, above it inf, NaN stays NaN.  NEG: the argument is <= 0 (or NaN).
template <bool NEG>
__device__ __forceinline__ double exp_any(double x, const double *tbl)
{
    x = x < -800.0 ? -800.0 : x;
    if (!NEG) x = x > 800.0 ? 800.0 : x;
    const double t = __builtin_fma(x, 64.0 * 1.4426950408889634074, kRoundMagic);
    const double n = t - kRoundMagic;
    const int ni = low_word(t);
    double r = __builtin_fma(-n, kLn2Hi64, x);
    r = __builtin_fma(-n, kLn2Lo64, r);
    double p = __builtin_fma(1.0 / 24.0, r, 1.0 / 6.0);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    return ldexp(tbl[ni & 63] * p, ni >> 6);
}

// log S for a softmax normaliser (1 <= S <= number of actions, or NaN): the fp32 logarithm y, off by less than 2e-6,
// corrected by log(S e^-y) = u - u^2 / 2 with u = S e^-y - 1 (u^3 / 3 < 3e-18).
__device__ __forceinline__ double log_normaliser(double S, const double *tbl)
{
    const double y = (double)(__builtin_amdgcn_logf((float)S) * 0.693147180559945309f);
    const double u = __builtin_fma(S, exp_any<true>(-y, tbl), -1.0);
    return y + __builtin_fma(-0.5 * u, u, u);
}

// ---- exchange between the P lanes of a step: P is a power of two, known at run time and the same for all lanes ------

// Every lane of the step ends with the same bits: each round combines two values that all lanes of a half hold alike.
template <typename T, int N, class Op>
__device__ __forceinline__ void across_lanes(T (&v)[N], int p_log2, Op op)
{
    if (p_log2 >= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = op(v[i], dpp<DPP_XOR1>(v[i]));
    if (p_log2 >= 2)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = op(v[i], dpp<DPP_XOR2>(v[i]));
    if (p_log2 >= 3)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = op(v[i], dpp<DPP_HALF_MIRROR>(v[i]));
    if (p_log2 >= 4)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = op(v[i], dpp<DPP_MIRROR>(v[i]));
    if (p_log2 >= 5)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = op(v[i], __shfl_xor(v[i], 16, 64));
    if (p_log2 >= 6)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = op(v[i], __shfl_xor(v[i], 32, 64));
}
template <int N>
__device__ __forceinline__ void lanes_max(float (&v)[N], int p_log2)
{
    across_lanes(v, p_log2, [](float x, float y) { return fmaxf(x, y); });
}
template <int N>
__device__ __forceinline__ void lanes_sum(double (&v)[N], int p_log2)
{
    across_lanes(v, p_log2, [](double x, double y) { return x + y; });
}

// ---- a lane's R elements -----------------------------------------------------------------------------------

template <typename E, int R>
__device__ __forceinline__ void load_elems(E (&x)[R], const char *p)
{
    __builtin_memcpy(x, p, sizeof(E) * R);
}
template <int R>
__device__ __forceinline__ void store_elems(float *p, const float (&x)[R])
{
    __builtin_memcpy(p, x, sizeof(float) * R);
}

// acc_t = delta_t + g_t acc_{t+1} for one chunk, by one wavefront.  2^l_log2 of its lanes share a trajectory, the first of them for
// the latest rows.  A lane walks its per_lane rows (read in blocks of SCAN_U, with padding that changes nothing up to
// per_lane_pad; row k of lane l lies at 64 k + l, which keeps every access free of bank conflicts and its address a constant away from
// the lane's own) first for their affine map (A, P), then, with the maps of the later rows composed across lanes, for the
// values themselves, which replace delta.  carry: the trajectory's value just after the chunk, the same in all its
// lanes, updated.
constexpr int SCAN_U = 4;

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or(double other, double x)     // lanes that have no source take `other`
{
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(other), __double2hiint(x), CTRL, ROWS, 0xF, false);
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(other), __double2loint(x), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ void compose(double &A, double &P, bool on)   // the map of the lane CTRL names comes first
{
    double Au = dpp_or<CTRL, ROWS>(0.0, A), Pu = dpp_or<CTRL, ROWS>(1.0, P);
    Au = on ? Au : 0.0;
    Pu = on ? Pu : 1.0;
    A = __builtin_fma(P, Au, A);
    P *= Pu;
}

__device__ __forceinline__ void lanes_scan(double *sd, const double *sg, int per_lane, int per_lane_pad, int l_log2, int lane, double &carry)
{
    const int j = lane & ((1 << l_log2) - 1);
    double *const d0 = sd + lane;
    const double *const g0 = sg + lane;
    double A = 0.0, P = 1.0;
    for (int k = 0; k < per_lane_pad; k += SCAN_U) {
        double d[SCAN_U], g[SCAN_U];
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) { d[u] = d0[64 * (k + u)]; g[u] = g0[64 * (k + u)]; }
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) { A = __builtin_fma(g[u], A, d[u]); P *= g[u]; }
    }
    if (l_log2 >= 1) compose<0x111 /* row_shr:1 */, 0xF>(A, P, j >= 1);
    if (l_log2 >= 2) compose<0x112, 0xF>(A, P, j >= 2);
    if (l_log2 >= 3) compose<0x114, 0xF>(A, P, j >= 4);
    if (l_log2 >= 4) compose<0x118, 0xF>(A, P, j >= 8);
    if (l_log2 >= 5) compose<0x142 /* row_bcast:15 */, 0xA>(A, P, true);
    if (l_log2 >= 6) compose<0x143 /* row_bcast:31 */, 0xC>(A, P, true);
    const double mine = __builtin_fma(P, carry, A), before = __shfl_up(mine, 1, 64);
    double acc = j == 0 ? carry : before;
    carry = __shfl(mine, lane | ((1 << l_log2) - 1), 64);
    for (int k = 0; k < per_lane_pad; k += SCAN_U) {
        double d[SCAN_U], g[SCAN_U];
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) { d[u] = d0[64 * (k + u)]; g[u] = g0[64 * (k + u)]; }
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) {
            acc = __builtin_fma(g[u], acc, d[u]);
            if (k + u < per_lane) d0[64 * (k + u)] = acc;      // (padding stays as it is, for the next chunk)
        }
    }
}

// The compiler may not carry anything it derived from these values past this point.
template <typename E, int N>
__device__ __forceinline__ void opaque(E (&x)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if constexpr (sizeof(E) == 4) {
            asm volatile("" : "+v"(x[i]));
        } else {
            unsigned v = x[i];
            asm volatile("" : "+v"(v));
            x[i] = (E)v;
        }
    }
}

template <typename T>
__device__ __forceinline__ void opaque(T &x) { asm volatile("" : "+v"(x)); }

// x where it counts, else 0; the computation of x is never put under the condition.
__device__ __forceinline__ double where(bool counts, double x)
{
    opaque(x);
    return counts ? x : 0.0;
}

// ---- the kernel --------------------------------------------------------------------------------------------

// MODE: where the behaviour side comes from (POLICY_FULL, POLICY_CACHED, POLICY_CACHED_TARGET).
template <int DIST, int MODE, typename ST, typename LT, int R>
__global__ __launch_bounds__(LANES_MAX_THREADS) void loss_lanes(const LossArgs a, const LanesShape g)
{
    constexpr bool CAT = DIST == IMPACT_CATEGORICAL, CACHED = MODE != POLICY_FULL, TGT = MODE != POLICY_CACHED;
    extern __shared__ double scan_lds[];           // delta and gamma lambda c of a chunk; two sets if there are several chunks
    __shared__ double tbl[LANES_TABLE];
    __shared__ float red[LANES_MAX_THREADS / 64][PARTIAL_STRIDE];
    __shared__ int slot_of[LANES_MAX_NB];

    touch_arguments();
    const int A = a.A, W = CAT ? A : 2 * A;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = 1 << g.nb_log2, P = 1 << g.p_log2;
    const int part = tid & (P - 1), step = tid >> g.p_log2;
    const bool lead = part == 0;
    // the step's place in the chunk: neighbouring lanes take neighbouring trajectories, or neighbouring time steps
    const int steps = g.rows << g.nb_log2;         // of a chunk
    const bool in_chunk = step < steps;            // (threads past the last step shadow it and drop their results)
    const int at_step = min(step, steps - 1);
    const int bl = g.t_fastest ? (at_step * g.rows_magic) >> 20 : at_step & (nb - 1);
    const int row = g.t_fastest ? at_step - bl * g.rows : at_step >> g.nb_log2;
    const int tile = tile_of_block((int)blockIdx.x, (int)gridDim.x);
    const int b0 = tile * nb;
    const bool mine = b0 + bl < a.B;
    const int b = min(b0 + bl, a.B - 1);           // (a missing trajectory shadows the last real one and drops its results)

    // my elements: `own` is the first; the last lane that has any starts early enough for R whole elements and leaves
    // the `dup` first ones, which its neighbour has too, out of the sums (their gradients come out the same twice)
    const int own = min(part * R, A - R), dup = part * R - own;
    const bool writes = mine && dup < R;

    float bad = 0.f;
    int at = b;                                    // the trajectory's index in the buffer-side tensors: itself, or its slot
    if (a.num_slots > 0) {
        if (a.slot_first >= 0) {                   // a run of consecutive slots: nothing to read
            at = a.slot_first + b;
            if (at >= a.num_slots) at -= a.num_slots;
        } else {
            if (tid < nb) slot_of[tid] = a.slots[min(b0 + tid, a.B - 1)];   // (once: they may lie across the bus)
            __syncthreads();
            at = slot_of[bl];
        }
        if (at < 0 || at >= a.num_slots) { bad = 1.f; at = min(max(at, 0), a.num_slots - 1); }
    }
    // where my step lies in the scan's arrays
    const int k = g.rows - 1 - row, scan_lane = (k * g.per_lane_magic) >> 16, spot = (k - scan_lane * g.per_lane) * 64 + (bl << g.l_log2) + scan_lane;
    const int set = 64 * g.per_lane_pad;
    const double ce = a.ent_coeff * a.inv_M, ck = a.kl_coeff * a.inv_M;

    double carry = 0.0;
    float sum_s = 0.f, sum_v = 0.f, sum_h = 0.f, sum_k = 0.f, n_clipped = 0.f, n_truncated = 0.f;
    for (int c = g.nchunk - 1; c >= 0; --c) {
        const int t = c * g.rows + row;
        // (addresses are formed afresh for every chunk: a pair of registers per tensor carried along would cost more)
        int p_log2 = g.p_log2;                     // (likewise the conditions on it: pairs of scalar registers)
        asm volatile("" : "+s"(p_log2));
        int tc = min(t, a.T - 1), at_c = at, b_c = b;
        opaque(tc); opaque(at_c); opaque(b_c);
        auto in_buffer = [&](const void *base, unsigned per_b, unsigned per_t) {
            return (const char *)base + ((size_t)(unsigned)at_c * per_b + (size_t)(unsigned)tc * per_t);
        };
        const bool valid = in_chunk && mine && t < a.T;
        double *sd = scan_lds + ((c & 1) ? 2 * set : 0), *sg = sd + set;

        // ---- loads: everything the chunk needs, at once ----
        const size_t s_ln = (size_t)(unsigned)tc * g.ln_t + (size_t)(unsigned)b_c * g.ln_b;
        const char *p_ln = (const char *)a.learner + (s_ln * W + own) * sizeof(LT);
        const char *p_act = in_buffer(a.actions, g.act_b, g.act_t);
        constexpr int R1 = CAT ? 1 : R;            // (the second half of a Gaussian record: log standard deviations)
        LT l0[R], l1[R1];
        ST t0[TGT ? R : 1], t1[TGT ? R1 : 1], w0[CACHED ? 1 : R], w1[CACHED ? 1 : R1], av[R1];
        load_elems(l0, p_ln);
        if constexpr (!CAT) load_elems(l1, p_ln + (size_t)A * sizeof(LT));
        if constexpr (TGT) {
            const char *p = in_buffer(a.target, g.dist_b, g.dist_t) + own * (int)sizeof(ST);
            load_elems(t0, p);
            if constexpr (!CAT) load_elems(t1, p + (size_t)A * sizeof(ST));
        }
        double lp_w = 0.0, lp_t = 0.0;
        if constexpr (CACHED) {
            const double *lp = (const double *)in_buffer(a.logp, g.lp_b, g.lp_t);
            lp_w = lp[0];
            lp_t = lp[1];
        } else {
            const char *p = in_buffer(a.worker, g.dist_b, g.dist_t) + own * (int)sizeof(ST);
            load_elems(w0, p);
            if constexpr (!CAT) load_elems(w1, p + (size_t)A * sizeof(ST));
        }
        int act = 0;
        if constexpr (CAT) act = a.act_bytes == 1 ? (int)*(const uint8_t *)p_act : *(const int *)p_act;
        else load_elems(av, p_act + (size_t)own * sizeof(ST));
        const float V = a.values[s_ln];
        const float *p_next = tc + 1 < a.T ? a.values + (s_ln + g.ln_t) : a.bootstrap + b_c;
        const float Vn = *p_next;
        const float rew = widen(*(const ST *)in_buffer(a.rewards, g.rew_b, g.rew_t));
        const bool done = *in_buffer(a.dones, g.done_b, g.done_t) != 0;

        if (c == g.nchunk - 1) {
            // while the first loads travel: the table, and zero advantage with coefficient one in the scan's arrays
            // wherever no step lies
            if (tid < LANES_TABLE) tbl[tid] = table_entry(tid);
            if (g.rows != (g.per_lane_pad << g.l_log2))
                for (int i = tid; i < set; i += 64 * g.waves)
                    for (int n = 0; n < (g.nchunk > 1 ? 2 : 1); ++n) { scan_lds[2 * n * set + i] = 0.0; scan_lds[(2 * n + 1) * set + i] = 1.0; }
            lds_barrier();
        }

        // ---- sums over the elements, of all the policies ----
        // el, et: the learner's and the target's unnormalised softmax (categorical); E, q: 1 / sigma^2 and
        // (sigma_t^2 + (mu - mu_t)^2) / sigma^2 (Gaussian; q = 1 without a target: no KL term)
        double el[CAT ? R : 1], et[CAT && TGT ? R : 1], E[R1], q[R1];
        float m[6];                                // categorical: maximum and the action's logit of learner, target, worker
        double S[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        if constexpr (CAT) {
            if (valid && (act < 0 || act >= A)) bad = 1.f;
            act = min(max(act, 0), A - 1);
#pragma unroll
            for (int j = 0; j < 6; ++j) m[j] = -__builtin_inff();
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const bool taken = own + i == act;
                m[0] = fmaxf(m[0], widen(l0[i]));
                if (taken) m[1] = widen(l0[i]);
                if constexpr (TGT) {
                    m[2] = fmaxf(m[2], widen(t0[i]));
                    if (taken) m[3] = widen(t0[i]);
                }
                if constexpr (!CACHED) {
                    m[4] = fmaxf(m[4], widen(w0[i]));
                    if (taken) m[5] = widen(w0[i]);
                }
            }
            if constexpr (!CACHED) {
                lanes_max(m, p_log2);
            } else {
                float k[4] = {m[0], m[1], m[2], m[3]};
                lanes_max(k, p_log2);
                m[0] = k[0]; m[1] = k[1]; m[2] = k[2]; m[3] = k[3];
            }
            // S: learner: sum e, the same without the action taken, sum e x; target: sum e, sum e x, sum e x_learner;
            // worker: sum e
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const bool counts = i >= dup;
                const double x = (double)widen(l0[i]) - (double)m[0];
                el[i] = exp_any<true>(x, tbl);
                const double e = where(counts, el[i]);
                S[0] += e;
                S[1] += where(own + i != act, e);
                S[2] += where(counts, e * x);
                if constexpr (TGT) {
                    const double xt = (double)widen(t0[i]) - (double)m[2];
                    et[i] = exp_any<true>(xt, tbl);
                    S[3] += where(counts, et[i]);
                    S[4] += where(counts, et[i] * xt);
                    S[5] += where(counts, et[i] * x);
                }
                if constexpr (!CACHED) {
                    const double ew = exp_any<true>((double)widen(w0[i]) - (double)m[4], tbl);
                    S[6] += where(counts, ew);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (!CACHED) {
                lanes_sum(S, p_log2);
            } else {
                double k[TGT ? 6 : 3];
#pragma unroll
                for (int j = 0; j < (TGT ? 6 : 3); ++j) k[j] = S[j];
                lanes_sum(k, p_log2);
#pragma unroll
                for (int j = 0; j < (TGT ? 6 : 3); ++j) S[j] = k[j];
            }
        } else {
            // S: learner: log pi(a) + D/2 log 2pi, sum of log-stds; target: sum of log-stds, sum q; log pi(a) + .. of target
            // and worker
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const bool counts = i >= dup;
                const double x = (double)widen(av[i]);
                const double mu = (double)widen(l0[i]), ls = (double)widen(l1[i]), d = x - mu;
                E[i] = exp_any<false>(-2.0 * ls, tbl);
                S[0] += where(counts, __builtin_fma(-0.5 * d * d, E[i], -ls));
                S[1] += where(counts, ls);
                q[i] = 1.0;
                if constexpr (TGT) {
                    const double dm = mu - (double)widen(t0[i]), lst = (double)widen(t1[i]);
                    q[i] = __builtin_fma(dm, dm, exp_any<false>(2.0 * lst, tbl)) * E[i];
                    S[2] += where(counts, lst);
                    S[3] += where(counts, q[i]);
                    if constexpr (!CACHED) {
                        const double dt = x - (double)widen(t0[i]);
                        S[4] += where(counts, __builtin_fma(-0.5 * dt * dt, exp_any<false>(-2.0 * lst, tbl), -lst));
                    }
                }
                if constexpr (!CACHED) {
                    const double dw = x - (double)widen(w0[i]), lsw = (double)widen(w1[i]);
                    S[5] += where(counts, __builtin_fma(-0.5 * dw * dw, exp_any<false>(-2.0 * lsw, tbl), -lsw));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            constexpr int N = !CACHED ? 6 : TGT ? 4 : 2;
            double k[N];
#pragma unroll
            for (int j = 0; j < N; ++j) k[j] = S[j];
            lanes_sum(k, p_log2);
#pragma unroll
            for (int j = 0; j < N; ++j) S[j] = k[j];
        }

        // ---- what the scan needs: w = pi_target(a) / pi_worker(a) ----
        double lw, lt, logSt = 0.0;                // log w; log pi_target(a) (Gaussian: + D/2 log 2pi)
        if constexpr (CAT && TGT) logSt = log_normaliser(S[3], tbl);
        if constexpr (CACHED) {
            lt = CAT ? lp_t : lp_t + A * kHalfLog2Pi;
            lw = lp_t - lp_w;
        } else if constexpr (CAT) {
            lt = ((double)m[3] - (double)m[2]) - logSt;
            lw = lt - (((double)m[5] - (double)m[4]) - log_normaliser(S[6], tbl));
        } else {
            lt = S[4];
            lw = S[4] - S[5];
        }
        const double w = exp_any<false>(lw, tbl);
        const ScanInputs sc = scan_inputs(a, w, rew, done, V, Vn);
        if (lead && in_chunk) {
            sd[spot] = valid ? sc.delta : 0.0;
            sg[spot] = valid ? sc.gco : 0.0;
        }
        lds_barrier();
        if (wave == 0) lanes_scan(sd, sg, g.per_lane, g.per_lane_pad, g.l_log2, lane, carry);

        // ---- ratio, entropy and KL, while the first wavefront scans ----
        double lr1, H, KL = 0.0, invSl = 0.0, invSt = 0.0, logSl = 0.0, others = 0.0;
        if constexpr (CAT) {
            logSl = log_normaliser(S[0], tbl);
            invSl = 1.0 / S[0];
            others = S[1] * invSl;                 // 1 - p_a without cancellation
            H = logSl - S[2] * invSl;
            if constexpr (TGT) {
                invSt = 1.0 / S[3];
                KL = ((S[4] - S[5]) * invSt - logSt) + logSl;
            }
            lr1 = (((double)m[1] - (double)m[0]) - logSl) - lt;
        } else {
            H = S[1] + A * (kHalfLog2Pi + 0.5);
            if constexpr (TGT) KL = (S[1] - S[2]) + 0.5 * (S[3] - A);
            lr1 = S[0] - lt;
        }
        const double Rt = exp_any<false>(surrogate_log_ratio(a, lr1, lw), tbl);
        lds_barrier();
        const double adv = sd[spot];

        // ---- gradients ----
        // (what they need of the elements is formed again from the tensors' own values, which take fewer registers than
        // the fp64 intermediates the compiler would otherwise keep across the scan)
        opaque(l0);
        if constexpr (!CAT) { opaque(av); if constexpr (TGT) opaque(t0); }
        double s, gp;
        const bool clipped = surrogate(a, Rt, adv, s, gp);
        if (valid && writes) {
            float *gd = a.grad_dist + s_ln * W + own;
            float o[R];
            if constexpr (CAT) {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const double x = (double)widen(l0[i]) - (double)m[0], p = el[i] * invSl;
                    double base = ce * p * ((x - logSl) + H);
                    if constexpr (TGT) base = __builtin_fma(ck, p - et[i] * invSt, base);
                    o[i] = (float)__builtin_fma(gp, own + i == act ? others : -p, base);
                    __builtin_amdgcn_sched_barrier(0);
                }
                store_elems(gd, o);
            } else {
                float o2[R];
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const double mu = (double)widen(l0[i]), d = (double)widen(av[i]) - mu;
                    double dm = 0.0;
                    if constexpr (TGT) dm = mu - (double)widen(t0[i]);
                    o[i] = (float)(__builtin_fma(gp, d, ck * dm) * E[i]);
                    o2[i] = (float)(gp * __builtin_fma(d * d, E[i], -1.0) + ck * (1.0 - q[i]) - ce);
                    __builtin_amdgcn_sched_barrier(0);
                }
                store_elems(gd, o);
                store_elems(gd + A, o2);
            }
        }
        if (valid && lead) {
            const float gV = (float)(-(double)a.vf_coeff * adv * a.inv_M);   // V - vs = -adv
            const float vs_t = (float)((double)V + adv), adv_t = (float)adv;
            if (a.step_out) {
                a.step_out[s_ln] = make_float4(gV, vs_t, adv_t, 0.f);
            } else {
                a.grad_values[s_ln] = gV;
                if (a.vs) a.vs[s_ln] = vs_t;
                if (a.adv) a.adv[s_ln] = adv_t;
            }
            sum_s += (float)s;
            sum_v += (float)(0.5 * adv * adv);
            sum_h += (float)H;
            sum_k += (float)KL;
            n_clipped += clipped ? 1.f : 0.f;
            n_truncated += w > (double)a.rho_bar ? 1.f : 0.f;
        }
    }

    // ---- loss terms ----
    const float mine7[7] = {sum_s, sum_v, sum_h, sum_k, bad, n_clipped, n_truncated};
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const float x = wave_sum_63(mine7[j]);
        if (lane == 63) red[wave][j] = x;
    }
    lds_barrier();                                 // (gradient stores may still be on their way)
    if (wave != 0) return;
    if (lane < 7) {
        float x = 0.f;
        for (int v = 0; v < g.waves; ++v) x += red[v][lane];
        __hip_atomic_store(a.partials + (size_t)tile * PARTIAL_STRIDE + lane, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!a.done_count) return;
    // (as in store_partials: the sums are acknowledged before the count, and the last workgroup drops stale copies)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    unsigned before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(a.done_count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(before) != gridDim.x - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    reduce_tiles<4, true>(a.partials, (int)gridDim.x, a.inv_M, a.vf_coeff, a.ent_coeff, a.kl_coeff, a.loss5, a.fractions, lane);
    if (lane == 0) *a.done_count = 0;
}

template <int DIST, int MODE, typename ST, int R>
void launch_lanes_r(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s)
{
    const dim3 grid(l.blocks), block(l.threads);
    if (a.learner_bf16) hipLaunchKernelGGL((loss_lanes<DIST, MODE, ST, bf16_t, R>), grid, block, l.lds_bytes, s, a, g);
    else hipLaunchKernelGGL((loss_lanes<DIST, MODE, ST, float, R>), grid, block, l.lds_bytes, s, a, g);
}

template <int DIST, int MODE, typename ST>
void launch_lanes_mode(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s)
{
    switch (l.R) {
    case 1: launch_lanes_r<DIST, MODE, ST, 1>(l, a, g, s); break;
    case 2: launch_lanes_r<DIST, MODE, ST, 2>(l, a, g, s); break;
    case 3: launch_lanes_r<DIST, MODE, ST, 3>(l, a, g, s); break;
    case 4: launch_lanes_r<DIST, MODE, ST, 4>(l, a, g, s); break;
    case 5: launch_lanes_r<DIST, MODE, ST, 5>(l, a, g, s); break;
    case 6: launch_lanes_r<DIST, MODE, ST, 6>(l, a, g, s); break;
    default: launch_lanes_r<DIST, MODE, ST, 8>(l, a, g, s); break;
    }
}

template <int DIST, typename ST>
void launch_lanes_typed(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s)
{
    if (!a.logp) launch_lanes_mode<DIST, POLICY_FULL, ST>(l, a, g, s);
    else if (a.target) launch_lanes_mode<DIST, POLICY_CACHED_TARGET, ST>(l, a, g, s);
    else launch_lanes_mode<DIST, POLICY_CACHED, ST>(l, a, g, s);
}

}  // namespace impact
