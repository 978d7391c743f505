// Data movement between time-major tensors and the slot-major planes of the circular buffer.
#include "loss_device.h"

namespace impact {

// bfloat16 from fp32: keep the upper 16 bits, round to nearest, ties to even; NaN stays NaN.
__device__ __forceinline__ bf16_t to_bf16(float x)
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

template <typename S, typename D>
__device__ __forceinline__ D convert(S x) { return (D)x; }
template <>
__device__ __forceinline__ bf16_t convert<float, bf16_t>(float x) { return to_bf16(x); }

// ---- into the ring: dst[slot0 + s][t][.] = src[t][i0 + s][.] for s < cnt, all fields in one launch ----------
//
// Every workgroup takes one tile of one field.  A field's records lie one after the other along the trajectories in the
// source and along the time steps in the ring, so a tile is a transpose through LDS, read and written in whole segments.
// What bounds it: memory for large batches (see launch_insert_plane), the launch for small ones.

constexpr int INSERT_NB = 8;                       // trajectories per tile of records
constexpr int INSERT_TILE_BYTES = 32768;
constexpr int INSERT_SCALAR_NB = 64, INSERT_SCALAR_ROWS = 32;     // tile of a field with one element per step

template <typename S, typename D>
__device__ __forceinline__ void insert_records(const PlaneCopyArgs &a, const PlaneTask &k, int block, S *tile)
{
    constexpr int VW = 16 / (int)sizeof(D);        // destination elements per 16-byte vector
    constexpr int SV = 16 / (int)sizeof(S);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int across = (a.cnt + INSERT_NB - 1) / INSERT_NB;
    const int ty = block / across, s0 = (block - ty * across) * INSERT_NB, t0 = ty * k.rows;
    const int nb = min(INSERT_NB, a.cnt - s0), rows = min(k.rows, a.T - t0);
    const int row_elems = nb * k.Wd;               // of the tile, in the source
    const int row_pitch = INSERT_NB * k.Wd;        // in LDS
    const S *src0 = (const S *)k.src + ((size_t)t0 * a.n + a.i0 + s0) * k.Wd;
    const size_t src_pitch = (size_t)a.n * k.Wd;
    // several loads in flight per thread before the first LDS store (the loop bounds are run-time values,
    // which would otherwise leave one load latency exposed per element)
    if (row_elems % SV == 0 && (size_t)src0 % 16 == 0 && src_pitch % SV == 0) {
        constexpr int U = 4;
        const int row_vecs = row_elems / SV, total = rows * row_vecs;
        const float inv_row = 1.0f / (float)row_vecs;
        for (int f0 = tid; f0 < total; f0 += 256 * U) {
            uint4 v[U];
            int at[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int f = min(f0 + 256 * u, total - 1);
                const int r = (int)(((float)f + 0.5f) * inv_row), i = (f - r * row_vecs) * SV;
                at[u] = r * row_pitch + i;
                v[u] = *(const uint4 *)(src0 + (size_t)r * src_pitch + i);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) *(uint4 *)(tile + at[u]) = v[u];       // (past the end: the last vector again)
        }
    } else {
        constexpr int U = 8;
        const int total = rows * row_elems;
        const float inv_row = 1.0f / (float)row_elems;
        for (int f0 = tid; f0 < total; f0 += 256 * U) {
            S v[U];
            int at[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int f = min(f0 + 256 * u, total - 1);
                const int r = (int)(((float)f + 0.5f) * inv_row), i = f - r * row_elems;
                at[u] = r * row_pitch + i;
                v[u] = src0[(size_t)r * src_pitch + i];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) tile[at[u]] = v[u];
        }
    }
    __syncthreads();
    const int piece = rows * k.Wd;                 // destination elements per trajectory
    const float inv_wd = 1.0f / (float)k.Wd;
    for (int j = wave; j < nb; j += 4) {
        D *dst = (D *)((char *)k.dst + (size_t)(a.slot0 + s0 + j) * k.slot_stride) + (size_t)t0 * k.Wd;
        const int nvec = (((size_t)dst % 16) == 0) ? piece / VW : 0;
        for (int v = lane; v < nvec; v += 64) {
            // element e of the trajectory's piece (below 8192: exact in float) is element c of row r
            const int e = v * VW, r = (int)(((float)e + 0.5f) * inv_wd);
            int c = e - r * k.Wd;
            const S *from = tile + r * row_pitch + j * k.Wd;
            D w[VW];
#pragma unroll
            for (int q = 0; q < VW; ++q) {
                w[q] = convert<S, D>(from[c]);
                if (++c == k.Wd) { c = 0; from += row_pitch; }
            }
            ((uint4 *)dst)[v] = *(const uint4 *)w;
        }
        for (int e = nvec * VW + lane; e < piece; e += 64) {
            const int r = (int)(((float)e + 0.5f) * inv_wd);
            dst[e] = convert<S, D>(tile[r * row_pitch + j * k.Wd + e - r * k.Wd]);
        }
    }
}

// One element per step: 64 trajectories x 32 steps, read along the trajectories, written along the steps.
template <typename S, typename D>
__device__ __forceinline__ void insert_scalars(const PlaneCopyArgs &a, const PlaneTask &k, int block, S *tile)
{
    constexpr int NB_ = INSERT_SCALAR_NB, ROWS = INSERT_SCALAR_ROWS, PITCH = NB_ + 1, U = NB_ * ROWS / 256;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int across = (a.cnt + NB_ - 1) / NB_;
    const int ty = block / across, s0 = (block - ty * across) * NB_, t0 = ty * ROWS;
    const int nb = min(NB_, a.cnt - s0), rows = min(ROWS, a.T - t0);
    const S *src0 = (const S *)k.src + (size_t)t0 * a.n + a.i0 + s0;
    S v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = src0[(size_t)min(wave + 4 * u, rows - 1) * a.n + min(lane, nb - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) tile[(wave + 4 * u) * PITCH + lane] = v[u];
    __syncthreads();
    const int t = tid & (ROWS - 1), j0 = tid / ROWS;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int j = j0 + u * (256 / ROWS);
        if (t < rows && j < nb) ((D *)((char *)k.dst + (size_t)(a.slot0 + s0 + j) * k.slot_stride))[t0 + t] = convert<S, D>(tile[t * PITCH + j]);
    }
}

// One element per thread, for records too long for the tile (thousands of actions).
template <typename S, typename D>
__device__ __forceinline__ void insert_elements(const PlaneCopyArgs &a, const PlaneTask &k, int block, int blocks)
{
    const size_t per_slot = (size_t)a.T * k.Wd, total = per_slot * a.cnt;
    for (size_t e = (size_t)block * 256 + threadIdx.x; e < total; e += (size_t)blocks * 256) {
        const int s = (int)(e / per_slot);
        const size_t rem = e - (size_t)s * per_slot;
        const int t = (int)(rem / k.Wd), c = (int)(rem - (size_t)t * k.Wd);
        ((D *)((char *)k.dst + (size_t)(a.slot0 + s) * k.slot_stride))[rem] = convert<S, D>(((const S *)k.src)[((size_t)t * a.n + a.i0 + s) * k.Wd + c]);
    }
}

// Lane q of every four adjacent ones.
template <int Q>
__device__ __forceinline__ double of_quad(double x) { return dpp<Q * 0x55 /* quad_perm Q,Q,Q,Q */>(x); }
// acc + the four lanes' terms in the order of the lanes
__device__ __forceinline__ double add_quad(double acc, double x)
{
    acc += of_quad<0>(x);
    acc += of_quad<1>(x);
    acc += of_quad<2>(x);
    return acc + of_quad<3>(x);
}

// log pi(a) of the action as the ring stores it, in fp64 with the library's exp and log: this runs once per trajectory, and
// is a chain of exponentials long (with one lane per step, 6.6 us for 128 trajectories of 50 steps, A = 18, which was the
// longest launch of that insert).  Four lanes share a step's exponentials; the sum goes through them in the order of the
// elements, so that the stored bits do not depend on the split.
template <typename ST>
__device__ __forceinline__ void insert_logp(const PlaneCopyArgs &a, const PlaneTask &k, int block)
{
    const LogpArgs &l = a.logp;
    const size_t total = (size_t)a.cnt * a.T;
    const int part = threadIdx.x & 3;
    const size_t e = min((size_t)block * 64 + (threadIdx.x >> 2), total - 1);
    // neighbouring steps are neighbouring trajectories of one time step: their records lie one after the other
    const int t = (int)(e / a.cnt), s = (int)(e - (size_t)t * a.cnt);
    const size_t from = (size_t)t * a.n + a.i0 + s;
    const float *z = (const float *)k.src + from * k.Wd;
    const size_t act_at = l.stride_act ? (size_t)t : from;
    const char *actions = (const char *)l.actions + (l.stride_act ? (size_t)(a.slot0 + s) * l.stride_act : 0);
    double lp;
    if (l.dist == IMPACT_CATEGORICAL) {
        const int given = l.act_bytes == 1 ? (int)((const uint8_t *)actions)[act_at] : ((const int *)actions)[act_at];
        const int act = min(max(given, 0), l.A - 1);         // (the loss flags an index out of range)
        float m = z[0];
        for (int c = part; c < l.A; c += 4) m = fmaxf(m, z[c]);
        m = fmaxf(m, dpp<DPP_XOR1>(m));
        m = fmaxf(m, dpp<DPP_XOR2>(m));
        double S = 0.0;
        for (int c = 0; c < l.A; c += 4) {
            const double x = exp((double)z[min(c + part, l.A - 1)] - (double)m);
            S = add_quad(S, c + part < l.A ? x : 0.0);
        }
        lp = ((double)z[act] - (double)m) - log(S);
    } else {
        lp = -l.A * (double)kHalfLog2Pi;
        for (int c = 0; c < l.A; c += 4) {
            const int d = min(c + part, l.A - 1);
            const double ls = (double)z[l.A + d];
            const double x = l.stride_act ? (double)widen(((const ST *)actions)[act_at * l.A + d])
                                          : (double)widen(convert<float, ST>(((const float *)actions)[act_at * l.A + d]));
            const double diff = x - (double)z[d];
            const double term = -0.5 * diff * diff * exp(-2.0 * ls) - ls;
            lp = add_quad(lp, c + part < l.A ? term : 0.0);
        }
    }
    if (part == 0) ((double *)((char *)k.dst + (size_t)(a.slot0 + s) * k.slot_stride))[2 * t + k.which] = lp;
}

template <typename ST>
__global__ __launch_bounds__(256) void insert_fields(const PlaneCopyArgs a)
{
    extern __shared__ __align__(16) unsigned char insert_tile[];
    int i = 0, first = 0;
    while (i < a.num - 1 && (int)blockIdx.x >= a.task[i].end) first = a.task[i++].end;
    const PlaneTask &k = a.task[i];
    const int block = (int)blockIdx.x - first;
    if (k.kind == INSERT_LOGP) insert_logp<ST>(a, k, block);
    else if (k.kind == INSERT_I32) insert_scalars<int32_t, int32_t>(a, k, block, (int32_t *)insert_tile);
    else if (k.kind == INSERT_U8) insert_scalars<uint8_t, uint8_t>(a, k, block, (uint8_t *)insert_tile);
    else if (k.Wd == 1) insert_scalars<float, ST>(a, k, block, (float *)insert_tile);
    else if (k.rows > 0) insert_records<float, ST>(a, k, block, (float *)insert_tile);
    else insert_elements<float, ST>(a, k, block, k.end - first);
}

// 4096 trajectories of 128 steps (D = 17, bf16 ring), 271 MB: 60 us, 4.5 TB/s; field by field 28 + 28 + 15 + 6 + 4 us in
// five launches, 88 us per call.
void launch_insert_plane(PlaneKind kind, const PlaneCopyArgs &given, hipStream_t s)
{
    PlaneCopyArgs a = given;
    const size_t steps = (size_t)a.T * a.cnt;
    if (steps == 0 || a.num == 0) return;
    size_t end = 0, lds = 0;
    for (int i = 0; i < a.num; ++i) {
        PlaneTask &k = a.task[i];
        const size_t across = (a.cnt + INSERT_NB - 1) / INSERT_NB;
        size_t blocks;
        k.rows = 0;
        if (k.kind == INSERT_LOGP) {
            blocks = (steps + 63) / 64;
        } else if (k.Wd == 1) {
            blocks = ((size_t)(a.cnt + INSERT_SCALAR_NB - 1) / INSERT_SCALAR_NB) * ((a.T + INSERT_SCALAR_ROWS - 1) / INSERT_SCALAR_ROWS);
            lds = max(lds, (size_t)INSERT_SCALAR_ROWS * (INSERT_SCALAR_NB + 1) * 4);
        } else {
            // rows per tile: a multiple of 8 (whole 16-byte vectors per trajectory's piece, whatever the record), as many
            // as the tile holds, or down to half as many if they divide the trajectories better
            const int most = (int)(INSERT_TILE_BYTES / ((size_t)INSERT_NB * k.Wd * 4));
            if (most >= 1) {
                k.rows = min(most, a.T);
                if (most >= 8) {
                    k.rows = min(most & ~7, (a.T + 7) & ~7);
                    for (int r = k.rows; r >= 8 && 2 * r >= k.rows; r -= 8)
                        if ((a.T + r - 1) / r * r < (a.T + k.rows - 1) / k.rows * k.rows) k.rows = r;
                }
                blocks = across * ((a.T + k.rows - 1) / k.rows);
                lds = max(lds, (size_t)INSERT_NB * k.rows * k.Wd * 4);
            } else {
                blocks = min((size_t)65536, (steps * k.Wd + 255) / 256);
            }
        }
        end += blocks;
        k.end = (int)end;
    }
    const dim3 grid((unsigned)end), block(256);
    if (kind == PLANE_F32) hipLaunchKernelGGL((insert_fields<float>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((insert_fields<bf16_t>), grid, block, lds, s, a);
}

// ---- out of the ring: dst[t][b][.] = plane[slots[b]][t][.], a byte copy of all fields in one launch -----------
//
// Every workgroup takes one tile of one field.  Records are copied in words of the largest of 4, 2, 1 bytes that divides
// one, transposed through LDS: each wavefront reads whole trajectories' pieces (contiguous in the plane), then each
// wavefront writes whole rows (GATHER_NB records, contiguous in the batch tensor).
constexpr int GATHER_NB = 16;
constexpr int GATHER_TILE_BYTES = 16384;
constexpr int GATHER_SCALAR_NB = 64, GATHER_SCALAR_ROWS = 32;     // tile of a field with one element per step

template <typename Word>
__device__ __forceinline__ void gather_records(const GatherArgs &a, const GatherTask &k, int block, Word *tile, const int *slot_of, int b0, int nb)
{
    constexpr int VW = 16 / (int)sizeof(Word);                 // words per 16-byte vector
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int across = (a.B + GATHER_NB - 1) / GATHER_NB, RT = k.rows;
    const int t0 = block / across * RT, rows = min(RT, a.T - t0);
    const int wpr = k.Wd * k.elem_bytes / (int)sizeof(Word);   // words per record
    // in: a trajectory's share of the tile is one contiguous piece of the plane, copied as it lies
    const int piece = rows * wpr;                  // words
    const int stride = RT * wpr;                   // words between trajectories in the tile
    const bool vec_in = (stride % VW) == 0 && (piece % VW) == 0;
    for (int j = wave; j < nb; j += 4) {
        const Word *src = (const Word *)((const char *)k.src + (size_t)slot_of[j] * k.slot_stride) + (size_t)t0 * wpr;
        if (vec_in && ((size_t)src % 16) == 0) {
            // two loads in flight per lane before the first LDS store (the bounds are run-time values)
            const int nvec = piece / VW;
            for (int i = lane; i < nvec; i += 128) {
                const uint4 v0 = ((const uint4 *)src)[i];
                const uint4 v1 = i + 64 < nvec ? ((const uint4 *)src)[i + 64] : make_uint4(0, 0, 0, 0);
                ((uint4 *)(tile + j * stride))[i] = v0;
                if (i + 64 < nvec) ((uint4 *)(tile + j * stride))[i + 64] = v1;
            }
        } else {
            for (int i = lane; i < piece; i += 64) tile[j * stride + i] = src[i];
        }
    }
    __syncthreads();
    // out: a row of the batch tensor is the tile's nb records of that time step, one after the other
    const int row_words = nb * wpr;
    const float inv_wpr = 1.0f / (float)wpr;
    for (int r = wave; r < rows; r += 4) {
        Word *dst = (Word *)k.dst + ((size_t)(t0 + r) * a.B + b0) * wpr;
        const Word *row = tile + r * wpr;
        if ((row_words % VW) == 0 && ((size_t)dst % 16) == 0) {
            for (int v = lane; v < row_words / VW; v += 64) {
                // word c of the row (below a few thousand: exact in float) is word w of record j
                const int c = v * VW, j = (int)(((float)c + 0.5f) * inv_wpr);
                int w = c - j * wpr;
                const Word *from = row + j * stride;
                Word x[VW];
#pragma unroll
                for (int q = 0; q < VW; ++q) {
                    x[q] = from[w];
                    if (++w == wpr) { w = 0; from += stride; }
                }
                ((uint4 *)dst)[v] = *(const uint4 *)x;
            }
        } else {
            for (int c = lane; c < row_words; c += 64) {
                const int j = (int)(((float)c + 0.5f) * inv_wpr);
                dst[c] = row[j * stride + c - j * wpr];
            }
        }
    }
}

// One element per step: 64 trajectories x 32 steps, read along the steps, written along the trajectories.
template <typename E>
__device__ __forceinline__ void gather_scalars(const GatherArgs &a, const GatherTask &k, int block, E *tile, const int *slot_of, int b0, int nb)
{
    constexpr int NB_ = GATHER_SCALAR_NB, ROWS = GATHER_SCALAR_ROWS, PITCH = NB_ + 1, U = NB_ * ROWS / 256;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int across = (a.B + NB_ - 1) / NB_, t0 = block / across * ROWS, rows = min(ROWS, a.T - t0);
    const int t = tid & (ROWS - 1), j0 = tid / ROWS;
    E v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        v[u] = ((const E *)((const char *)k.src + (size_t)slot_of[min(j0 + u * (256 / ROWS), nb - 1)] * k.slot_stride))[t0 + min(t, rows - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) tile[t * PITCH + j0 + u * (256 / ROWS)] = v[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = wave + 4 * u;
        if (r < rows && lane < nb) ((E *)k.dst)[(size_t)(t0 + r) * a.B + b0 + lane] = tile[r * PITCH + lane];
    }
}

// One element per thread: records too long for the tile (thousands of actions), and small fields, where its short chain wins.
template <typename E>
__device__ __forceinline__ void gather_elements(const GatherArgs &a, const GatherTask &k, int block, int blocks)
{
    const size_t row = (size_t)a.B * k.Wd, total = row * a.T;
    for (size_t e = (size_t)block * 256 + threadIdx.x; e < total; e += (size_t)blocks * 256) {
        const int t = (int)(e / row);
        const size_t rem = e - (size_t)t * row;
        const int b = (int)(rem / k.Wd), c = (int)(rem - (size_t)b * k.Wd);
        const int slot = min(max(a.slots[b], 0), a.num_slots - 1);
        ((E *)k.dst)[e] = ((const E *)((const char *)k.src + (size_t)slot * k.slot_stride))[(size_t)t * k.Wd + c];
    }
}

__global__ __launch_bounds__(256) void gather_fields(const GatherArgs a)
{
    __shared__ __align__(16) unsigned char tile[GATHER_TILE_BYTES];
    __shared__ int slot_of[GATHER_SCALAR_NB];
    int i = 0, first = 0;
    while (i < a.num - 1 && (int)blockIdx.x >= a.task[i].end) first = a.task[i++].end;
    const GatherTask &k = a.task[i];
    const int block = (int)blockIdx.x - first;
    if (k.rows == 0) {
        if (k.elem_bytes == 4) gather_elements<uint32_t>(a, k, block, k.end - first);
        else if (k.elem_bytes == 2) gather_elements<uint16_t>(a, k, block, k.end - first);
        else gather_elements<uint8_t>(a, k, block, k.end - first);
        return;
    }
    const int per = k.rows < 0 ? GATHER_SCALAR_NB : GATHER_NB;
    const int b0 = block % ((a.B + per - 1) / per) * per, nb = min(per, a.B - b0);
    if ((int)threadIdx.x < per) slot_of[threadIdx.x] = min(max(a.slots[min(b0 + (int)threadIdx.x, a.B - 1)], 0), a.num_slots - 1);
    __syncthreads();
    if (k.rows < 0) {
        if (k.elem_bytes == 4) gather_scalars<uint32_t>(a, k, block, (uint32_t *)tile, slot_of, b0, nb);
        else if (k.elem_bytes == 2) gather_scalars<uint16_t>(a, k, block, (uint16_t *)tile, slot_of, b0, nb);
        else gather_scalars<uint8_t>(a, k, block, tile, slot_of, b0, nb);
    } else {
        if (k.word_bytes == 4) gather_records<uint32_t>(a, k, block, (uint32_t *)tile, slot_of, b0, nb);
        else if (k.word_bytes == 2) gather_records<uint16_t>(a, k, block, (uint16_t *)tile, slot_of, b0, nb);
        else gather_records<uint8_t>(a, k, block, tile, slot_of, b0, nb);
    }
}

// 8192 trajectories of 100 steps (A = 18, fp32 ring, slots in no order), 250 MB: 59 us, 4.3 TB/s; field by field 23 + 23 + 7
// + 7 + 5 us in five launches, 83 us per call.
void launch_gather_plane(const GatherArgs &given, hipStream_t s)
{
    GatherArgs a = given;
    if (a.num == 0) return;
    size_t end = 0;
    for (int i = 0; i < a.num; ++i) {
        GatherTask &k = a.task[i];
        const size_t rec = (size_t)k.Wd * k.elem_bytes, total = (size_t)a.T * a.B * k.Wd;
        const bool small = total * k.elem_bytes < (k.Wd == 1 ? (size_t)1 << 20 : (size_t)4 << 20);
        size_t blocks;
        if (small || GATHER_NB * rec > GATHER_TILE_BYTES) {
            k.rows = 0;
            blocks = min((size_t)65536, (total + 255) / 256);
        } else if (k.Wd == 1) {
            k.rows = -1;
            blocks = ((size_t)(a.B + GATHER_SCALAR_NB - 1) / GATHER_SCALAR_NB) * ((a.T + GATHER_SCALAR_ROWS - 1) / GATHER_SCALAR_ROWS);
        } else {
            k.word_bytes = rec % 4 == 0 ? 4 : rec % 2 == 0 ? 2 : 1;
            int RT = max(1, (int)(GATHER_TILE_BYTES / (GATHER_NB * rec)));
            // whole 16-byte vectors per trajectory piece: a multiple of 16 / gcd(record bytes, 16) rows
            int unit = 1;
            while ((rec * unit) % 16 != 0) unit <<= 1;
            if (RT >= unit) RT -= RT % unit;
            k.rows = min(RT, a.T);
            blocks = ((size_t)(a.B + GATHER_NB - 1) / GATHER_NB) * ((a.T + k.rows - 1) / k.rows);
        }
        end += blocks;
        k.end = (int)end;
    }
    hipLaunchKernelGGL(gather_fields, dim3((unsigned)end), dim3(256), 0, s, a);
}

__global__ void zero_words(unsigned *p, int n)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

void launch_zero_words(unsigned *p, int n, hipStream_t s)
{
    hipLaunchKernelGGL(zero_words, dim3(1), dim3(64), 0, s, p, n);
}

}  // namespace impact
