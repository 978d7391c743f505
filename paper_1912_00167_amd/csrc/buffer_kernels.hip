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

// log pi(a) of the action as the ring stores it, in fp64 with the library's exp and log, four lanes per step: this runs
// once per trajectory, and is a chain of exponentials long (with one lane per step, 6.6 us for 128 trajectories of 50 steps,
// A = 18, which was the longest launch of that insert).
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
        for (int c = part; c < l.A; c += 4) S += exp((double)z[c] - (double)m);
        S += dpp<DPP_XOR1>(S);
        S += dpp<DPP_XOR2>(S);
        lp = ((double)z[act] - (double)m) - log(S);
    } else {
        lp = 0.0;
        for (int d = part; d < l.A; d += 4) {
            const double ls = (double)z[l.A + d];
            const double x = l.stride_act ? (double)widen(((const ST *)actions)[act_at * l.A + d])
                                          : (double)widen(convert<float, ST>(((const float *)actions)[act_at * l.A + d]));
            const double diff = x - (double)z[d];
            lp += -0.5 * diff * diff * exp(-2.0 * ls) - ls;
        }
        lp += dpp<DPP_XOR1>(lp);
        lp += dpp<DPP_XOR2>(lp);
        lp -= l.A * (double)kHalfLog2Pi;
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

// dst[t][b][.] = plane[slots[b]][t][.]: a byte copy, done in words of WB bytes (the largest of 4, 2, 1
// that divides a record).  A workgroup transposes a tile of GATHER_NB (16) trajectories x RT rows through
// LDS: each wavefront reads whole trajectories' pieces (RT records, contiguous in the plane), then
// each wavefront writes whole rows (GATHER_NB records, contiguous in the batch tensor).
#ifndef IMPACT_GATHER_NB
#define IMPACT_GATHER_NB 16
#endif
#ifndef IMPACT_GATHER_TILE_BYTES
#define IMPACT_GATHER_TILE_BYTES 16384
#endif
constexpr int GATHER_NB = IMPACT_GATHER_NB;
constexpr int GATHER_TILE_BYTES = IMPACT_GATHER_TILE_BYTES;

template <typename Word>
__global__ __launch_bounds__(256) void gather_tiles(const GatherArgs a, int wpr, int RT, size_t slot_words)
{
    __shared__ __align__(16) unsigned char tile_bytes[GATHER_TILE_BYTES];
    __shared__ int slot_of[GATHER_NB];
    Word *tile = (Word *)tile_bytes;
    constexpr int WB = (int)sizeof(Word), VW = 16 / WB;        // words per 16-byte vector
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b0 = blockIdx.x * GATHER_NB, t0 = blockIdx.y * RT;
    const int nb = min(GATHER_NB, a.B - b0), rows = min(RT, a.T - t0);
    if (tid < GATHER_NB) slot_of[tid] = min(max(a.slots[min(b0 + tid, a.B - 1)], 0), a.num_slots - 1);
    __syncthreads();
    // in: a trajectory's share of the tile is one contiguous piece of the plane, copied as it lies
    const int piece = rows * wpr;                  // words
    const int stride = RT * wpr;                   // words between trajectories in the tile
    const bool vec_in = (stride % VW) == 0 && (piece % VW) == 0;
    for (int j = wave; j < nb; j += 4) {
        const Word *src = (const Word *)a.src + (size_t)slot_of[j] * slot_words + (size_t)t0 * wpr;
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
    auto from_tile = [&](int r, int c) {           // word c of row r (c below a few thousand: exact in float)
        const int j = (int)(((float)c + 0.5f) * inv_wpr), k = c - j * wpr;
        return tile[j * stride + r * wpr + k];
    };
    for (int r = wave; r < rows; r += 4) {
        Word *dst = (Word *)a.dst + ((size_t)(t0 + r) * a.B + b0) * wpr;
        if ((row_words % VW) == 0 && ((size_t)dst % 16) == 0) {
            for (int v = lane; v < row_words / VW; v += 64) {
                Word w[VW];
#pragma unroll
                for (int q = 0; q < VW; ++q) w[q] = from_tile(r, v * VW + q);
                ((uint4 *)dst)[v] = *(const uint4 *)w;
            }
        } else {
            for (int c = lane; c < row_words; c += 64) dst[c] = from_tile(r, c);
        }
    }
}

// The same copy one element per thread, for records too long for the tile (thousands of actions).
template <typename E>
__global__ __launch_bounds__(256) void gather_elements(const GatherArgs a)
{
    const size_t row = (size_t)a.B * a.Wd;
    const size_t total = row * a.T;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (size_t)gridDim.x * 256) {
        const int t = (int)(e / row);
        const size_t rem = e - (size_t)t * row;
        const int b = (int)(rem / a.Wd), k = (int)(rem - (size_t)b * a.Wd);
        const int slot = min(max(a.slots[b], 0), a.num_slots - 1);
        ((E *)a.dst)[e] = ((const E *)a.src)[(size_t)slot * a.slot_stride + (size_t)t * a.Wd + k];
    }
}

void launch_gather_plane(const GatherArgs &a, hipStream_t s)
{
    const size_t rec = (size_t)a.Wd * a.elem_bytes;           // bytes of one record
    const size_t total = (size_t)a.T * a.B * a.Wd;
    if (total == 0) return;
    // (also for the per-step scalars: a tile of 8 trajectories' rewards or flags is too little work per workgroup)
    // ... and small planes, where the element-wise kernel's shorter dependency chain wins
    if (GATHER_NB * rec > GATHER_TILE_BYTES || a.T > 65535 || rec < 16 || total * a.elem_bytes < ((size_t)4 << 20)) {
        const unsigned blocks = (unsigned)min((size_t)65536, (total + 255) / 256);
        switch (a.elem_bytes) {
        case 4: hipLaunchKernelGGL((gather_elements<uint32_t>), dim3(blocks), dim3(256), 0, s, a); break;
        case 2: hipLaunchKernelGGL((gather_elements<uint16_t>), dim3(blocks), dim3(256), 0, s, a); break;
        default: hipLaunchKernelGGL((gather_elements<uint8_t>), dim3(blocks), dim3(256), 0, s, a); break;
        }
        return;
    }
    const int WB = rec % 4 == 0 ? 4 : rec % 2 == 0 ? 2 : 1;
    const int wpr = (int)(rec / WB);
    const size_t slot_words = a.slot_stride * a.elem_bytes / WB;   // (a stride is T records, or a multiple of 16 bytes)
    int RT = max(1, (int)(GATHER_TILE_BYTES / (GATHER_NB * rec)));
    // whole 16-byte vectors per trajectory piece: a multiple of 16 / gcd(record bytes, 16) rows
    int unit = 1;
    while ((rec * unit) % 16 != 0) unit <<= 1;
    if (RT >= unit) RT -= RT % unit;
    RT = min(RT, a.T);
    const dim3 grid((a.B + GATHER_NB - 1) / GATHER_NB, (a.T + RT - 1) / RT), block(256);
    switch (WB) {
    case 4: hipLaunchKernelGGL((gather_tiles<uint32_t>), grid, block, 0, s, a, wpr, RT, slot_words); break;
    case 2: hipLaunchKernelGGL((gather_tiles<uint16_t>), grid, block, 0, s, a, wpr, RT, slot_words); break;
    default: hipLaunchKernelGGL((gather_tiles<uint8_t>), grid, block, 0, s, a, wpr, RT, slot_words); break;
    }
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
