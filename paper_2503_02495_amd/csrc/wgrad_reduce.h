// Reduction of split weight-gradient tiles, shared by the backward passes.
#pragma once
#include "common.h"
#include "gemm_mfma.h"

namespace uoe {

constexpr int RED_T = 64;
template <typename T> __device__ __forceinline__ void store4_as(T *p, float4 v);
template <> __device__ __forceinline__ void store4_as<float>(float *p, float4 v) { *reinterpret_cast<float4 *>(p) = v; }
template <> __device__ __forceinline__ void store4_as<bf16_t>(bf16_t *p, float4 v)
{
    *reinterpret_cast<uint2 *>(p) = make_uint2(pack2_bf16(v.x, v.y), pack2_bf16(v.z, v.w));
}
typedef float (*RedTile)[RED_T + 1];   // the workgroup's RED_T x RED_T tile in LDS
constexpr size_t RED_LDS = sizeof(float) * RED_T * (RED_T + 1);
// partial [sets*chunks*parts][M][N] fp32 -> storage dtype, an expert's parts added in order and rounded once.
// Set s goes to dst[s], stored as [n][M][N] or transposed as [n][N][M].  64x64 tiles, 16-byte loads with four rows of
// a part in flight per thread, 8-byte stores (bf16; straight, or transposed through LDS): the launch is a plain stream
// of the partial tiles (134 MB on the largest shape: 47.7 us with 32x32 tiles and 4-byte loads).
// CHUNKED: more than 128 samples are possible
template <typename T, bool CHUNKED> __device__ __forceinline__ void wgrad_reduce_tile(const WgradReduceArgs &a, RedTile tile, int bx, int by, int bz)
{
    const int set = bz / a.n, e = bz - set * a.n, r0 = by * RED_T, c0 = bx * RED_T;
    const int tx = (threadIdx.x & 15) * 4, ty = threadIdx.x >> 4;
    const int col = c0 + tx;                 // M and N are multiples of 8
    const size_t part = (size_t)a.M * a.N;
    float4 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
    for (int chunk = 0; chunk < (CHUNKED ? a.w.chunks : 1); ++chunk) {
        int first, parts;
        if (__builtin_expect(a.w.each != 0, 1)) {
            first = e * a.w.each;
            parts = a.w.each;
        } else {
            const int32_t *end = a.part_end + chunk * 32 + e;
            first = e ? end[-1] : 0;
            parts = end[0] - first;
        }
        const float *src = a.partial + ((size_t)(CHUNKED ? set * a.w.chunks + chunk : set) * a.w.parts + first) * part + min(col, a.N - 4);
#pragma unroll 2
        for (int j = 0; j < parts; ++j) {
            float4 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const float4 *>(src + (size_t)j * part + (size_t)min(r0 + ty + 16 * q, a.M - 1) * a.N);
#pragma unroll
            for (int q = 0; q < 4; ++q) { acc[q].x += v[q].x; acc[q].y += v[q].y; acc[q].z += v[q].z; acc[q].w += v[q].w; }
        }
    }
    T *dst = static_cast<T *>(a.dst[set]) + (size_t)e * part;
    if (!a.transposed[set]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = r0 + ty + 16 * q;
            if (r < a.M && col < a.N) store4_as<T>(dst + (size_t)r * a.N + col, acc[q]);
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float *t = &tile[ty + 16 * q][tx];
        t[0] = acc[q].x; t[1] = acc[q].y; t[2] = acc[q].z; t[3] = acc[q].w;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {            // 16 rows of the transposed tile per pass, 4 of its columns per thread
        const int rn = ty + 16 * q, n = c0 + rn, m = r0 + tx;
        if (n < a.N && m < a.M)
            store4_as<T>(dst + (size_t)n * a.M + m, make_float4(tile[tx][rn], tile[tx + 1][rn], tile[tx + 2][rn], tile[tx + 3][rn]));
    }
}

// Gate gradients of one unit (sample, slot) of a data-selected block from the row sums r_t = dL/dw_t, by NT threads: wave w takes
// picks w, w + waves, ...; d_patch_gate of the unit's expert [m] (zero where it picked nothing) and its d_expert_gate.  The
// unit of slot 0 also writes the zeros of the experts its sample did not select.
struct UnitGateLds {
    float ps[1024], row[1024];
    uint32_t chosen;
};
template <int NT> __device__ __forceinline__ void unit_gate_block(const SmhaBwdArgs &a, int g, void *lds)
{
    float *const ps = static_cast<UnitGateLds *>(lds)->ps, *const row = static_cast<UnitGateLds *>(lds)->row;
    uint32_t &chosen = static_cast<UnitGateLds *>(lds)->chosen;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = a.f.n, m = a.f.m, c = a.f.c;
    const int l_p = a.f.l / m, l_a = c * l_p;
    const int bb = g / a.f.k, i = clampi(a.f.expert_idx[g], n);
    const bool ge_on = a.flags & F_GATE_EXPERT, gp_on = a.flags & F_GATE_PATCH;
    if (g % a.f.k == 0) {
        if (tid == 0) chosen = 0;
        __syncthreads();
        if (tid < a.f.k) atomicOr(&chosen, 1u << clampi(a.f.expert_idx[g + tid], n));
        __syncthreads();
        for (int e = 0; e < n; ++e) {
            if (chosen >> e & 1u) continue;
            if (a.d_expert_gate && tid == 0) a.d_expert_gate[(size_t)bb * n + e] = 0.f;
            if (a.d_patch_gate)
                for (int j = tid; j < m; j += NT) a.d_patch_gate[((size_t)bb * n + e) * m + j] = 0.f;
        }
    }
    for (int j = tid; j < m; j += NT) row[j] = 0.f;
    if (!ge_on && !gp_on) {
        if (a.d_expert_gate && tid == 0) a.d_expert_gate[(size_t)bb * n + i] = 0.f;
        if (a.d_patch_gate)
            for (int j = tid; j < m; j += NT) a.d_patch_gate[((size_t)bb * n + i) * m + j] = 0.f;
        return;
    }
    const float *rt = a.rt + (size_t)g * l_a;
    const int parts = a.rt_parts > 1 ? a.rt_parts : 1;
    const size_t part_stride = (size_t)a.f.b * a.f.k * l_a;
    for (int t = wave; t < c; t += NT / 64) {
        float v = 0.f;
        for (int q = lane; q < l_p; q += 64)
#pragma unroll 4
            for (int part = 0; part < parts; ++part) v += rt[part * part_stride + t * l_p + q];
        v = wave_sum(v);
        if (lane == 0) ps[t] = v;
    }
    __syncthreads();
    const int32_t *pid = a.f.patch_idx + ((size_t)bb * n + i) * c;
    const float *gp = gp_on ? a.patch_gate + ((size_t)bb * n + i) * m : nullptr;
    if (a.d_patch_gate) {
        const float ge = ge_on ? a.expert_gate[(size_t)bb * n + i] : 1.0f;
        if (gp_on)
            for (int t = tid; t < c; t += NT) row[clampi(pid[t], m)] = ge * ps[t];
        __syncthreads();
        for (int j = tid; j < m; j += NT) a.d_patch_gate[((size_t)bb * n + i) * m + j] = row[j];
    }
    if (a.d_expert_gate && wave == 0) {
        float v = 0.f;
        if (ge_on)
            for (int t = lane; t < c; t += 64) v = fmaf(gp ? gp[clampi(pid[t], m)] : 1.0f, ps[t], v);
        v = wave_sum(v);
        if (lane == 0) a.d_expert_gate[(size_t)bb * n + i] = v;
    }
}

// Gate gradients beside another launch's work: `units` workgroups behind its own
struct UnitGates {
    static constexpr size_t LDS = sizeof(UnitGateLds);
    SmhaBwdArgs a;
    int units;
    template <int NT> __device__ __forceinline__ void run(int block, void *lds) const
    {
        if (block < units) unit_gate_block<NT>(a, block, lds);
    }
    static __host__ int count(const SmhaBwdArgs &a) { return a.d_expert_gate || a.d_patch_gate ? a.f.b * a.f.k : 0; }
};

// d_gate [b,n]: block (slot s, sample b) adds the slot's partial sums (256 strided subsets in index order, then a fixed tree: one order for
// any number of threads) into the entry of the slot's expert; the block of slot 0
// also writes the zeros of the experts the sample did not select (all of them without the gate flag).
constexpr int GATE_SUMS = 256;
template <int NT> __device__ __forceinline__ void uome_bwd_gate_block(const UomeBwdArgs &a, int s, int bb, float *red)   // NT threads, red: GATE_SUMS floats of LDS
{
    const int tid = threadIdx.x;
    const bool gated = a.flags & F_GATE_EXPERT;
    if (s == 0 && tid < a.n) {
        bool chosen = false;
#pragma unroll 8
        for (int q = 0; q < a.k; ++q) chosen |= clampi(a.expert_idx[bb * a.k + q], a.n) == tid;
        if (!chosen || !gated) a.d_gate[(size_t)bb * a.n + tid] = 0.f;
    }
    if (!gated) return;
    const float *src = a.gpart + ((size_t)bb * a.k + s) * a.gchunks;
    for (int i = tid; i < GATE_SUMS; i += NT) {
        float v = 0.f;
        for (int c = i; c < a.gchunks; c += GATE_SUMS) v += src[c];
        red[i] = v;
    }
    __syncthreads();
    for (int st = GATE_SUMS / 2; st > 0; st >>= 1) {
        for (int i = tid; i < st; i += NT) red[i] += red[i + st];
        __syncthreads();
    }
    if (tid == 0) a.d_gate[(size_t)bb * a.n + clampi(a.expert_idx[bb * a.k + s], a.n)] = red[0];
}

// the gate gradient's blocks behind the tiles of another launch
struct UomeGates {
    static constexpr int THREADS = 0;
    static constexpr bool OPTIONAL = false;
    static constexpr size_t LDS = GATE_SUMS * sizeof(float);
    UomeBwdArgs a;
    template <int NT> __device__ __forceinline__ void run(int block, void *lds) const
    {
        static_assert(NT >= 64, "a wave for the experts");
        uome_bwd_gate_block<NT>(a, block % a.k, block / a.k, static_cast<float *>(lds));
    }
};

// tiles of a reduction: columns, rows, all
struct RedGrid {
    int nx, ny, tiles;
    RedGrid(const WgradReduceArgs &ra, int sets) : nx((ra.N + RED_T - 1) / RED_T), ny((ra.M + RED_T - 1) / RED_T), tiles(nx * ny * sets * ra.n) {}
};

// the last launch of a data-selected MLP block whose gates did not fit beside another (at most 128 samples): the gate gradients' units
// (the longer chains, hence first) and the weight-gradient tiles
template <typename T> __global__ __launch_bounds__(256) void wgrad_reduce_gates_kernel(WgradReduceArgs ra, SmhaBwdArgs ga, int nx, int ny, int units)
{
    __shared__ __align__(16) unsigned char lds[RED_LDS > sizeof(UnitGateLds) ? RED_LDS : sizeof(UnitGateLds)];
    const int id = (int)blockIdx.x - units;
    if (id >= 0) wgrad_reduce_tile<T, false>(ra, reinterpret_cast<RedTile>(lds), id % nx, id / nx % ny, id / (nx * ny));
    else unit_gate_block<256>(ga, blockIdx.x, lds);
}

template <typename T> static inline hipError_t launch_wgrad_reduce_gates(const WgradReduceArgs &ra, int sets, const SmhaBwdArgs &ga, hipStream_t st)
{
    const RedGrid g(ra, sets);
    const int units = UnitGates::count(ga);
    hipLaunchKernelGGL((wgrad_reduce_gates_kernel<T>), dim3(g.tiles + units), dim3(256), 0, st, ra, ga, g.nx, g.ny, units);
    return hipGetLastError();
}

template <typename T> __global__ __launch_bounds__(256) void wgrad_reduce_kernel(WgradReduceArgs a, int nx, int ny)
{
    __shared__ __align__(16) unsigned char lds[RED_LDS];
    const int id = blockIdx.x;
    wgrad_reduce_tile<T, true>(a, reinterpret_cast<RedTile>(lds), id % nx, id / nx % ny, id / (nx * ny));
}

// tail not NULL: left to the launch that follows
template <typename T> static inline hipError_t launch_wgrad_reduce(const WgradReduceArgs &a, int sets, hipStream_t st, BwdTail *tail)
{
    if (tail && a.w.chunks == 1) {
        tail->reduce = a;
        tail->sets = sets;
        return hipSuccess;
    }
    const RedGrid g(a, sets);
    hipLaunchKernelGGL((wgrad_reduce_kernel<T>), dim3(g.tiles), dim3(256), 0, st, a, g.nx, g.ny);
    return hipGetLastError();
}

}  // namespace uoe
