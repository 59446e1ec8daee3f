// The expert selection (Eq. 21, 22): a launch of its own (route_select), or beside the first contraction of a block that selects experts only.
//
// As a launch it is 4 to 5 us of a chain of launches of 4 to 12 us, most of that its start, and the contraction behind it
// begins with lookups of what it wrote.  Every workgroup of the UoME block's first layer can instead add up its sample's partial logits
// (16 KB from L2 on the small shapes) and rank them for itself; the first one of a sample also writes the
// results.  Forward of 8 x 512 x 512 59.2 -> 57.4 us (5.0 + 12.2 -> 14.6 traced), 6 x 1000 x 360 76.1 -> 73.2.  With the patches as well (the SMHA block's projection) the chain was as long as the
// launch: 8 x 512 x 512, 8 x 16 logits 7.1 + 5.8 -> 13.2 us, 16 x 4096 x 256, 8 x 64 6.6 + 6.7 -> 23.
#pragma once
#include "common.h"

namespace uoe {

constexpr int SELECT_THREADS = 512;

// Where a chunk's partial expert logits lie: a sample's and expert's of all chunks in a row
__device__ __forceinline__ size_t zpart_at(const RouteArgs &a, int chunk, int bb, int e) { return ((size_t)bb * a.n + e) * a.nchunks + chunk; }

// a lane's value plus that of the lane whose number differs in one bit, 16 lanes at a time: after the steps before, all lanes of a quad (and of
// half a row) hold the same, so that the mirrored lane's is the same number
template <int CTRL> __device__ __forceinline__ float add_dpp(float v)
{
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_sum(float v)
{
    v = add_dpp<0xB1>(v);      // quad_perm 1 0 3 2
    v = add_dpp<0x4E>(v);      // quad_perm 2 3 0 1
    v = add_dpp<0x141>(v);     // row_half_mirror
    return add_dpp<0x140>(v);  // row_mirror
}

// The logits of a sample (without the noise) from its chunks' partials, by NT threads, in one order whoever selects: chunks whose numbers are equal
// modulo zgroups (512 / n of them) one after the other, then the sums of groups equal modulo 16, then these 16 by halves.  A thread has 512 / NT
// (expert, group) pairs, neighbours' groups side by side as their chunks in memory, and all their partials in flight up to 32 or 16 each (as many as
// leave a contraction's occupancy alone).  sums: 512 floats of LDS.
// (In rows sorted by group a thread has 16 bytes a load, but the expert router then either writes its partials scattered or takes its chunks out of
// order: forward of 4 x 8192 x 1024 520.9 -> 525.0 us, 20 x 1440 x 704 158.6 -> 163.7.  A wave an expert and 16 in flight: 2 x 960 x 160, 10 and 13
// experts, 52.5 us.)
template <int NT> __device__ __forceinline__ void expert_logits(const RouteArgs &a, int bb, float *sums, float *logit, int tid)
{
    constexpr int ITEMS = SELECT_THREADS / NT, PASSES = ITEMS > 2 ? 4 : 8;
    const int n = a.n, step = a.zgroups;
    const float inv = __builtin_amdgcn_rcpf((float)step);   // (good enough for quotients of up to 512)
    int left[ITEMS];   // chunks of the row from the pair's first on; 0: none of its own
    const float *src[ITEMS];
    float s[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int p = tid + i * NT, e = (int)((p + 0.5f) * inv), g = p - e * step;
        left[i] = e < n ? max(a.nchunks - g, 0) : 0;
        src[i] = a.zpart + zpart_at(a, min(g, a.nchunks - 1), bb, min(e, n - 1));
        s[i] = 0.f;
    }
    for (int at = 0; at < a.nchunks; at += PASSES * 4 * step) {
        float v[ITEMS][PASSES][4];
#pragma unroll
        for (int q = 0; q < PASSES; ++q)
            if (q == 0 || at + q * 4 * step < a.nchunks)
#pragma unroll
                for (int i = 0; i < ITEMS; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[i][q][c] = src[i][at + (q * 4 + c) * step < left[i] ? at + (q * 4 + c) * step : 0];
#pragma unroll
        for (int q = 0; q < PASSES; ++q)
            if (q == 0 || at + q * 4 * step < a.nchunks)
#pragma unroll
                for (int i = 0; i < ITEMS; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c) s[i] += at + (q * 4 + c) * step < left[i] ? v[i][q][c] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) sums[tid + i * NT] = s[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int e = (tid + i * NT) / 16, l16 = tid & 15;
        if (e >= n) break;
        float z = 0.f;
#pragma unroll 4
        for (int g = l16; g < step; g += 16) z += sums[e * step + g];
        z = row_sum(z);
        if (l16 == 0) logit[e] = z;
    }
}

// the noise on a lane's expert, to be fetched before the sums are waited for
__device__ __forceinline__ float expert_noise(const RouteArgs &a, int bb, int lane)
{
    return a.noise_e && lane < a.n ? a.noise_e[(size_t)bb * a.n + lane] : 0.f;
}

// what a workgroup keeps of its own selection: the sample's experts by slot and their gates
struct SelectedExperts {
    int expert[32];
    float gate[32];
};
struct NoSelect {};

// Eq. 21 softmax -> Eq. 22 top-k of one sample by one wave, to `out` (may be NULL) and, `write`, to the routing results.  The softmax is
// strictly increasing in the logit within a sample, so the k largest gates are the k largest logits: rank on the
// logits, which cannot underflow.
__device__ __forceinline__ void rank_experts(const RouteArgs &a, int bb, int has_e, const float *logit, float noise, bool write, SelectedExperts *out, int lane)
{
    const int n = a.n;
    const bool in = lane < n;
    const float z = !in ? -INFINITY : (has_e ? logit[lane] + noise : 0.f);
    float mx = z;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    const float own = in ? expf(z - mx) : 0.f;
    float den = own;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) den += __shfl_xor(den, off, 64);
    const float gate = has_e ? own / den : 1.0f;
    if (in && write && a.expert_gate) a.expert_gate[(size_t)bb * n + lane] = gate;
    int rank = 0;
#pragma unroll
    for (int ii = 0; ii < 32; ++ii) {
        const float w = __shfl(z, ii, 64);
        rank += ii < n && (w > z || (w == z && ii < lane)) ? 1 : 0;
    }
    const bool kept = in && rank < a.k;
    const uint64_t mask = __ballot(kept);
    const int pos = __popcll(mask & ((1ull << lane) - 1));
    if (!kept || pos >= a.k) return;
    if (out) {
        out->expert[pos] = lane;
        out->gate[pos] = gate;
    }
    if (write && a.expert_idx) a.expert_idx[(size_t)bb * a.k + pos] = lane;
}

// The selection of sample bb by a workgroup of NT threads for itself; `write`: also to the routing results.  scratch: 544 floats of LDS.
// Ends on a barrier.
template <int NT>
__device__ __forceinline__ void select_experts_beside(const RouteSelect &s, int bb, float *scratch, SelectedExperts &out, bool write, int tid)
{
    const float noise = expert_noise(s.r, bb, tid);
    if (s.has_e) {
        expert_logits<NT>(s.r, bb, scratch, scratch + SELECT_THREADS, tid);
        __syncthreads();
    }
    if (tid < 64) rank_experts(s.r, bb, s.has_e, scratch + SELECT_THREADS, noise, write, &out, tid);
    // Nothing of it may be in flight for the compiler (vmcnt 0, in a form that it reads): partials that not all lanes' sums took stay so, and its
    // wait before their registers' next use stood in the contraction's loop, where it waits for the copies of every K-step
    // (30 x 156 tokens, d 928, 96 hidden columns: the layer's forward 68.4 us, 66.1 with the selection as a launch).
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
}

}  // namespace uoe
