// The expert selection (Eq. 21, 22): a launch of its own (route_select), or beside the first contraction of a block that selects experts only.
//
// As a launch it is 4 to 5 us of a chain of launches of 4 to 12 us, most of that its start, and the contraction behind it
// begins with lookups of what it wrote.  Every workgroup of the UoME block's first layer can instead add up its sample's partial logits
// (16 KB from L2 on the small shapes, four chunks a lane and load) and rank them for itself; the first one of a sample also writes the
// results.  Forward of 8 x 512 x 512 59.2 -> 57.2 us (5.0 + 12.2 -> 14.6 traced), 6 x 1000 x 360 76.1 -> 73.2.  With the patches as well (the SMHA block's projection) the chain was as long as the
// launch: 8 x 512 x 512, 8 x 16 logits 7.1 + 5.8 -> 13.2 us, 16 x 4096 x 256, 8 x 64 6.6 + 6.7 -> 23.
#pragma once
#include "common.h"

namespace uoe {

constexpr int SELECT_THREADS = 512;
constexpr int SELECT_BESIDE_VALUES = 16 * 1024;   // partial logits of a sample that a workgroup adds up beside its work
typedef float part4_t __attribute__((ext_vector_type(4), aligned(4)));   // four partials in a row, from any of them on

// Where a chunk's partial expert logits lie: a sample's and expert's of all chunks in a row, as the selection adds them up
__device__ __forceinline__ size_t zpart_at(const RouteArgs &a, int chunk, int bb, int e) { return ((size_t)bb * a.n + e) * a.nchunks + chunk; }

// The logits of a sample (without the noise) from its chunks' partials, by NT threads: a wave takes every NT/64th expert, a lane four chunks and the
// wave 256 a pass, then the lanes' sums are added.  The order does not depend on NT.
template <int NT> __device__ __forceinline__ void expert_logits(const RouteArgs &a, int bb, float *logit, int tid)
{
    constexpr int W = NT / 64, E = W >= 8 ? 1 : 2, PASSES = 2;   // E x PASSES loads in flight
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), at = (tid & 63) * 4, chunks = a.nchunks;
    for (int e0 = wave; e0 < a.n; e0 += E * W) {
        const float *src[E];
        float s[E];
#pragma unroll
        for (int i = 0; i < E; ++i) {
            src[i] = a.zpart + zpart_at(a, 0, bb, min(e0 + i * W, a.n - 1));
            s[i] = 0.f;
        }
        for (int c0 = at; c0 < chunks; c0 += PASSES * 256) {
            part4_t v[E][PASSES];
#pragma unroll
            for (int j = 0; j < PASSES; ++j)
                // the last lane's load may reach three values behind its row: the next row, or the workspace's next array
#pragma unroll
                for (int i = 0; i < E; ++i) v[i][j] = *reinterpret_cast<const part4_t *>(src[i] + (c0 + j * 256 < chunks ? c0 + j * 256 : c0));
#pragma unroll
            for (int j = 0; j < PASSES; ++j) {
                const int c = c0 + j * 256;
#pragma unroll
                for (int i = 0; i < E; ++i) {
                    const float two = (c + 2 < chunks ? v[i][j].z : 0.f) + (c + 3 < chunks ? v[i][j].w : 0.f);
                    s[i] += c < chunks ? (v[i][j].x + (c + 1 < chunks ? v[i][j].y : 0.f)) + two : 0.f;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const float z = wave_sum(s[i]);
            if ((tid & 63) == 0 && e0 + i * W < a.n) logit[e0 + i * W] = z;
        }
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

// The selection of sample bb by a workgroup of NT threads for itself; `write`: also to the routing results.  scratch: 32 floats of LDS.
// Ends on a barrier.
template <int NT>
__device__ __forceinline__ void select_experts_beside(const RouteSelect &s, int bb, float *scratch, SelectedExperts &out, bool write, int tid)
{
    const float noise = expert_noise(s.r, bb, tid);
    if (s.has_e) {
        expert_logits<NT>(s.r, bb, scratch, tid);
        __syncthreads();
    }
    if (tid < 64) rank_experts(s.r, bb, s.has_e, scratch, noise, write, &out, tid);
    __syncthreads();
}

}  // namespace uoe
