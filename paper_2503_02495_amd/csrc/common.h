// Shared device helpers and the internal launcher interface of libuoe (gfx950 only).
#pragma once
#include <cstdlib>
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "wgrad_plan.h"

namespace uoe {

// ---------------------------------------------------------------- storage types
struct bf16_t {
    uint16_t v;
};

// 16-byte accesses with the non-temporal hint, for bytes a call touches once: an output nobody reads
// again before the call ends, a residual at its last use.  Without the hint such streams displace, in L2
// and in the memory-side cache, the tensors that later kernels of the same call do read again
// (x, u, the hidden activations).  Operands that several workgroups share must NOT take it.
// `once` is decided on the host (stream_once): tensors that fit the caches keep the plain accesses, which
// let the next kernel find them there.
typedef unsigned int once_u32x4 __attribute__((ext_vector_type(4)));
template <bool ONCE> __device__ __forceinline__ void store16(void *p, uint4 v)
{
    const once_u32x4 w = {v.x, v.y, v.z, v.w};
    if constexpr (ONCE) __builtin_nontemporal_store(w, reinterpret_cast<once_u32x4 *>(p));
    else *reinterpret_cast<once_u32x4 *>(p) = w;
}
template <bool ONCE> __device__ __forceinline__ uint4 load16(const void *p)
{
    once_u32x4 w;
    if constexpr (ONCE) w = __builtin_nontemporal_load(reinterpret_cast<const once_u32x4 *>(p));
    else w = *reinterpret_cast<const once_u32x4 *>(p);
    return make_uint4(w.x, w.y, w.z, w.w);
}
// a tensor of this many bytes is streamed past the caches (measured: 67 MB and up gain, 34 MB and down lose);
// UOE_STREAM_ONCE_MIN_BYTES in the environment overrides the threshold (0: always, for tests of the hinted paths)
inline bool stream_once(size_t bytes)
{
    const char *env = getenv("UOE_STREAM_ONCE_MIN_BYTES");
    const double min_bytes = env ? atof(env) : 48.0 * 1048576.0;
    return (double)bytes >= min_bytes;
}

// Tile of a contraction of any size or in fp32 (launch_gemm_tail).  km: both operands along rows and columns (weight gradients);
// gaps_nk: rows that are absent from K segments, against [n][k] (d_x).
// bf16: 128x128 tiles (eight waves of 64x32, 16 waves a compute unit; four waves of 64x64 took 32.5 against 29.5 us on 128 x 196 x 768 x
// 384) once they give every compute unit one (fewer operand bytes per product), 64-row tiles below that, 32-row tiles where groups are
// that short.
// fp32, us on rows x K x columns (x: on the fp32 instruction); no tile that pads more than a tenth beyond 64x64:
//   128x128, four waves  512 and more: 16384 x 512 x 1024 114, 64x128 133, 64x64 143, with eight waves 147.  Two sets of accumulators leave 44
//                        to 60 bytes of scratch a lane, against [n][k] 164 to 224: a backward pass with d_u on it still 677 against 693 and
//                        704, but d_x, whose segments are two K-steps long, not (128 samples of 14 x 14 tokens 333 against 308 and 304)
//   64x128               512 and more: 4096 x 512 x 1024 38.1, 128x128 38.7, 64x64 40.8 (x 45.5)
//   64x64                4096 x 1024 x 512 39.5, 64x128 42.9 (x 44.7); 128 groups of 128 x 512 x 192 32.7, 64x128 40.2; groups of up to 64 rows: 512 of
//                        64 x 256 37.5, 64x128 41.5
//   64x64 x              up to 256 of them: a wave a SIMD cannot hide the chain read -> split -> product (1280 x 384 x 512 11.6 against 12.2; 24
//                        groups of 240 x 360 x 120 12.9 against 14.7)
//   32x64 x              up to 128 (2048 x 512 x 256 13.7 against 14.0; 160 of them 17.2 against 11.6), and short groups
// fp32 weight gradients (whole backward passes): 64x128 from 385 of them (504: 318 against 333 with 64x64; 512 of 32 rows 189 against 199; 216: 163
// against 158), 128x128 as above; the fp32 instruction gains nothing on few tiles.
struct TailTile {
    int rows, cols;
    bool exact;   // fp32: on the fp32 instruction
};
inline TailTile tail_tile(bool f32, bool km, bool gaps_nk, long groups, int rows, int cols)
{
    const auto up = [](int v, int to) { return (long)((v + to - 1) / to); };
    const auto tiles = [&](int bm, int bn) { return groups * up(rows, bm) * up(cols, bn); };
    if (!f32) {
        if (rows > 64 && tiles(128, 128) >= 256) return {128, 128, false};
        return {rows <= 32 && !km ? 32 : 64, 128, false};
    }
    const auto padded = [&](int bm, int bn) { return (double)tiles(bm, bn) * bm * bn / ((double)tiles(64, 64) * 64 * 64); };
    if (km) {
        if (rows > 64 && tiles(128, 128) >= 512 && padded(128, 128) <= 1.1) return {128, 128, false};
        if (tiles(64, 128) > 384 && padded(64, 128) <= 1.25) return {64, 128, false};
        return {64, 64, false};
    }
    if (rows <= 32 || tiles(64, 64) <= 128) return {32, 64, true};
    if (tiles(64, 64) <= 256) return {64, 64, true};
    if (rows > 64 && tiles(128, 128) >= 512 && padded(128, 128) <= 1.1 && !gaps_nk) return {128, 128, false};
    if (rows > 64 && tiles(64, 128) >= 512 && padded(64, 128) <= 1.1) return {64, 128, false};
    return {64, 64, false};
}

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return __uint_as_float(((uint32_t)x.v) << 16); }

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// two fp32 -> packed bf16, round to nearest even (one v_cvt_pk_bf16_f32 on gfx950; the same in integer arithmetic is four
// instructions a value)
__device__ __forceinline__ uint32_t pack2_bf16(float a, float b)
{
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

template <typename T> __device__ __forceinline__ T from_f32(float f);
template <> __device__ __forceinline__ float from_f32<float>(float f) { return f; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float f)
{
    bf16_t r;
    r.v = (uint16_t)pack2_bf16(f, f);
    return r;
}

// 8 consecutive elements (16-byte aligned for bf16, 32-byte span for fp32) -> fp32
__device__ __forceinline__ void load8(const float *p, float (&o)[8])
{
    const float4 a = *reinterpret_cast<const float4 *>(p);
    const float4 b = *reinterpret_cast<const float4 *>(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16_t *p, float (&o)[8])
{
    const uint4 a = *reinterpret_cast<const uint4 *>(p);
    o[0] = __uint_as_float(a.x << 16); o[1] = __uint_as_float(a.x & 0xFFFF0000u);
    o[2] = __uint_as_float(a.y << 16); o[3] = __uint_as_float(a.y & 0xFFFF0000u);
    o[4] = __uint_as_float(a.z << 16); o[5] = __uint_as_float(a.z & 0xFFFF0000u);
    o[6] = __uint_as_float(a.w << 16); o[7] = __uint_as_float(a.w & 0xFFFF0000u);
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Routing indices are caller data: clamp them into [0, count) so that a corrupt index can read the
// wrong row but never leave the tensor.
__device__ __forceinline__ int clampi(int v, int count) { return min(max(v, 0), count - 1); }

__device__ __forceinline__ float silu(float z) { return z / (1.0f + __expf(-z)); }
// The backward passes' sigmoid, 1 / (1 + e) with e = exp(-z): the hardware reciprocal and one step of Newton's iteration on (1 + e) 2^-32,
// scaled back at the end, so that results below 2^-126 (z <= -87.4, where the reciprocal alone is zero) come out as a division
// rounds them and infinite e gives 0.  The reciprocal is good to an ulp, the step squares that: what is left is one rounding, as in a
// division, with five instructions less (layer forward + backward of the lm shape 215.9 -> 214.9 us).  The minimum hands NaN through.
__device__ __forceinline__ float sigmoid_of(float e)   // 1 / (1 + e), e >= 0
{
    constexpr float scale = 2.3283064365386963e-10f;   // 2^-32
    const float d = __builtin_elementwise_minimum(fmaf(e, scale, scale), 8.507059173023462e37f), r = __builtin_amdgcn_rcpf(d);
    return fmaf(r, fmaf(-d, r, 1.0f), r) * scale;
}
__device__ __forceinline__ float sigmoid(float z) { return sigmoid_of(__expf(-z)); }
// SiLU with the hardware exp2 and reciprocal (about 1 ulp each): for epilogues that round the
// result to bf16 anyway
__device__ __forceinline__ float silu_fast(float z)
{
    return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}

// Sine and cosine of the rotary angle pos * theta (Eq. 32): the angle as the rounded product and its rounding error (angles
// reach thousands of radians), reduced by multiples of pi/2 held in three parts (Cody and Waite), Taylor polynomials of
// degree 9 and 10 on what is left, at most pi/4.  Largest and rms error against fp64 over the pairs of a head, sincosf of the rounded
// angle / the hardware's sine and cosine / this: rope_dim 2, 128 positions 5.1e-8 1.8e-8 / 1.9e-7 6.7e-8 / 5.0e-8 1.7e-8;
// rope_dim 32, 1024 positions 3.3e-5 2.1e-6 / 3.3e-5 2.1e-6 / 7.3e-6 9.7e-7; no range from 32 to 8192 positions and rope_dim 2
// to 128 where it is the larger one.
__device__ __forceinline__ void rope_sincos(float pos, float theta, float &sn, float &cs)
{
    constexpr double pio2 = 1.57079632679489661923;
    constexpr float p1 = (float)pio2, p2 = (float)(pio2 - (double)p1), p3 = (float)(pio2 - (double)p1 - (double)p2);
    const float angle = pos * theta, rest = fmaf(pos, theta, -angle), n = rintf(angle * (float)(1.0 / pio2));
    const float r = fmaf(-n, p3, fmaf(-n, p2, fmaf(-n, p1, angle))) + rest, z = r * r;
    const float s = fmaf(r * z, fmaf(z, fmaf(z, fmaf(z, 1.f / 362880.f, -1.f / 5040.f), 1.f / 120.f), -1.f / 6.f), r);
    const float c = fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, -1.f / 3628800.f, 1.f / 40320.f), -1.f / 720.f), 1.f / 24.f), -0.5f), 1.f);
    const int q = (int)n;
    const float a = q & 1 ? c : s, b = q & 1 ? s : c;
    sn = q & 2 ? -a : a;
    cs = (q + 1) & 2 ? -b : b;
}
// theta_i of the pair at offset 2i of the rotary part
__device__ __forceinline__ float rope_theta(int offset, int rope_dim)
{
    return exp2f(-((float)offset / (float)rope_dim) * 13.287712379549449f);  // log2(10000)
}

// ---------------------------------------------------------------- flags (mirror of the ABI values)
constexpr uint32_t F_RESIDUAL = 1u, F_GATE_EXPERT = 2u, F_GATE_PATCH = 4u, F_CAUSAL = 8u;

// ---------------------------------------------------------------- launcher arguments
struct RouteArgs {
    const void *x, *w_e, *w_b, *w_a;          // w_e NULL: no expert router; w_b NULL: no data router
    const float *noise_e, *noise_p;
    int b, l, d, n, k, m, c;
    int tc, nchunks;                          // expert router: tokens per chunk, chunks per sample
    int tc_d, nchunks_d;                      // data router: the same
    int zgroups;                              // 512 / n: the order of the logits' sums (select.h)
    float *zpart, *gpart;                     // [b, n, nchunks], [nchunks_d, b, n*m]
    float *gred;                              // [b, n*m]
    float *t1;                                // [b, l, n]: per-token expert scores x W_B of the one-pass kernel
    int32_t *expert_idx, *patch_idx;          // outputs (any may be NULL)
    float *expert_gate, *patch_gate;
    // dynamic capacity (Eq. 15-16) and balance statistics (Eq. 43-44): capacity NULL = not asked for
    int patch_k;                              // experts each patch names in stage 1
    int32_t *capacity;                        // [b]
    float *load_f, *load_p;                   // [b,n] each, or NULL
};
// An expert selection that the block's first contraction makes beside its own work (select.h); on 0: it has been launched
struct RouteSelect {
    RouteArgs r;
    int on, has_e;
    int most;   // in: with more partial logits a sample it is launched (uome_select_values)
};

struct SmhaArgs {
    const void *x, *wq, *wk, *wv, *wo;
    const int32_t *expert_idx, *patch_idx;
    const float *expert_gate, *patch_gate;    // NULL when the matching flag is off
    void *out;
    int b, l, d, n, k, m, c, d_h;
    uint32_t flags;
    int rope_dim;                             // rotary dims at the end of a head (Eq. 32), 0 = none
    const unsigned char *pad_mask;            // [b,l] 1 = token, 0 = padding (Eq. 41), or NULL
    // workspace
    void *q, *kk, *v, *o, *o_lo;              // [b*k, l_a, d_h] each, storage dtype (o_lo: low part of o, bf16 storage)
    float *lse;                               // [b*k, l_a] or NULL: base-2 log-sum-exp of each query's scaled logits
                                              // (MFMA attention only; kept for the backward pass)
    // also written when not NULL (bf16 MFMA path): a bf16 copy of v and the attention output without its gate weight as a
    // (hi, lo) pair.  With lse they are what the backward pass of the same call needs of the forward one
    void *v_copy, *o_raw, *o_raw_lo;
    int keep_v_bf16;                          // 1: the MFMA path leaves v in bf16 (the backward pass reads it); 0: it
                                              // writes v as fp16, the operand format of the attention kernel's P V
    uint32_t skip;                            // steps NOT to run (SMHA_STEP_* bits; 0 = the whole block): a caller
                                              // that times one step runs it on what the others left in the workspace
};
constexpr uint32_t SMHA_STEP_QKV = 1u, SMHA_STEP_ATTENTION = 2u, SMHA_STEP_OUT = 4u;

struct UomeArgs {
    const void *u, *a_in, *a_out;
    const int32_t *expert_idx;
    const float *expert_gate;                 // NULL when GATE_EXPERT is off
    void *out;
    int b, l, d, n, k, d_e;
    uint32_t flags;
    void *hidden;                             // [b, l, k*d_e], storage dtype
    const RouteSelect *select;                // the block's selection, to be made by the first layer's launch; NULL: it is there
};

// UoME with patch-wise data selection (Eq. 37-40): routing as for SMHA, hidden per active unit
struct UomeDsArgs {
    const void *u, *a_in, *a_out;
    const int32_t *expert_idx, *patch_idx;
    const float *expert_gate, *patch_gate;    // NULL when the matching flag is off
    void *out;
    int b, l, d, n, k, m, c, d_e;
    uint32_t flags;
    void *hidden;                             // [b*k, l_a, d_e], storage dtype
};

// Backward pass of the expert-selection UoME block
struct UomeBwdArgs {
    const void *u, *a_in, *a_out, *d_out;
    const int32_t *expert_idx;
    const float *expert_gate;                 // NULL when GATE_EXPERT is off
    void *d_u, *d_a_in, *d_a_out;             // [b,l,d], [n,d,d_e], [n,d_e,d], storage dtype
    float *d_gate;                            // [b,n] or NULL
    int b, l, d, n, k, d_e;
    uint32_t flags;
    // workspace, storage dtype unless noted
    void *z, *dz, *h;                         // [b, l, k*d_e] each
    void *dh;                                 // any-shape path: dH, fp32
    float *gpart;                             // [b, k, gchunks] partial sums of d_gate
    float *partial;                           // [2*chunks*parts, d_e, d] partial tiles of the two weight gradients
    int32_t *part_end;                        // [chunks, 32] first part id behind an expert's
    int gchunks;
    WgradPlan wgrad;
    void *h_op, *dz_op;                       // any-shape path: H and dZ as left operands (may be z and dh themselves)
    // data-selection mode (patch_idx != NULL): units = (sample, slot) with l_a = c*l/m gathered rows;
    // z, dz, h are [units, l_a, d_e]
    const int32_t *patch_idx;
    const float *patch_gate;                  // NULL when GATE_PATCH is off
    float *d_patch_gate;                      // [b,n,m] or NULL
    float *rt;                                // [parts, units, l_a]: parts of dL/d(weight of row t)
    int m, c;
};

// Backward pass of the SMHA block
struct SmhaBwdArgs {
    SmhaArgs f;                               // the forward call that is recomputed: no gates in f.flags, f.lse set
    int kept;                                 // 1: its q, k, v (and o, o_lo, lse on the bf16 path) are there already
    const void *d_out;                        // [b,l,d]
    const float *expert_gate, *patch_gate;    // as in the forward call (NULL when the flag is off)
    uint32_t flags;                           // the block's flags
    void *d_x, *d_wq, *d_wk, *d_wv, *d_wo;    // [b,l,d], 3 x [n,d,d_h], [n,d_h,d], storage dtype
    float *d_expert_gate, *d_patch_gate;      // [b,n], [b,n,m], or NULL
    // workspace, storage dtype unless noted
    float *do_raw;                            // any-shape path: [units, l_a, d_h] fp32
    void *d_o;                                // [units, l_a, d_h]
    void *dqkv;                               // [units, l_a, 3*d_h]
    float *rt, *dd;                           // [units, l_a] each: dL/dw_t and the softmax row term
    float *inv_sum;                           // any-shape path: [units, l_a] 1 / softmax row sum; f.lse holds the row maximum there
    int rt_parts;                             // rt is that many arrays to be added (0: one), set by the launcher
    float *partial;                           // [4*chunks*parts, d_h, d] partial tiles of the four weight gradients
    int32_t *part_end;                        // [chunks, 32] first part id behind an expert's
    WgradPlan wgrad;
    void *og;                                 // w o [units, l_a, d_h]; any-shape path: [units, l_a, parts, d_h], do_raw, q, k, v are
                                              // fp32 there and dqkv is [units, l_a, parts, 3*d_h]
};

// Reduction of split weight-gradient tiles (wgrad_reduce.h): partial [sets*chunks*parts][M][N] fp32 -> storage dtype
struct WgradReduceArgs {
    const float *partial;
    void *dst[4];   // storage type T of the launch
    int transposed[4];
    int n, M, N;
    const int32_t *part_end;   // [chunks, 32] first part id behind an expert's
    WgradPlan w;
};

// Launch shape of the routers' backward pass: d_x in chunks of pieces (8 columns) x groups of samples, dW_E in chunks
// of pieces x groups of 8 experts, t1 and dW_B in chunks of the b*l tokens x slices of columns
constexpr int ROUTE_BWD_TILE = 32, ROUTE_BWD_SLICE = 256;
struct RouteBwdPlan {
    int data_blocks, wb_chunks, chunk_tokens, slices, slice_w;
    int dx_blocks, dx_chunks, dx_groups, dx_bg, dx_pieces, dx_reps;
    int w_blocks, w_chunks, w_groups, wsplit, w_reps;
};
RouteBwdPlan route_bwd_plan(int b, int l, int d, int n, bool has_e, bool has_d);

// Backward pass of the routers of one block
struct RouteBwdArgs {
    const void *x, *w_e, *w_b, *w_a;          // w_e NULL: no expert router; w_b NULL: no data router
    const float *g_e, *g_p;                   // gates of the forward pass [b,n], [b,n,m]
    const float *d_g_e, *d_g_p;               // their gradients
    void *d_x;                                // [b,l,d] in/out: the routers' contribution is added
    void *d_w_e, *d_w_b, *d_w_a;              // [n,l*d], [d,n], [l,m], storage dtype
    int b, l, d, n, m;
    // workspace (fp32 but wbt), used by the data router only
    float *dl;                                // [b,n,m]: gradients of the patch logits
    float *u;                                 // [b,l,n]: W_A dL^T
    float *t1;                                // [slices,b,l,n]: x W_B, one part per slice of columns
    float *wb_part;                           // [wb_chunks,d,n] partial sums of dW_B
    void *wbt;                                // [n,d] W_B transposed, storage dtype
    RouteBwdPlan plan;                        // set by the launcher
};

// What a block's backward pass leaves to, or does for, the routers' backward pass that follows it in a chain of calls: the reduction of the
// weight gradients runs beside that pass's main launch, and where the block's last launch has room, that pass's first one beside it
struct BwdTail {
    WgradReduceArgs reduce;
    int sets;                  // of the reduction, 0: it has been launched
    const RouteBwdArgs *prep;  // in: the routers' pass, NULL: it has no data router
    int prep_done;
};

struct GatherArgs {
    const void *x;
    const int32_t *expert_idx, *patch_idx;
    void *h;
    int b, l, d, n, k, m, c;
};

// Launchers: enqueue on `st`, return the runtime's launch status.
// `beside` not NULL: the block's first contraction can make the selection; where that pays *beside says so and it is not launched
hipError_t launch_route(const RouteArgs &a, bool bf16, hipStream_t st, RouteSelect *beside = nullptr);
hipError_t launch_balance_loss(const float *load_f, const float *load_p, float alpha, float *loss, float *d_patch_gate,
                               int b, int n, int m, hipStream_t st);
hipError_t launch_gather(const GatherArgs &a, bool bf16, hipStream_t st);
hipError_t launch_smha(const SmhaArgs &a, bool bf16, hipStream_t st);
// Eq. 28-34 of the MFMA path only (projections, rotary embedding, attention into a.o / a.o_lo / a.lse);
// the caller has checked bf16 storage, d % 32 == 0 and d_h in {32, 64, 128}
hipError_t launch_smha_qkv_attention(const SmhaArgs &a, hipStream_t st);
hipError_t launch_uome(const UomeArgs &a, bool bf16, hipStream_t st);
int uome_mlp_waves(const UomeArgs &a);                                      // not 0: both layers in one launch (uome_mlp.hip), bf16
hipError_t launch_uome_mlp(const UomeArgs &a, hipStream_t st);
int uome_select_values(const UomeArgs &a, bool bf16);                       // RouteSelect::most for the block's first launch; 0: never
hipError_t launch_uome_up(const UomeArgs &a, bool bf16, hipStream_t st);    // Eq. 38 only
hipError_t launch_uome_down(const UomeArgs &a, bool bf16, hipStream_t st);  // Eq. 39-40 only
hipError_t launch_uome_ds(const UomeDsArgs &a, bool bf16, hipStream_t st);
hipError_t launch_uome_backward(const UomeBwdArgs &a, hipStream_t st, BwdTail *tail = nullptr);
hipError_t launch_smha_backward(const SmhaBwdArgs &a, hipStream_t st, BwdTail *tail = nullptr);
// rotary embedding (Eq. 32) of fp32 q and k with rows of d_h
hipError_t launch_rope_f32(const SmhaArgs &a, hipStream_t st);
// backward passes for the shapes and storage types the 32-multiple bf16 kernels do not take
hipError_t launch_uome_backward_any(const UomeBwdArgs &a, bool bf16, hipStream_t st, BwdTail *tail = nullptr);
hipError_t launch_smha_backward_any(const SmhaBwdArgs &a, bool bf16, hipStream_t st, BwdTail *tail = nullptr);
constexpr int BWD_ANY_SEGMENTS = 1024;        // (unit, pick) entries one part of an expert's weight gradient holds
// `tail`: of the block's backward pass before it (at most 128 samples)
hipError_t launch_route_backward(const RouteBwdArgs &a, bool bf16, hipStream_t st, const BwdTail *tail = nullptr);
int uome_backward_gate_chunks(int l, int d_e);

// measurement probes (probe.hip)
constexpr unsigned PROBE_READ_BLOCKS = 256 * 16, PROBE_MFMA_BLOCKS = 256 * 2;
hipError_t launch_probe_copy(const void *src, void *dst, size_t bytes, hipStream_t st);
hipError_t launch_probe_read(const void *src, size_t bytes, uint32_t *sink, hipStream_t st);
hipError_t launch_probe_mfma(const void *operands, int iters, float *sink, hipStream_t st);

// host-side sizing shared by api.hip and the launchers
int route_tokens_per_chunk(int b, int l, int d, int n, int m, bool bf16);
int route_expert_mfma_tokens_per_chunk(int b, int l, int d, int n);
int route_data_tokens_per_chunk(int b, int l, int d, int n, int m, bool bf16);
// streaming router kernel: applicability and launch shape (host side)
constexpr int ROUTE_STREAM_CHUNKS = 256;      // one workgroup per compute unit
struct RouteStreamPlan {
    bool ok;             // the kernel applies to this shape
    int rt, ct, rb;      // 16-sample tiles per workgroup, 16-expert tiles, bytes per row per stage
    int tpc, nchunks;    // tokens per chunk, chunks
    int ipw;             // load instructions per wave per stage
    size_t lds;          // dynamic LDS bytes
};
RouteStreamPlan route_stream_plan(int b, int l, int d, int n, bool bf16, bool has_d);
struct RouteFoldPlan {
    int tr, ranges;      // tokens per range, ranges per sample
};
RouteFoldPlan route_fold_plan(int b, int l);

}  // namespace uoe
