// Backward pass of the two routers (Eq. 21 and Eq. 13-14) for given gradients of their gates.
//   expert router: z = W_E vec(x), g = softmax_n(z):  dz = g * (dg - sum_i g_i dg_i),
//                  dW_E = dz^T vec(x),  d_x += dz W_E
//   data router:   L = (x W_B)^T W_A per sample, gate = softmax over experts for each patch:
//                  dL = gate * (dgate - sum_i gate_i dgate_i),  U = W_A dL^T [l,n],
//                  dW_A = sum_b (x W_B) dL,  dW_B = sum_b x^T U,  d_x += U W_B^T
// All of it is streaming over x, W_E, dW_E and d_x with n <= 32 outputs per element: bound by HBM on large
// tensors and by the depth of the chain of launches on small ones.  Hence at most three launches:
//   prep    dL, U and W_B^T (nothing of size l*d; skipped without a data router),
//   main    three independent kinds of workgroup side by side: dW_E from x; d_x from W_E, U and W_B^T, read and
//           written once for both routers; t1 = x W_B and partial sums of dW_B from x,
//   finish  dW_A from t1 and dL, the ordered sum of the dW_B partials (skipped without a data router).
// The thin contractions (K = tokens, d, m or b*n; n columns) run on v_mfma_f32_16x16x4_f32, which multiplies and
// adds in fp32 and takes one scalar per lane and operand, so a plain row-major LDS tile serves as left operand
// in either orientation.  Summation orders are fixed: no atomics.
#include "common.h"
#include "route_prep.h"
#include "wgrad_reduce.h"
#include <type_traits>

namespace uoe {

// pack2_bf16 for the ends of long sums: with the conversion in sight the compiler sums pairs of values as vectors and keeps the
// loads of the whole unrolled loop in registers (592 bytes of scratch a lane, 158 -> 932 us on the largest shape)
__device__ __forceinline__ uint32_t pack2_sums(float a, float b)
{
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

template <typename T> __device__ __forceinline__ void store8(T *p, const float (&v)[8]);
template <> __device__ __forceinline__ void store8<float>(float *p, const float (&v)[8])
{
    *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4 *>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
template <> __device__ __forceinline__ void store8<bf16_t>(bf16_t *p, const float (&v)[8])
{
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = pack2_sums(v[2 * e], v[2 * e + 1]);
    *reinterpret_cast<uint4 *>(p) = make_uint4(w[0], w[1], w[2], w[3]);
}

// W_E and its gradient are read or written once per call and are larger than the memory-side cache on the
// big shapes: with ONCE (chosen per launch, stream_once) their 16-byte accesses carry the non-temporal hint,
// so that they do not push x and d_x out of the caches.  fp32 storage keeps the plain accesses.
template <bool ONCE> __device__ __forceinline__ void load8_w(const float *p, float (&o)[8]) { load8(p, o); }
template <bool ONCE> __device__ __forceinline__ void load8_w(const bf16_t *p, float (&o)[8])
{
    const uint4 a = load16<ONCE>(p);
    o[0] = __uint_as_float(a.x << 16); o[1] = __uint_as_float(a.x & 0xFFFF0000u);
    o[2] = __uint_as_float(a.y << 16); o[3] = __uint_as_float(a.y & 0xFFFF0000u);
    o[4] = __uint_as_float(a.z << 16); o[5] = __uint_as_float(a.z & 0xFFFF0000u);
    o[6] = __uint_as_float(a.w << 16); o[7] = __uint_as_float(a.w & 0xFFFF0000u);
}
template <bool ONCE> __device__ __forceinline__ void store8_w(float *p, const float (&v)[8]) { store8<float>(p, v); }
template <bool ONCE> __device__ __forceinline__ void store8_w(bf16_t *p, const float (&v)[8])
{
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = pack2_sums(v[2 * e], v[2 * e + 1]);
    store16<ONCE>(p, make_uint4(w[0], w[1], w[2], w[3]));
}

template <typename T> struct RawPiece;   // 8 elements as loaded
template <> struct RawPiece<bf16_t> { uint4 v[1]; };
template <> struct RawPiece<float> { uint4 v[2]; };

template <typename T> __global__ __launch_bounds__(256) void route_bwd_prep_kernel(RoutePrep<T> p)
{
    __shared__ __align__(16) unsigned char lds[RoutePrep<T>::LDS];
    p.template run<256>(blockIdx.x, lds);
}

// gates and gate gradients of nb samples into LDS: softmax_bwd walks a row n times
__device__ __forceinline__ void stage_gates(const RouteBwdArgs &a, float *gs, int b0, int nb)
{
    for (int idx = threadIdx.x; idx < nb * a.n; idx += 256) {
        gs[idx] = a.g_e[(size_t)b0 * a.n + idx];
        gs[nb * a.n + idx] = a.d_g_e[(size_t)b0 * a.n + idx];
    }
    __syncthreads();
}

// ---- main launch, kind 1: dW_E[i, q] = sum_b dz[b,i] x[b,q], 8 consecutive q and 8 experts per thread.
// With split (few columns, many samples) eight lanes of a wave share the samples of one 8-column piece and end up
// with one expert each: three halving exchanges instead of eight times as long a chain of loads (b 128, l*d 75264:
// the whole launch 53 + 15 -> 24 us).
template <typename T, bool ONCE> __device__ __forceinline__ void bwd_wexpert(const RouteBwdArgs &a, float *dzs, int chunk0, int e0)
{
    constexpr int EG = 8;
    const long ld = (long)a.l * a.d;
    const int tid = threadIdx.x, lane = tid & 63, ne = min(EG, a.n - e0);
    float *gs = dzs + a.b * EG;
    stage_gates(a, gs, 0, a.b);
    for (int idx = tid; idx < a.b * EG; idx += 256) {
        const int bb = idx / EG, e = idx % EG;
        dzs[idx] = e < ne ? softmax_bwd(gs + bb * a.n, gs + (a.b + bb) * a.n, a.n, 1, e0 + e) : 0.f;
    }
    __syncthreads();
    const bool split = a.plan.wsplit;
    const int last = min(chunk0 + 8 * a.plan.w_reps, a.plan.w_chunks);
    for (int chunk = chunk0; chunk < last; chunk += 8) {
        const long q = split ? ((long)chunk * 32 + (tid >> 6) * 8 + (lane & 7)) * 8 : ((long)chunk * 256 + tid) * 8;
        const bool live = q < ld;
        const T *x = static_cast<const T *>(a.x) + (live ? q : 0);
        float acc[EG][8];
#pragma unroll
        for (int e = 0; e < EG; ++e)
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[e][c] = 0.f;
        const int b0 = split ? lane >> 3 : 0, bs = split ? 8 : 1;
#pragma unroll 4
        for (int bb = b0; bb < a.b; bb += bs) {
            float xv[8];
            load8(x + (size_t)bb * ld, xv);
#pragma unroll
            for (int e = 0; e < EG; ++e) {
                const float w = dzs[bb * EG + e];
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[e][c] = fmaf(w, xv[c], acc[e][c]);
            }
        }
        T *dw = static_cast<T *>(a.d_w_e) + q;
        if (!split) {
#pragma unroll
            for (int e = 0; e < EG; ++e)
                if (live && e < ne) store8_w<ONCE>(dw + (size_t)(e0 + e) * ld, acc[e]);
            continue;
        }
#pragma unroll
        for (int half = 4; half >= 1; half >>= 1) {
            const bool upper = (lane >> 3) & half;
#pragma unroll
            for (int e = 0; e < half; ++e)
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const float lo = acc[e][c], hi = acc[e + half][c];
                    acc[e][c] = (upper ? hi : lo) + __shfl_xor(upper ? lo : hi, half * 8, 64);
                }
        }
        if (live && (lane >> 3) < ne) store8_w<ONCE>(dw + (size_t)(e0 + (lane >> 3)) * ld, acc[0]);
    }
}

// ---- kind 2: d_x[b, (t,e)] += sum_i dz[b,i] W_E[i,(t,e)] + sum_i U[b,t,i] W_B[e,i]: 8 consecutive e and BG samples
// per thread, so W_E is read once per BG samples and d_x read, updated and rounded once for both routers.
template <typename T, int BG, bool ONCE> __device__ __forceinline__ void bwd_dx(const RouteBwdArgs &a, float *smem, int chunk0, int b0)
{
    const long ld = (long)a.l * a.d;
    const int tid = threadIdx.x, nb = min(BG, a.b - b0), pieces = a.plan.dx_pieces, P = a.d / 8;
    float *dzs = smem, *us = smem + a.n * BG;  // [n][BG], [n][tokens][BG]
    if (a.w_e) {
        stage_gates(a, us, b0, nb);
        for (int idx = tid; idx < a.n * BG; idx += 256) {
            const int i = idx / BG, s = idx % BG;
            dzs[idx] = s < nb ? softmax_bwd(us + s * a.n, us + (nb + s) * a.n, a.n, 1, i) : 0.f;
        }
        __syncthreads();
    }
    const int last = min(chunk0 + 8 * a.plan.dx_reps, a.plan.dx_chunks);
    for (int chunk = chunk0; chunk < last; chunk += 8) {
        const long p0 = (long)chunk * pieces, p = p0 + tid, q = p * 8;
        const int t0 = (int)(p0 / P), t1 = (int)min((p0 + pieces - 1) / P, (long)a.l - 1), nt = t1 - t0 + 1;
        if (a.w_b) {
            if (chunk != chunk0) __syncthreads();
            for (int idx = tid; idx < nt * a.n * BG; idx += 256) {
                const int s = idx / (nt * a.n), k = idx - s * nt * a.n, tk = k / a.n, i = k - tk * a.n;
                us[(i * nt + tk) * BG + s] = a.u[((size_t)(b0 + min(s, nb - 1)) * a.l + t0) * a.n + k];
            }
            __syncthreads();
        }
        if (tid >= pieces || q >= ld) continue;
        const int t = (int)(p / P), e = (int)(p - (long)t * P) * 8;
        T *dx = static_cast<T *>(a.d_x) + (size_t)b0 * ld + q;
        RawPiece<T> cur[BG];
        float de[BG][8];
#pragma unroll
        for (int s = 0; s < BG; ++s) {
#pragma unroll
            for (int c = 0; c < 8; ++c) de[s][c] = 0.f;
            cur[s] = *reinterpret_cast<const RawPiece<T> *>(dx + (size_t)(s < nb ? s : 0) * ld);
        }
        if (a.w_e) {
            const T *w = static_cast<const T *>(a.w_e) + q;
#pragma unroll 4
            for (int i = 0; i < a.n; ++i) {
                float wv[8];
                load8_w<ONCE>(w + (size_t)i * ld, wv);
#pragma unroll
                for (int s = 0; s < BG; ++s) {
                    const float z = dzs[i * BG + s];
#pragma unroll
                    for (int c = 0; c < 8; ++c) de[s][c] = fmaf(z, wv[c], de[s][c]);
                }
            }
        }
        if (a.w_b) {
            const T *w = static_cast<const T *>(a.wbt) + e;
            const float *ut = us + (t - t0) * BG;
#pragma unroll 4
            for (int i = 0; i < a.n; ++i) {
                float wv[8];
                load8(w + (size_t)i * a.d, wv);
#pragma unroll
                for (int s = 0; s < BG; ++s) {
                    const float z = ut[i * nt * BG + s];
#pragma unroll
                    for (int c = 0; c < 8; ++c) de[s][c] = fmaf(z, wv[c], de[s][c]);
                }
            }
        }
#pragma unroll
        for (int s = 0; s < BG; ++s)
            if (s < nb) {
                float o[8];
                load8(reinterpret_cast<const T *>(cur[s].v), o);
#pragma unroll
                for (int c = 0; c < 8; ++c) o[c] += de[s][c];
                store8<T>(dx + (size_t)s * ld, o);
            }
    }
}

// ---- kind 3: a chunk of tokens (all b*l in one row) x a slice of at most 256 columns of x: the slice's part of
// t1 = x W_B and the chunk's part of dW_B = x^T U.  32 tokens at a time go through one fp32 LDS tile that both
// products read; a wave owns every fourth 16-column tile, keeps its W_B fragments and dW_B sums in registers, and
// the next tile's loads are in flight under the matrix instructions.
// The tile is held in the storage type and converted on the way out (exact): all kinds of workgroup carry its LDS, and 44 KB of fp32
// let three of them on a compute unit where the registers allow four (4 x 8192 x 1024, 16 experts: 203 -> 171 us).
constexpr int BT = ROUTE_BWD_TILE, BS = ROUTE_BWD_SLICE;
// row stride: fp32 20 mod 64 banks, conflict-free by rows, 2-way by columns; bf16 12 mod 64 banks, conflict-free either way
template <typename T> constexpr int bwd_stride() { return BS + (sizeof(T) == 4 ? 20 : 24); }
template <typename T, int NT> __device__ __forceinline__ void bwd_data(const RouteBwdArgs &a, float *smem, int chunk, int slice)
{
    constexpr int BST = bwd_stride<T>();
    T *xs = reinterpret_cast<T *>(smem);
    const int tid = threadIdx.x, wave = tid >> 6, r = tid & 15, q = (tid & 63) >> 4;
    const int e0 = slice * a.plan.slice_w, ew = min(a.plan.slice_w, a.d - e0), rst = ((a.n + 15) & ~15) + 1;
    const long tokens = (long)a.b * a.l, tok0 = (long)chunk * a.plan.chunk_tokens;
    const long tok1 = min(tokens, tok0 + a.plan.chunk_tokens);
    float *red = reinterpret_cast<float *>(xs + BT * BST);  // [4 waves][BT][rst]
    float *t1 = a.t1 + (size_t)slice * tokens * a.n;
    float wb[4][4][NT];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int e = (wave + 4 * k) * 16 + 4 * s + q, i = 16 * nt + r;
                const float v = to_f32(static_cast<const T *>(a.w_b)[(size_t)(e0 + min(e, ew - 1)) * a.n + min(i, a.n - 1)]);
                wb[k][s][nt] = (e < ew && i < a.n) ? v : 0.f;
            }
    rb_f32x4 wacc[4][NT];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wacc[k][nt] = {0.f, 0.f, 0.f, 0.f};
    RawPiece<T> pre[4];
    const int row0 = tid / 32, pc = (tid % 32) * 8;
    auto fetch = [&](long t) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const long tk = t + row0 + 8 * v;
            const bool in = tk < tok1 && pc < ew;
            const uint4 *src = reinterpret_cast<const uint4 *>(static_cast<const T *>(a.x) + (size_t)(in ? tk : tok0) * a.d + (in ? e0 + pc : 0));
#pragma unroll
            for (int h = 0; h < (int)(sizeof(RawPiece<T>) / 16); ++h) {
                const uint4 w = src[h];
                pre[v].v[h] = in ? w : make_uint4(0, 0, 0, 0);
            }
        }
    };
    fetch(tok0);
    for (long t = tok0; t < tok1; t += BT) {
        float ub[8][NT];
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const long tk = t + 4 * s + q;
                const int i = 16 * nt + r;
                const float v = a.u[min(tk, tok1 - 1) * a.n + min(i, a.n - 1)];
                ub[s][nt] = (tk < tok1 && i < a.n) ? v : 0.f;
            }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            *reinterpret_cast<RawPiece<T> *>(xs + (row0 + 8 * v) * BST + pc) = pre[v];
        }
        __syncthreads();
        if (t + BT < tok1) fetch(t + BT);
        rb_f32x4 ta[2][NT];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) ta[tt][nt] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int et = (wave + 4 * k) * 16;
            if (et >= ew) continue;
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    const float xv = to_f32(xs[(tt * 16 + r) * BST + et + 4 * s + q]);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) ta[tt][nt] = mfma_f32(xv, wb[k][s][nt], ta[tt][nt]);
                }
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const float xv = to_f32(xs[(4 * s + q) * BST + et + r]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) wacc[k][nt] = mfma_f32(xv, ub[s][nt], wacc[k][nt]);
            }
        }
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 4; ++e) red[(wave * BT + tt * 16 + 4 * q + e) * rst + nt * 16 + r] = ta[tt][nt][e];
        __syncthreads();
        const int ntok = (int)min((long)BT, tok1 - t);
        for (int idx = tid; idx < ntok * a.n; idx += 256) {
            const int tk = idx / a.n, i = idx - tk * a.n;
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) s += red[(w * BT + tk) * rst + i];
            t1[(size_t)t * a.n + idx] = s;
        }
    }
    float *dst = a.wb_part + (size_t)chunk * a.d * a.n;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ee = (wave + 4 * k) * 16 + 4 * q + e, i = 16 * nt + r;
                if (ee < ew && i < a.n) dst[(size_t)(e0 + ee) * a.n + i] = wacc[k][nt][e];
            }
}

// The three kinds side by side.  Consecutive groups of a column chunk (experts of dW_E, samples of d_x) get block
// ids 8 apart, so that they run on one XCD and its L2 serves the second reading of x or W_E.
// NT: 16-expert tiles of the data router, 0 without one.  Registers are capped so that a compute unit holds 16 waves
// of the 4-sample form and 12 of the 8-sample form (fewer in fp32 and with a second expert tile, which would spill):
// the two streaming kinds live on loads in flight.
constexpr int main_waves(int bg, bool f32, int nt) { return (bg == 4 ? 4 : 3) - f32 - (nt == 2) < 2 ? 2 : (bg == 4 ? 4 : 3) - f32 - (nt == 2); }
template <typename T, int BG, bool ONCE, int NT>
__global__ __launch_bounds__(256, main_waves(BG, sizeof(T) == 4, NT)) void route_bwd_main_kernel(RouteBwdArgs a, WgradReduceArgs ra, int rx, int ry)
{
    extern __shared__ __align__(16) float smem[];
    const RouteBwdPlan &p = a.plan;
    int id = blockIdx.x;
    if constexpr (NT > 0) {  // first: its chains are the longest (last: 211 -> 235 us on the largest shape)
        if (id < p.data_blocks) {
            if (id < p.wb_chunks * p.slices) bwd_data<T, NT>(a, smem, id / p.slices, id % p.slices);
            return;
        }
        id -= p.data_blocks;
    }
    if (id < p.dx_blocks) {
        const int o = id / 8, chunk = (o / p.dx_groups) * 8 * p.dx_reps + id % 8;
        if (chunk < p.dx_chunks) bwd_dx<T, BG, ONCE>(a, smem, chunk, (o % p.dx_groups) * BG);
        return;
    }
    id -= p.dx_blocks;
    if (id < p.w_blocks) {
        const int o = id / 8, chunk = (o / p.w_groups) * 8 * p.w_reps + id % 8;
        if (chunk < p.w_chunks) bwd_wexpert<T, ONCE>(a, smem, chunk, (o % p.w_groups) * 8);
        return;
    }
    id -= p.w_blocks;   // the block's weight gradients (BwdTail)
    wgrad_reduce_tile<T, false>(ra, reinterpret_cast<RedTile>(smem), id % rx, id / rx % ry, id / (rx * ry));
}

// dW_A[t,j] = sum over k = (sample, expert) of t1[t,k] dL[k,j]: block = 16 tokens x up to 128 patches; its 8 waves
// are 1, 2 or 4 pairs of 16-patch tiles x parts of k, added in order.  The blocks behind them add the chunks'
// partials of dW_B: 32 outputs x 16 lanes (lane q takes chunks q, q+16, ...), then the lanes in order.
template <typename T> __global__ __launch_bounds__(512) void route_bwd_finish_kernel(RouteBwdArgs a, int wa_x, int wa_y, int jw)
{
    __shared__ float red[8][16][33];
    const int tid = threadIdx.x, id = blockIdx.x;
    if (id < wa_x * wa_y) {
        const int wave = tid >> 6, r = tid & 15, q = (tid & 63) >> 4, K = a.b * a.n, slices = a.plan.slices;
        const int kw = 8 / jw, t0 = (id % wa_x) * 16, j00 = (id / wa_x) * 32 * jw, j0 = j00 + 32 * (wave % jw);
        const int t = min(t0 + r, a.l - 1), ja = min(j0 + r, a.m - 1), jb = min(j0 + 16 + r, a.m - 1);
        const size_t slice = (size_t)a.b * a.l * a.n;
        rb_f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        for (int k0 = 4 * (wave / jw); k0 < K; k0 += 16 * kw) {  // four steps' loads in flight
            float v[4] = {0.f, 0.f, 0.f, 0.f}, da[4], db[4];
            const float *src[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = min(k0 + q + 4 * kw * u, K - 1), bb = k / a.n, i = k - bb * a.n;
                src[u] = a.t1 + ((size_t)bb * a.l + t) * a.n + i;
                da[u] = a.dl[(size_t)k * a.m + ja];
                db[u] = a.dl[(size_t)k * a.m + jb];
            }
            for (int s = 0; s < slices; ++s)
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] += src[u][(size_t)s * slice];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (k0 + q + 4 * kw * u >= K) v[u] = da[u] = db[u] = 0.f;
                acc[0] = mfma_f32(v[u], da[u], acc[0]);
                acc[1] = mfma_f32(v[u], db[u], acc[1]);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave][4 * q + e][16 * h + r] = acc[h][e];
        __syncthreads();
        for (int idx = tid; idx < 16 * 32 * jw; idx += 512) {
            const int tk = idx / (32 * jw), jj = idx - tk * 32 * jw;
            if (t0 + tk >= a.l || j00 + jj >= a.m) continue;
            float s = 0.f;
            for (int w = 0; w < kw; ++w) s += red[w * jw + jj / 32][tk][jj % 32];
            static_cast<T *>(a.d_w_a)[(size_t)(t0 + tk) * a.m + j00 + jj] = from_f32<T>(s);
        }
        return;
    }
    const int ol = tid & 31, ql = tid >> 5, total = a.d * a.n, idx = (id - wa_x * wa_y) * 32 + ol, chunks = a.plan.wb_chunks;
    const float *part = a.wb_part + min(idx, total - 1);
    float s = 0.f;
    for (int p = ql; p < chunks; p += 8 * 16) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(size_t)min(p + 16 * u, chunks - 1) * total];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += p + 16 * u < chunks ? v[u] : 0.f;
    }
    float *col = &red[0][0][0];
    col[ql * 33 + ol] = s;
    __syncthreads();
    if (ql == 0 && idx < total) {
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < 16; ++q) v += col[q * 33 + ol];
        static_cast<T *>(a.d_w_b)[idx] = from_f32<T>(v);
    }
}

// Launch shape: chunks and groups of the three kinds of workgroup.
RouteBwdPlan route_bwd_plan(int b, int l, int d, int n, bool has_e, bool has_d)
{
    RouteBwdPlan p{};
    const long pieces = (long)l * d / 8, tokens = (long)b * l;
    const int P = d / 8;
    auto up8 = [](long v) { return (int)((v + 7) & ~7L); };
    // chunks per block: the gates are staged once for all of them; 2048 blocks keep every compute unit's slots filled
    auto reps = [](long blocks) { return (int)(blocks < 4096 ? 1 : (blocks > 8 * 2048 ? 8 : blocks / 2048)); };
    // d_x: 4 samples per thread, 16 waves a compute unit; 8, with 12 waves, where W_E is long enough that its second reading costs more than
    // that gives (launch of 128 x 196 x 384, 6 experts, W_E 0.9 MB: 48.7 us with 8, 47.8 with 4; 16 x 4096 x 256, 8, 17 MB: 61.8 and 58.1;
    // 32 x 1024 x 512, 8, 8 MB: 62.0 and 56.7; 16 x 2048 x 1024, 16, 67 MB: 142.4 and 146.4; 12 x 4096 x 512, 32, 134 MB: 202.9 and 197.5,
    // two expert tiles leaving 8 samples 8 waves).  At most 32 tokens per block (their rows of U are staged in LDS)
    p.dx_pieces = 30 * P < 256 ? 30 * P : 256;
    p.dx_chunks = (int)((pieces + p.dx_pieces - 1) / p.dx_pieces);
    p.dx_bg = b > 4 && n <= 16 && pieces * n >= 3L << 20 ? 8 : 4;   // W_E of 48 MB in bf16
    p.dx_groups = (b + p.dx_bg - 1) / p.dx_bg;
    p.dx_reps = reps((long)p.dx_chunks * p.dx_groups);
    p.dx_blocks = up8((p.dx_chunks + p.dx_reps - 1) / p.dx_reps) * p.dx_groups;
    if (has_e) {
        p.w_groups = (n + 7) / 8;
        p.wsplit = b >= 16 && pieces * p.w_groups < 512L * 256;
        p.w_chunks = (int)((pieces + (p.wsplit ? 31 : 255)) / (p.wsplit ? 32 : 256));
        p.w_reps = reps((long)p.w_chunks * p.w_groups);
        p.w_blocks = up8((p.w_chunks + p.w_reps - 1) / p.w_reps) * p.w_groups;
    }
    if (has_d) {
        p.slices = (d + ROUTE_BWD_SLICE - 1) / ROUTE_BWD_SLICE;
        p.slice_w = ((d + p.slices - 1) / p.slices + 15) & ~15;
        // about 512 workgroups, each at least one tile of tokens
        const long want = (tokens * p.slices + 511) / 512;
        p.chunk_tokens = (int)((want + ROUTE_BWD_TILE - 1) / ROUTE_BWD_TILE) * ROUTE_BWD_TILE;
        p.wb_chunks = (int)((tokens + p.chunk_tokens - 1) / p.chunk_tokens);
        p.data_blocks = up8((long)p.wb_chunks * p.slices);
    }
    return p;
}

template <typename T> static hipError_t route_backward(RouteBwdArgs a, hipStream_t st, const BwdTail *tail)
{
    hipError_t err;
    a.plan = route_bwd_plan(a.b, a.l, a.d, a.n, a.w_e != nullptr, a.w_b != nullptr);
    const RouteBwdPlan &p = a.plan;
    if (a.w_b && !(tail && tail->prep_done)) {
        const RoutePrep<T> prep(a);
        hipLaunchKernelGGL((route_bwd_prep_kernel<T>), dim3(prep.blocks()), dim3(256), 0, st, prep);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    size_t floats = 0;
    auto need = [&](size_t v) { floats = v > floats ? v : floats; };
    if (a.w_e) need((size_t)a.b * 8 + 2 * (size_t)a.b * a.n);
    if (a.w_e) need((size_t)a.n * p.dx_bg * 3);
    const int P = a.d / 8, ntok = (p.dx_pieces + P - 2) / P + 1;  // tokens a d_x block can touch
    need((size_t)a.n * p.dx_bg * (1 + (a.w_b ? ntok : 0)));
    if (a.w_b) need((size_t)BT * bwd_stride<T>() * sizeof(T) / 4 + 4 * BT * (((a.n + 15) & ~15) + 1));
    WgradReduceArgs ra{};
    int rx = 1, ry = 1, tiles = 0;
    if (tail && tail->sets) {
        const RedGrid g(tail->reduce, tail->sets);
        ra = tail->reduce;
        rx = g.nx; ry = g.ny; tiles = g.tiles;
        need(RED_LDS / sizeof(float));
    }
    const dim3 grid(p.data_blocks + p.dx_blocks + p.w_blocks + tiles);
    const bool once = a.w_e && sizeof(T) == 2 && stream_once((size_t)a.n * a.l * a.d * sizeof(T));
    const size_t lds = floats * sizeof(float);
    auto launch = [&](auto bg, auto hint) {
        constexpr int BG = decltype(bg)::value;
        constexpr bool ONCE = decltype(hint)::value && sizeof(T) == 2;
        if (!a.w_b) hipLaunchKernelGGL((route_bwd_main_kernel<T, BG, ONCE, 0>), grid, dim3(256), lds, st, a, ra, rx, ry);
        else if (a.n <= 16) hipLaunchKernelGGL((route_bwd_main_kernel<T, BG, ONCE, 1>), grid, dim3(256), lds, st, a, ra, rx, ry);
        else hipLaunchKernelGGL((route_bwd_main_kernel<T, BG, ONCE, 2>), grid, dim3(256), lds, st, a, ra, rx, ry);
    };
    using std::integral_constant;
    if (p.dx_bg == 4) once ? launch(integral_constant<int, 4>{}, std::true_type{}) : launch(integral_constant<int, 4>{}, std::false_type{});
    else once ? launch(integral_constant<int, 8>{}, std::true_type{}) : launch(integral_constant<int, 8>{}, std::false_type{});
    if ((err = hipGetLastError()) != hipSuccess) return err;
    if (a.w_b) {
        const int jw = a.m <= 32 ? 1 : (a.m <= 64 ? 2 : 4), wa_x = (a.l + 15) / 16, wa_y = (a.m + 32 * jw - 1) / (32 * jw);
        hipLaunchKernelGGL((route_bwd_finish_kernel<T>), dim3(wa_x * wa_y + (a.d * a.n + 31) / 32), dim3(512), 0, st, a, wa_x, wa_y, jw);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    return hipSuccess;
}

hipError_t launch_route_backward(const RouteBwdArgs &a, bool bf16, hipStream_t st, const BwdTail *tail)
{
    return bf16 ? route_backward<bf16_t>(a, st, tail) : route_backward<float>(a, st, tail);
}

}  // namespace uoe
