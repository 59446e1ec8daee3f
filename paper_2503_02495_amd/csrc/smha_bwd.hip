// Backward pass of the SMHA block (Eq. 27-36 with the partial RoPE of Eq. 32 and the masks of
// Sec. III-C.3), bf16 storage, MFMA shapes.  For an upstream gradient G = dL/du [b,l,d], per active unit (sample b,
// slot s, expert i) with gathered token positions T, gate weight w_t of row t (Eq. 36 with the
// gate flags), o = softmax(q k^T / sqrt(d_h)) v and y = o W^O_i (u[T_t] += w_t y_t):
//   dO_raw = G[T] W^O_i^T,   r_t = dO_raw_t . o_t  (= dL/dw_t),   dO = w * dO_raw
//   dW^O_i += (w * o)^T G[T]
//   d_expert_gate[b,i] = sum_t g_patch(t) r_t,  d_patch_gate[b,i,p] = g_expert * sum_{t in p} r_t
//   P = softmax(...), dV = P^T dO, dP = dO V^T, dS = P * (dP - D) with D_i = sum_j P_ij dP_ij,
//   dQ = dS K / sqrt(d_h), dK = dS^T Q / sqrt(d_h)  (both rotated back when q, k were rotated)
//   dW^{q,k,v}_i += x[T]^T d{Q,K,V},   d_x[T] += dQ W^q_i^T + dK W^k_i^T + dV W^v_i^T  (+ G: residual)
// The forward intermediates are recomputed with the forward's own kernels (projections and
// attention, which also keeps each query's log-sum-exp); the contractions with the weights run on
// the pipelined GEMM engine (gathers folded into operand addressing as in the forward pass; the
// scatter-add of d_x output-stationary per patch, no atomics); the attention backward is a pair of
// MFMA kernels (one owning query rows, one owning key rows) that never materialise P.
#include "common.h"
#include "problems.h"
#include "gemm_mfma.h"
#include "gemm_dma.h"
#include "wgrad_reduce.h"
#include "route_prep.h"

namespace uoe {

// dO_raw = G[T] W^O_i^T (W^O_i [d_h, d] read as [n][k]) and what the attention gradient and dW^O need of it, straight
// from the fp32 accumulators: r_t = dO_raw_t . o_t (one part per WN columns), dO = w dO_raw (rounded once) and w o.  A lane
// owns a row and groups of 4 columns of it, so o arrives and dO leaves in 8-byte pieces that complete 64-byte runs of a
// row in L2.  (A row kernel between the two contractions read dO_raw back in fp32: 9.2 + 3.9 us on the lm shape.)
template <typename T> struct SmhaDoProblem {
    typedef typename storage_elem<T>::type Elem;
    const T *d_out, *wo, *o, *o_lo;
    const int32_t *expert_idx, *patch_idx;
    const float *expert_gate, *patch_gate;   // NULL: weight 1
    T *d_o, *og;                             // [units, l_a, d_h]
    float *rt;                               // [ceil(d_h / WN)][units*l_a]
    size_t rt_stride;
    int l, d, n, kact, m, c, l_p, l_a, d_h;
    static constexpr bool kAccOut = true, kPrepare = false, kRowScale = true, kColScale = false;
    __device__ int rows(int) const { return l_a; }
    __device__ int kdim(int) const { return d; }
    __device__ int ncols() const { return d_h; }
    __host__ __device__ int kseg(int) const { return d; }
    __device__ long b_stride() const { return 0; }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ int expert(int g) const { return clampi(expert_idx[g], n); }
    __device__ int patch(int g, int r) const { return clampi(patch_idx[((size_t)(g / kact) * n + expert(g)) * c + r / l_p], m); }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t) const
    {
        return d_out + ((size_t)(g / kact) * l + patch(g, r) * l_p + r % l_p) * d;
    }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t) const { return wo + ((size_t)expert(g) * d_h + nn) * d; }
    __device__ float row_scale(int g, int r) const
    {
        const size_t e = (size_t)(g / kact) * n + expert(g);
        return (expert_gate ? expert_gate[e] : 1.0f) * (patch_gate ? patch_gate[e * m + patch(g, r)] : 1.0f);
    }
    template <int TM, int TN>
    __device__ void acc_out(f32x16_t (&acc)[TM][TN], const float (&rs)[TM], int g, int grow0, int gcol0, int M, int N, int lane) const
    {
        const int lr = lane & 31, lh = lane >> 5;
        if (gcol0 >= N) return;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int grow = grow0 + i * 32 + lr;
            const size_t base = ((size_t)g * M + min(grow, M - 1)) * N + gcol0 + lh * 4;
            uint2 oh[TN * 4], ol[TN * 4];
#pragma unroll
            for (int q = 0; q < TN * 4; ++q) {   // 8-column group q of the wave tile (N is a multiple of 32)
                const size_t at = base + (gcol0 + q * 8 < N ? q * 8 : 0);
                oh[q] = *reinterpret_cast<const uint2 *>(o + at);
                ol[q] = *reinterpret_cast<const uint2 *>(o_lo + at);
            }
            float dot = 0.f;
#pragma unroll
            for (int q = 0; q < TN * 4; ++q) {
                if (gcol0 + q * 8 >= N) continue;
                const float w = rs[i];
                const uint32_t h[2] = {oh[q].x, oh[q].y}, lo[2] = {ol[q].x, ol[q].y};
                uint32_t od[2], ov[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float d0 = acc[i][q / 4][(q % 4) * 4 + 2 * e], d1 = acc[i][q / 4][(q % 4) * 4 + 2 * e + 1];
                    const float o0 = __uint_as_float(h[e] << 16) + __uint_as_float(lo[e] << 16);
                    const float o1 = __uint_as_float(h[e] & 0xFFFF0000u) + __uint_as_float(lo[e] & 0xFFFF0000u);
                    dot = fmaf(d0, o0, dot);
                    dot = fmaf(d1, o1, dot);
                    od[e] = pack2_bf16(d0 * w, d1 * w);
                    ov[e] = pack2_bf16(o0 * w, o1 * w);
                }
                if (grow < M) {
                    *reinterpret_cast<uint2 *>(d_o + base + q * 8) = make_uint2(od[0], od[1]);
                    *reinterpret_cast<uint2 *>(og + base + q * 8) = make_uint2(ov[0], ov[1]);
                }
            }
            dot += __shfl_xor(dot, 32, 64);
            if (grow < M && lh == 0) rt[gcol0 / (TN * 32) * rt_stride + (size_t)g * M + grow] = dot;
        }
    }
};

// ---------------------------------------------------------------------------------------------
// Attention backward.  One wave owns 32 rows of one unit ("own" rows) and walks the unit's other
// axis in tiles of 64 ("streamed" rows): KV = false owns queries and streams keys (dQ), KV = true
// owns keys and streams queries (dK, dV).  Everything is computed transposed, as in the forward
// kernel, so that an accumulator lane holds one own row:
//   S^T [streamed x own] = TA fa^T,  dP^T = TB fb^T      (TA/TB streamed tiles, fa/fb own fragments)
//   P^T = exp2(S^T - lse[query]),  dS^T = P^T * (dP^T - D[query]),  D[i] = sum_j P_ij dP_ij
//   accA^T [d_h x own] += TA^T dS^T        (dQ = K^T-contraction; dK = Q^T-contraction)
//   accB^T [d_h x own] += TB^T P^T         (KV only: dV = dO^T-contraction)
// with (TA, TB, fa, fb) = (k, v, q, dO) for KV = false and (q, dO, k, v) for KV = true.  q arrives
// scaled by log2(e)/sqrt(d_h) (base-2 softmax), so dK = ln 2 * accA and dQ = accA / sqrt(d_h).
// P^T and dS^T, as (hi, lo) bf16 pairs made in place, are the B operands of the second products; the A
// operands come out of the [row][d_h] LDS tiles through the transposing read.  Outputs go to the
// [dq | dk | dv] buffer, token-major: the left operand of the d_x contraction and of the weight gradients.
// KS = 2: two groups of NW waves own the same rows and take the streamed tiles in turn, each with LDS tiles of its own;
// their sums (D, then the accumulators) meet in LDS in group order.  A wave alternates between matrix, exponential and
// packing phases, so a SIMD needs two of them, and with one wave per 32 own rows most shapes give it one or none.
// (32 units of 1024 rows, d_h 64: 76.6 + 64.3 -> 55.0 + 47.8 us for the two kernels; 32 units of 128 rows 15.8 + 13.9 ->
// 14.3 + 12.7 us.)
struct AttnBwdArgs {
    const bf16_t *q, *k, *v, *d_o;
    const float *lse;
    float *dd;              // [units, l_a]: written by the query-owning kernel, read by the key-owning one
    bf16_t *dqkv;           // [units, l_a, 3*d_h]
    int units, l_a, causal;
    int rope_dim;           // Eq. 32: dq and dk are rotated back (the transposed rotation) on the way out
    // Eq. 41: padded keys are out of every softmax.  pad_mask [b,l] (1 = token) or NULL, looked up
    // through the unit's patch indices
    const unsigned char *pad_mask;
    const int32_t *expert_idx, *patch_idx;
    int l, n, kact, c, m, l_p;
};

__device__ __forceinline__ bool bwd_key_is_token(const AttnBwdArgs &a, int g, int key)
{
    const int bb = g / a.kact, i = clampi(a.expert_idx[g], a.n);
    const int p = clampi(a.patch_idx[((size_t)bb * a.n + i) * a.c + key / a.l_p], a.m);
    return a.pad_mask[(size_t)bb * a.l + p * a.l_p + key % a.l_p] != 0;
}

template <int DH, int NW, int KS, bool KV, bool PAD> __global__ __launch_bounds__(NW * KS * 64, DH <= 64 && NW == 4 ? 2 : 1) void attention_bwd_kernel(AttnBwdArgs a, UnitGates gates)
{
    constexpr int BT = 64, KP = DH + 8, VP = 2 * b_pitch_dwords(DH), NT = NW * 64;
    constexpr int CHUNKS = BT * DH / 8, PER_T = (CHUNKS + NT - 1) / NT;
    struct alignas(16) Tiles {
        uint16_t TAr[BT][KP], TAt[BT][VP], TBr[BT][KP], TBt[KV ? BT : 1][VP];
        float Ls[BT], Ds[BT];
        unsigned char Km[PAD ? BT : 16];  // streamed key admissible under the padding mask (KV = false)
    };
    constexpr int ACCS = KV ? 2 : 1, MERGE = NW * (DH / 32) * 16 * 64;  // floats of one accumulator of a group
    static_assert(sizeof(Tiles) % 16 == 0, "the groups' tiles keep 16-byte rows");
    static_assert(KS == 1 || (KS == 2 && ACCS * MERGE * sizeof(float) <= KS * sizeof(Tiles)), "accumulators meet in the tiles' space");
    __shared__ __align__(16) unsigned char lds[KS * sizeof(Tiles)];
    __shared__ float Dred[KV ? 1 : KS][NW * 32];

    const int g = blockIdx.y, l_a = a.l_a;
    if constexpr (KV) {   // the block's gate gradients, behind the units' rows of workgroups (r_t is there since dO was formed)
        static_assert(UnitGates::LDS <= sizeof(lds), "the gate gradients' LDS");
        if (g >= a.units) {
            gates.run<NW * KS * 64>((g - a.units) * gridDim.x + blockIdx.x, lds);
            return;
        }
    }
    const int split = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NT) : 0;
    const int tid = threadIdx.x - split * NT, lane = tid & 63, wave = tid >> 6;   // within the group
    Tiles &T = reinterpret_cast<Tiles *>(lds)[split];
    auto &TAr = T.TAr; auto &TAt = T.TAt; auto &TBr = T.TBr; auto &TBt = T.TBt;
    auto &Ls = T.Ls; auto &Ds = T.Ds; auto &Km = T.Km;
    const int lr = lane & 31, lh = lane >> 5;
    const int orow = blockIdx.x * (32 * NW) + wave * 32 + lr;
    const size_t ubase = (size_t)g * l_a * DH;
    const bf16_t *own_a = (KV ? a.k : a.q) + ubase, *own_b = (KV ? a.v : a.d_o) + ubase;
    const bf16_t *str_a = (KV ? a.q : a.k) + ubase, *str_b = (KV ? a.d_o : a.v) + ubase;

    bf16x8_t fa[DH / 16], fb[DH / 16];
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
        uint4 va = make_uint4(0, 0, 0, 0), vb = make_uint4(0, 0, 0, 0);
        if (orow < l_a) {
            va = *reinterpret_cast<const uint4 *>(own_a + (size_t)orow * DH + ks * 16 + lh * 8);
            vb = *reinterpret_cast<const uint4 *>(own_b + (size_t)orow * DH + ks * 16 + lh * 8);
        }
        fa[ks] = __builtin_bit_cast(bf16x8_t, va);
        fb[ks] = __builtin_bit_cast(bf16x8_t, vb);
    }
    float lse_o = 0.f, d_own = 0.f;
    if (!KV && orow < l_a) lse_o = a.lse[(size_t)g * l_a + orow];
    constexpr bool padded = PAD;  // compile-time: the unmasked kernels keep two waves per SIMD
    const bool own_key_ok = !(KV && padded) || bwd_key_is_token(a, g, min(orow, l_a - 1));

    f32x16_t acc_a[DH / 32], acc_b[DH / 32];
#pragma unroll
    for (int t = 0; t < DH / 32; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc_a[t][q] = acc_b[t][q] = 0.f;

    // streamed tiles: under the causal mask a query sees keys <= itself
    const int blk0 = blockIdx.x * 32 * NW, blk1 = min(l_a, blk0 + 32 * NW);
    int t_begin = 0, t_end = (l_a + BT - 1) / BT;
    if (a.causal) {
        if (KV) t_begin = blk0 / BT;
        else t_end = (blk1 + BT - 1) / BT;
    }

    uint4 ra[PER_T], rb[PER_T];
    float lreg = 0.f, dreg = 0.f;
    unsigned char kmreg = 1;
    auto load_global = [&](int row0) {
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
            const int c = tid + i * NT;
            const int row = c / (DH / 8), kc = c % (DH / 8);
            uint4 va = make_uint4(0, 0, 0, 0), vb = make_uint4(0, 0, 0, 0);
            if (c < CHUNKS && row0 + row < l_a) {
                va = *reinterpret_cast<const uint4 *>(str_a + (size_t)(row0 + row) * DH + kc * 8);
                vb = *reinterpret_cast<const uint4 *>(str_b + (size_t)(row0 + row) * DH + kc * 8);
            }
            ra[i] = va;
            rb[i] = vb;
        }
        if (KV && tid < BT) {
            const bool in = row0 + tid < l_a;
            lreg = in ? a.lse[(size_t)g * l_a + row0 + tid] : 0.f;
            dreg = in ? a.dd[(size_t)g * l_a + row0 + tid] : 0.f;
        }
        if (!KV && padded && tid < BT) kmreg = row0 + tid < l_a && bwd_key_is_token(a, g, min(row0 + tid, l_a - 1));
    };
    auto store_lds = [&]() {
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
            const int c = tid + i * NT;
            if (c < CHUNKS) {
                const int row = c / (DH / 8), col = (c % (DH / 8)) * 8;
                *reinterpret_cast<uint4 *>(&TAr[row][col]) = ra[i];
                *reinterpret_cast<uint4 *>(&TAt[row][col]) = ra[i];
                *reinterpret_cast<uint4 *>(&TBr[row][col]) = rb[i];
                if (KV) *reinterpret_cast<uint4 *>(&TBt[row][col]) = rb[i];
            }
        }
        if (KV && tid < BT) {
            Ls[tid] = lreg;
            Ds[tid] = dreg;
        }
        if (!KV && padded && tid < BT) Km[tid] = kmreg;
    };

    // first products of one tile and the probabilities: leaves P^T in sacc and dP^T in pacc
    auto scores = [&](int kt, f32x16_t (&sacc)[2], f32x16_t (&pacc)[2]) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 16; ++q) sacc[t][q] = pacc[t][q] = 0.f;
#pragma unroll
        for (int ks = 0; ks < DH / 16; ++ks)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const bf16x8_t ta = *reinterpret_cast<const bf16x8_t *>(&TAr[t * 32 + lr][ks * 16 + lh * 8]);
                sacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ta, fa[ks], sacc[t], 0, 0, 0);
                const bf16x8_t tb = *reinterpret_cast<const bf16x8_t *>(&TBr[t * 32 + lr][ks * 16 + lh * 8]);
                pacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tb, fb[ks], pacc[t], 0, 0, 0);
            }
        // accumulator register q of tile t is streamed row kt*64 + t*32 + (q/4)*8 + lh*4 + q%4
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int qg = 0; qg < 4; ++qg) {
                const int cl0 = t * 32 + qg * 8 + lh * 4;
                float l4[4] = {lse_o, lse_o, lse_o, lse_o};
                if (KV) {
                    const float4 lv = *reinterpret_cast<const float4 *>(&Ls[cl0]);
                    l4[0] = lv.x; l4[1] = lv.y; l4[2] = lv.z; l4[3] = lv.w;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = qg * 4 + e, crow = kt * BT + cl0 + e;
                    const int query = KV ? crow : orow, key = KV ? orow : crow;
                    const float p = __builtin_amdgcn_exp2f(sacc[t][q] - l4[e]);
                    bool key_ok = true;
                    if constexpr (PAD) key_ok = KV ? own_key_ok : Km[cl0 + e] != 0;
                    sacc[t][q] = (crow >= l_a || (a.causal && key > query) || !key_ok) ? 0.f : p;
                }
            }
    };

    // Owning the queries, a first walk over the keys forms the softmax row term from the very
    // values the second walk uses, D = sum_j P_ij dP_ij, so that the rows of dS cancel to zero
    // as they do in exact arithmetic (a row that attends to one key gets dS = 0, not the rounding
    // difference of two separately rounded numbers); it is kept for the key-owning kernel.
    if (!KV) {
        float dsum = 0.f;
        if (t_begin + split < t_end) load_global((t_begin + split) * BT);
        for (int kt0 = t_begin; kt0 < t_end; kt0 += KS) {
            const int kt = kt0 + split;
            __syncthreads();
            if (kt < t_end) store_lds();
            __syncthreads();
            if (kt >= t_end) continue;
            if (kt + KS < t_end) load_global((kt + KS) * BT);
            f32x16_t sacc[2], pacc[2];
            scores(kt, sacc, pacc);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 16; ++q) dsum = fmaf(sacc[t][q], pacc[t][q], dsum);
        }
        dsum += __shfl_xor(dsum, 32, 64);
        if constexpr (KS > 1) {
            if (lh == 0) Dred[split][wave * 32 + lr] = dsum;
            __syncthreads();
            dsum = Dred[0][wave * 32 + lr] + Dred[KS - 1][wave * 32 + lr];
        }
        d_own = dsum;
        if (orow < l_a && lh == 0 && split == 0) a.dd[(size_t)g * l_a + orow] = dsum;
    }

    if (t_begin + split < t_end) load_global((t_begin + split) * BT);
    for (int kt0 = t_begin; kt0 < t_end; kt0 += KS) {
        const int kt = kt0 + split;
        __syncthreads();  // the previous tile has been consumed
        if (kt < t_end) store_lds();
        __syncthreads();
        if (kt >= t_end) continue;
        if (kt + KS < t_end) load_global((kt + KS) * BT);

        f32x16_t sacc[2], pacc[2];
        scores(kt, sacc, pacc);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int qg = 0; qg < 4; ++qg) {
                float d4[4] = {d_own, d_own, d_own, d_own};
                if (KV) {
                    const float4 dv = *reinterpret_cast<const float4 *>(&Ds[t * 32 + qg * 8 + lh * 4]);
                    d4[0] = dv.x; d4[1] = dv.y; d4[2] = dv.z; d4[3] = dv.w;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) pacc[t][qg * 4 + e] = sacc[t][qg * 4 + e] * (pacc[t][qg * 4 + e] - d4[e]);
            }
        // second products over the 64 streamed rows: four k-steps of 16; dS^T and P^T enter as
        // (hi, lo) bf16 pairs, which keeps ~16 of their bits
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const int t = s4 >> 1, r0 = (s4 & 1) * 8;
            uint32_t dsh[4], dsl[4], ph[4], pl[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x0 = pacc[t][r0 + 2 * e], x1 = pacc[t][r0 + 2 * e + 1];
                dsh[e] = pack2_bf16(x0, x1);
                dsl[e] = pack2_bf16(x0 - __uint_as_float(dsh[e] << 16), x1 - __uint_as_float(dsh[e] & 0xFFFF0000u));
                if (KV) {
                    const float p0 = sacc[t][r0 + 2 * e], p1 = sacc[t][r0 + 2 * e + 1];
                    ph[e] = pack2_bf16(p0, p1);
                    pl[e] = pack2_bf16(p0 - __uint_as_float(ph[e] << 16), p1 - __uint_as_float(ph[e] & 0xFFFF0000u));
                }
            }
            const bf16x8_t ds_hi = __builtin_bit_cast(bf16x8_t, make_uint4(dsh[0], dsh[1], dsh[2], dsh[3]));
            const bf16x8_t ds_lo = __builtin_bit_cast(bf16x8_t, make_uint4(dsl[0], dsl[1], dsl[2], dsl[3]));
            const int trow = s4 * 16 + lh * 4 + ((lane & 15) >> 2);
#pragma unroll
            for (int td = 0; td < DH / 32; ++td) {
                const int tcol = td * 32 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
                const uint2 a0 = lds_read_tr4(&TAt[trow][tcol]);
                const uint2 a1 = lds_read_tr4(&TAt[trow + 8][tcol]);
                const bf16x8_t taf = __builtin_bit_cast(bf16x8_t, make_uint4(a0.x, a0.y, a1.x, a1.y));
                acc_a[td] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(taf, ds_hi, acc_a[td], 0, 0, 0);
                acc_a[td] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(taf, ds_lo, acc_a[td], 0, 0, 0);
                if (KV) {
                    const bf16x8_t p_hi = __builtin_bit_cast(bf16x8_t, make_uint4(ph[0], ph[1], ph[2], ph[3]));
                    const bf16x8_t p_lo = __builtin_bit_cast(bf16x8_t, make_uint4(pl[0], pl[1], pl[2], pl[3]));
                    const uint2 b0 = lds_read_tr4(&TBt[trow][tcol]);
                    const uint2 b1 = lds_read_tr4(&TBt[trow + 8][tcol]);
                    const bf16x8_t tbf = __builtin_bit_cast(bf16x8_t, make_uint4(b0.x, b0.y, b1.x, b1.y));
                    acc_b[td] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tbf, p_hi, acc_b[td], 0, 0, 0);
                    acc_b[td] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tbf, p_lo, acc_b[td], 0, 0, 0);
                }
            }
        }
    }

    if constexpr (KS > 1) {
        float *meet = reinterpret_cast<float *>(lds) + wave * (DH / 32) * 16 * 64 + lane;
        __syncthreads();  // every wave is done with the tiles
        if (split != 0) {
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    meet[(td * 16 + q) * 64] = acc_a[td][q];
                    if (KV) meet[MERGE + (td * 16 + q) * 64] = acc_b[td][q];
                }
        }
        __syncthreads();
        if (split != 0) return;
#pragma unroll
        for (int td = 0; td < DH / 32; ++td)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                acc_a[td][q] += meet[(td * 16 + q) * 64];
                if (KV) acc_b[td][q] += meet[MERGE + (td * 16 + q) * 64];
            }
    }
    if (orow >= l_a) return;
    // accumulator register q of tile td is head-dim index td*32 + (q/4)*8 + lh*4 + q%4
    const float scale_a = KV ? 0.6931471805599453f : rsqrtf((float)DH);
    bf16_t *row_out = a.dqkv + ((size_t)g * l_a + orow) * (3 * DH);
    // q and k were rotated in adjacent pairs (2i, 2i+1) of the last rope_dim dims, row r by r * theta_i;
    // the gradient of the unrotated projection is the gradient rotated by -r * theta_i.  A lane's four
    // consecutive head dims hold two whole pairs (rope_dim and d_h are even).
    const int rope_first = DH - a.rope_dim;
    auto put = [&](const f32x16_t (&acc)[DH / 32], int block, float scale) {
#pragma unroll
        for (int td = 0; td < DH / 32; ++td)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const int dh0 = td * 32 + i4 * 8 + lh * 4;
                float v[4] = {acc[td][i4 * 4 + 0] * scale, acc[td][i4 * 4 + 1] * scale, acc[td][i4 * 4 + 2] * scale,
                              acc[td][i4 * 4 + 3] * scale};
                if (block < 2 && a.rope_dim > 0) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int dh = dh0 + 2 * h;
                        if (dh >= rope_first) {
                            float sn, cs;
                            rope_sincos((float)orow, rope_theta(dh - rope_first, a.rope_dim), sn, cs);
                            const float ga = v[2 * h], gb = v[2 * h + 1];
                            v[2 * h] = ga * cs + gb * sn;
                            v[2 * h + 1] = gb * cs - ga * sn;
                        }
                    }
                }
                const uint32_t w0 = pack2_bf16(v[0], v[1]);
                const uint32_t w1 = pack2_bf16(v[2], v[3]);
                *reinterpret_cast<uint2 *>(row_out + block * DH + dh0) = make_uint2(w0, w1);
            }
    };
    if (KV) {
        put(acc_a, 1, scale_a);
        put(acc_b, 2, 1.0f);
    } else {
        put(acc_a, 0, scale_a);
    }
}

template <int DH, int NW, int KS, bool PAD> static hipError_t launch_attention_bwd_as(const AttnBwdArgs &a, const UnitGates &gates, hipStream_t st)
{
    const int blocks = (a.l_a + 32 * NW - 1) / (32 * NW), more = (gates.units + blocks - 1) / blocks;
    hipLaunchKernelGGL((attention_bwd_kernel<DH, NW, KS, false, PAD>), dim3(blocks, a.units), dim3(NW * KS * 64), 0, st, a, gates);
    hipLaunchKernelGGL((attention_bwd_kernel<DH, NW, KS, true, PAD>), dim3(blocks, a.units + more), dim3(NW * KS * 64), 0, st, a, gates);
    return hipGetLastError();
}

// Two groups of waves per own block while one would leave SIMDs with less than two waves (2048 on the chip) and there
// is a second tile to stream; then as many own blocks per workgroup (they share the streamed tiles) as still give every
// compute unit a workgroup.  Heads of 128 stay with one group: two would not fit the register file.
template <int DH, bool PAD> static hipError_t launch_attention_bwd_dh(const AttnBwdArgs &a, const UnitGates &gates, hipStream_t st)
{
    const int units = a.units;
    const long wide = (long)((a.l_a + 127) / 128) * units, mid = (long)((a.l_a + 63) / 64) * units;
    if constexpr (DH <= 64) {
        if (a.l_a > 64 && (long)((a.l_a + 31) / 32) * units < 2048) {
            if (wide >= 256) return launch_attention_bwd_as<DH, 4, 2, PAD>(a, gates, st);
            if (mid >= 256) return launch_attention_bwd_as<DH, 2, 2, PAD>(a, gates, st);
            return launch_attention_bwd_as<DH, 1, 2, PAD>(a, gates, st);
        }
    }
    if (wide >= 128) return launch_attention_bwd_as<DH, 4, 1, PAD>(a, gates, st);
    if (mid >= 64) return launch_attention_bwd_as<DH, 2, 1, PAD>(a, gates, st);
    return launch_attention_bwd_as<DH, 1, 1, PAD>(a, gates, st);
}

template <bool PAD> static hipError_t launch_attention_bwd(const AttnBwdArgs &a, int dh, const UnitGates &gates, hipStream_t st)
{
    if (dh == 32) return launch_attention_bwd_dh<32, PAD>(a, gates, st);
    if (dh == 64) return launch_attention_bwd_dh<64, PAD>(a, gates, st);
    return launch_attention_bwd_dh<128, PAD>(a, gates, st);
}

hipError_t launch_smha_backward(const SmhaBwdArgs &a_in, hipStream_t st, BwdTail *tail)
{
    typedef bf16_t T;
    SmhaBwdArgs a = a_in;
    const SmhaArgs &f = a.f;
    const int l_p = f.l / f.m, l_a = f.c * l_p, units = f.b * f.k, dh = f.d_h;
    hipError_t err;
    if (a.wgrad.parts > WGRAD_MAX_PARTS) return hipErrorInvalidValue;

    // forward intermediates: q (scaled for the base-2 softmax), k, v, ungated o = hi + lo, lse
    if (!a.kept && (err = launch_smha_qkv_attention(f, st)) != hipSuccess) return err;

    SmhaDoProblem<T> dp;
    dp.d_out = static_cast<const T *>(a.d_out); dp.wo = static_cast<const T *>(f.wo);
    dp.o = static_cast<const T *>(f.o); dp.o_lo = static_cast<const T *>(f.o_lo);
    dp.expert_idx = f.expert_idx; dp.patch_idx = f.patch_idx;
    dp.expert_gate = (a.flags & F_GATE_EXPERT) ? a.expert_gate : nullptr;
    dp.patch_gate = (a.flags & F_GATE_PATCH) ? a.patch_gate : nullptr;
    dp.d_o = static_cast<T *>(a.d_o); dp.og = static_cast<T *>(a.og);
    dp.rt = a.rt; dp.rt_stride = (size_t)units * l_a;
    dp.l = f.l; dp.d = f.d; dp.n = f.n; dp.kact = f.k; dp.m = f.m; dp.c = f.c; dp.l_p = l_p; dp.l_a = l_a; dp.d_h = dh;
    // 32x64 tiles of two 32-column waves while 64-row tiles would leave compute units without one
    if ((long)units * ((l_a + 63) / 64) < 256) {
        a.rt_parts = (dh + 31) / 32;
        err = f.d % 64 == 0 ? launch_gemm_dma<SmhaDoProblem<T>, 32, 64, 64, 1, 2, 4, 2, GEMM_B_NK>(dp, units, l_a, dh, st)
                            : launch_gemm_dma<SmhaDoProblem<T>, 32, 64, 32, 1, 2, 4, 2, GEMM_B_NK>(dp, units, l_a, dh, st);
    } else {
        int wave_cols;
        err = launch_gemm_dma_auto<GEMM_B_NK>(dp, units, l_a, dh, f.d, f.d, st, &wave_cols);
        a.rt_parts = (dh + wave_cols - 1) / wave_cols;
    }
    if (err != hipSuccess) return err;

    AttnBwdArgs ab;
    ab.q = static_cast<const T *>(f.q); ab.k = static_cast<const T *>(f.kk); ab.v = static_cast<const T *>(f.v);
    ab.d_o = static_cast<const T *>(a.d_o); ab.lse = f.lse; ab.dd = a.dd;
    ab.dqkv = static_cast<T *>(a.dqkv);
    ab.units = units; ab.l_a = l_a; ab.causal = (f.flags & F_CAUSAL) ? 1 : 0; ab.rope_dim = f.rope_dim;
    ab.pad_mask = f.pad_mask; ab.expert_idx = f.expert_idx; ab.patch_idx = f.patch_idx;
    ab.l = f.l; ab.n = f.n; ab.kact = f.k; ab.c = f.c; ab.m = f.m; ab.l_p = l_p;
    const UnitGates gates{a, UnitGates::count(a)};
    err = ab.pad_mask ? launch_attention_bwd<true>(ab, dh, gates, st) : launch_attention_bwd<false>(ab, dh, gates, st);
    if (err != hipSuccess) return err;

    // d_x = (G) + scatter-add of dq W^q^T + dk W^k^T + dv W^v^T
    SmhaDxProblem<T, 1> xp;
    xp.o = static_cast<const T *>(a.dqkv); xp.o_lo = nullptr; xp.parts = 1; xp.wo = nullptr;
    xp.w[0] = static_cast<const T *>(f.wq); xp.w[1] = static_cast<const T *>(f.wk); xp.w[2] = static_cast<const T *>(f.wv);
    xp.x = static_cast<const T *>(a.d_out);
    xp.expert_idx = f.expert_idx; xp.patch_idx = f.patch_idx;
    xp.out = static_cast<T *>(a.d_x);
    xp.l = f.l; xp.d = f.d; xp.n = f.n; xp.kact = f.k; xp.m = f.m; xp.c = f.c;
    xp.l_p = l_p; xp.l_a = l_a; xp.d_h = dh; xp.o_row = 3 * dh; xp.flags = a.flags & F_RESIDUAL;

    // weight gradients, all four in one launch (M = d_h each): sets 0-2 = (dW^q, dW^k, dW^v)^T from
    // [dq|dk|dv]^T against gathered x, set 3 = dW^O from (w*o)^T against gathered d_out
    SmhaWgradProblem<T> wp;
    for (int q = 0; q < 3; ++q) {
        wp.left[q] = static_cast<const T *>(a.dqkv); wp.right[q] = static_cast<const T *>(f.x);
        wp.row_len[q] = 3 * dh; wp.col0[q] = q * dh;
    }
    wp.left[3] = static_cast<const T *>(a.og); wp.right[3] = static_cast<const T *>(a.d_out);
    wp.row_len[3] = dh; wp.col0[3] = 0;
    wp.expert_idx = f.expert_idx; wp.patch_idx = f.patch_idx; wp.partial = a.partial;
    wp.b = f.b; wp.l = f.l; wp.d = f.d; wp.n = f.n; wp.kact = f.k; wp.m = f.m; wp.c = f.c;
    wp.l_p = l_p; wp.l_a = l_a; wp.parts = {4, DEALT, a.wgrad, a.part_end}; wp.M = dh;
    // one launch with d_x while the weight gradients do not fill the chip's slots (two per compute unit)
    const int groups = wp.parts.groups();
    typedef GemmTile<SmhaDxProblem<T, 1>, 32, 128, 32, 1, 4, 4, GEMM_B_NK> Dx32;
    typedef GemmTile<SmhaDxProblem<T, 1>, 64, 128, 32, 2, 2, 4, GEMM_B_NK> Dx64;
    typedef GemmTile<SmhaWgradProblem<T>, 64, 128, 32, 2, 2, 4, GEMM_A_KM> Wg;
    if ((long)groups * ((dh + 63) / 64) * ((f.d + 127) / 128) <= 512) {
        RoutePrep<T> prep{};   // and with the first launch of the data router's pass, whose gate gradients are there
        int prep_blocks = 0;
        if (tail && tail->prep) {
            prep = RoutePrep<T>(*tail->prep);
            prep_blocks = prep.blocks();
            tail->prep_done = 1;
        }
        err = l_p <= 32 ? launch_gemm_dma_pair<Wg, Dx32, 2>(wp, groups, dh, f.d, xp, f.b * f.m, l_p, f.d, st, prep, prep_blocks)
                        : launch_gemm_dma_pair<Wg, Dx64, 2>(wp, groups, dh, f.d, xp, f.b * f.m, l_p, f.d, st, prep, prep_blocks);
    } else {
        if (l_p <= 32) err = launch_gemm_dma<SmhaDxProblem<T, 1>, 32, 128, 32, 1, 4, 4, 2, GEMM_B_NK>(xp, f.b * f.m, l_p, f.d, st);
        else err = launch_gemm_dma<SmhaDxProblem<T, 1>, 64, 128, 32, 2, 2, 4, 2, GEMM_B_NK>(xp, f.b * f.m, l_p, f.d, st);
        if (err == hipSuccess) err = launch_gemm_dma_auto<GEMM_A_KM>(wp, groups, dh, f.d, 0, l_p, st);
    }
    if (err != hipSuccess) return err;
    WgradReduceArgs ra{};
    ra.partial = a.partial; ra.n = f.n; ra.M = dh; ra.N = f.d;
    ra.w = a.wgrad; ra.part_end = a.part_end;
    ra.dst[0] = a.d_wq; ra.dst[1] = a.d_wk;
    ra.dst[2] = a.d_wv; ra.dst[3] = a.d_wo;
    ra.transposed[0] = ra.transposed[1] = ra.transposed[2] = 1; ra.transposed[3] = 0;
    return launch_wgrad_reduce<T>(ra, 4, st, tail);
}

}  // namespace uoe
