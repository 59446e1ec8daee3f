// Selective Multi-Head Attention on given routing results (Eq. 27-36).
//
// Pipeline per call (all on one stream):
//   QKV projection   : grouped GEMM over active units, Eq. 18 gather folded into the A rows.
//   attention        : softmax(q k^T / sqrt(d_h)) v per unit over its l_a tokens (Eq. 33-34),
//                      rows scaled by their gate weight on the way out.
//   out-projection   : output-stationary grouped GEMM over (sample, patch) that concatenates the
//                      contributions of every expert that picked the patch along K and writes
//                      each output row once, residual included (Eq. 35-36).
#include "common.h"
#include "problems.h"
#include "gemm_mfma.h"
#include "gemm_dma.h"

namespace uoe {

// Partial RoPE of Eq. 32 for fp32 storage, in place on the q and k workspaces (the projections of bf16 storage rotate in
// their epilogue): the last rope_dim dims of a head are
// rotated in adjacent pairs (2i, 2i+1) by position * 10000^(-2i/rope_dim); the position of a row
// is its index in the unit's compacted sequence.  One thread per (unit row, pair).
__global__ __launch_bounds__(256) void smha_rope_kernel(SmhaArgs a)
{
    const int l_a = a.c * (a.l / a.m), half = a.rope_dim >> 1;
    const long total = (long)a.b * a.k * l_a * half;
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int i = (int)(idx % half);
    const long row = idx / half;              // unit * l_a + r
    const int r = (int)(row % l_a);
    const float theta = exp2f(-(2.0f * (float)i / (float)a.rope_dim) * 13.287712379549449f);  // log2(10000)
    float sn, cs;
    sincosf((float)r * theta, &sn, &cs);
    const size_t at = (size_t)row * a.d_h + (a.d_h - a.rope_dim) + 2 * i;
    float *q = static_cast<float *>(a.q) + at, *k = static_cast<float *>(a.kk) + at;
    const float q0 = q[0], q1 = q[1], k0 = k[0], k1 = k[1];
    q[0] = q0 * cs - q1 * sn;
    q[1] = q0 * sn + q1 * cs;
    k[0] = k0 * cs - k1 * sn;
    k[1] = k0 * sn + k1 * cs;
}

hipError_t launch_rope_f32(const SmhaArgs &a, hipStream_t st)
{
    if (a.rope_dim <= 0) return hipSuccess;
    const long total = (long)a.b * a.k * a.c * (a.l / a.m) * (a.rope_dim >> 1);
    hipLaunchKernelGGL(smha_rope_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError();
}

// padding flag of key `key` of unit g (Eq. 41: the mask is gathered with the unit's indices)
__device__ __forceinline__ bool key_is_token(const SmhaArgs &a, int g, int key, int l_p)
{
    const int bb = g / a.k, i = clampi(a.expert_idx[g], a.n);
    const int p = clampi(a.patch_idx[((size_t)bb * a.n + i) * a.c + key / l_p], a.m);
    return a.pad_mask[(size_t)bb * a.l + p * l_p + key % l_p] != 0;
}

// Attention with fp32 products and fp32 probabilities (Eq. 33-34): fp32 storage, and bf16 storage where the bf16 kernels do
// not apply (launch_smha), whose q, k and v are widened on the way into LDS and whose o leaves as a (hi, lo) pair.  One wave
// owns 32 query rows of one unit and walks key tiles of 32, online softmax in base 2.
// Layout as in the bf16 kernel: the scores are computed transposed, S^T = K Q^T, so that a lane holds one query;
// accumulator register q is key (q/4)*8 + lh*4 + q%4, and that key order is the one of both operands of the second
// product, P^T and V.  K rows are padded by 4 floats (16-byte fragment reads of 16 consecutive rows
// hit all banks once), V rows by 8 (the half-waves' rows are 4 apart: 32 banks).
// Products.  fp32 storage: v_mfma_f32_32x32x2_f32 (six bf16 products of operands split in three took registers, two waves a SIMD
// became one: 384 units of 56 rows, d_h 64, 18.9 us against 14.3, 64 units of 400 rows 50 against 46, though 32 of 1600 rows 221
// against 271; and they lost the last bits of v below 2^-110).  bf16 storage: q, k and v are exact as one bf16 part, so that a score is one bf16
// product (q enters unscaled, the score is scaled) and P V three, P in three parts (SplitF32): 32 and 96 cycles of the matrix pipe
// for what takes 512.  The bf16 instruction rounds its sum towards minus infinity: odd pairs of sub-steps of a score are summed negated, and
// O takes half of its key tiles with each sign, whatever the number of splits (in the multiplication that rescales it anyway).  P
// is multiplied by 2^24 and O divided by it, so that no part of P times v falls below the normal numbers.
// us, before -> now (four key splits instead of two on short grids in both types): 6 x 1000 x 360 in bf16, heads of 40 (18 units of 240 rows)
// 18.6 -> 11.4, 384 units of 112 rows, d_h 56, 28.4 -> 19.7; fp32, 32 units of 128 rows, d_h 64: 13.8 -> 11.1, 18 of 240 19.5 -> 13.2.  What is
// left is the chain of a tile: staging, scores, maximum, exponentials, second product, two barriers.
// KSPLIT waves share a query block and take key tiles KSPLIT apart (merged through LDS) so that short grids
// still give most SIMDs a wave.
template <typename T, int DH, int NQ, int KSPLIT>
__global__ __launch_bounds__(NQ *KSPLIT * 64) void attention_f32_kernel(SmhaArgs a)
{
    constexpr int BT = 32, KP = DH + 4, VP = DH + 8, NTH = NQ * 64;   // NTH: threads that stage one split's tiles
    constexpr int EP = 16 / sizeof(T), CHUNKS = BT * DH / EP, PER_T = (CHUNKS + NTH - 1) / NTH;
    constexpr int SPLIT_FLOATS = BT * KP + BT * VP + BT;
    constexpr int SLOT = DH / 2 + 2, MERGE_FLOATS = (KSPLIT - 1) * NQ * 64 * SLOT;
    constexpr int LDS_FLOATS = KSPLIT * SPLIT_FLOATS > MERGE_FLOATS ? KSPLIT * SPLIT_FLOATS : MERGE_FLOATS;
    __shared__ __align__(16) float lds[LDS_FLOATS];

    const int l_p = a.l / a.m, l_a = a.c * l_p, d_h = a.d_h, g = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int split = wave / NQ, qg = wave - split * NQ, stid = tid - split * NTH;
    const int lr = lane & 31, lh = lane >> 5;
    const int qrow = blockIdx.x * (32 * NQ) + qg * 32 + lr;
    float *Ks = lds + split * SPLIT_FLOATS, *Vs = Ks + BT * KP, *Km = Vs + BT * VP;   // Km: 1 = admissible key
    const size_t ubase = (size_t)g * l_a * d_h;
    const T *Q = static_cast<const T *>(a.q) + ubase, *Kg = static_cast<const T *>(a.kk) + ubase, *Vg = static_cast<const T *>(a.v) + ubase;

    const float scale = 1.4426950408889634f * rsqrtf((float)d_h);   // base-2 softmax
    constexpr float P_SCALE = 16777216.0f;
    auto q_at = [&](int ks, int e) -> float {   // own query, k of sub-step ks of the fp32 instruction
        const int dh = ks * 8 + lh * 4 + e;
        return qrow < l_a && dh < d_h ? to_f32(Q[(size_t)qrow * d_h + dh]) : 0.f;
    };
    f32x16_t oacc[DH / 32];
    float mrun, lsum;
    const bool causal = (a.flags & F_CAUSAL) != 0;
    // under the causal mask no query of this workgroup sees keys past its last row
    const int key_end = causal ? min(l_a, (int)(blockIdx.x + 1) * 32 * NQ) : l_a;
    const int nkt = (key_end + BT - 1) / BT, nit = (nkt + KSPLIT - 1) / KSPLIT;

    uint4 kr[PER_T], vr[PER_T];
    float kmreg = 0.f;
    auto load_global = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
            const int c = stid + i * NTH, row = c / (DH / EP), col = (c % (DH / EP)) * EP, key = kt * BT + row;
            kr[i] = vr[i] = make_uint4(0, 0, 0, 0);
            if (c < CHUNKS && key < l_a && col < d_h) {
                kr[i] = *reinterpret_cast<const uint4 *>(Kg + (size_t)key * d_h + col);
                vr[i] = *reinterpret_cast<const uint4 *>(Vg + (size_t)key * d_h + col);
            }
        }
        if (stid < BT) {
            const int key = kt * BT + stid;
            kmreg = key < l_a && (!a.pad_mask || key_is_token(a, g, key, l_p)) ? 1.f : 0.f;
        }
    };
    auto put_row = [](float *dst, uint4 v) {
        if constexpr (sizeof(T) == 4) *reinterpret_cast<uint4 *>(dst) = v;
        else {
            const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dst[2 * e] = __uint_as_float(u[e] << 16);
                dst[2 * e + 1] = __uint_as_float(u[e] & 0xFFFF0000u);
            }
        }
    };
    auto store_lds = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
            const int c = stid + i * NTH, row = c / (DH / EP), col = (c % (DH / EP)) * EP;
            if (c < CHUNKS) {
                put_row(Ks + row * KP + col, kr[i]);
                put_row(Vs + row * VP + col, vr[i]);
            }
        }
        if (stid < BT) Km[stid] = kmreg;
    };

    auto walk = [&](auto exact_c) __attribute__((always_inline)) {
        constexpr bool EXACT = decltype(exact_c)::value;
        static_assert(EXACT || sizeof(T) == 2, "one bf16 part holds q, k and v");
        // the query as second operand: fp32 and scaled; or as it is in bf16, odd pairs of sub-steps negated, the scores scaled instead
        float qf[EXACT ? DH / 8 : 1][4];
        bf16x8_t qb[EXACT ? 1 : DH / 16];
        if constexpr (EXACT) {
#pragma unroll
            for (int ks = 0; ks < DH / 8; ++ks)
#pragma unroll
                for (int e = 0; e < 4; ++e) qf[ks][e] = q_at(ks, e) * scale;
        } else {
#pragma unroll
            for (int s = 0; s < DH / 16; ++s) {
                f32x4_t q0, q1;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    q0[e] = q_at(2 * s, e);
                    q1[e] = q_at(2 * s + 1, e);
                }
                qb[s] = pack8_bf16(q0, q1, s & 1 ? -1.0f : 1.0f);
            }
        }
#pragma unroll
        for (int t = 0; t < DH / 32; ++t)
#pragma unroll
            for (int q = 0; q < 16; ++q) oacc[t][q] = 0.f;
        mrun = -INFINITY;
        lsum = 0.f;
        float sign = split & 1 ? -1.0f : 1.0f;   // of O in its accumulators
        bool unseen = false;                     // an admissible key, and none with a score above -inf
        if (split < nkt) load_global(split);
        for (int it = 0; it < nit; ++it) {   // nit is uniform over the workgroup
            const int kt = it * KSPLIT + split;
            __syncthreads();   // the previous tiles have been consumed
            if (kt < nkt) store_lds();
            __syncthreads();
            if (kt + KSPLIT < nkt) load_global(kt + KSPLIT);
            if (kt >= nkt) continue;
            f32x16_t sacc, sneg;
#pragma unroll
            for (int q = 0; q < 16; ++q) sacc[q] = sneg[q] = 0.f;
#pragma unroll
            for (int s = 0; s < DH / 16; ++s) {
                const f32x4_t k0 = *reinterpret_cast<const f32x4_t *>(Ks + lr * KP + s * 16 + lh * 4);
                const f32x4_t k1 = *reinterpret_cast<const f32x4_t *>(Ks + lr * KP + s * 16 + 8 + lh * 4);
                if constexpr (EXACT) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(k0[e], qf[2 * s][e], sacc, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(k1[e], qf[2 * s + 1][e], sacc, 0, 0, 0);
                } else {
                    f32x16_t &sum = s & 1 ? sneg : sacc;
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pack8_bf16(k0, k1, 1.0f), qb[s], sum, 0, 0, 0);
                }
            }
            if constexpr (!EXACT) {
#pragma unroll
                for (int q = 0; q < 16; ++q) sacc[q] = (sacc[q] - sneg[q]) * scale;
            }
            float tmax = -INFINITY;
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const float4 ok4 = *reinterpret_cast<const float4 *>(Km + q4 * 8 + lh * 4);
                const float okv[4] = {ok4.x, ok4.y, ok4.z, ok4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int key = kt * BT + q4 * 8 + lh * 4 + e;
                    const bool ok = okv[e] != 0.f && (!causal || key <= qrow);
                    sacc[q4 * 4 + e] = ok ? sacc[q4 * 4 + e] : -INFINITY;
                    tmax = fmaxf(tmax, sacc[q4 * 4 + e]);
                }
            }
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
            const float mnew = fmaxf(mrun, tmax), msub = mnew == -INFINITY ? 0.f : mnew;   // nothing admissible yet: exp2(-inf - 0) = 0
            if constexpr (!EXACT) {
                if (mnew == -INFINITY) {
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const int at = (q >> 2) * 8 + lh * 4 + (q & 3);
                        unseen |= Km[at] != 0.f && (!causal || kt * BT + at <= qrow);
                    }
                } else unseen = false;
            }
            const float corr = __builtin_amdgcn_exp2f(mrun - msub);   // 0 before the first admissible key
            mrun = mnew;
            float psum = 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                sacc[q] = __builtin_amdgcn_exp2f(sacc[q] - msub);
                psum += sacc[q];
            }
            lsum = fmaf(lsum, corr, psum);
            if constexpr (!EXACT) sign = -sign;
            const float oc = EXACT ? corr : -corr;
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) oacc[td][q] *= oc;
            // key of accumulator register q: it is, with the lane halves' keys 4 apart, the order of the second product's operands
            auto v_at = [&](int q, int td) { return Vs[((q >> 2) * 8 + lh * 4 + (q & 3)) * VP + td * 32 + lr]; };
            if constexpr (EXACT) {
#pragma unroll
                for (int q = 0; q < 16; ++q)
#pragma unroll
                    for (int td = 0; td < DH / 32; ++td) oacc[td] = __builtin_amdgcn_mfma_f32_32x32x2f32(v_at(q, td), sacc[q], oacc[td], 0, 0, 0);
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    f32x4_t p0, p1;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        p0[e] = sacc[h * 8 + e];
                        p1[e] = sacc[h * 8 + 4 + e];
                    }
                    SplitF32 pp;
                    pp.set(p0, p1, sign * P_SCALE);
#pragma unroll
                    for (int td = 0; td < DH / 32; ++td) {
                        f32x4_t v0, v1;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            v0[e] = v_at(h * 8 + e, td);
                            v1[e] = v_at(h * 8 + 4 + e, td);
                        }
                        oacc[td] = mfma_split(pack8_bf16(v0, v1, 1.0f), pp, oacc[td]);
                    }
                }
            }
        }
        float bad = unseen ? NAN : 0.f;
        if constexpr (!EXACT) {
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    oacc[td][q] *= sign * (1.0f / P_SCALE);
                    bad = fmaf(oacc[td][q], 0.f, bad);
                }
        }
        return bad != bad;
    };
    // bf16: parts of an infinity are infinity and NaN, and an unscaled score may overflow where the scaled one does not: a block whose O
    // is not finite, or with a row whose scores are all -inf, is walked again on fp32 products
    if constexpr (sizeof(T) == 4) walk(std::true_type{});
    else if (__builtin_expect(__syncthreads_or(walk(std::false_type{})), 0)) walk(std::true_type{});
    if constexpr (KSPLIT > 1) {   // split 0 folds the others' (max, sum, O) in, in split order
        __syncthreads();
        if (split > 0) {
            float *dst = lds + ((size_t)((split - 1) * NQ + qg) * 64 + lane) * SLOT;
            dst[0] = mrun;
            dst[1] = lsum;
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) dst[2 + td * 16 + q] = oacc[td][q];
        }
        __syncthreads();
        if (split > 0) return;
#pragma unroll
        for (int s = 1; s < KSPLIT; ++s) {
            const float *src = lds + ((size_t)((s - 1) * NQ + qg) * 64 + lane) * SLOT;
            const float m1 = src[0], mf = fmaxf(mrun, m1);
            const float c0 = mrun == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrun - mf);
            const float c1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m1 - mf);
            lsum = lsum * c0 + src[1] * c1;
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) oacc[td][q] = oacc[td][q] * c0 + src[2 + td * 16 + q] * c1;
            mrun = mf;
        }
    }
    if (qrow >= l_a) return;
    lsum += __shfl_xor(lsum, 32, 64);
    // gate weight of this row (Eq. 36 with the optional gate flags)
    const int bb = g / a.k, i = clampi(a.expert_idx[g], a.n);
    float w = 1.0f;
    if ((a.flags & F_GATE_EXPERT) && a.expert_gate) w *= a.expert_gate[(size_t)bb * a.n + i];
    if ((a.flags & F_GATE_PATCH) && a.patch_gate) {
        const int p = clampi(a.patch_idx[((size_t)bb * a.n + i) * a.c + qrow / l_p], a.m);
        w *= a.patch_gate[((size_t)bb * a.n + i) * a.m + p];
    }
    const float inv = lsum > 0.f ? w / lsum : 0.f;  // a row with no admissible key contributes nothing
    const size_t row = ubase + (size_t)qrow * d_h;
#pragma unroll
    for (int td = 0; td < DH / 32; ++td)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const int dh = td * 32 + q4 * 8 + lh * 4;
            if (dh >= d_h) continue;
            const float v[4] = {oacc[td][q4 * 4] * inv, oacc[td][q4 * 4 + 1] * inv, oacc[td][q4 * 4 + 2] * inv, oacc[td][q4 * 4 + 3] * inv};
            if constexpr (sizeof(T) == 4) *reinterpret_cast<float4 *>(static_cast<float *>(a.o) + row + dh) = make_float4(v[0], v[1], v[2], v[3]);
            else {   // hi = bf16(o), lo = bf16(o - hi): the out-projection contracts both
                uint32_t hi[2], lo[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    hi[e] = pack2_bf16(v[2 * e], v[2 * e + 1]);
                    lo[e] = pack2_bf16(v[2 * e] - __uint_as_float(hi[e] << 16), v[2 * e + 1] - __uint_as_float(hi[e] & 0xFFFF0000u));
                }
                *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(a.o) + row + dh) = make_uint2(hi[0], hi[1]);
                *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(a.o_lo) + row + dh) = make_uint2(lo[0], lo[1]);
            }
        }
}

template <typename T, int DH> static void launch_attention_f32_dh(const SmhaArgs &a, hipStream_t st)
{
    const int l_a = a.c * (a.l / a.m), units = a.b * a.k;
    // two query blocks per workgroup once that leaves a workgroup for every compute unit; key splits while the
    // grid has fewer waves than the chip has SIMDs
    const int nq = (long)((l_a + 63) / 64) * units >= 256 ? 2 : 1;
    const long blocks = (long)((l_a + 31) / 32) * units;
    const int ks = blocks >= 1024 || l_a <= 32 ? 1 : (blocks >= 512 || l_a <= 64 ? 2 : 4);
    const dim3 grid((l_a + 32 * nq - 1) / (32 * nq), units);
    if (nq == 2 && ks >= 2) hipLaunchKernelGGL((attention_f32_kernel<T, DH, 2, 2>), grid, dim3(256), 0, st, a);
    else if (nq == 2) hipLaunchKernelGGL((attention_f32_kernel<T, DH, 2, 1>), grid, dim3(128), 0, st, a);
    else if (ks == 4) hipLaunchKernelGGL((attention_f32_kernel<T, DH, 1, 4>), grid, dim3(256), 0, st, a);
    else if (ks == 2) hipLaunchKernelGGL((attention_f32_kernel<T, DH, 1, 2>), grid, dim3(128), 0, st, a);
    else hipLaunchKernelGGL((attention_f32_kernel<T, DH, 1, 1>), grid, dim3(64), 0, st, a);
}

template <typename T> static hipError_t launch_attention_f32(const SmhaArgs &a, hipStream_t st)
{
    if (a.d_h <= 32) launch_attention_f32_dh<T, 32>(a, st);
    else if (a.d_h <= 64) launch_attention_f32_dh<T, 64>(a, st);
    else launch_attention_f32_dh<T, 128>(a, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// MFMA attention (bf16, d_h in {32, 64, 128}), Eq. 33-34.  One wave owns 32 query rows of one unit and
// walks key tiles of 64, online softmax in fp32 (base 2: q arrives pre-scaled by log2(e)/sqrt(d_h)).
//
// Layout.  The scores are computed TRANSPOSED, S^T = K Q^T (v_mfma_f32_32x32x16_bf16), so that an
// accumulator lane holds one query column: the row max / row sum of the softmax are in-lane
// reductions plus one exchange with the partner lane (lane ^ 32), and the probabilities, converted
// in place, already ARE the B operand of the second product O^T = V^T P^T (the k-slots of an MFMA
// operand may hold any permutation of K as long as both operands agree, so V^T is read with the
// accumulator's key order: keys 16s+4h..+4 and 16s+8+4h..+4 for k-step s, half-wave h).
//
// What the kernel is bound by is the vector ALU work of the softmax, not the matrix pipe, so that work
// is kept to a max, an exp2, an add and half a convert per score:
//  * P V runs in fp16 (v_mfma_f32_32x32x16_f16): probabilities carry 11 significant bits, enough for
//    the 2e-2 bound with one MFMA pass (a bf16 P needs a (hi, lo) pair: twice the MFMAs plus the split
//    arithmetic).  The projection kernel writes V as fp16 straight from its fp32 accumulators (VF16;
//    11 significant bits instead of bf16's 8, |v| up to 65504).  When the caller needs V in bf16 (the
//    backward pass) the kernel converts bf16 -> fp16 while it stages the tile instead (exact for
//    |v| in [6.1e-5, 65504]).
//  * The running maximum is subtracted by the matrix pipe: the score accumulators are initialised
//    with -m instead of 0.  As long as no score of a tile exceeds the running maximum by more than
//    2^8 the tile needs no rescaling at all (p = exp2(s - m) <= 256 fits fp16 and fp32 sums); only
//    when one does (always on the first tile) the maximum moves and O and the row sum are rescaled.
//  * KSPLIT waves share a query block and take key tiles KSPLIT apart, so that a compute unit holds
//    two waves per SIMD also when the grid has only one wave of queries per SIMD: one wave's softmax
//    then runs under another's MFMAs.  Their (max, sum, O) triples are merged through LDS at the end.
// K and V tiles [key][d_h] are staged through double-buffered LDS as 16-byte row copies; the V^T
// fragments come out of the [key][d_h] tile through the transposing LDS read.
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint32_t pack2_f16(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));  // toward zero: never rounds up to inf
}

// One key tile of 64 keys for the 32 queries of a wave: scores, masks, the lazy running maximum, probabilities and
// O^T += V^T P^T.  kfrag(t, ks) gives the K fragment of accumulator tile t (keys t*32 + lane%32) for k-step ks,
// vfrag(s4, td) the V^T fragment of key step s4 for head-dim block td; km points at the tile's padding flags
// (one byte per key) or is NULL.  The staging of K and V is the caller's.
template <int DH, typename KF, typename VF>
__device__ __forceinline__ void attention_tile(const bf16x8_t (&qf)[DH / 16], f32x16_t (&oacc)[DH / 32], float &mrun, float &lsum, int kt,
                                               int l_a, int qrow, int qrow_first, bool causal, const unsigned char *km, int lane,
                                               KF kfrag, VF vfrag)
{
    constexpr int BKV = 64;
    constexpr float TAU = 8.0f;
    const int lh = lane >> 5;
    const bool masked = km != nullptr;
    // S^T tile: [64 keys x 32 queries] as two 32x32 accumulators, started at -m
    const float moff = mrun == -INFINITY ? 0.f : mrun;
    f32x16_t sacc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) sacc[t][q] = -moff;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bf16x8_t kf = kfrag(t, ks);
            sacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], sacc[t], 0, 0, 0);
        }
    // accumulator register q of tile t is key kt*64 + t*32 + (q/4)*8 + lh*4 + q%4.  Masks: a wave-uniform
    // test whether the tile can hold an inadmissible key for any query of the wave, then straight-line
    // selects (accumulators must not cross divergent branches).
    if ((kt + 1) * BKV > l_a || masked || (causal && (kt + 1) * BKV > qrow_first + 1)) {
        uint32_t kmw[2][4];   // the padding flags of this lane's keys, four consecutive keys per word
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq)
                kmw[t][gq] = masked ? *reinterpret_cast<const uint32_t *>(km + t * 32 + gq * 8 + lh * 4) : 0x01010101u;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int key = kt * BKV + t * 32 + (q >> 2) * 8 + lh * 4 + (q & 3);
                const bool ok = key < l_a && (!causal || key <= qrow) && ((kmw[t][q >> 2] >> ((q & 3) * 8)) & 0xFFu) != 0;
                sacc[t][q] = ok ? sacc[t][q] : -INFINITY;
            }
    }
    float tmax = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) tmax = fmaxf(tmax, sacc[t][q]);
    {   // largest score of the tile, relative to the running maximum: the other half-wave's value through
        // v_permlane32_swap (lanes 32-63 of the first result and lanes 0-31 of the second hold the partner's)
        const uint32_t tb = __float_as_uint(tmax);
        const auto sw = __builtin_amdgcn_permlane32_swap(tb, tb, false, false);
        tmax = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    // the maximum moves only when a score exceeds it by more than 2^TAU, or when there is none yet
    const bool move = tmax > TAU || (mrun == -INFINITY && tmax > -INFINITY);
    if (__builtin_amdgcn_ballot_w64(move) != 0) {   // wave-uniform: rare after the first tile
        if (move) {
            const float corr = mrun == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(-tmax);
            mrun = moff + tmax;
            lsum *= corr;
#pragma unroll
            for (int t = 0; t < DH / 32; ++t)
#pragma unroll
                for (int q = 0; q < 16; ++q) oacc[t][q] *= corr;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 16; ++q) sacc[t][q] -= tmax;
        }
    }
    float psum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const float pv = __builtin_amdgcn_exp2f(sacc[t][q]);   // exp2(-inf) = 0 for masked keys
            sacc[t][q] = pv;
            psum += pv;
        }
    lsum += psum;

    // O^T += V^T P^T over the 64 keys of the tile: four k-steps of 16 keys
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
        const int t = s4 >> 1, r0 = (s4 & 1) * 8;
        uint32_t ph[4];  // two probabilities per word, fp16
#pragma unroll
        for (int e = 0; e < 4; ++e) ph[e] = pack2_f16(sacc[t][r0 + 2 * e], sacc[t][r0 + 2 * e + 1]);
        const f16x8_t pf = __builtin_bit_cast(f16x8_t, make_uint4(ph[0], ph[1], ph[2], ph[3]));
#pragma unroll
        for (int td = 0; td < DH / 32; ++td) {
            const f16x8_t vf = vfrag(s4, td);
            oacc[td] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pf, oacc[td], 0, 0, 0);
        }
    }
}

// End of an attention workgroup: the key splits are merged (splits 1.. park their (max, row sum, O^T) in LDS, whose
// tile buffers are free once the key loop has ended on a barrier; split 0 folds them in, in split order), then
// split 0 normalises, applies the row's gate weight and writes o as a (hi, lo) bf16 pair and, if asked, the
// base-2 log-sum-exp of the row.
template <int DH, int NQ, int KSPLIT>
__device__ __forceinline__ void attention_finish(const SmhaArgs &a, unsigned char *lds_raw, int split, int qg, int lane, int g, int qrow,
                                                 int l_a, float w, f32x16_t (&oacc)[DH / 32], float mrun, float lsum)
{
    const int lh = lane >> 5;
    if constexpr (KSPLIT > 1) {
        float *mg = reinterpret_cast<float *>(lds_raw);
        constexpr int SLOT = DH / 2 + 2;   // floats per lane
        if (split > 0) {
            float *dst = mg + ((size_t)((split - 1) * NQ + qg) * 64 + lane) * SLOT;
            dst[0] = mrun;
            dst[1] = lsum;
#pragma unroll
            for (int t = 0; t < DH / 32; ++t)
#pragma unroll
                for (int q = 0; q < 16; ++q) dst[2 + t * 16 + q] = oacc[t][q];
        }
        __syncthreads();
        if (split > 0) return;
#pragma unroll
        for (int s = 1; s < KSPLIT; ++s) {
            const float *src = mg + ((size_t)((s - 1) * NQ + qg) * 64 + lane) * SLOT;
            const float m1 = src[0], l1 = src[1];
            const float mf = fmaxf(mrun, m1);
            // a side that has seen no admissible key (max = -inf) contributes nothing
            const float c0 = mrun == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrun - mf);
            const float c1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m1 - mf);
            lsum = lsum * c0 + l1 * c1;
#pragma unroll
            for (int t = 0; t < DH / 32; ++t)
#pragma unroll
                for (int q = 0; q < 16; ++q) oacc[t][q] = oacc[t][q] * c0 + src[2 + t * 16 + q] * c1;
            mrun = mf;
        }
    }

    if (qrow >= l_a) return;
    lsum += __shfl_xor(lsum, 32, 64);
    const float inv = lsum > 0.f ? w / lsum : 0.f;  // a row with no admissible key contributes nothing
    if (a.lse && lh == 0) a.lse[(size_t)g * l_a + qrow] = lsum > 0.f ? mrun + log2f(lsum) : 0.f;
    if (a.o_raw) {
        const float raw = lsum > 0.f ? 1.0f / lsum : 0.f;
        const size_t row = ((size_t)g * l_a + qrow) * DH;
        bf16_t *r_hi = static_cast<bf16_t *>(a.o_raw) + row, *r_lo = static_cast<bf16_t *>(a.o_raw_lo) + row;
#pragma unroll
        for (int td = 0; td < DH / 32; ++td)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                uint32_t hi[2], lo[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float v0 = oacc[td][i4 * 4 + 2 * e] * raw, v1 = oacc[td][i4 * 4 + 2 * e + 1] * raw;
                    hi[e] = pack2_bf16(v0, v1);
                    lo[e] = pack2_bf16(v0 - __uint_as_float(hi[e] << 16), v1 - __uint_as_float(hi[e] & 0xFFFF0000u));
                }
                *reinterpret_cast<uint2 *>(r_hi + td * 32 + i4 * 8 + lh * 4) = make_uint2(hi[0], hi[1]);
                *reinterpret_cast<uint2 *>(r_lo + td * 32 + i4 * 8 + lh * 4) = make_uint2(lo[0], lo[1]);
            }
    }
    bf16_t *o = static_cast<bf16_t *>(a.o) + ((size_t)g * l_a + qrow) * DH;
    bf16_t *o_lo = static_cast<bf16_t *>(a.o_lo) + ((size_t)g * l_a + qrow) * DH;
    // accumulator register q of tile td is head-dim index td*32 + (q/4)*8 + lh*4 + q%4.
    // o is written as hi = bf16(o) and lo = bf16(o - hi): the out-projection contracts both.
#pragma unroll
    for (int td = 0; td < DH / 32; ++td)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            uint32_t hi[2], lo[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float v0 = oacc[td][i4 * 4 + 2 * e] * inv, v1 = oacc[td][i4 * 4 + 2 * e + 1] * inv;
                hi[e] = pack2_bf16(v0, v1);
                lo[e] = pack2_bf16(v0 - __uint_as_float(hi[e] << 16), v1 - __uint_as_float(hi[e] & 0xFFFF0000u));
            }
            *reinterpret_cast<uint2 *>(o + td * 32 + i4 * 8 + lh * 4) = make_uint2(hi[0], hi[1]);
            *reinterpret_cast<uint2 *>(o_lo + td * 32 + i4 * 8 + lh * 4) = make_uint2(lo[0], lo[1]);
        }
}

template <int DH, int NQ, int KSPLIT, bool VF16>
__global__ __launch_bounds__(NQ *KSPLIT * 64) void attention_mfma_kernel(SmhaArgs a)
{
    constexpr int BKV = 64, KP = DH + 8, VP = 2 * b_pitch_dwords(DH), NTH = NQ * 64;  // NTH: threads that stage one split's tiles
    constexpr int CHUNKS = BKV * DH / 8, PER_T = (CHUNKS + NTH - 1) / NTH;
    constexpr int PD = 3;   // register sets of the K/V prefetch
    constexpr int K_BYTES = 2 * BKV * KP * 2, V_BYTES = 2 * BKV * VP * 2, SPLIT_BYTES = K_BYTES + V_BYTES + 2 * BKV;
    constexpr int MERGE_BYTES = (KSPLIT - 1) * NQ * 64 * (DH / 2 + 2) * 4;
    constexpr int LDS_BYTES = KSPLIT * SPLIT_BYTES > MERGE_BYTES ? KSPLIT * SPLIT_BYTES : MERGE_BYTES;
    __shared__ __align__(16) unsigned char lds_raw[LDS_BYTES];

    const int l_p = a.l / a.m, l_a = a.c * l_p;
    // Workgroup -> (unit, query block).  Hardware deals consecutive workgroup ids round-robin over the 8
    // XCDs, each with its own L2: the query blocks of one unit are given ids 8 apart, so that a unit's K and
    // V are fetched into one L2 only (units in groups of 8; a ragged last group keeps the plain order).
    int g, qblk;
    {
        const int nqb = (l_a + 32 * NQ - 1) / (32 * NQ), units = a.b * a.k, id = blockIdx.x;
        const int full = (units / 8) * 8 * nqb;   // ids that belong to whole groups of 8 units
        if (id < full) {
            const int grp = id / (8 * nqb), rem = id - grp * 8 * nqb;
            g = grp * 8 + (rem & 7);
            qblk = rem >> 3;
        } else {
            const int rem = id - full;
            g = (units / 8) * 8 + rem / nqb;
            qblk = rem % nqb;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: tile tests stay scalar
    const int split = wave / NQ, qg = wave - split * NQ, stid = tid - split * NTH;  // key split, query group, thread within the split
    const int lr = lane & 31, lh = lane >> 5;
    const int qrow = qblk * (32 * NQ) + qg * 32 + lr;
    unsigned char *sbase = lds_raw + (size_t)split * SPLIT_BYTES;
    uint16_t(*Ks)[BKV][KP] = reinterpret_cast<uint16_t(*)[BKV][KP]>(sbase);
    uint16_t(*Vs)[BKV][VP] = reinterpret_cast<uint16_t(*)[BKV][VP]>(sbase + K_BYTES);   // fp16, [key][d_h]
    unsigned char(*Km)[BKV] = reinterpret_cast<unsigned char(*)[BKV]>(sbase + K_BYTES + V_BYTES);
    const bf16_t *Q = static_cast<const bf16_t *>(a.q) + (size_t)g * l_a * DH;
    const bf16_t *Kg = static_cast<const bf16_t *>(a.kk) + (size_t)g * l_a * DH;
    const bf16_t *Vg = static_cast<const bf16_t *>(a.v) + (size_t)g * l_a * DH;

    // gate weight of this row (Eq. 36 with the optional gate flags): two dependent lookups, started
    // here so that they complete under the key loop instead of in front of the output stores
    float w = 1.0f;
    if (split == 0) {
        const int bb = g / a.k, i = clampi(a.expert_idx[g], a.n);
        if ((a.flags & F_GATE_EXPERT) && a.expert_gate) w *= a.expert_gate[(size_t)bb * a.n + i];
        if ((a.flags & F_GATE_PATCH) && a.patch_gate) {
            const int p = clampi(a.patch_idx[((size_t)bb * a.n + i) * a.c + min(qrow, l_a - 1) / l_p], a.m);
            w *= a.patch_gate[((size_t)bb * a.n + i) * a.m + p];
        }
    }

    bf16x8_t qf[DH / 16];
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (qrow < l_a) v = *reinterpret_cast<const uint4 *>(Q + (size_t)qrow * DH + ks * 16 + lh * 8);
        qf[ks] = __builtin_bit_cast(bf16x8_t, v);
    }

    f32x16_t oacc[DH / 32];
#pragma unroll
    for (int t = 0; t < DH / 32; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) oacc[t][q] = 0.f;
    float mrun = -INFINITY, lsum = 0.f;   // running maximum of this query (both half-waves agree), this lane's part of the row sum

    const bool causal = (a.flags & F_CAUSAL) != 0, masked = a.pad_mask != nullptr;
    const int nkt_all = (l_a + BKV - 1) / BKV;
    // K/V tiles travel global -> registers -> LDS.  A tile's loads are issued PD - 1 iterations before the
    // tile is used (PD register sets): one iteration of a key split is shorter than a memory round trip.
    struct Staged {   // plain words, moved one by one: whole-vector copies of a local array would be a memcpy, which
        uint32_t k[PER_T][4], v[PER_T][4];   // keeps the array out of the register file
        unsigned char km;
    };
    Staged set0, set1, set2;   // separate objects: each one small enough to live in registers
    // Loads are issued for every iteration, also past the last tile (the last tile again, never stored),
    // with clamped addresses instead of guards: straight-line code whose outstanding loads the
    // compiler can count, so a wait for one tile leaves the younger tiles in flight.
    static_assert(CHUNKS % NTH == 0, "every staging thread moves the same number of pieces");
    // Element offset of piece i in tile t: ((t * BKV + row_i) * DH + kc_i * 8), clamped to the same piece of
    // the last key (keys past l_a repeat the last key: their scores are masked to -inf below, so they get
    // probability 0 against finite V rows; zeroing the registers instead would make every load wait).
    uint32_t piece[PER_T], piece_last[PER_T];
#pragma unroll
    for (int i = 0; i < PER_T; ++i) {
        const int c = stid + i * NTH;
        piece[i] = (uint32_t)(c / (DH / 8)) * DH + (c % (DH / 8)) * 8;
        piece_last[i] = (uint32_t)(l_a - 1) * DH + (c % (DH / 8)) * 8;
    }
    auto load_global = [&](Staged &sr, int tile) {
        if (masked && stid < BKV) {
            const int key = tile * BKV + stid;
            sr.km = key < l_a && key_is_token(a, g, min(key, l_a - 1), l_p);
        }
        const uint32_t t0 = (uint32_t)min(tile, nkt_all) * (BKV * DH);   // a tile past the end: clamped below, never stored
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
            const uint32_t at = min(t0 + piece[i], piece_last[i]);
            const uint4 kq = *reinterpret_cast<const uint4 *>(Kg + at), vq = *reinterpret_cast<const uint4 *>(Vg + at);
            sr.k[i][0] = kq.x; sr.k[i][1] = kq.y; sr.k[i][2] = kq.z; sr.k[i][3] = kq.w;
            sr.v[i][0] = vq.x; sr.v[i][1] = vq.y; sr.v[i][2] = vq.z; sr.v[i][3] = vq.w;
        }
    };
    auto store_lds = [&](const Staged &sr, int buf) {
        if (masked && stid < BKV) Km[buf][stid] = sr.km;
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
            const int c = stid + i * NTH;
            {
                *reinterpret_cast<uint4 *>(&Ks[buf][c / (DH / 8)][(c % (DH / 8)) * 8]) = make_uint4(sr.k[i][0], sr.k[i][1], sr.k[i][2], sr.k[i][3]);
                const uint32_t u[4] = {sr.v[i][0], sr.v[i][1], sr.v[i][2], sr.v[i][3]};
                uint32_t h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // a bf16 v: widen to fp32 (a shift), then narrow; exact whenever fp16 can hold the value
                    if constexpr (VF16) h[e] = u[e];
                    else h[e] = pack2_f16(__uint_as_float(u[e] << 16), __uint_as_float(u[e] & 0xFFFF0000u));
                }
                *reinterpret_cast<uint4 *>(&Vs[buf][c / (DH / 8)][(c % (DH / 8)) * 8]) = make_uint4(h[0], h[1], h[2], h[3]);
            }
        }
    };

    // under the causal mask no query of this workgroup sees keys past the workgroup's last row
    const int key_end = causal ? min(l_a, (qblk + 1) * 32 * NQ) : l_a;
    const int nkt = (key_end + BKV - 1) / BKV;
    const int nit = (nkt + KSPLIT - 1) / KSPLIT;   // iterations: split s takes tiles s, s + KSPLIT, ...
    auto tile_of = [&](int it) { return it * KSPLIT + split; };   // this split's it-th tile (exists if < nkt)
    set0.km = set1.km = set2.km = 1;
    load_global(set0, tile_of(0));
    load_global(set1, tile_of(1));
    store_lds(set0, 0);
    __syncthreads();
    // one iteration; J = it % PD picks the register sets at compile time (arrays indexed by a run-time
    // value would leave the register file)
    auto iteration = [&](auto jc, int it) {
        constexpr int J = decltype(jc)::value;
        const int kt = tile_of(it), buf = it & 1;
        Staged &fill = J == 0 ? set2 : (J == 1 ? set0 : set1), &drain = J == 0 ? set1 : (J == 1 ? set2 : set0);
        load_global(fill, tile_of(it + PD - 1));
        if (kt < nkt) {
            attention_tile<DH>(qf, oacc, mrun, lsum, kt, l_a, qrow, qblk * (32 * NQ) + qg * 32, causal, masked ? &Km[buf][0] : nullptr, lane,
                               [&](int t, int ks) { return *reinterpret_cast<const bf16x8_t *>(&Ks[buf][t * 32 + lr][ks * 16 + lh * 8]); },
                               [&](int s4, int td) {
                                   // V^T fragment for head-dim column td*32 + lr: keys 16*s4 + 4*lh + 0..3, then + 8
                                   const uint16_t *vsrc = &Vs[buf][s4 * 16 + lh * 4 + ((lane & 15) >> 2)][td * 32 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4];
                                   const uint2 v0 = lds_read_tr4(vsrc);
                                   const uint2 v1 = lds_read_tr4(vsrc + 8 * VP);
                                   return __builtin_bit_cast(f16x8_t, make_uint4(v0.x, v0.y, v1.x, v1.y));
                               });
        }
        if (tile_of(it + 1) < nkt) store_lds(drain, buf ^ 1);
        __syncthreads();
    };
    static_assert(PD == 3, "the loop below names the register sets");
    for (int it0 = 0; it0 < nit; it0 += PD) {   // nit is uniform over the workgroup
        iteration(std::integral_constant<int, 0>{}, it0);
        if (it0 + 1 < nit) iteration(std::integral_constant<int, 1>{}, it0 + 1);
        if (it0 + 2 < nit) iteration(std::integral_constant<int, 2>{}, it0 + 2);
    }

    attention_finish<DH, NQ, KSPLIT>(a, lds_raw, split, qg, lane, g, qrow, l_a, w, oacc, mrun, lsum);
}

// The same kernel with K and V tiles copied from global memory straight into LDS (global_load_lds_dwordx4:
// 16 bytes per lane, the 64 lanes of an instruction fill 1 KiB of consecutive LDS), three tiles deep: no
// staging registers, no LDS store instructions and no converts in the loop, and a wave waits for a tile only
// when it needs it.  What that takes: V already in fp16 in memory (the projection kernel writes it so), the
// padding flags of all the unit's keys in LDS before the loop (PAD, up to DMA_PAD_KEYS of them: their lookups are ordinary
// loads, whose compiler-placed waits would drain the copies in flight; longer masked units take the register-staged
// kernel), and unpadded tiles, so bank conflicts are avoided
// by permuting which 16-byte piece of a row an LDS slot receives (every lane supplies its own global
// address): K slot (r, pos) <- piece pos ^ ((r / (16/CK)) % CK), the rule for tiles read as row fragments; V
// slot (r, pos) <- piece pos ^ ((r & 3) << 2) for 256-byte rows (d_h = 128) and pos ^ (((r >> 1) & 1) << 2) for
// 128-byte rows (d_h = 64), the rule for tiles read with the transposing LDS read.  The copies are inline
// assembly that the compiler cannot count, so their completion is waited for by hand (they complete in
// issue order): at the top of an iteration at most the copies of the STAGES-2 younger tiles may be
// outstanding, then one barrier publishes every wave's part of the tile and frees the buffer of the tile
// before for the copies issued right after it.
// 4096 flags: a choice, not a bound (160 KiB hold 128 KiB of tiles and four times as many); longer masked units were not
// measured on this kernel and stay on the register-staged one.  The masked lm forward, 32 units of 128 keys at d_h 64, goes
// 65.6 -> 64.4 us in all.
constexpr int DMA_PAD_KEYS = 4096;
template <int DH, int NQ, int KSPLIT, bool PAD>
__global__ __launch_bounds__(NQ *KSPLIT * 64) void attention_dma_kernel(SmhaArgs a)
{
    static_assert(DH == 64 || DH == 128, "piece permutations are written for 128- and 256-byte rows");
    constexpr int BKV = 64, STAGES = 4;
    constexpr int CK = DH / 8;                        // 16-byte pieces per row
    constexpr int RPI = 64 / CK;                      // rows one copy instruction covers
    constexpr int TILE_BYTES = BKV * DH * 2, INSTR = TILE_BYTES / 1024;
    constexpr int PER_W = INSTR / NQ;                 // copy instructions per wave, tile and operand
    static_assert(INSTR % NQ == 0, "every wave of a split issues the same number of copies");
    constexpr int SPLIT_BYTES = STAGES * 2 * TILE_BYTES;
    constexpr int MERGE_BYTES = (KSPLIT - 1) * NQ * 64 * (DH / 2 + 2) * 4;
    constexpr int LDS_BYTES = KSPLIT * SPLIT_BYTES > MERGE_BYTES ? KSPLIT * SPLIT_BYTES : MERGE_BYTES;
    __shared__ __align__(1024) unsigned char lds_raw[LDS_BYTES];
    __shared__ __align__(16) unsigned char Km[PAD ? DMA_PAD_KEYS : 16];   // key admissible under the padding mask

    const int l_p = a.l / a.m, l_a = a.c * l_p;
    int g, qblk;   // workgroup -> (unit, query block): the query blocks of a unit share an XCD (see attention_mfma_kernel)
    {
        const int nqb = (l_a + 32 * NQ - 1) / (32 * NQ), units = a.b * a.k, id = blockIdx.x;
        const int full = (units / 8) * 8 * nqb;
        if (id < full) {
            const int grp = id / (8 * nqb), rem = id - grp * 8 * nqb;
            g = grp * 8 + (rem & 7);
            qblk = rem >> 3;
        } else {
            const int rem = id - full;
            g = (units / 8) * 8 + rem / nqb;
            qblk = rem % nqb;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int split = wave / NQ, qg = wave - split * NQ;
    const int lr = lane & 31, lh = lane >> 5;
    const int qrow = qblk * (32 * NQ) + qg * 32 + lr;
    unsigned char *sbase = lds_raw + (size_t)split * SPLIT_BYTES;   // stage s: K tile at s * 2 * TILE_BYTES, V tile after it
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)sbase;
    const bf16_t *Q = static_cast<const bf16_t *>(a.q) + (size_t)g * l_a * DH;
    const uint16_t *Kg = static_cast<const uint16_t *>(a.kk) + (size_t)g * l_a * DH;
    const uint16_t *Vg = static_cast<const uint16_t *>(a.v) + (size_t)g * l_a * DH;

    float w = 1.0f;   // gate weight of this row (Eq. 36), looked up early
    if (split == 0) {
        const int bb = g / a.k, i = clampi(a.expert_idx[g], a.n);
        if ((a.flags & F_GATE_EXPERT) && a.expert_gate) w *= a.expert_gate[(size_t)bb * a.n + i];
        if ((a.flags & F_GATE_PATCH) && a.patch_gate) {
            const int p = clampi(a.patch_idx[((size_t)bb * a.n + i) * a.c + min(qrow, l_a - 1) / l_p], a.m);
            w *= a.patch_gate[((size_t)bb * a.n + i) * a.m + p];
        }
    }
    bf16x8_t qf[DH / 16];
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (qrow < l_a) v = *reinterpret_cast<const uint4 *>(Q + (size_t)qrow * DH + ks * 16 + lh * 8);
        qf[ks] = __builtin_bit_cast(bf16x8_t, v);
    }
    f32x16_t oacc[DH / 32];
#pragma unroll
    for (int t = 0; t < DH / 32; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) oacc[t][q] = 0.f;
    float mrun = -INFINITY, lsum = 0.f;

    auto v_swz = [](int r) { return (DH == 128 ? (r & 3) : ((r >> 1) & 1)) << 2; };
    // Copy roles.  Instruction j of this wave fills 1 KiB block qg * PER_W + j of a tile: lane -> slot (row, pos).
    // Element offsets inside the unit's K (V) array, for tile 0; a tile adds BKV * DH.  Keys past l_a repeat
    // the last key (their scores are masked, so they get probability 0 against finite V rows).
    uint32_t k_off[PER_W], v_off[PER_W], k_last[PER_W], v_last[PER_W];
#pragma unroll
    for (int j = 0; j < PER_W; ++j) {
        const int r = (qg * PER_W + j) * RPI + lane / CK, pos = lane % CK;
        const int kp = pos ^ ((r / (16 / CK)) % CK), vp = pos ^ v_swz(r);
        k_off[j] = (uint32_t)r * DH + kp * 8;
        v_off[j] = (uint32_t)r * DH + vp * 8;
        k_last[j] = (uint32_t)(l_a - 1) * DH + kp * 8;
        v_last[j] = (uint32_t)(l_a - 1) * DH + vp * 8;
    }
    const bool causal = (a.flags & F_CAUSAL) != 0;
    const int nkt_all = (l_a + BKV - 1) / BKV;
    const int key_end = causal ? min(l_a, (qblk + 1) * 32 * NQ) : l_a;   // no query of this workgroup sees later keys
    const int nkt = (key_end + BKV - 1) / BKV;
    const int nit = (nkt + KSPLIT - 1) / KSPLIT;   // iterations: split s takes tiles s, s + KSPLIT, ...
    auto tile_of = [&](int it) { return it * KSPLIT + split; };
    // copies are issued for every iteration, also past the last tile (clamped to the end, never read): the
    // number outstanding is then the same in every iteration
    auto issue = [&](int it, int stage) {
        const uint32_t t0 = (uint32_t)min(tile_of(it), nkt_all) * (BKV * DH);
        const uint32_t dst = lds_base + stage * (2 * TILE_BYTES) + qg * PER_W * 1024;
#pragma unroll
        for (int j = 0; j < PER_W; ++j) {
            dma_load16(Kg + min(t0 + k_off[j], k_last[j]), dst + j * 1024);
            dma_load16(Vg + min(t0 + v_off[j], v_last[j]), dst + TILE_BYTES + j * 1024);
        }
    };
#pragma unroll
    for (int q = 0; q < STAGES - 1; ++q) issue(q, q);
    if constexpr (PAD)   // under the first copies; published by the loop's first barrier
        for (int key = tid; key < nkt_all * BKV; key += NQ * KSPLIT * 64) Km[key] = key < l_a && key_is_token(a, g, min(key, l_a - 1), l_p);
    // fragment offsets (bytes inside a stage): K row fragments, V^T through the transposing read
    const int vx = (lane & 15) >> 2;   // row of the 4-row group this lane points at
    int stage = 0, fill = STAGES - 1;
    for (int it = 0; it < nit; ++it) {   // nit is uniform over the workgroup
        dma_wait<(STAGES - 2) * 2 * PER_W>();
        __syncthreads();
        issue(it + STAGES - 1, fill);
        const int kt = tile_of(it);
        if (kt < nkt) {
            const unsigned char *kb = sbase + stage * (2 * TILE_BYTES), *vb = kb + TILE_BYTES;
            attention_tile<DH>(qf, oacc, mrun, lsum, kt, l_a, qrow, qblk * (32 * NQ) + qg * 32, causal, PAD ? Km + kt * BKV : nullptr, lane,
                               [&](int t, int ks) {
                                   const int r = t * 32 + lr;
                                   return *reinterpret_cast<const bf16x8_t *>(kb + r * (DH * 2) + (((ks * 2 + lh) ^ ((r / (16 / CK)) % CK)) * 16));
                               },
                               [&](int s4, int td) {
                                   // keys 16*s4 + 4*lh + vx, then + 8 (the same permutation of both rows), head-dim columns
                                   // td*32 + ((lane>>4)&1)*16 + (lane&3)*4 .. +3
                                   const int r = s4 * 16 + lh * 4 + vx;
                                   const int piece = (td * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ v_swz(r);
                                   const uint16_t *vsrc = reinterpret_cast<const uint16_t *>(vb + r * (DH * 2) + piece * 16 + (lane & 1) * 8);
                                   const uint2 v0 = lds_read_tr4(vsrc);
                                   const uint2 v1 = lds_read_tr4(vsrc + 8 * DH);
                                   return __builtin_bit_cast(f16x8_t, make_uint4(v0.x, v0.y, v1.x, v1.y));
                               });
        }
        stage = stage + 1 == STAGES ? 0 : stage + 1;
        fill = fill + 1 == STAGES ? 0 : fill + 1;
    }
    dma_wait<0>();     // the copies past the last tile
    __syncthreads();   // every wave is done with the tiles: LDS is free for the merge
    attention_finish<DH, NQ, KSPLIT>(a, lds_raw, split, qg, lane, g, qrow, l_a, w, oacc, mrun, lsum);
}

// Launch shape: NQ waves of 32 queries per workgroup (more share K/V tiles, fewer give more workgroups:
// at least one workgroup per compute unit if possible), KSPLIT key splits so that the grid holds two
// waves per SIMD (2048 waves) where the key tiles allow it.
template <int DH, int NQ, int KSPLIT> static void launch_attention_shape(const SmhaArgs &a, hipStream_t st)
{
    const int l_a = a.c * (a.l / a.m), units = a.b * a.k;
    const dim3 grid(((l_a + 32 * NQ - 1) / (32 * NQ)) * units), block(NQ * KSPLIT * 64);
    if (a.keep_v_bf16) {
        hipLaunchKernelGGL((attention_mfma_kernel<DH, NQ, KSPLIT, false>), grid, block, 0, st, a);
        return;
    }
    // (LDS: stages x (K + V tile) per split, and the flags; every wave the same number of copies; the wait count fits its field)
    if constexpr ((DH == 64 || DH == 128) && KSPLIT * 4 * 2 * 64 * DH * 2 + DMA_PAD_KEYS <= 160 * 1024 && (64 * DH * 2 / 1024) % NQ == 0 &&
                  2 * 2 * (64 * DH * 2 / 1024 / NQ) <= 63) {
        if (!a.pad_mask) {   // V in fp16: tiles copied straight into LDS
            hipLaunchKernelGGL((attention_dma_kernel<DH, NQ, KSPLIT, false>), grid, block, 0, st, a);
            return;
        }
        if (l_a <= DMA_PAD_KEYS) {
            hipLaunchKernelGGL((attention_dma_kernel<DH, NQ, KSPLIT, true>), grid, block, 0, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((attention_mfma_kernel<DH, NQ, KSPLIT, true>), grid, block, 0, st, a);
}

template <int DH> static hipError_t launch_attention_mfma_dh(const SmhaArgs &a, hipStream_t st)
{
    const int l_a = a.c * (a.l / a.m), units = a.b * a.k;
    const long waves = (long)units * ((l_a + 31) / 32);
    const int nkt = (l_a + 63) / 64;
    int ks = 1;
    while (ks < 4 && waves * ks < 2048 && 2 * ks <= nkt) ks *= 2;
    if (DH > 32 && ks > 2) ks = 2;     // LDS: four splits fit a compute unit only with d_h = 32 tiles
    int nq = 4;
    while (nq > 1 && ((l_a + 32 * nq - 1) / (32 * nq)) * (long)units < 256) nq >>= 1;
    if (nq == 4 && ks == 4) ks = 2;    // at most 8 waves per workgroup
#define UOE_ATT(NQ, KS) launch_attention_shape<DH, NQ, KS>(a, st)
    if (nq == 4) { if (ks == 1) UOE_ATT(4, 1); else UOE_ATT(4, 2); }
    else if (nq == 2) {
        if (ks == 1) UOE_ATT(2, 1);
        else if (ks == 2) UOE_ATT(2, 2);
        else if constexpr (DH == 32) UOE_ATT(2, 4);
    } else {
        if (ks == 1) UOE_ATT(1, 1);
        else if (ks == 2) UOE_ATT(1, 2);
        else if constexpr (DH == 32) UOE_ATT(1, 4);
    }
#undef UOE_ATT
    return hipGetLastError();
}

static hipError_t launch_attention_mfma(const SmhaArgs &a, hipStream_t st)
{
    if (a.d_h == 32) return launch_attention_mfma_dh<32>(a, st);
    if (a.d_h == 64) return launch_attention_mfma_dh<64>(a, st);
    return launch_attention_mfma_dh<128>(a, st);
}

template <typename T, bool ROPE> static QkvProblem<T, false, ROPE> make_qkv(const SmhaArgs &a)
{
    QkvProblem<T, false, ROPE> qp;
    qp.x = static_cast<const T *>(a.x);
    qp.wq = static_cast<const T *>(a.wq);
    qp.wk = static_cast<const T *>(a.wk);
    qp.wv = static_cast<const T *>(a.wv);
    qp.expert_idx = a.expert_idx;
    qp.patch_idx = a.patch_idx;
    qp.q = static_cast<T *>(a.q);
    qp.k = static_cast<T *>(a.kk);
    qp.v = static_cast<T *>(a.v);
    qp.l = a.l; qp.d = a.d; qp.n = a.n; qp.kact = a.k; qp.m = a.m; qp.c = a.c;
    qp.l_p = a.l / a.m; qp.l_a = a.c * qp.l_p; qp.d_h = a.d_h;
    qp.q_scale = 1.0f;
    qp.nout = 3;
    qp.rope_dim = ROPE ? a.rope_dim : 0;
    qp.q32 = nullptr;
    return qp;
}

template <typename T> static OutProjProblem<T> make_outproj(const SmhaArgs &a)
{
    OutProjProblem<T> op;
    op.o = static_cast<const T *>(a.o);
    op.o_lo = nullptr;
    op.parts = 1;
    op.wo = static_cast<const T *>(a.wo);
    op.x = static_cast<const T *>(a.x);
    op.expert_idx = a.expert_idx;
    op.patch_idx = a.patch_idx;
    op.out = static_cast<T *>(a.out);
    op.l = a.l; op.d = a.d; op.n = a.n; op.kact = a.k; op.m = a.m; op.c = a.c;
    op.l_p = a.l / a.m; op.l_a = a.c * op.l_p; op.d_h = op.o_row = a.d_h; op.flags = a.flags;
    return op;
}

// fp32 storage, and bf16 storage where the bf16 attention kernels do not apply: any width, attention in
// fp32 products (attention_f32_kernel)
template <typename T> static hipError_t smha_f32(const SmhaArgs &a, hipStream_t st)
{
    constexpr bool BF = std::is_same<T, bf16_t>::value;
    const int l_p = a.l / a.m, l_a = a.c * l_p, units = a.b * a.k;
    hipError_t err;
    if (!(a.skip & SMHA_STEP_QKV)) {
        if (BF && a.rope_dim > 0) err = launch_gemm_tail<0>(make_qkv<T, BF>(a), units, l_a, 3 * a.d_h, st);
        else err = launch_gemm_tail<0>(make_qkv<T, false>(a), units, l_a, 3 * a.d_h, st);
        if (err != hipSuccess) return err;
        if (!BF && (err = launch_rope_f32(a, st)) != hipSuccess) return err;
    }
    if (!(a.skip & SMHA_STEP_ATTENTION) && (err = launch_attention_f32<T>(a, st)) != hipSuccess) return err;
    if (a.skip & SMHA_STEP_OUT) return hipSuccess;
    OutProjProblem<T> op = make_outproj<T>(a);
    if (BF) {
        op.o_lo = static_cast<const T *>(a.o_lo);
        op.parts = 2;
    }
    const int groups = a.b * op.set_patch_groups(a.b);
    return launch_gemm_tail<0>(op, groups, op.gp * l_p, a.d, st);
}

// Tile choice of the pipelined output-stationary contraction (out-projection of SMHA, second layer
// of the data-selected UoME).  A group is a short chain of dependent steps (find the experts that picked its patches,
// fetch their rows, a few K-steps, add the residual), so with many groups what counts is how many of them a CU holds at
// once, and with few that every K-step is in flight.  us, out-projection alone, looped:
//   groups of 65 rows and more (several short patches): 128x128, eight waves (14-token patches 17.8, 32-row tiles 21.6)
//   64-row patches: two stage buffers and four workgroups a CU while that gives 2048 of them, else four stage buffers
//   32-row tiles: 512 groups and more two-wave workgroups with two stage buffers, else four waves and four buffers
template <typename OP> static hipError_t launch_outproj_dma(const OP &op, int groups, int rows, int d, hipStream_t st)
{
    if (rows > 64) return launch_gemm_dma<OP, 128, 128, 32, 2, 4, 3, 4>(op, groups, rows, d, st);
    if (rows <= 32 && groups >= 512) return launch_gemm_dma<OP, 32, 128, 32, 1, 2, 2, 4>(op, groups, rows, d, st);
    if (rows <= 32) return launch_gemm_dma<OP, 32, 128, 32, 1, 4, 4, 2>(op, groups, rows, d, st);
    if ((long)groups * ((d + 127) / 128) >= 2048) return launch_gemm_dma<OP, 64, 128, 32, 2, 2, 2, 4>(op, groups, rows, d, st);
    return launch_gemm_dma<OP, 64, 128, 32, 2, 2, 4, 2>(op, groups, rows, d, st);
}

// Projections of the MFMA path.  ROPE apart at compile time: with the rotation behind a run-time test calls without it were
// 1.2 % slower (the layer at 8 x 512 x 512 62.2 -> 62.9 us; apart 61.0).
template <bool ROPE> static hipError_t launch_projections(const SmhaArgs &a, hipStream_t st)
{
    typedef QkvProblem<bf16_t, false, ROPE> QP;
    const int l_p = a.l / a.m, l_a = a.c * l_p, units = a.b * a.k;
    QP qp = make_qkv<bf16_t, ROPE>(a);
    qp.q_scale = 1.4426950408889634f / sqrtf((float)a.d_h);  // base-2 softmax in the MFMA kernel
    qp.v_f16 = !a.keep_v_bf16;
    qp.v_copy = static_cast<bf16_t *>(a.v_copy);
    // 64x64 tiles (one 64-column stretch of q, k or v: the gathered rows are read three times, out of L2, for three times
    // the workgroups, three per compute unit) up to 1024 of them; one workgroup for q, k and v beyond.  us, looped:
    // 32 units of 128 rows x 512 x 192 5.9 (32x64 tiles 7.0), 32 of 512 x 256 x 96 5.9 (128x128 8.9), 64 of 256 x 768 x 192 11.6
    // (64x192 13.2), 384 of 56 x 384 x 192 11.9 against 11.7, 32 of 1024 x 1024 x 192 24.2 with 128x192 (64x64 26.5)
    const int N = 3 * a.d_h;
    const bool k64 = a.d % 64 == 0;
    const long t64 = (long)units * ((l_a + 63) / 64) * ((N + 63) / 64);
    if (k64 && l_a > 32 && t64 <= 1024) return launch_gemm_dma<QP, 64, 64, 64, 2, 2, 3, 3>(qp, units, l_a, N, st);
    if (a.d_h == 64) {
        if (l_a >= 256) return k64 ? launch_gemm_dma<QP, 128, 192, 64, 2, 2, 3>(qp, units, l_a, N, st)
                                   : launch_gemm_dma<QP, 128, 192, 32, 2, 2, 3, 2>(qp, units, l_a, N, st);
        if (l_a > 32) return launch_gemm_dma<QP, 64, 192, 32, 2, 2, 3, 2>(qp, units, l_a, N, st);
        if (k64 && (long)units < 256) return launch_gemm_dma<QP, 32, 64, 64, 1, 2, 4>(qp, units, l_a, N, st);
        return k64 ? launch_gemm_dma<QP, 32, 192, 64, 1, 2, 4>(qp, units, l_a, N, st)
                   : launch_gemm_dma<QP, 32, 192, 32, 1, 2, 4>(qp, units, l_a, N, st);
    }
    if (l_a > 32) return l_a > 64 ? launch_gemm_dma<QP, 128, 128, 32, 2, 4, 3, 4>(qp, units, l_a, N, st)
                                  : launch_gemm_dma<QP, 64, 128, 32, 2, 4, 4, 4>(qp, units, l_a, N, st);
    return k64 ? launch_gemm_dma<QP, 32, 128, 64, 1, 2, 4>(qp, units, l_a, N, st)
               : launch_gemm_dma<QP, 32, 128, 32, 1, 2, 4>(qp, units, l_a, N, st);
}

// projections, rotary embedding and attention of the MFMA path
hipError_t launch_smha_qkv_attention(const SmhaArgs &a, hipStream_t st)
{
    hipError_t err;
    if (!(a.skip & SMHA_STEP_QKV)
        && (err = a.rope_dim > 0 ? launch_projections<true>(a, st) : launch_projections<false>(a, st)) != hipSuccess) return err;
    if (a.skip & SMHA_STEP_ATTENTION) return hipSuccess;
    return launch_attention_mfma(a, st);
}

static hipError_t smha_mfma(const SmhaArgs &a, hipStream_t st)
{
    typedef OutProjProblem<bf16_t> OP;
    const int l_p = a.l / a.m;
    hipError_t err;
    if ((err = launch_smha_qkv_attention(a, st)) != hipSuccess) return err;
    if (a.skip & SMHA_STEP_OUT) return hipSuccess;
    OP op = make_outproj<bf16_t>(a);
    op.once = stream_once((size_t)a.b * a.l * a.d * sizeof(bf16_t));
    op.o_lo = static_cast<const bf16_t *>(a.o_lo);   // the MFMA attention kernel writes o as a (hi, lo) bf16 pair
    op.parts = 2;
    const int groups = a.b * op.set_patch_groups(a.b);
    return launch_outproj_dma(op, groups, op.gp * l_p, a.d, st);
}

// ---------------------------------------------------------------------------------------------
// UoME with patch-wise data selection (Eq. 37-40).  Same skeleton as SMHA without the attention:
// first layer per active unit on its gathered rows (UomeDsUpProblem), second layer + index add as
// the output-stationary contraction over the experts that picked each patch (OutProjProblem with
// A^O in the place of W^o and the hidden activations in the place of o).
template <typename T, bool EXACT> static UomeDsUpProblem<T, EXACT> make_ds_up(const UomeDsArgs &a)
{
    UomeDsUpProblem<T, EXACT> up;
    up.u = static_cast<const T *>(a.u);
    up.a_in = static_cast<const T *>(a.a_in);
    up.expert_idx = a.expert_idx;
    up.patch_idx = a.patch_idx;
    up.expert_gate = (a.flags & F_GATE_EXPERT) ? a.expert_gate : nullptr;
    up.patch_gate = (a.flags & F_GATE_PATCH) ? a.patch_gate : nullptr;
    up.hidden = static_cast<T *>(a.hidden);
    up.l = a.l; up.d = a.d; up.n = a.n; up.kact = a.k; up.m = a.m; up.c = a.c;
    up.l_p = a.l / a.m; up.l_a = a.c * up.l_p; up.d_e = a.d_e;
    return up;
}

template <typename T> static OutProjProblem<T> make_ds_down(const UomeDsArgs &a)
{
    OutProjProblem<T> op;
    op.o = static_cast<const T *>(a.hidden);
    op.o_lo = nullptr;
    op.parts = 1;
    op.wo = static_cast<const T *>(a.a_out);
    op.x = static_cast<const T *>(a.u);
    op.expert_idx = a.expert_idx;
    op.patch_idx = a.patch_idx;
    op.out = static_cast<T *>(a.out);
    op.l = a.l; op.d = a.d; op.n = a.n; op.kact = a.k; op.m = a.m; op.c = a.c;
    op.l_p = a.l / a.m; op.l_a = a.c * op.l_p; op.d_h = op.o_row = a.d_e; op.flags = a.flags;
    return op;
}

// any width, either storage type; SiLU by a division
template <typename T> static hipError_t uome_ds_tail(const UomeDsArgs &a, hipStream_t st)
{
    const int l_p = a.l / a.m, l_a = a.c * l_p;
    hipError_t err;
    if ((err = launch_gemm_tail<0>(make_ds_up<T, true>(a), a.b * a.k, l_a, a.d_e, st)) != hipSuccess) return err;
    OutProjProblem<T> op = make_ds_down<T>(a);
    const int groups = a.b * op.set_patch_groups(a.b);
    return launch_gemm_tail<0>(op, groups, op.gp * l_p, a.d, st);
}

static hipError_t uome_ds_mfma(const UomeDsArgs &a, hipStream_t st)
{
    typedef UomeDsUpProblem<bf16_t> UP;
    typedef OutProjProblem<bf16_t> OP;
    const int l_p = a.l / a.m, l_a = a.c * l_p, units = a.b * a.k;
    hipError_t err;
    const UP up = make_ds_up<bf16_t, false>(a);
    if ((err = launch_gemm_dma_auto(up, units, l_a, a.d_e, a.d, a.d, st)) != hipSuccess) return err;
    OP op = make_ds_down<bf16_t>(a);
    op.once = stream_once((size_t)a.b * a.l * a.d * sizeof(bf16_t));   // u's last use, the block's output
    const int groups = a.b * op.set_patch_groups(a.b);
    return launch_outproj_dma(op, groups, op.gp * l_p, a.d, st);
}

hipError_t launch_uome_ds(const UomeDsArgs &a, bool bf16, hipStream_t st)
{
    if (bf16 && a.d % 32 == 0 && a.d_e % 32 == 0) return uome_ds_mfma(a, st);
    return bf16 ? uome_ds_tail<bf16_t>(a, st) : uome_ds_tail<float>(a, st);
}

// The bf16 kernels (bf16 products, probabilities and v in fp16) take widths that are multiples of 32, heads of 32, 64 or 128
// and units whose keys 32-bit element offsets reach.  Everything else runs on fp32 products: padding the other heads
// into the bf16 kernels is faster (6 x 1000 tokens, d 360, heads of 40: the layer's forward 76 us against 87), but it held their
// probabilities in 16 bits and v in fp16, where |v| above 65504 is infinite and below 6e-8 zero.
hipError_t launch_smha(const SmhaArgs &a, bool bf16, hipStream_t st)
{
    if (!bf16) return smha_f32<float>(a, st);
    const bool heads = a.d_h == 32 || a.d_h == 64 || a.d_h == 128;
    if (a.d % 32 == 0 && heads && (long)a.c * (a.l / a.m) * a.d_h < (1L << 31)) return smha_mfma(a, st);
    return smha_f32<bf16_t>(a, st);
}

}  // namespace uoe
