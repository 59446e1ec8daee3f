// Backward passes of the SMHA block (Eq. 27-36, Eq. 32 RoPE, the masks of Sec. III-C.3) and of the UoME block
// in expert-selection mode (Eq. 38-40 with Eq. 24-26) for every shape and storage type the kernels of
// smha_bwd.hip / uome_bwd.hip do not take: fp32 storage, head or expert widths and token counts that are not
// multiples of 32 (a 14-token patch, a 196-token sequence).  Same formulas, on the matrix cores, with
// intermediates as exact as fp32 storage (or the final bf16 rounding) can show:
//  * fp32 storage: every contraction through the pipelined engine, operands split in three bf16 parts (SplitF32).
//  * bf16 storage: x, u, the upstream gradient and the weights enter as they are; what the pass computes in between
//    stays in fp32 or, where it is the operand of another contraction, is a pair of bf16 values hi + lo
//    (16 significant bits, 2^-17 relative, against the 2^-9 of the rounded outputs), contracted as two K
//    segments that share the other operand.  Over 45 drawn SMHA and 40 drawn UoME shapes every gradient is as far from
//    fp64 as with fp32 operands, to four digits; the gate gradients, outputs in fp32, are formed before the split.
//  * attention: both products of every tile in fp32 (v_mfma_f32_32x32x2_f32), probabilities never stored.
// The vector-ALU kernels before it took one thread per output element (SMHA) or 64x64 tiles fetched element by
// element (UoME): vit shape, bf16, layer forward + backward 4617 us, lm shape in fp32 2423 us; here 700 and 558 us.
// Every sum has a fixed order (no atomics: results do not depend on scheduling).
#include "common.h"
#include "problems.h"
#include "gemm_mfma.h"
#include "gemm_dma.h"
#include "wgrad_reduce.h"
#include "route_prep.h"
#include "unit_grid.h"

namespace uoe {

namespace {

// parts of a left operand the pass computed: one fp32 value, or bf16 hi and lo
template <typename T> struct parts_of {
    static constexpr int value = 2;
};
template <> struct parts_of<float> {
    static constexpr int value = 1;
};

// four values as they enter the next contraction: fp32, or hi at `dst` and lo `plane` elements behind it
__device__ __forceinline__ void put4_operand(float *dst, long, float4 v) { *reinterpret_cast<float4 *>(dst) = v; }
__device__ __forceinline__ void put4_operand(bf16_t *dst, long plane, float4 v)
{
    const uint32_t h0 = pack2_bf16(v.x, v.y), h1 = pack2_bf16(v.z, v.w);
    const uint32_t l0 = pack2_bf16(v.x - __uint_as_float(h0 << 16), v.y - __uint_as_float(h0 & 0xFFFF0000u));
    const uint32_t l1 = pack2_bf16(v.z - __uint_as_float(h1 << 16), v.w - __uint_as_float(h1 & 0xFFFF0000u));
    *reinterpret_cast<uint2 *>(dst) = make_uint2(h0, h1);
    *reinterpret_cast<uint2 *>(dst + plane) = make_uint2(l0, l1);
}

// members every problem below shares: no residual, no factors
struct PlainEpilogue {
    static constexpr bool kRowScale = false, kColScale = false;
    __device__ float col_scale(int, int) const { return 1.0f; }
    __device__ float epi(float v, float) const { return v; }
    __device__ float epi_f32(float v, float) const { return v; }
    __device__ bool has_residual() const { return false; }
    __device__ uint4 res8(int, int, int) const { return make_uint4(0, 0, 0, 0); }
    __device__ void put8(int, int, int, uint4) const {}
};

// ------------------------------------------------------------------------------------------ UoME

// Z = u W1_b and dH = d_out W2_b^T, fp32 out: group = sample, M = l, N = k*d_e, K = d.  The weight of the first is
// A^I_i [d, d_e], of the second A^O_i [d_e, d], read as [n][k].
template <typename T, bool NK> struct UomeBwdProj : PlainEpilogue {
    typedef typename storage_elem<T>::type Elem;
    const T *left, *w;
    const int32_t *expert_idx;
    float *out;   // [b, l, k*d_e]
    int l, d, n, kact, d_e;
    static constexpr bool kF32Out = true, kPrepare = false;
    __device__ int rows(int) const { return l; }
    __device__ int ncols() const { return kact * d_e; }
    __host__ __device__ int kseg(int) const { return d; }
    __device__ int kdim(int) const { return d; }
    __device__ long b_stride() const { return d_e; }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t) const { return left + ((size_t)g * l + r) * d; }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t) const
    {
        const int s = nn / d_e, e = nn - s * d_e, i = clampi(expert_idx[g * kact + s], n);
        return w + (size_t)i * d * d_e + (NK ? (size_t)e * d : (size_t)e);
    }
    __device__ void put4(int g, int r, int nn, float4 v) const
    {
        *reinterpret_cast<float4 *>(out + ((size_t)g * l + r) * ((size_t)kact * d_e) + nn) = v;
    }
    __device__ void put4_f32(int g, int r, int nn, float4 v) const { put4(g, r, nn, v); }
};

// dH again, with the tile of Z in the accumulators beside it: H = w SiLU(Z), dZ = w dH SiLU'(Z) (operand layout [b, l, k,
// parts, d_e]) and the sums of dH SiLU(Z) for the gate gradient, one per wave's rows and 8 columns (a wave's 32 columns may
// belong to several experts, 8 never do).  Neither Z nor dH reaches memory: 8 bytes written per element instead of
// 8 written, 8 read and 8 written (uome_bwd_any_mid): 128 x 196 x 384 x 768 in bf16 34.9 + 42.9 + 56.9 -> 88 us, bound by the
// epilogue's arithmetic (exact exponential and reciprocal) and its stores; with 8-byte stores straight from the
// accumulators, 16 bytes of a row at a time, the vit layer's forward + backward gained 11 us instead of 34.
template <typename T> struct UomeBwdDhPair : UomeBwdProj<T, true> {
    static constexpr bool kPairOut = true, kColScale = true;
    const float *expert_gate;   // NULL: weight 1
    T *h, *dz;
    float *gpart;               // [b, k, gchunks], gchunks = row blocks * d_e / 8
    int gchunks;
    __device__ float col_scale(int g, int nn) const
    {
        return expert_gate ? expert_gate[(size_t)g * this->n + clampi(this->expert_idx[g * this->kact + nn / this->d_e], this->n)] : 1.0f;
    }
    template <int TM, int TN, int SPITCH>
    __device__ void pair_out(f32x16_t (&acc)[TM][TN], f32x16_t *z, uint16_t (*stage)[SPITCH], const float *colw, int g, int grow0, int gcol0, int M, int N,
                             int lane) const
    {
        constexpr int PARTS = parts_of<T>::value, WC = TN * 4;
        const int lr = lane & 31, lh = lane >> 5, d_e = this->d_e, rows = M - grow0;
        if (rows <= 0) return;
        // operand layout, first part: the tile's rows from `first` on, `step` apart, and a place in a row.  Divisions by d_e are vector work of 20
        // instructions each: one a lane, and a walk over the wave's columns (with one for each 16-byte piece, the sigmoid by a
        // division and the blocks of rows behind the sample's end worked as well, Z and dH of 128 x 196 x 384 x 768 took 98 us, vector instructions issuing
        // 74 % of it; 88 so)
        const uint32_t step = (uint32_t)this->kact * PARTS * d_e;
        const size_t first = ((size_t)g * this->l + grow0) * step;
        // in place: z becomes H, the accumulators dZ
        int s = gcol0 / d_e, c = gcol0 - s * d_e;   // the slot and its column of 8 columns of the wave's (uniform)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (gcol0 + j * 32 + q * 8 >= N) continue;
                const float w = colw[j * 4 + q];
                float part = 0.f;
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    if (i && i * 32 >= rows) break;
                    float ps = 0.f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float zv = z[i * TN + j][q * 4 + e], dv = acc[i][j][q * 4 + e];
                        const float sig = sigmoid_of(expf(-zv)), v = zv * sig;
                        ps = fmaf(dv, v, ps);
                        z[i * TN + j][q * 4 + e] = v * w;
                        acc[i][j][q * 4 + e] = dv * w * (sig * (1.0f + zv * (1.0f - sig)));
                    }
                    if (i * 32 + lr < rows) part += ps;
                }
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) part += __shfl_xor(part, off, 64);
                if (lane == 0) gpart[((size_t)g * this->kact + s) * gchunks + (size_t)(grow0 / (TM * 32)) * (d_e / 8) + c / 8] = part;
                c += 8;
                if (c >= d_e) {
                    c = 0;
                    ++s;
                }
            }
        if constexpr (PARTS == 1) {
            s = gcol0 / d_e;
            c = gcol0 - s * d_e;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        if (i * 32 + lr >= rows || gcol0 + j * 32 + q * 8 >= N) continue;
                        const size_t to = first + (size_t)(i * 32 + lr) * step + s * d_e + c + lh * 4;
                        const f32x16_t &hv = z[i * TN + j], &gv = acc[i][j];
                        *reinterpret_cast<float4 *>(h + to) = make_float4(hv[q * 4], hv[q * 4 + 1], hv[q * 4 + 2], hv[q * 4 + 3]);
                        *reinterpret_cast<float4 *>(dz + to) = make_float4(gv[q * 4], gv[q * 4 + 1], gv[q * 4 + 2], gv[q * 4 + 3]);
                    }
                    c += 8;
                    if (c >= d_e) {
                        c = 0;
                        ++s;
                    }
                }
        } else {
            const int col = gcol0 + lane % WC * 8, sl = col / d_e;
            const uint32_t place = sl * PARTS * d_e + (col - sl * d_e);
            auto plane = [&](T *dst, auto value, bool low) {
                stage_plane<TM, TN, SPITCH>(
                    stage, lane, rows,
                    [&](int i, int j, int q) {
                        const f32x16_t &v = value(i, j);
                        uint32_t o[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const float a = v[q * 4 + 2 * e], b = v[q * 4 + 2 * e + 1];
                            o[e] = pack2_bf16(a, b);
                            if (low) o[e] = pack2_bf16(a - __uint_as_float(o[e] << 16), b - __uint_as_float(o[e] & 0xFFFF0000u));
                        }
                        return make_uint2(o[0], o[1]);
                    },
                    [&](int row, int, uint4 piece) {
                        if (row < rows && col < N) store16<false>(dst + first + (size_t)row * step + place + (low ? d_e : 0), piece);
                    });
            };
            auto hv = [&](int i, int j) -> const f32x16_t & { return z[i * TN + j]; };
            auto gv = [&](int i, int j) -> const f32x16_t & { return acc[i][j]; };
            plane(h, hv, false);
            plane(h, hv, true);
            plane(dz, gv, false);
            plane(dz, gv, true);
        }
    }
};

// d_u = (d_out) + dZ W1_b^T: group = sample, M = l, N = d, K segments = (slot, part) of d_e; A^I_i [d, d_e] is [n][k]
template <typename T> struct UomeBwdDu : PlainEpilogue {
    typedef typename storage_elem<T>::type Elem;
    static constexpr int kSegParts = parts_of<T>::value;
    const T *dz, *a_in, *d_out;   // dz [b, l, k, parts, d_e]
    const int32_t *expert_idx;
    T *d_u;
    int l, d, n, kact, d_e;
    uint32_t flags;
    static constexpr bool kPrepare = false;
    __device__ int rows(int) const { return l; }
    __device__ int ncols() const { return d; }
    __host__ __device__ int kseg(int) const { return d_e; }
    __device__ int kdim(int) const { return kact * kSegParts * d_e; }
    __device__ long b_stride() const { return 0; }
    // the engine asks for segment `seg`'s context directly before its loop and for table entry e = seg / parts in it:
    // both are the expert of a slot
    __device__ uint32_t seg_ctx(int g, int s) const { return (uint32_t)clampi(expert_idx[g * kact + clampi(s, kact)], n); }
    __device__ const T *a_ptr_ctx(int g, int r, int seg, uint32_t) const
    {
        return dz + (((size_t)g * l + r) * kact * kSegParts + seg) * d_e;   // seg = slot * parts + part
    }
    __device__ const T *b_ptr_ctx(int, int, int nn, uint32_t i) const { return a_in + ((size_t)i * d + nn) * d_e; }
    __device__ bool has_residual() const { return flags & F_RESIDUAL; }
    __device__ uint4 res8(int g, int r, int nn) const { return load16<false>(d_out + ((size_t)g * l + r) * d + nn); }
    __device__ void put8(int g, int r, int nn, uint4 piece) const { store16<false>(d_u + ((size_t)g * l + r) * d + nn, piece); }
    __device__ void put4(int g, int r, int nn, float4 v) const
    {
        const size_t at = ((size_t)g * l + r) * d + nn;
        if (flags & F_RESIDUAL) v = add4_f32(v, reinterpret_cast<const float *>(d_out) + at);
        *reinterpret_cast<float4 *>(d_u + at) = v;
    }
};

// Weight gradients: dA^O_i [d_e, d] = sum H_{b,s}^T d_out_b (set 0), (dA^I_i)^T [d_e, d] = sum dZ_{b,s}^T u_b (set 1)
// over the (sample, slot) pairs of expert i, both operands token-major ([k][m] and [k][n]), in parts of the expert's list of ranges of
// tokens (uome_any_wgrad; whole pairs where there are many).  A K segment costs its lookups and
// addresses once, so long ones pay: 128 samples of 196 tokens in 8 parts of pairs instead of 32 tokens 150 -> 103 us.
template <typename T> struct UomeBwdWgrad : PlainEpilogue {
    typedef typename storage_elem<T>::type Elem;
    static constexpr int kSegParts = parts_of<T>::value;
    const T *left[2], *right[2];   // left [b, l, k, parts, d_e], right [b, l, d]
    const int32_t *expert_idx;
    float *partial;                // [2*chunks*parts, d_e, d]
    int b, l, d, n, kact, d_e, range;   // range: tokens of an item, fewer in a pair's last one
    WgradOrder<true, false> parts;
    Divider items;
    static constexpr bool kF32Out = true, kPrepare = true;
    __device__ int rows(int) const { return d_e; }
    __device__ int ncols() const { return d; }
    __host__ __device__ int kseg(int) const { return range; }
    __device__ int seg_len(uint32_t ctx) const { return min(range, l - (int)(ctx >> 12) * range); }
    // (range is a multiple of 32, or l; one short K-step in 16 and more unbalances the sums of either sign too little to matter)
    __device__ int seg_tail(int step) const { return range < l && l >= 512 ? 0 : l % step; }
    __device__ int kdim(int) const { return 0; }
    __device__ long b_stride() const { return d; }
    __device__ long a_stride(int) const { return (long)kact * kSegParts * d_e; }
    // context of a segment: slot in bits 0-4, sample of the chunk in bits 5-11, range above
    __device__ int decode(int g) const { return parts.decode(g); }
    __device__ int prepare(int &g, uint32_t *segtab, void *scratch, int tid, int) const
    {
        PartList &list = *static_cast<PartList *>(scratch);
        const int base = parts.chunk(g) * 128, nb = min(128, b - base);
        int expert, first, last;
        if (!list.fill(expert_idx + (size_t)base * kact, nb, kact, n, parts, g, tid, expert, first, last)) return -1;
        if (tid < nb && list.slot_of[tid] >= 0) {
            const int at = list.before(expert, tid) * parts.w.items - first;
            for (int r = max(0, -at); r < min(parts.w.items, last - first - at); ++r)
                segtab[at + r] = ((uint32_t)r << 12) | ((uint32_t)tid << 5) | (uint32_t)list.slot_of[tid];
        }
        __syncthreads();
        // a K-step is 32 tokens; a pair's last range is shorter
        const int steps = (range + 31) / 32, steps_last = (l - (parts.w.items - 1) * range + 31) / 32;
        return ((last - first) * steps - (items.of(last) - items.of(first)) * (steps - steps_last)) * kSegParts * 32;
    }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ size_t token(int g, uint32_t ctx) const
    {
        return (size_t)(parts.chunk(g) * 128 + (int)(ctx >> 5 & 0x7Fu)) * l + (size_t)(ctx >> 12) * range;
    }
    __device__ const T *a_ptr_ctx(int g, int m, int seg, uint32_t ctx) const
    {
        return (parts.set(g) ? left[1] : left[0]) + ((token(g, ctx) * kact + (ctx & 0x1Fu)) * kSegParts + seg % kSegParts) * d_e + m;
    }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t ctx) const { return (parts.set(g) ? right[1] : right[0]) + token(g, ctx) * d + nn; }
    __device__ void put4(int g, int r, int nn, float4 v) const
    {
        *reinterpret_cast<float4 *>(partial + (parts.tile(g) * d_e + r) * d + nn) = v;
    }
    __device__ void put4_f32(int g, int r, int nn, float4 v) const { put4(g, r, nn, v); }
};

// Where Z and dH are formed by two launches.  Elementwise middle: H = w SiLU(Z) into `h`, dZ = w dH SiLU'(Z) into `dz` (operand layout [b, l, k, parts, d_e]) and
// the slot's partial sums of dH SiLU(Z).  Block = (chunk of tokens, slot, sample); a group of `lpr` lanes of one
// wave takes a (token, slot) row of d_e values in blocks of 4*8*lpr columns: a row of at most one block (d_e <= 2048)
// is read by its lanes before they write it, so it may be written in place (h == z, dz == dh: an fp32 value and a
// (hi, lo) pair take the same four bytes).  Bound by its traffic, 16 bytes per element.
template <typename T> __global__ __launch_bounds__(256) void uome_bwd_any_mid(UomeBwdArgs a, T *h, T *dz, int lpr, int per_chunk)
{
    constexpr int PARTS = parts_of<T>::value;
    __shared__ float red[256];
    const int chunk = blockIdx.x, s = blockIdx.y, bb = blockIdx.z, tid = threadIdx.x;
    const int i = clampi(a.expert_idx[bb * a.k + s], a.n);
    const float w = ((a.flags & F_GATE_EXPERT) && a.expert_gate) ? a.expert_gate[(size_t)bb * a.n + i] : 1.0f;
    const int rpb = 256 / lpr, sub = tid % lpr;
    const float *z = static_cast<const float *>(a.z), *dh = static_cast<const float *>(a.dh);
    const int t_end = min(a.l, (chunk + 1) * per_chunk);
    float part = 0.f;
    for (int t = chunk * per_chunk + tid / lpr; t < t_end; t += rpb) {
        const size_t row = (((size_t)bb * a.l + t) * a.k + s) * a.d_e;
        for (int c0 = 0; c0 < a.d_e; c0 += 32 * lpr) {
            float4 zv[8], dv[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int col = c0 + (q * lpr + sub) * 4;
                if (col < a.d_e) {
                    zv[q] = *reinterpret_cast<const float4 *>(z + row + col);
                    dv[q] = *reinterpret_cast<const float4 *>(dh + row + col);
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // every lane of the row holds its values before any is overwritten
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int col = c0 + (q * lpr + sub) * 4;
                if (col >= a.d_e) continue;
                const float zq[4] = {zv[q].x, zv[q].y, zv[q].z, zv[q].w}, dq[4] = {dv[q].x, dv[q].y, dv[q].z, dv[q].w};
                float hq[4], gq[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float sig = 1.0f / (1.0f + expf(-zq[e])), v = zq[e] * sig;
                    part = fmaf(dq[e], v, part);
                    hq[e] = v * w;
                    gq[e] = dq[e] * w * (sig * (1.0f + zq[e] * (1.0f - sig)));
                }
                put4_operand(h + row * PARTS + col, a.d_e, make_float4(hq[0], hq[1], hq[2], hq[3]));
                put4_operand(dz + row * PARTS + col, a.d_e, make_float4(gq[0], gq[1], gq[2], gq[3]));
            }
        }
    }
    if (!a.d_gate) return;
    red[tid] = part;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) red[tid] += red[tid + st];
        __syncthreads();
    }
    if (tid == 0) a.gpart[((size_t)bb * a.k + s) * a.gchunks + chunk] = red[0];
}

template <typename T> hipError_t uome_backward_any(const UomeBwdArgs &a, hipStream_t st, BwdTail *tail)
{
    if (a.wgrad.parts > WGRAD_MAX_PARTS) return hipErrorInvalidValue;
    const int W = a.k * a.d_e;
    hipError_t err;
    const T *u = static_cast<const T *>(a.u), *a_in = static_cast<const T *>(a.a_in), *a_out = static_cast<const T *>(a.a_out);
    const T *d_out = static_cast<const T *>(a.d_out);
    UomeBwdProj<T, false> zp;
    zp.left = u; zp.w = a_in; zp.expert_idx = a.expert_idx; zp.out = static_cast<float *>(a.z);
    zp.l = a.l; zp.d = a.d; zp.n = a.n; zp.kact = a.k; zp.d_e = a.d_e;
    UomeBwdDhPair<T> hp;
    hp.left = d_out; hp.w = a_out; hp.expert_idx = a.expert_idx; hp.out = static_cast<float *>(a.dh);
    hp.l = a.l; hp.d = a.d; hp.n = a.n; hp.kact = a.k; hp.d_e = a.d_e;

    T *h = static_cast<T *>(a.h_op), *dz = static_cast<T *>(a.dz_op);
    UomeBwdArgs ga = a;   // for the gate gradient
    constexpr bool F32 = std::is_same<T, float>::value;
    const bool large = a.l > 64 && (long)a.b * ((a.l + 127) / 128) * ((W + 127) / 128) >= 256;
    // one launch for Z, dH and what becomes of them, where tiles of 64 rows and more are the choice anyway and the gate
    // gradient's sums fit the room they have (a wave's rows: 64 of the large tiles, 32 of the small ones)
    const long row_blocks = large ? (a.l + 63) / 64 : (a.l + 31) / 32;
    const long sums = row_blocks * (a.d_e / 8), room = (long)2 * a.wgrad.chunks * a.wgrad.parts * a.d * a.d_e / ((long)a.b * a.k);
    if (a.l > 32 && sums <= room) {
        hp.expert_gate = (a.flags & F_GATE_EXPERT) ? a.expert_gate : nullptr;
        hp.h = h; hp.dz = dz; hp.gpart = a.gpart; hp.gchunks = ga.gchunks = (int)sums;
        const auto both = [&](auto tail) {
            constexpr int FZ = decltype(tail)::value, FH = FZ | GEMM_B_NK;
            if constexpr (F32) {
                // (few tiles, on the fp32 instruction as in tail_tile: 8 x 77 x 200 x 272 47.3 -> 44.8 us for the pass)
                const bool few = (long)a.b * ((a.l + 63) / 64) * ((W + 63) / 64) <= 256;
                return large ? launch_gemm_dma_dual<FZ, FH, 128, 128, 32, 2, 4, 2, 2>(zp, hp, a.b, a.l, W, st)
                      : few ? launch_gemm_dma_dual<FZ | GEMM_EXACT, FH | GEMM_EXACT, 64, 64, 32, 2, 2, 3, 2>(zp, hp, a.b, a.l, W, st)
                            : launch_gemm_dma_dual<FZ, FH, 64, 64, 32, 2, 2, 3, 2>(zp, hp, a.b, a.l, W, st);
            }
            else
                return large ? launch_gemm_dma_dual<FZ, FH, 128, 128, 32, 2, 4, 3, 4>(zp, hp, a.b, a.l, W, st)
                            : launch_gemm_dma_dual<FZ, FH, 64, 128, 32, 2, 2, 4, 2>(zp, hp, a.b, a.l, W, st);
        };
        err = a.d % 32 ? both(std::integral_constant<int, GEMM_TAIL>{}) : both(std::integral_constant<int, 0>{});   // (as launch_gemm_tail)
        if (err != hipSuccess) return err;
    } else {
        if ((err = launch_gemm_tail<0>(zp, a.b, a.l, W, st)) != hipSuccess) return err;
        if ((err = launch_gemm_tail<GEMM_B_NK>(static_cast<const UomeBwdProj<T, true> &>(hp), a.b, a.l, W, st)) != hipSuccess) return err;
        int lpr = 2;
        while (lpr < 64 && lpr * 4 < a.d_e) lpr *= 2;
        const int per_chunk = (a.l + a.gchunks - 1) / a.gchunks;
        hipLaunchKernelGGL((uome_bwd_any_mid<T>), dim3(a.gchunks, a.k, a.b), dim3(256), 0, st, a, h, dz, lpr, per_chunk);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    UomeBwdDu<T> up;
    up.dz = dz; up.a_in = a_in; up.d_out = d_out; up.expert_idx = a.expert_idx; up.d_u = static_cast<T *>(a.d_u);
    up.l = a.l; up.d = a.d; up.n = a.n; up.kact = a.k; up.d_e = a.d_e; up.flags = a.flags;
    Beside<UomeGates> gates{{ga}, a.d_gate ? a.b * a.k : 0};   // (before the weight gradients, whose partial tiles take the place of its sums)
    if ((err = launch_gemm_tail<GEMM_B_NK>(up, a.b, a.l, a.d, st, &gates)) != hipSuccess) return err;

    UomeBwdWgrad<T> wp;
    wp.left[0] = h; wp.right[0] = d_out;
    wp.left[1] = dz; wp.right[1] = u;
    wp.expert_idx = a.expert_idx; wp.partial = a.partial;
    wp.b = a.b; wp.l = a.l; wp.d = a.d; wp.n = a.n; wp.kact = a.k; wp.d_e = a.d_e; wp.parts = {2, BY_SAMPLE, a.wgrad, a.part_end};
    wp.range = uome_any_range(a.l, a.wgrad.items); wp.items = Divider(a.wgrad.items);
    if ((err = launch_gemm_tail<GEMM_A_KM>(wp, wp.parts.groups(), a.d_e, a.d, st)) != hipSuccess) return err;
    WgradReduceArgs ra{};
    ra.partial = a.partial; ra.n = a.n; ra.M = a.d_e; ra.N = a.d;
    ra.w = a.wgrad; ra.part_end = a.part_end;
    ra.dst[0] = a.d_a_out; ra.transposed[0] = 0;
    ra.dst[1] = a.d_a_in; ra.transposed[1] = 1;
    return launch_wgrad_reduce<T>(ra, 2, st, tail);
}

// ------------------------------------------------------------------------------------------ SMHA
// Workspace: q, k, v and do_raw fp32 [units, l_a, d_h]; og = w o, operand layout [units, l_a, parts, d_h]; dqkv, operand
// layout [units, l_a, parts, 3*d_h] as [dq | dk | dv]; f.lse, inv_sum, dd, rt fp32 [units, l_a].

// weight of row r of unit g in the block's output (Eq. 36 with the gate flags)
__device__ __forceinline__ float row_weight(const SmhaBwdArgs &a, int g, int r, int l_p)
{
    const SmhaArgs &f = a.f;
    const int bb = g / f.k, i = clampi(f.expert_idx[g], f.n);
    float w = 1.0f;
    if (a.flags & F_GATE_EXPERT) w *= a.expert_gate[(size_t)bb * f.n + i];
    if (a.flags & F_GATE_PATCH) {
        const int p = clampi(f.patch_idx[((size_t)bb * f.n + i) * f.c + r / l_p], f.m);
        w *= a.patch_gate[((size_t)bb * f.n + i) * f.m + p];
    }
    return w;
}

// a product that is rounded by itself (not fused into a later subtraction): w dP enters D and dS as the same number
__device__ __forceinline__ float mul_rounded(float a, float b)
{
#pragma clang fp contract(off)
    return a * b;
}

__device__ __forceinline__ bool any_key_ok(const SmhaArgs &f, int g, int key, int l_p)
{
    if (!f.pad_mask) return true;
    const int bb = g / f.k, i = clampi(f.expert_idx[g], f.n);
    const int p = clampi(f.patch_idx[((size_t)bb * f.n + i) * f.c + key / l_p], f.m);
    return f.pad_mask[(size_t)bb * f.l + p * l_p + key % l_p] != 0;   // Eq. 41: padded keys are out of every softmax
}

// Attention backward in fp32.  One wave owns 32 rows of one unit and walks the unit's other axis in tiles of 32:
// KV = false owns queries (softmax statistics and o, then D, then dQ: three walks over the keys), KV = true owns
// keys (dK, dV: one walk over the queries).  Everything is transposed as in the forward kernels, so that a lane
// holds one own row; an accumulator register of a [streamed x own] tile is by itself the second operand of the
// next product (attention_f32_kernel).  q enters scaled by log2(e)/sqrt(d_h), dO as w * dO_raw with the row's
// weight applied to the products; P and dP are formed the same way in both kernels and by both walks that use
// them, so that the rows of dS cancel as in exact arithmetic (a row that attends to one key has dS = 0).  P is formed from the
// row's maximum and the reciprocal of its sum: a log-sum-exp of 10 is held to 2^-21, which every P of the row would be off
// by (weight gradients 2 to 3 percent further from fp64 over 18 drawn fp32 shapes).
// KS waves share an own block and take streamed tiles KS apart; sums are merged through LDS in wave order: with one
// wave per block the lm shape in fp32 has 128 of them for 1024 SIMDs.
// ONE: one tile a wave (units of up to 32 KS rows).  The query-owning kernel stages it once (the merges take the place of TB, which
// only the first walk reads) and keeps its scores and dP in registers: four products instead of seven, the same bits.  No tile is
// in flight during the products: 302 / 423 registers -> 156 to 158 at d_h 64, where LDS lets two waves on a SIMD (36 KiB for two waves, 72
// for four) and the general form's registers one (at 128 no scratch, 156 / 884 bytes before); 384 units of 56 rows, d_h 64: 44.4 -> 27.3
// us owning queries, 27.1 -> 22.0 owning keys.  vit shape forward + backward 712 -> 698 us.
template <typename T, int DH, int NQ, int KS, bool KV, bool ONE>
__global__ __launch_bounds__(NQ *KS * 64, (ONE && DH <= 64) || DH == 32 ? 2 : 1) void attention_bwd_f32_kernel(SmhaBwdArgs a, UnitGrid grid)
{
    constexpr int BT = 32, P = DH + 4, NTH = NQ * 64, NP = BT * DH / 4 / NTH;   // NP: 16-byte pieces per staging thread
    constexpr int TILE = BT * P, SPLIT = 2 * TILE + 4 * BT, SLOT = (KV ? DH : DH / 2) + 2, MERGE = (KS - 1) * NQ * 64 * SLOT;
    __shared__ __align__(16) float lds[KS * SPLIT > MERGE ? KS * SPLIT : MERGE];
    constexpr bool KEEP = ONE && !KV;
    static_assert(!KEEP || (KS * TILE >= MERGE && TILE >= NQ * 64), "merges in the place of TB");
    float *const merged = KEEP ? lds + KS * TILE : lds;
    constexpr int PARTS = parts_of<T>::value;
    const SmhaArgs &f = a.f;
    if constexpr (KV) {   // the block's gate gradients, behind the units' workgroups (r_t: of the query-owning kernel)
        static_assert(UnitGates::LDS <= sizeof(lds), "the gate gradients' LDS");
        if (blockIdx.x >= grid.own()) {
            unit_gate_block<NQ * KS * 64>(a, (int)(blockIdx.x - grid.own()), lds);
            return;
        }
    }
    const int l_p = f.l / f.m, l_a = f.c * l_p, d_h = f.d_h, g = grid.unit(blockIdx.x), block = grid.block(blockIdx.x);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int split = wave / NQ, qg = wave - split * NQ, stid = tid - split * NTH;
    const int lr = lane & 31, lh = lane >> 5;
    const int own = block * (32 * NQ) + qg * 32 + lr, own_c = min(own, l_a - 1);
    // [TA of every split][TB][R0 to R3]
    float *TA = lds + split * TILE, *TB = TA + KS * TILE, *R0 = lds + 2 * KS * TILE + split * 4 * BT, *R1 = R0 + BT, *R2 = R1 + BT, *R3 = R2 + BT;
    const size_t ubase = (size_t)g * l_a * d_h;
    const float *Q = static_cast<const float *>(f.q) + ubase, *K = static_cast<const float *>(f.kk) + ubase;
    const float *V = static_cast<const float *>(f.v) + ubase, *DO = a.do_raw + ubase;
    const float *own_a = KV ? K : Q, *own_b = KV ? V : DO, *str_a = KV ? Q : K, *str_b = KV ? DO : V;
    const float qscale = 1.4426950408889634f * rsqrtf((float)d_h);
    const bool causal = (f.flags & F_CAUSAL) != 0;

    float fa[DH / 8][4], fb[DH / 8][4];   // own rows as second operands: k of sub-step ks is ks*8 + lh*4 + e
#pragma unroll
    for (int ks = 0; ks < DH / 8; ++ks) {
        const int dh = ks * 8 + lh * 4;
        float4 va = make_float4(0, 0, 0, 0), vb = va;
        if (dh < d_h) {
            va = *reinterpret_cast<const float4 *>(own_a + (size_t)own_c * d_h + dh);
            vb = *reinterpret_cast<const float4 *>(own_b + (size_t)own_c * d_h + dh);
        }
        fa[ks][0] = va.x; fa[ks][1] = va.y; fa[ks][2] = va.z; fa[ks][3] = va.w;
        fb[ks][0] = vb.x; fb[ks][1] = vb.y; fb[ks][2] = vb.z; fb[ks][3] = vb.w;
        if (!KV)
#pragma unroll
            for (int e = 0; e < 4; ++e) fa[ks][e] *= qscale;
    }
    const float w_own = KV ? 1.0f : row_weight(a, g, own_c, l_p);
    const bool own_ok = own < l_a && (!KV || any_key_ok(f, g, own_c, l_p));

    // streamed tiles: under the causal mask a query sees keys <= itself
    const int blk0 = block * 32 * NQ, blk1 = min(l_a, blk0 + 32 * NQ);
    int t_begin = 0, t_end = (l_a + BT - 1) / BT;
    if (causal) {
        if (KV) t_begin = blk0 / BT;
        else t_end = (blk1 + BT - 1) / BT;
    }
    const int nit = ONE ? 1 : (t_end - t_begin + KS - 1) / KS;   // uniform over the workgroup
    auto tile_of = [&](int it) { return t_begin + it * KS + split; };

    float4 ra[NP], rb[NP];
    float r0 = 0.f, r1 = 0.f, r2 = 0.f, r3 = 0.f;
    auto load_global = [&](int kt) {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int c = stid + q * NTH, row = kt * BT + c / (DH / 4), col = (c % (DH / 4)) * 4;
            ra[q] = rb[q] = make_float4(0, 0, 0, 0);
            if (row < l_a && col < d_h) {
                ra[q] = *reinterpret_cast<const float4 *>(str_a + (size_t)row * d_h + col);
                rb[q] = *reinterpret_cast<const float4 *>(str_b + (size_t)row * d_h + col);
            }
        }
        if (stid < BT) {
            const int row = kt * BT + stid;
            if (KV) {   // streamed queries: softmax maximum, D, weight, softmax 1 / sum
                r0 = row < l_a ? a.f.lse[(size_t)g * l_a + row] : 0.f;
                r3 = row < l_a ? a.inv_sum[(size_t)g * l_a + row] : 0.f;
                r1 = row < l_a ? a.dd[(size_t)g * l_a + row] : 0.f;
                r2 = row < l_a ? row_weight(a, g, row, l_p) : 0.f;
            } else r0 = row < l_a && any_key_ok(f, g, row, l_p) ? 1.f : 0.f;   // streamed keys: admissible
        }
    };
    auto store_lds = [&]() {
        const float s = KV ? qscale : 1.0f;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int c = stid + q * NTH, row = c / (DH / 4), col = (c % (DH / 4)) * 4;
            *reinterpret_cast<float4 *>(TA + row * P + col) =
                KV ? make_float4(ra[q].x * s, ra[q].y * s, ra[q].z * s, ra[q].w * s) : ra[q];
            *reinterpret_cast<float4 *>(TB + row * P + col) = rb[q];
        }
        if (stid < BT) {
            R0[stid] = r0;
            if (KV) {
                R1[stid] = r1;
                R2[stid] = r2;
                R3[stid] = r3;
            }
        }
    };
    // [streamed x own] product of a tile with own rows
    auto product = [&](const float *tile, const float (&fr)[DH / 8][4]) {
        f32x16_t acc;
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] = 0.f;
#pragma unroll
        for (int ks = 0; ks < DH / 8; ++ks) {
            const float4 t = *reinterpret_cast<const float4 *>(tile + lr * P + ks * 8 + lh * 4);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(t.x, fr[ks][0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(t.y, fr[ks][1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(t.z, fr[ks][2], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(t.w, fr[ks][3], acc, 0, 0, 0);
        }
        return acc;
    };
    // out^T [d_h x own] += tile^T x (streamed x own)
    auto accumulate = [&](f32x16_t (&out)[DH / 32], const float *tile, const f32x16_t &x) {
#pragma unroll
        for (int q = 0; q < 16; ++q)
#pragma unroll
            for (int td = 0; td < DH / 32; ++td) {
                const float t = tile[((q >> 2) * 8 + lh * 4 + (q & 3)) * P + td * 32 + lr];
                out[td] = __builtin_amdgcn_mfma_f32_32x32x2f32(t, x[q], out[td], 0, 0, 0);
            }
    };
    auto admissible = [&](int kt, int q, const float *okv) {   // accumulator register q of tile kt
        const int row = kt * BT + (q >> 2) * 8 + lh * 4 + (q & 3);
        const int query = KV ? row : own, key = KV ? own : row;
        return own_ok && row < l_a && (!causal || key <= query) && (KV || okv[(q >> 2) * 8 + lh * 4 + (q & 3)] != 0.f);
    };
    // adds every split's array into split 0's, in split order; ALL: the sums go back to every split
    auto merge = [&](auto &v, auto all_splits) {
        if constexpr (KS > 1) {
            constexpr int COUNT = sizeof(v) / sizeof(float);
            constexpr size_t STEP = (size_t)NQ * 64 * SLOT;
            float *slot = merged + ((size_t)qg * 64 + lane) * SLOT;
            __syncthreads();
            if (split > 0) {
#pragma unroll
                for (int q = 0; q < COUNT; ++q) slot[(split - 1) * STEP + q] = v[q];
            }
            __syncthreads();
            if (split == 0) {
#pragma unroll
                for (int s = 1; s < KS; ++s)
#pragma unroll
                    for (int q = 0; q < COUNT; ++q) v[q] += slot[(s - 1) * STEP + q];
            }
            if constexpr (decltype(all_splits)::value) {
                __syncthreads();
                if (split == 0) {
#pragma unroll
                    for (int q = 0; q < COUNT; ++q) slot[q] = v[q];
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < COUNT; ++q) v[q] = slot[q];
            }
        }
    };

    f32x16_t acc_a[DH / 32], acc_b[KV ? DH / 32 : 1];
#pragma unroll
    for (int t = 0; t < DH / 32; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            acc_a[t][q] = 0.f;
            if (KV) acc_b[t][q] = 0.f;
        }
    float max_own = 0.f, inv_own = 0.f, d_own = 0.f;
    f32x16_t s1, dp1;

    if constexpr (!KV) {
        // walk 1: softmax statistics and o
        float mrun = -INFINITY, lsum = 0.f;
        if (tile_of(0) < t_end) load_global(tile_of(0));
        for (int it = 0; it < nit; ++it) {
            const int kt = tile_of(it);
            __syncthreads();
            if (kt < t_end) store_lds();
            __syncthreads();
            if (!ONE && kt + KS < t_end) load_global(kt + KS);
            if (kt >= t_end) continue;
            f32x16_t s = product(TA, fa);
            if constexpr (KEEP) {
                s1 = s;
                dp1 = product(TB, fb);
            }
            float tmax = -INFINITY;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                s[q] = admissible(kt, q, R0) ? s[q] : -INFINITY;
                tmax = fmaxf(tmax, s[q]);
            }
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
            const float mnew = fmaxf(mrun, tmax), msub = mnew == -INFINITY ? 0.f : mnew;
            const float corr = __builtin_amdgcn_exp2f(mrun - msub);
            mrun = mnew;
            float psum = 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                s[q] = __builtin_amdgcn_exp2f(s[q] - msub);
                psum += s[q];
            }
            lsum = fmaf(lsum, corr, psum);
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc_a[td][q] *= corr;
            accumulate(acc_a, TB, s);
        }
        lsum += __shfl_xor(lsum, 32, 64);
        if constexpr (KS > 1) {   // merge (max, sum, o): rescale to the common maximum, then add
            float mall = mrun;
            __syncthreads();
            merged[((size_t)split * NQ + qg) * 64 + lane] = mrun;
            __syncthreads();
#pragma unroll
            for (int s = 0; s < KS; ++s) mall = fmaxf(mall, merged[((size_t)s * NQ + qg) * 64 + lane]);
            const float c = mrun == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrun - mall);
            lsum *= c;
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc_a[td][q] *= c;
            mrun = mall;
            float v[1] = {lsum};
            merge(v, std::true_type{});
            lsum = v[0];
            float o[DH / 2];
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) o[td * 16 + q] = acc_a[td][q];
            merge(o, std::false_type{});
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc_a[td][q] = o[td * 16 + q];
        }
        max_own = lsum > 0.f ? mrun : 0.f;
        inv_own = lsum > 0.f ? 1.0f / lsum : 0.f;
        if (split == 0) {
            const float inv = inv_own;
            const size_t row = (size_t)g * l_a + own_c;
            float dot = 0.f;
#pragma unroll
            for (int td = 0; td < DH / 32; ++td)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const int dh = td * 32 + q4 * 8 + lh * 4;
                    if (dh >= d_h) continue;
                    const float4 dr = *reinterpret_cast<const float4 *>(DO + (size_t)own_c * d_h + dh);
                    const float4 o = make_float4(acc_a[td][q4 * 4] * inv, acc_a[td][q4 * 4 + 1] * inv, acc_a[td][q4 * 4 + 2] * inv,
                                                 acc_a[td][q4 * 4 + 3] * inv);
                    dot = fmaf(dr.x, o.x, dot);
                    dot = fmaf(dr.y, o.y, dot);
                    dot = fmaf(dr.z, o.z, dot);
                    dot = fmaf(dr.w, o.w, dot);
                    if (own < l_a)
                        put4_operand(static_cast<T *>(a.og) + row * PARTS * d_h + dh, d_h,
                                     make_float4(o.x * w_own, o.y * w_own, o.z * w_own, o.w * w_own));
                }
            dot += __shfl_xor(dot, 32, 64);
            if (own < l_a && lh == 0) {
                a.rt[row] = dot;
                a.f.lse[row] = max_own;
                a.inv_sum[row] = inv_own;
            }
        }
        // walk 2: D = sum_j P_j dP_j
        auto add_to_d = [&](int kt, const f32x16_t &s, const f32x16_t &dp) {
#pragma unroll
            for (int q = 0; q < 16; ++q)
                d_own = fmaf(admissible(kt, q, R0) ? __builtin_amdgcn_exp2f(s[q] - max_own) * inv_own : 0.f, mul_rounded(dp[q], w_own), d_own);
        };
        if constexpr (KEEP) {
            if (tile_of(0) < t_end) add_to_d(tile_of(0), s1, dp1);
        } else {
            if (tile_of(0) < t_end) load_global(tile_of(0));
            for (int it = 0; it < nit; ++it) {
                const int kt = tile_of(it);
                __syncthreads();
                if (kt < t_end) store_lds();
                __syncthreads();
                if (kt + KS < t_end) load_global(kt + KS);
                if (kt >= t_end) continue;
                add_to_d(kt, product(TA, fa), product(TB, fb));
            }
        }
        d_own += __shfl_xor(d_own, 32, 64);
        float v[1] = {d_own};
        merge(v, std::true_type{});
        d_own = v[0];
        if (split == 0 && own < l_a && lh == 0) a.dd[(size_t)g * l_a + own] = d_own;
#pragma unroll
        for (int t = 0; t < DH / 32; ++t)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc_a[t][q] = 0.f;
    }

    // last walk: dQ, or dK and dV
    if (!KEEP && tile_of(0) < t_end) load_global(tile_of(0));
    for (int it = 0; it < nit; ++it) {
        const int kt = tile_of(it);
        if constexpr (!KEEP) {
            __syncthreads();
            if (kt < t_end) store_lds();
            __syncthreads();
            if (!ONE && kt + KS < t_end) load_global(kt + KS);
        }
        if (kt >= t_end) continue;
        f32x16_t s, dp;
        if constexpr (KEEP) {
            s = s1;
            dp = dp1;
        } else {
            s = product(TA, fa);
            dp = product(TB, fb);
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int at = (q >> 2) * 8 + lh * 4 + (q & 3);
            const float mx = KV ? R0[at] : max_own, inv = KV ? R3[at] : inv_own, dd = KV ? R1[at] : d_own, w = KV ? R2[at] : w_own;
            const float p = admissible(kt, q, R0) ? __builtin_amdgcn_exp2f(s[q] - mx) * inv : 0.f;
            dp[q] = p * (mul_rounded(dp[q], w) - dd);
            s[q] = p * w;   // dV contracts P with dO = w dO_raw
        }
        accumulate(acc_a, TA, dp);
        if constexpr (KV) accumulate(acc_b, TB, s);
    }
    constexpr int COUNT = KV ? DH : DH / 2;
    float out[COUNT];
#pragma unroll
    for (int td = 0; td < DH / 32; ++td)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            out[td * 16 + q] = acc_a[td][q];
            if constexpr (KV) out[DH / 2 + td * 16 + q] = acc_b[td][q];
        }
    merge(out, std::false_type{});
    if (split > 0 || own >= l_a) return;
    // q' = q log2(e)/sqrt(d_h): dK = dS^T q / sqrt(d_h) = ln(2) dS^T q'
    const float scale = KV ? 0.6931471805599453f : rsqrtf((float)d_h);
    T *row_out = static_cast<T *>(a.dqkv) + ((size_t)g * l_a + own) * PARTS * 3 * d_h;
    const int rope_first = d_h - f.rope_dim;
    auto put = [&](const float *v, int block, float sc) {
#pragma unroll
        for (int td = 0; td < DH / 32; ++td)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int dh0 = td * 32 + q4 * 8 + lh * 4;
                if (dh0 >= d_h) continue;
                float x[4] = {v[td * 16 + q4 * 4] * sc, v[td * 16 + q4 * 4 + 1] * sc, v[td * 16 + q4 * 4 + 2] * sc, v[td * 16 + q4 * 4 + 3] * sc};
                if (block < 2 && f.rope_dim > 0) {   // the transposed rotation of Eq. 32
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh) {
                        const int dh = dh0 + 2 * hh;
                        if (dh >= rope_first) {
                            const float theta = exp2f(-((float)(dh - rope_first) / (float)f.rope_dim) * 13.287712379549449f);
                            float sn, cs;
                            sincosf((float)own * theta, &sn, &cs);
                            const float ga = x[2 * hh], gb = x[2 * hh + 1];
                            x[2 * hh] = ga * cs + gb * sn;
                            x[2 * hh + 1] = gb * cs - ga * sn;
                        }
                    }
                }
                put4_operand(row_out + block * d_h + dh0, 3 * d_h, make_float4(x[0], x[1], x[2], x[3]));
            }
    };
    if (KV) {
        put(out, 1, scale);
        put(out + (KV ? DH / 2 : 0), 2, 1.0f);
    } else put(out, 0, scale);
}

template <typename T, int DH> void launch_attention_bwd_f32_dh(const SmhaBwdArgs &a, hipStream_t st)
{
    const int l_a = a.f.c * (a.f.l / a.f.m), units = a.f.b * a.f.k;
    const long blocks = (long)((l_a + 31) / 32) * units;
    // up to 128 rows a wave for every streamed tile, however many blocks there are (owning queries / keys, us; a wave per block
    // with all tiles -> this): 768 units of 56 rows 82 / 48 -> 50 / 44, 384 of 112 136 / 76 -> 80 / 64, 768 of 126 and d_h 40 202 / 108
    // -> 125 / 106, 768 of 56 and d_h 128 169 / 157 -> 102 / 84; 192 of 112, two waves -> four, 81 / 41 -> 51 / 41.  From 65 rows on some
    // of four waves have no tile, and under the causal mask more: the whole backward pass in bf16, d_h 40, 384 units of 65 rows, one wave a
    // block 207, two 214, four 154; causal 169, 182, 155; 768 units, causal 229, 271, 222; in fp32, d_h 120, causal 615, 701, 604.  Longer units:
    // splits while the launch has fewer waves than SIMDs.
    const int ks = l_a <= 32 ? 1 : l_a <= 64 ? 2 : l_a <= 128 || blocks < 512 ? 4 : blocks < 1024 ? 2 : 1;
    const UnitGrid grid{(l_a + 31) / 32, units, 0}, grid_kv{grid.rows, units, UnitGates::count(a)};
#define UOE_ABW(KS, ONE)                                                                                            \
    hipLaunchKernelGGL((attention_bwd_f32_kernel<T, DH, 1, KS, false, ONE>), dim3(grid.workgroups()), dim3(KS * 64), 0, st, a, grid);     \
    hipLaunchKernelGGL((attention_bwd_f32_kernel<T, DH, 1, KS, true, ONE>), dim3(grid_kv.workgroups()), dim3(KS * 64), 0, st, a, grid_kv)
    const bool one = l_a <= 32 * ks;   // a tile a wave
    if (ks == 1 && one) { UOE_ABW(1, true); }
    else if (ks == 1) { UOE_ABW(1, false); }
    else if (ks == 2 && one) { UOE_ABW(2, true); }
    else if (ks == 2) { UOE_ABW(2, false); }
    else if (one) { UOE_ABW(4, true); }
    else { UOE_ABW(4, false); }
#undef UOE_ABW
}

// Weight gradients of the SMHA block: sets 0-2 (dW^{q,k,v}_i)^T [d_h, d] = sum d{Q,K,V}^T x[T], set 3 dW^O_i [d_h, d] =
// sum (w o)^T G[T], both operands token-major, right rows gathered patch by patch.  K segments = (unit, pick) of
// l_p tokens x parts, in order, cut as WgradPlan says.
template <typename T> struct SmhaBwdWgrad : PlainEpilogue {
    typedef typename storage_elem<T>::type Elem;
    static constexpr int kSegParts = parts_of<T>::value;
    const T *dqkv, *og, *x, *d_out;   // dqkv [units, l_a, parts, 3*d_h], og [units, l_a, parts, d_h]
    const int32_t *expert_idx, *patch_idx;
    float *partial;                   // [4*chunks*parts, d_h, d]
    int b, l, d, n, kact, m, c, l_p, l_a, d_h;
    WgradOrder<true, true> parts;
    static constexpr bool kF32Out = true, kPrepare = true;
    static constexpr int kMaxSegments = BWD_ANY_SEGMENTS;
    __device__ int rows(int) const { return d_h; }
    __device__ int ncols() const { return d; }
    __host__ __device__ int kseg(int) const { return l_p; }
    __device__ int kdim(int) const { return 0; }
    __device__ long b_stride() const { return d; }
    __device__ int width(int g) const { return parts.set(g) < 3 ? 3 * d_h : d_h; }
    __device__ long a_stride(int g) const { return (long)kSegParts * width(g); }
    // context of a segment: sample of the chunk in bits 0-6, slot in bits 7-11, pick in bits 12-21, patch in bits 22-31
    __device__ int decode(int g) const { return parts.decode(g); }
    __device__ int prepare(int &g, uint32_t *segtab, void *scratch, int tid, int nthreads) const
    {
        PartList &list = *static_cast<PartList *>(scratch);
        const int base = parts.chunk(g) * 128, nb = min(128, b - base);
        int expert, first, last;
        if (!list.fill(expert_idx + (size_t)base * kact, nb, kact, n, parts, g, tid, expert, first, last)) return -1;
        for (int idx = tid; idx < nb * c; idx += nthreads) {
            const int bb = idx / c, t = idx - bb * c;
            if (list.slot_of[bb] < 0) continue;
            const int pos = list.before(expert, bb) * c + t;
            if (pos < first || pos >= last) continue;
            const int p = clampi(patch_idx[((size_t)(base + bb) * n + expert) * c + t], m);
            segtab[pos - first] = (uint32_t)bb | ((uint32_t)list.slot_of[bb] << 7) | ((uint32_t)t << 12) | ((uint32_t)p << 22);
        }
        __syncthreads();
        return (last - first) * kSegParts * l_p;
    }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ size_t sample(int g, uint32_t ctx) const { return (size_t)(parts.chunk(g) * 128) + (ctx & 0x7Fu); }
    __device__ const T *a_ptr_ctx(int g, int mm, int seg, uint32_t ctx) const
    {
        const size_t row = (sample(g, ctx) * kact + ((ctx >> 7) & 0x1Fu)) * l_a + (size_t)((ctx >> 12) & 0x3FFu) * l_p;
        const int st = parts.set(g);
        return (st < 3 ? dqkv + st * d_h : og) + (row * kSegParts + seg % kSegParts) * width(g) + mm;
    }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t ctx) const
    {
        return (parts.set(g) < 3 ? x : d_out) + (sample(g, ctx) * l + (size_t)(ctx >> 22) * l_p) * d + nn;
    }
    __device__ void put4(int g, int r, int nn, float4 v) const
    {
        *reinterpret_cast<float4 *>(partial + (parts.tile(g) * d_h + r) * d + nn) = v;
    }
    __device__ void put4_f32(int g, int r, int nn, float4 v) const { put4(g, r, nn, v); }
};

template <typename T> hipError_t smha_backward_any(const SmhaBwdArgs &a, hipStream_t st, BwdTail *tail)
{
    if (a.wgrad.parts > WGRAD_MAX_PARTS) return hipErrorInvalidValue;
    const SmhaArgs &f = a.f;
    const int l_p = f.l / f.m, l_a = f.c * l_p, units = f.b * f.k, dh = f.d_h;
    hipError_t err;
    // q, k, v in fp32
    QkvProblem<T, parts_of<T>::value == 2> qp;
    qp.x = static_cast<const T *>(f.x);
    qp.wq = static_cast<const T *>(f.wq); qp.wk = static_cast<const T *>(f.wk); qp.wv = static_cast<const T *>(f.wv);
    qp.expert_idx = f.expert_idx; qp.patch_idx = f.patch_idx;
    qp.q = static_cast<T *>(f.q); qp.k = static_cast<T *>(f.kk); qp.v = static_cast<T *>(f.v);
    qp.q32 = static_cast<float *>(f.q); qp.q32_plane = static_cast<float *>(f.kk) - static_cast<float *>(f.q);
    qp.l = f.l; qp.d = f.d; qp.n = f.n; qp.kact = f.k; qp.m = f.m; qp.c = f.c;
    qp.l_p = l_p; qp.l_a = l_a; qp.d_h = dh; qp.q_scale = 1.0f; qp.nout = 3;
    if (!a.kept) {
        if ((err = launch_gemm_tail<0>(qp, units, l_a, 3 * dh, st)) != hipSuccess) return err;
        if ((err = launch_rope_f32(f, st)) != hipSuccess) return err;
    }
    // dO_raw = G[T] W^O^T
    auto dp = qp;
    dp.x = static_cast<const T *>(a.d_out);
    dp.wq = dp.wk = dp.wv = static_cast<const T *>(f.wo);
    dp.w_nk = 1; dp.nout = 1;
    dp.q = dp.k = dp.v = reinterpret_cast<T *>(a.do_raw);
    dp.q32 = a.do_raw;
    if ((err = launch_gemm_tail<GEMM_B_NK>(dp, units, l_a, dh, st)) != hipSuccess) return err;

    if (dh <= 32) launch_attention_bwd_f32_dh<T, 32>(a, st);
    else if (dh <= 64) launch_attention_bwd_f32_dh<T, 64>(a, st);
    else launch_attention_bwd_f32_dh<T, 128>(a, st);
    if ((err = hipGetLastError()) != hipSuccess) return err;

    SmhaDxProblem<T, parts_of<T>::value> xp;
    xp.o = static_cast<const T *>(a.dqkv); xp.o_lo = nullptr; xp.parts = 1; xp.wo = nullptr;
    xp.w[0] = static_cast<const T *>(f.wq); xp.w[1] = static_cast<const T *>(f.wk); xp.w[2] = static_cast<const T *>(f.wv);
    xp.x = static_cast<const T *>(a.d_out);
    xp.expert_idx = f.expert_idx; xp.patch_idx = f.patch_idx; xp.out = static_cast<T *>(a.d_x);
    xp.l = f.l; xp.d = f.d; xp.n = f.n; xp.kact = f.k; xp.m = f.m; xp.c = f.c;
    xp.l_p = l_p; xp.l_a = l_a; xp.d_h = dh; xp.o_row = parts_of<T>::value * 3 * dh; xp.flags = a.flags & F_RESIDUAL;
    const int groups = f.b * xp.set_patch_groups(f.b);
    if ((err = launch_gemm_tail<GEMM_B_NK>(xp, groups, xp.gp * l_p, f.d, st)) != hipSuccess) return err;

    SmhaBwdWgrad<T> wp;
    wp.dqkv = static_cast<const T *>(a.dqkv); wp.og = static_cast<const T *>(a.og);
    wp.x = static_cast<const T *>(f.x); wp.d_out = static_cast<const T *>(a.d_out);
    wp.expert_idx = f.expert_idx; wp.patch_idx = f.patch_idx; wp.partial = a.partial;
    wp.b = f.b; wp.l = f.l; wp.d = f.d; wp.n = f.n; wp.kact = f.k; wp.m = f.m; wp.c = f.c;
    wp.l_p = l_p; wp.l_a = l_a; wp.d_h = dh; wp.parts = {4, DEALT, a.wgrad, a.part_end};
    Beside<RoutePrep<T>> prep{};
    if (tail && tail->prep) {
        prep.side = RoutePrep<T>(*tail->prep);
        prep.blocks = prep.side.blocks();
    }
    if ((err = launch_gemm_tail<GEMM_A_KM>(wp, wp.parts.groups(), dh, f.d, st, &prep)) != hipSuccess) return err;
    if (tail && tail->prep && !prep.blocks) tail->prep_done = 1;
    WgradReduceArgs ra{};
    ra.partial = a.partial; ra.n = f.n; ra.M = dh; ra.N = f.d;
    ra.w = a.wgrad; ra.part_end = a.part_end;
    ra.dst[0] = a.d_wq; ra.dst[1] = a.d_wk; ra.dst[2] = a.d_wv; ra.dst[3] = a.d_wo;
    ra.transposed[0] = ra.transposed[1] = ra.transposed[2] = 1; ra.transposed[3] = 0;
    return launch_wgrad_reduce<T>(ra, 4, st, tail);
}

}  // namespace

hipError_t launch_uome_backward_any(const UomeBwdArgs &a, bool bf16, hipStream_t st, BwdTail *tail)
{
    return bf16 ? uome_backward_any<bf16_t>(a, st, tail) : uome_backward_any<float>(a, st, tail);
}

hipError_t launch_smha_backward_any(const SmhaBwdArgs &a, bool bf16, hipStream_t st, BwdTail *tail)
{
    return bf16 ? smha_backward_any<bf16_t>(a, st, tail) : smha_backward_any<float>(a, st, tail);
}

}  // namespace uoe
