// The contractions of the layer, each stated as a grouped GEMM "problem":
// for a group g, C[M(g), N] = A[M(g), K(g)] * B[K(g), N] with an epilogue, where the rows of A and
// the rows/columns of B are resolved through the routing indices.  A problem is a small POD
// passed by value to the engine (gemm_dma.h), which asks it for
//   rows(g), kdim(g), ncols()            problem extents
//   kseg(g)                              length of one K segment (one expert's slice, or all of K)
//   seg_ctx(g, seg)                      32 bits of routing context of a K segment, looked up once per tile (the engine may not
//                                        touch global memory through the compiler inside its K loop)
//   a_ptr_ctx(g, m, seg, ctx)            pointer to A[m][seg*kseg], from that context; the segment's elements are contiguous
//   b_ptr_ctx(g, seg, nn, ctx)           pointer to B[seg*kseg][nn..nn+8)  (nn % 8 == 0)
//   b_stride()                           elements between consecutive K rows of B inside a segment
//   kPrepare / prepare(g, segtab, scratch, tid, nthreads)  the workgroup builds its segment list itself (scratch: the stage buffers' LDS,
//                                        behind a last barrier theirs again) and returns K (out-projection: which experts picked this patch); -1: there is no such tile
//   kSelects / select<NT>(g, tile, scratch, tid)  (optional) the workgroup, `tile` of its group, selects for the group itself first
//                                        (select.h), in the stage buffers' LDS; NT threads, ends on a barrier
//   decode(g)                            (optional) what the problem calls the launch's group g
//   seg_len(ctx), seg_tail(step)         (optional, GEMM_A_KM and GEMM_TAIL) a segment's own length, at most kseg(g), and what the longest tail of one
//                                        is in a K-step; K is then the sum of the lengths in whole K-steps
// Its fp32 form writes four columns of a row at a time:
//   epi_f32(v, scale), put4(g, m, nn, v4)   per-element math; the store (residual included)
// and its bf16 form 16-byte pieces of output rows:
//   kColScale / col_scale(g, nn)  a per-column factor (constant over 8-column groups), fetched
//                                 once per tile before the K loop
//   epi(v, scale)                 per-element math
//   kRowScale / row_scale(g, m)   a per-row factor, fetched once per tile before the K loop; the
//                                 epilogue passes col_scale * row_scale to epi
//   has_residual() / res8(g, m, nn)  the 16-byte piece of the residual row, loaded in batches
//   put8(g, m, nn, piece)         plain store of a finished piece
//   once, res8_as<ONCE> / put8_as<ONCE>  (optional) a problem with a `once` member lets the launch choose the
//                                 non-temporal versions of the two accesses above, for outputs and
//                                 residuals that this call touches exactly once and that are too large
//                                 for the caches
// K and N are concatenations of per-expert segments of length `width`; since width % 8 == 0 an
// 8-element run never straddles two experts.
#pragma once
#include "common.h"
#include "select.h"
#include <type_traits>

namespace uoe {

// what the engines call the elements of a storage type
template <typename T> struct storage_elem {
    typedef uint16_t type;
};
template <> struct storage_elem<float> {
    typedef float type;
};

__device__ __forceinline__ float4 add4_f32(float4 a, const float *r)
{
    const float4 b = *reinterpret_cast<const float4 *>(r);
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// 8 bf16 (one 16-byte piece of an output row) + 8 bf16 of a residual row, added in fp32
__device__ __forceinline__ uint4 add8_bf16(uint4 v, uint4 r)
{
    const uint32_t a[4] = {v.x, v.y, v.z, v.w}, b[4] = {r.x, r.y, r.z, r.w};
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float lo = __uint_as_float(a[i] << 16) + __uint_as_float(b[i] << 16);
        const float hi = __uint_as_float(a[i] & 0xFFFF0000u) + __uint_as_float(b[i] & 0xFFFF0000u);
        o[i] = pack2_bf16(lo, hi);
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
}

// ---------------------------------------------------------------------------------------------
// SMHA Eq. 28-30 with the index selection of Eq. 18 folded into the A-row lookup.
// group = active unit (b, slot s); M = l_a; K = d; N = 3*d_h laid out [q | k | v].
// F32: bf16 operands, fp32 rows into q32 (projection w at q32 + w * q32_plane) instead.
// w_nk: the single projection (nout = 1) multiplies by the transpose of wq [n, d_h, d] (engine flag GEMM_B_NK).
template <typename T, bool F32 = false, bool ROPE = false> struct QkvProblem {
    typedef typename storage_elem<T>::type Elem;
    const T *x, *wq, *wk, *wv;
    const int32_t *expert_idx, *patch_idx;
    T *q, *k, *v;  // [units, l_a, d_h]
    float *q32;    // nout x [units, l_a, d_h] (F32 only)
    size_t q32_plane = 0;
    int w_nk = 0;
    static constexpr bool kF32Out = F32;
    __device__ void put4_f32(int g, int r, int nn, float4 val) const
    {
        const int which = nn / d_h;
        *reinterpret_cast<float4 *>(q32 + which * q32_plane + ((size_t)g * l_a + r) * d_h + (nn - which * d_h)) = val;
    }
    int l, d, n, kact, m, c, l_p, l_a, d_h;
    float q_scale;  // folded into q on the way out (1 for the plain layout)
    int nout;       // 3: q, k and v; 1: the first projection only (N = d_h)
    // ROPE, bf16 rows: the last rope_dim dims of q and k rotated by the row's position in the compacted sequence (Eq. 32),
    // in fp32 before the one rounding (an in-place kernel behind the projection took 2.8-3.7 us and rounded twice)
    static constexpr bool kRotates = ROPE;
    int rope_dim = 0;
    __device__ bool rotates(int col8) const
    {
        const int which = col8 / d_h, dh = col8 - which * d_h;
        return which < 2 && dh + 8 > d_h - rope_dim;
    }
    __device__ void rotate(int r, int col, float &e0, float &e1, float &e2, float &e3) const
    {
        const int dh = col % d_h, first = d_h - rope_dim;
        float sn, cs, t;
        if (dh >= first) {
            rope_sincos((float)r, rope_theta(dh - first, rope_dim), sn, cs);
            t = e0; e0 = t * cs - e1 * sn; e1 = t * sn + e1 * cs;
        }
        if (dh + 2 >= first) {
            rope_sincos((float)r, rope_theta(dh + 2 - first, rope_dim), sn, cs);
            t = e2; e2 = t * cs - e3 * sn; e3 = t * sn + e3 * cs;
        }
    }
    int v_f16 = 0;  // bf16 storage: v is written as fp16 (what the attention kernel's P V product takes)
    __device__ bool f16_col(int nn) const { return v_f16 && nn >= 2 * d_h; }
    T *v_copy = nullptr;   // with v_f16: v in bf16 as well (the backward pass's operand)
    __device__ void put4_copy(int g, int r, int nn, uint2 piece) const
    {
        *reinterpret_cast<uint2 *>(v_copy + ((size_t)g * l_a + r) * d_h + (nn - 2 * d_h)) = piece;
    }

    __device__ int rows(int) const { return l_a; }
    __device__ int kdim(int) const { return d; }
    __device__ int ncols() const { return nout * d_h; }
    __device__ int expert(int g) const { return clampi(expert_idx[g], n); }
    __device__ int token(int g, int r) const
    {
        const int bb = g / kact;
        const int i = expert(g);
        const int t = r / l_p;
        return clampi(patch_idx[((size_t)bb * n + i) * c + t], m) * l_p + (r - t * l_p);
    }
    __host__ __device__ int kseg(int) const { return d; }
    __device__ long b_stride() const { return d_h; }
    // K is one segment, rows and columns are resolved once before the loop
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t) const
    {
        const int bb = g / kact;
        return x + ((size_t)bb * l + token(g, r)) * d;
    }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t) const
    {
        const int i = expert(g);
        if (w_nk) return wq + ((size_t)i * d_h + nn) * d;
        const int which = nn / d_h;
        const T *w = which == 0 ? wq : (which == 1 ? wk : wv);
        return w + (size_t)i * d * d_h + (nn - which * d_h);
    }
    __device__ float epi_f32(float val, float scale) const { return val * scale; }
    __device__ void put4(int g, int r, int nn, float4 val) const
    {
        const int which = nn / d_h;
        T *o = which == 0 ? q : (which == 1 ? k : v);
        *reinterpret_cast<float4 *>(o + ((size_t)g * l_a + r) * d_h + (nn - which * d_h)) = val;
    }
    static constexpr bool kPrepare = false;
    static constexpr bool kRowScale = false;
    static constexpr bool kColScale = true;
    __device__ float col_scale(int, int nn) const { return nn < d_h ? q_scale : 1.0f; }
    __device__ float epi(float val, float scale) const { return val * scale; }
    __device__ bool has_residual() const { return false; }
    __device__ uint4 res8(int, int, int) const { return make_uint4(0, 0, 0, 0); }
    __device__ void put8(int g, int r, int nn, uint4 piece) const
    {
        const int which = nn / d_h;
        T *o = which == 0 ? q : (which == 1 ? k : v);
        *reinterpret_cast<uint4 *>(o + ((size_t)g * l_a + r) * d_h + (nn - which * d_h)) = piece;
    }
};

// ---------------------------------------------------------------------------------------------
// SMHA Eq. 35 + Eq. 36, output-stationary: group = (b, gp consecutive patches); M = gp * l_p; N = d;
// K = (number of active experts that picked any of them) * d_h, rows of the patches an expert did not pick read zeros.
// gp > 1 (set_patch_groups) where patches are shorter than a tile is high: one 14-token patch in a 32-row tile left half of it
// empty.  The per-expert products o_i W^o_i that land
// on the same patch are summed as one contraction over the concatenated K, so each output row is
// written exactly once (residual added in the epilogue) and no atomics are needed.
// o already carries the gate weight of its row.  In the bf16 MFMA path o arrives as two bf16
// buffers, o = hi + lo, so that the attention output enters this contraction with ~16 significant
// bits instead of 8 (the rows of W^o are simply visited twice).
template <typename T> struct OutProjProblem {
    typedef typename storage_elem<T>::type Elem;
    bool once = false;   // this launch streams its output (and residual) past the caches: see store16, wave_write_out
    const T *o, *o_lo, *wo, *x;
    const int32_t *expert_idx, *patch_idx;
    T *out;
    int l, d, n, kact, m, c, l_p, l_a, d_h;
    int o_row;  // elements between rows of o (d_h, or more where they hold other columns too)
    int parts;  // 1: o only; 2: o is a (hi, lo) pair of buffers, contracted as [hi | lo] x [W^o ; W^o]
    uint32_t flags;
    int w_nk = 0;   // wo is [n, d, d_h] (engine flag GEMM_B_NK)
    int gp = 1;     // patches per group, at most 32
    static constexpr bool kRowGaps = true;

    // Patches per group for 32-row tiles, or for 128-row ones where those still fill the chip's slots (two workgroups of
    // eight waves per compute unit) and the experts' rows are not spread too thin: a group multiplies all its rows
    // with every expert that picked any of its patches, 1 - (1 - c/m)^gp of them.  Up to twice the products of 32-row
    // groups are repaid by a quarter of the workgroups and of their lookup chains (128 samples of 14 x 14 tokens, 4 of 14
    // patches, three experts: 21.6 us with two patches, 17.8 us with nine); patches that fill a 64-row tile gain nothing (two
    // of 64 tokens on the largest shape 37 -> 51 us).  Returns the groups per sample.
    __host__ int set_patch_groups(int b)
    {
        const auto fit = [&](int tile) { const int g = 2 * l_p <= tile ? tile / l_p : 1; return g < m ? g : m; };
        const auto products = [&](int g, int tile) {
            double none = 1.0;
            for (int i = 0; i < g && none > 1e-3; ++i) none *= 1.0 - (double)c / m;
            return (double)((g * l_p + tile - 1) / tile * tile) / g * (1.0 - none);
        };
        gp = fit(32);
        const int g128 = fit(128) < 32 ? fit(128) : 32;
        const long tiles = (long)b * ((m + g128 - 1) / g128) * ((d + 127) / 128);
        if (l_p <= 32 && g128 > gp && g128 * l_p > 64 && tiles >= 512 && products(g128, 128) <= 2.0 * products(gp, 32)) gp = g128;
        return groups_per_sample();
    }
    __host__ __device__ int groups_per_sample() const { return (m + gp - 1) / gp; }
    __device__ int first_patch(int g) const { return g % groups_per_sample() * gp; }
    __device__ int rows(int g) const { return min(gp, m - first_patch(g)) * l_p; }
    __device__ int kdim(int) const { return 0; }  // prepare() supplies K
    __device__ int ncols() const { return d; }
    __host__ __device__ int kseg(int) const { return d_h; }
    __device__ long b_stride() const { return d; }
    __device__ float epi_f32(float val, float) const { return val; }
    __device__ void put4(int g, int r, int nn, float4 val) const
    {
        const size_t at = at8(g, r, nn);
        if (flags & F_RESIDUAL) val = add4_f32(val, reinterpret_cast<const float *>(x) + at);
        *reinterpret_cast<float4 *>(out + at) = val;
    }
    // per K segment, the slot in bits 0-4, the expert in bits 20-25 and the hi/lo part in bit 26.
    // The workgroup builds the list of its group's segments itself (prepare), straight from the routing indices:
    // thread (slot s, pick t) notes which of the group's patches slot s picked as which pick (at most one t per slot and
    // patch), then the slots that picked any are listed in slot order, which fixes the summation order.  Returns K;
    // ends on a barrier.
    static constexpr bool kPrepare = true;
    static constexpr bool kRowScale = false;
    __device__ static int16_t *pick_table()   // [slot][patch of the group] -> pick, or -1
    {
        __shared__ int16_t tab[32 * 32];
        return tab;
    }
    __device__ int prepare(int g, uint32_t *segtab, void *, int tid, int nthreads) const
    {
        __shared__ int slot_any[32], slot_e[32];
        int16_t *pick = pick_table();
        const int bb = g / groups_per_sample(), p0 = first_patch(g);
        if (tid < kact) slot_any[tid] = 0;
        for (int idx = tid; idx < kact * gp; idx += nthreads) pick[idx] = -1;
        __syncthreads();
        for (int idx = tid; idx < kact * c; idx += nthreads) {
            const int s = idx / c, t = idx - s * c;
            const int i = clampi(expert_idx[bb * kact + s], n);
            if (t == 0) slot_e[s] = i;
            const int pp = clampi(patch_idx[((size_t)bb * n + i) * c + t], m) - p0;
            if (pp >= 0 && pp < gp) {
                pick[s * gp + pp] = (int16_t)t;
                slot_any[s] = 1;
            }
        }
        __syncthreads();
        int cnt = 0;
        for (int s = 0; s < kact; ++s) {  // every thread walks the (at most 32) slots: cnt is uniform
            if (!slot_any[s]) continue;
            if (tid == 0)
                for (int part = 0; part < parts; ++part)
                    segtab[cnt * parts + part] = (uint32_t)s | ((uint32_t)slot_e[s] << 20) | ((uint32_t)part << 26);
            ++cnt;
        }
        __syncthreads();
        return cnt * parts * d_h;
    }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t ctx) const
    {
        const int bb = g / groups_per_sample(), s = (int)(ctx & 0x1Fu), pr = gp > 1 ? r / l_p : 0;
        const int t = pick_table()[s * gp + pr];
        if (t < 0) return nullptr;
        const T *src = (ctx >> 26) & 1u ? o_lo : o;
        return src + (((size_t)bb * kact + s) * l_a + t * l_p + (r - pr * l_p)) * o_row;
    }
    __device__ const T *b_ptr_ctx(int, int, int nn, uint32_t ctx) const
    {
        return wo + (size_t)((ctx >> 20) & 0x3Fu) * d_h * d + (size_t)nn * (w_nk ? d_h : 1);
    }
    static constexpr bool kColScale = false;
    __device__ float col_scale(int, int) const { return 1.0f; }
    __device__ float epi(float val, float) const { return val; }
    __device__ size_t at8(int g, int r, int nn) const
    {
        return ((size_t)(g / groups_per_sample()) * l + (size_t)first_patch(g) * l_p + r) * d + nn;
    }
    __device__ bool has_residual() const { return flags & F_RESIDUAL; }
    __device__ uint4 res8(int g, int r, int nn) const { return res8_as<false>(g, r, nn); }
    __device__ void put8(int g, int r, int nn, uint4 piece) const { put8_as<false>(g, r, nn, piece); }
    // ONCE: the residual is this tensor's last use in the call and every output piece is written once
    template <bool ONCE> __device__ uint4 res8_as(int g, int r, int nn) const { return load16<ONCE>(x + at8(g, r, nn)); }
    template <bool ONCE> __device__ void put8_as(int g, int r, int nn, uint4 piece) const { store16<ONCE>(out + at8(g, r, nn), piece); }
};

// d_x = (G) + sum over the experts that picked the patch of [dq|dk|dv] [W^q|W^k|W^v]^T: the out-projection's
// output-stationary contraction; K segments of an entry: parts x (q, k, v) of d_h, W [d, d_h] is [n][k].  PARTS = 2:
// rows of dqkv are (hi, lo) pairs.
template <typename T, int PARTS> struct SmhaDxProblem : OutProjProblem<T> {
    const T *w[3];   // wq, wk, wv
    static constexpr int kSegParts = 3 * PARTS;
    __device__ int prepare(int g, uint32_t *segtab, void *scratch, int tid, int nthreads) const
    {
        return OutProjProblem<T>::prepare(g, segtab, scratch, tid, nthreads) * kSegParts;   // this->parts is 1: one table entry per expert
    }
    __device__ const T *a_ptr_ctx(int g, int r, int seg, uint32_t ctx) const
    {
        const T *row = OutProjProblem<T>::a_ptr_ctx(g, r, seg, ctx);
        return row ? row + (size_t)(seg % kSegParts) * this->d_h : row;   // [parts][3][d_h] in a row
    }
    __device__ const T *b_ptr_ctx(int, int seg, int nn, uint32_t ctx) const
    {
        const int which = (seg % kSegParts) % 3;
        const T *base = which == 0 ? w[0] : which == 1 ? w[1] : w[2];
        return base + ((size_t)((ctx >> 20) & 0x3Fu) * this->d + nn) * this->d_h;
    }
};

// ---------------------------------------------------------------------------------------------
// UoME Eq. 38: group = sample b; M = l; K = d; N = k*d_e (the sample's active experts side by
// side); epilogue SiLU and the expert's gate.  EXACT: SiLU by a division also for bf16 storage.  SEL: the sample's experts and gates come
// from a selection of the workgroup's own.
template <typename T, bool RAW = false, bool EXACT = false, bool SEL = false> struct UomeUpProblem {
    typedef typename storage_elem<T>::type Elem;
    bool once = false;   // this launch streams its output (and residual) past the caches: see store16, wave_write_out
    const T *u, *a_in;
    const int32_t *expert_idx;
    const float *expert_gate;  // NULL: weight 1
    T *hidden;                 // [b, l, k*d_e]
    int l, d, n, kact, d_e;
    static constexpr bool raw = RAW;   // true: store the plain product (backward pass), no SiLU, no gate
    std::conditional_t<SEL, RouteSelect, NoSelect> sel;
    static constexpr bool kSelects = SEL;
    __device__ static SelectedExperts &selected()
    {
        __shared__ SelectedExperts s;
        return s;
    }
    template <int NT> __device__ void select(int g, int tile, unsigned char *scratch, int tid) const
    {
        select_experts_beside<NT>(sel, g, reinterpret_cast<float *>(scratch), selected(), tile == 0, tid);
    }
    __device__ int expert(int g, int slot) const
    {
        if constexpr (SEL) return clampi(selected().expert[slot], n);
        else return clampi(expert_idx[g * kact + slot], n);
    }

    __device__ int rows(int) const { return l; }
    __device__ int kdim(int) const { return d; }
    __device__ int ncols() const { return kact * d_e; }
    __host__ __device__ int kseg(int) const { return d; }
    __device__ long b_stride() const { return d_e; }
    // no per-segment lookups (K is one segment; the column's expert is resolved once, before the loop)
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t) const { return u + ((size_t)g * l + r) * d; }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t) const
    {
        const int s = nn / d_e;
        return a_in + (size_t)expert(g, s) * d * d_e + (nn - s * d_e);
    }
    __device__ float epi_f32(float val, float gate) const { return raw ? val : silu(val) * gate; }
    __device__ void put4(int g, int r, int nn, float4 val) const
    {
        *reinterpret_cast<float4 *>(hidden + ((size_t)g * l + r) * ((size_t)kact * d_e) + nn) = val;
    }
    static constexpr bool kPrepare = false;
    static constexpr bool kRowScale = false;
    static constexpr bool kColScale = true;
    __device__ float col_scale(int g, int nn) const   // the gate of the column's expert
    {
        if (!expert_gate || raw) return 1.0f;
        if constexpr (SEL) return selected().gate[nn / d_e];
        else return expert_gate[(size_t)g * n + expert(g, nn / d_e)];
    }
    __device__ float epi(float val, float gate) const { return raw ? val : (EXACT ? silu(val) : silu_fast(val)) * gate; }
    __device__ bool has_residual() const { return false; }
    __device__ uint4 res8(int, int, int) const { return make_uint4(0, 0, 0, 0); }
    __device__ void put8(int g, int r, int nn, uint4 piece) const { put8_as<false>(g, r, nn, piece); }
    template <bool ONCE> __device__ uint4 res8_as(int, int, int) const { return make_uint4(0, 0, 0, 0); }
    template <bool ONCE> __device__ void put8_as(int g, int r, int nn, uint4 piece) const   // ONCE: 134 MB on the largest shape, streamed past L2
    {
        store16<ONCE>(hidden + ((size_t)g * l + r) * ((size_t)kact * d_e) + nn, piece);
    }
};

// UoME with patch-wise data selection, first layer (Eq. 37-38): group = active unit (b, slot s);
// M = l_a rows gathered through the unit's patch indices (Eq. 18 folded into the A-row lookup, as
// for QKV); K = d; N = d_e.  Epilogue: SiLU, times the weight of the row's contribution (expert
// gate and/or the gate of the row's patch): the second layer is linear, so the weight can ride on
// the hidden activations and the output-stationary second GEMM needs no per-segment scale.
template <typename T, bool EXACT = false> struct UomeDsUpProblem {
    typedef typename storage_elem<T>::type Elem;
    const T *u, *a_in;
    const int32_t *expert_idx, *patch_idx;
    const float *expert_gate, *patch_gate;  // NULL: weight 1
    T *hidden;                              // [units, l_a, d_e]
    int l, d, n, kact, m, c, l_p, l_a, d_e;

    __device__ int rows(int) const { return l_a; }
    __device__ int kdim(int) const { return d; }
    __device__ int ncols() const { return d_e; }
    __host__ __device__ int kseg(int) const { return d; }
    __device__ long b_stride() const { return d_e; }
    __device__ int expert(int g) const { return clampi(expert_idx[g], n); }
    __device__ int patch(int g, int r) const
    {
        return clampi(patch_idx[((size_t)(g / kact) * n + expert(g)) * c + r / l_p], m);
    }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t) const
    {
        return u + ((size_t)(g / kact) * l + patch(g, r) * l_p + r % l_p) * d;
    }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t) const { return a_in + (size_t)expert(g) * d * d_e + nn; }
    __device__ float row_scale(int g, int r) const
    {
        const int bb = g / kact, i = expert(g);
        float w = expert_gate ? expert_gate[(size_t)bb * n + i] : 1.0f;
        if (patch_gate) w *= patch_gate[((size_t)bb * n + i) * m + patch(g, r)];
        return w;
    }
    __device__ float epi_f32(float val, float w) const { return silu(val) * w; }
    __device__ void put4(int g, int r, int nn, float4 val) const
    {
        *reinterpret_cast<float4 *>(hidden + ((size_t)g * l_a + r) * d_e + nn) = val;
    }
    static constexpr bool kPrepare = false;
    static constexpr bool kRowScale = true;
    static constexpr bool kColScale = false;
    __device__ float col_scale(int, int) const { return 1.0f; }
    __device__ float epi(float val, float w) const { return (EXACT ? silu(val) : silu_fast(val)) * w; }
    __device__ bool has_residual() const { return false; }
    __device__ uint4 res8(int, int, int) const { return make_uint4(0, 0, 0, 0); }
    __device__ void put8(int g, int r, int nn, uint4 piece) const
    {
        *reinterpret_cast<uint4 *>(hidden + ((size_t)g * l_a + r) * d_e + nn) = piece;
    }
};

// UoME Eq. 39 + Eq. 40: group = sample b; M = l; K = k*d_e (row slices of A^O of the active
// experts stacked); N = d; epilogue adds the residual.  One write per output element.
template <typename T> struct UomeDownProblem {
    typedef typename storage_elem<T>::type Elem;
    bool once = false;   // this launch streams its output (and residual) past the caches: see store16, wave_write_out
    const T *hidden, *a_out, *u;
    const int32_t *expert_idx;
    T *out;
    int l, d, n, kact, d_e;
    uint32_t flags;
    int w_nk = 0;        // a_out is [n, d, d_e] (engine flag GEMM_B_NK)

    __device__ int rows(int) const { return l; }
    __device__ int kdim(int) const { return kact * d_e; }
    __device__ int ncols() const { return d; }
    __host__ __device__ int kseg(int) const { return d_e; }
    __device__ long b_stride() const { return d; }
    // the segment's expert, looked up once before the loop
    __device__ uint32_t seg_ctx(int g, int seg) const { return (uint32_t)clampi(expert_idx[g * kact + clampi(seg, kact)], n); }
    __device__ const T *a_ptr_ctx(int g, int r, int seg, uint32_t) const
    {
        return hidden + ((size_t)g * l + r) * ((size_t)kact * d_e) + (size_t)clampi(seg, kact) * d_e;
    }
    __device__ const T *b_ptr_ctx(int, int, int nn, uint32_t i) const { return a_out + (size_t)i * d_e * d + (size_t)nn * (w_nk ? d_e : 1); }
    __device__ float epi_f32(float val, float) const { return val; }
    __device__ void put4(int g, int r, int nn, float4 val) const
    {
        const size_t at = ((size_t)g * l + r) * d + nn;
        if (flags & F_RESIDUAL) val = add4_f32(val, reinterpret_cast<const float *>(u) + at);
        *reinterpret_cast<float4 *>(out + at) = val;
    }
    static constexpr bool kPrepare = false;
    static constexpr bool kRowScale = false;
    static constexpr bool kColScale = false;
    __device__ float col_scale(int, int) const { return 1.0f; }
    __device__ float epi(float val, float) const { return val; }
    __device__ bool has_residual() const { return flags & F_RESIDUAL; }
    __device__ uint4 res8(int g, int r, int nn) const { return res8_as<false>(g, r, nn); }
    __device__ void put8(int g, int r, int nn, uint4 piece) const { put8_as<false>(g, r, nn, piece); }
    __device__ bool has_early() const { return has_residual(); }
    template <bool ONCE> __device__ uint4 early8(int g, int r, int nn) const { return res8_as<ONCE>(g, r, nn); }
    // ONCE: u's last use and the block's output
    template <bool ONCE> __device__ uint4 res8_as(int g, int r, int nn) const { return load16<ONCE>(u + ((size_t)g * l + r) * d + nn); }
    template <bool ONCE> __device__ void put8_as(int g, int r, int nn, uint4 piece) const { store16<ONCE>(out + ((size_t)g * l + r) * d + nn, piece); }
};

// Which of up to 128 samples selected each expert: two ballots an expert give its count and every sample's place in its list
// (counting through LDS sample by sample took longer than a short contraction).  Called by the whole workgroup of at least
// 128 threads; ends on a barrier.
constexpr int KEPT_IDX = 8;   // of a sample's indices, what stays in registers
__device__ __forceinline__ void expert_masks(uint64_t (*mask)[2], int (&idx)[KEPT_IDX], const int32_t *expert_idx, int nb, int kact, int n, int tid)
{
    uint32_t mine = 0;
#pragma unroll
    for (int s = 0; s < KEPT_IDX; ++s) {
        idx[s] = clampi(expert_idx[min(tid, nb - 1) * kact + min(s, kact - 1)], n);   // (unconditional: all in flight together)
        mine |= 1u << idx[s];
    }
    for (int s = KEPT_IDX; s < kact; ++s) mine |= 1u << clampi(expert_idx[min(tid, nb - 1) * kact + s], n);
    if (tid >= nb) mine = 0;
    if (tid < 128) {
        uint64_t keep = 0;
        for (int e = 0; e < n; ++e) {
            const uint64_t m = __ballot(mine >> e & 1u);
            if ((tid & 63) == e) keep = m;
        }
        if ((tid & 63) < n) mask[tid & 63][tid >> 6] = keep;
    }
    __syncthreads();
}

// Where an expert's parts lie among a chunk's part ids (lane e of a wave holds expert e's; n <= 32), `each` being 0.  Each lane tries one value
// of `per` from lo to hi, every one where there are at most 64 and equally spaced ones (hi among them) otherwise; the least that fits the budget is taken.
struct PartScan {
    int count, parts, behind;   // selecting samples; parts; first id behind them
    __device__ PartScan(const uint64_t (*mask)[2], const WgradPlan &w, int n, int lane)
    {
        const int e = lane & 31;
        count = e < n ? __popcll(mask[e][0]) + __popcll(mask[e][1]) : 0;
        const int items = count * w.items, step = (w.hi - w.lo + 62) / 63;
        const int per = min(w.lo + lane * step, w.hi);
        const float inv = __builtin_amdgcn_rcpf((float)per);
        auto cuts = [](int of, int by, float by_inv) {   // ceil(of / by) for of < 2^23
            const int x = of + by - 1;
            int q = (int)((float)x * by_inv);
            const int r = x - q * by;
            q += r >= by ? 1 : (r < 0 ? -1 : 0);
            return q;
        };
        int sum = 0;
        for (int i = 0; i < n; ++i) sum += cuts(__builtin_amdgcn_readlane(items, i), per, inv);
        const uint64_t fits = __ballot(sum <= w.parts);
        const int at = fits ? __ffsll((unsigned long long)fits) - 1 : 63;
        const int best = __builtin_amdgcn_readlane(per, at);
        parts = cuts(items, best, __builtin_amdgcn_rcpf((float)best));
        behind = parts;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const int t = __shfl_up(behind, off, 32);
            if (e >= off) behind += t;
        }
    }
};

// x / by for x * by < 2^32 by the reciprocal rounded up
struct Divider {
    int by;
    uint32_t inv;   // 0: by one
    Divider() = default;
    explicit Divider(int by_) : by(by_), inv(by_ > 1 ? 0xFFFFFFFFu / (uint32_t)by_ + 1u : 0u) {}
    __device__ int of(int x) const { return inv ? (int)__umulhi((uint32_t)x, inv) : x; }
};

// A launch's groups: (set, chunk, place) for gradient tensors of one shape.  Each XCD works on a contiguous eighth of the groups.
//   IN_ORDER   expert by expert
//   BY_SAMPLE  places follow where in the sample axis a part begins: the parts that run on an XCD at one time are those of different experts
//              over the same tokens, whose right operands are the same rows (4 x 8192 tokens, 16 experts of 1024 x 256: 272 -> 254 us)
//   DEALT      dealt round-robin over the eighths, so that each gets parts of all experts: short parts of patches, where finding the order
//              by samples takes longer than it saves (8 x 512 tokens, 8 experts, with d_x: 15.0 us in order, 17.8 by sample, 13.3 dealt)
// CHUNKED: more than 128 samples are possible; MAY_DEAL: the problem asks for DEALT
enum { IN_ORDER, BY_SAMPLE, DEALT };
template <bool CHUNKED, bool MAY_DEAL> struct WgradOrder {
    int sets_log2, by;
    WgradPlan w;
    int32_t *part_end;   // [chunks, 32] first part id behind an expert's, for the reduction
    Divider parts, eighth, each;   // (five divisions one behind the other were half a microsecond at the start of a short launch)
    WgradOrder() = default;
    WgradOrder(int sets, int by_, const WgradPlan &w_, int32_t *part_end_)
        : sets_log2(sets == 4 ? 2 : 1), by(w_.each || (by_ == BY_SAMPLE && w_.parts > 256) ? IN_ORDER : by_), w(w_), part_end(part_end_), parts(w_.parts), eighth((sets * w_.chunks * w_.parts + 7) / 8),
          each(w_.each ? w_.each : 1) {}
    int groups() const { const int g = (w.chunks * w.parts) << sets_log2; return by == DEALT ? (g + 7) / 8 * 8 : g; }
    // Set in bits 0-1, place in bits 2-14, chunk above: up to WGRAD_MAX_PARTS parts a chunk.  Lists of patches come to that many, n x c of them, with 128 samples of
    // which each part holds 128 entries; n x m <= 8192 is what the entry points accept.
    __device__ int decode(int g) const
    {
        if (CHUNKED && w.chunks > 1) {
            if (MAY_DEAL && by == DEALT) {
                const int o = g % eighth.by * 8 + g / eighth.by, r = o >> sets_log2, c = r % w.chunks;
                return (o - (r << sets_log2)) | (r / w.chunks) << 2 | c << 15;
            }
            const int s = g / (w.chunks * w.parts), r = g - s * (w.chunks * w.parts), c = r / w.parts;
            return s | (r - c * w.parts) << 2 | c << 15;
        }
        if (MAY_DEAL && by == DEALT) {   // (fewer than 2^15 groups)
            const int q = eighth.of(g), o = (g - q * eighth.by) * 8 + q, r = o >> sets_log2;
            return (o - (r << sets_log2)) | r << 2;
        }
        const int s = parts.of(g);
        return s | (g - s * w.parts) << 2;
    }
    __device__ int set(int g) const { return g & 3; }
    __device__ int place(int g) const { return g >> 2 & 0x1FFF; }   // (prepare() puts the part's id there)
    __device__ int chunk(int g) const { return CHUNKED ? g >> 15 : 0; }
    __device__ size_t tile(int g) const { return (size_t)(CHUNKED ? set(g) * w.chunks + chunk(g) : set(g)) * w.parts + place(g); }   // its partial tile
};

// The workgroup's part of an expert's list: its partial tile, items [first, last) of the expert, the expert's samples and slots
struct PartList {
    uint64_t mask[32][2];
    uint32_t key[256];
    int32_t end[32];
    int16_t slot_of[128];
    int32_t found;
    // first item of a part (at most 2^17 items and 2^13 parts; 64-bit divisions took 2 us here)
    static __device__ int begin_of(int items, int part, int parts) { return (int)((uint32_t)items * (uint32_t)part / (uint32_t)parts); }
    // false: no such part; else g's place becomes the part's id.  Ends on a barrier.
    template <typename ORDER> __device__ bool fill(const int32_t *expert_idx, int nb, int kact, int n, const ORDER &o, int &g, int tid, int &expert, int &first, int &last)
    {
        const WgradPlan &w = o.w;
        int idx[KEPT_IDX];
        if (__builtin_expect(w.each != 0, 1)) {   // the expert is known: one ballot, and the slots with it (what follows lies out of the way)
            expert = o.each.of(o.place(g));
            const int part = o.place(g) - expert * w.each, at = min(tid, nb - 1) * kact;
            int slot = -1;
            for (int s = kact - 1; s >= KEPT_IDX; --s) slot = clampi(expert_idx[at + s], n) == expert ? s : slot;
#pragma unroll
            for (int s = KEPT_IDX - 1; s >= 0; --s) {
                const int t = min(s, kact - 1);
                slot = clampi(expert_idx[at + t], n) == expert ? t : slot;
            }
            if (tid >= nb) slot = -1;
            const uint64_t m = __ballot(slot >= 0);
            if (tid < 128 && (tid & 63) == 0) mask[expert][tid >> 6] = m;
            if (tid < nb) slot_of[tid] = (int16_t)slot;
            __syncthreads();
            const int items = (__popcll(mask[expert][0]) + __popcll(mask[expert][1])) * w.items, per = o.each.of(items + w.each - 1);
            first = __builtin_amdgcn_readfirstlane(min(items, part * per));
            last = __builtin_amdgcn_readfirstlane(min(items, (part + 1) * per));
            return true;
        }
        expert_masks(mask, idx, expert_idx, nb, kact, n, tid);
        const PartScan scan(mask, w, n, tid & 63);
        const int total = __builtin_amdgcn_readlane(scan.behind, 31), q = o.place(g);
        if (q == 0 && o.set(g) == 0 && tid < 32) o.part_end[o.chunk(g) * 32 + tid] = scan.behind;
        int mine = q;
        if (o.by != BY_SAMPLE) {
            if (q >= total) return false;
        } else {   // (at most 256 parts) the places that hold a part are spread evenly
            const int rank = begin_of(total, q, w.parts);
            if (begin_of(total, q + 1, w.parts) == rank) return false;
            if (tid < 32) end[tid] = scan.behind;
            __syncthreads();
            if (tid < 256) {
                uint32_t k = ~0u;
                if (tid < total) {
                    int e = 0;
#pragma unroll
                    for (int s = 16; s; s >>= 1) e += end[e + s - 1] <= tid ? s : 0;
                    const uint64_t m0 = mask[e][0], m1 = mask[e][1];
                    const int c0 = __popcll(m0), items = (c0 + __popcll(m1)) * w.items, begin = e ? end[e - 1] : 0;
                    const int at = begin_of(items, tid - begin, end[e] - begin);
                    int nth = at / w.items, sample = 0;   // of its first item: the nth listed sample
                    const int range = at - nth * w.items;
                    uint64_t m = m0;
                    if (nth >= c0) { m = m1; nth -= c0; sample = 64; }
#pragma unroll
                    for (int s = 32; s; s >>= 1) {
                        const int low = __popcll(m & ((1ull << s) - 1));
                        if (nth >= low) { nth -= low; m >>= s; sample += s; }
                    }
                    k = (uint32_t)(sample * w.items + range) << 8 | (uint32_t)tid;
                }
                key[tid] = k;
            }
            __syncthreads();
            if (tid < total) {
                const uint32_t k = key[tid];
                int below = 0;
                for (int j = 0; j < total; j += 4) {   // (what lies behind the keys is the largest value)
                    const uint4 v = *reinterpret_cast<const uint4 *>(&key[j]);
                    below += (v.x < k) + (v.y < k) + (v.z < k) + (v.w < k);
                }
                if (below == rank) found = tid;
            }
            __syncthreads();
            mine = found;
        }
        mine = __builtin_amdgcn_readfirstlane(mine);
        expert = __builtin_amdgcn_readfirstlane(__ffs((uint32_t)__ballot(mine < scan.behind)) - 1);
        const int parts = __builtin_amdgcn_readlane(scan.parts, expert), items = __builtin_amdgcn_readlane(scan.count, expert) * w.items;
        const int part = mine - (__builtin_amdgcn_readlane(scan.behind, expert) - parts);
        first = __builtin_amdgcn_readfirstlane(begin_of(items, part, parts));
        last = __builtin_amdgcn_readfirstlane(begin_of(items, part + 1, parts));
        g = (g & 3) | mine << 2 | o.chunk(g) << 15;
        if (tid < nb) {
            int slot = -1;
#pragma unroll
            for (int s = KEPT_IDX - 1; s >= 0; --s) slot = idx[s] == expert ? s : slot;
            if (slot < 0 && (mask[expert][tid >> 6] >> (tid & 63) & 1ull))
                for (int s = kact - 1; s >= KEPT_IDX; --s) slot = clampi(expert_idx[tid * kact + s], n) == expert ? s : slot;
            slot_of[tid] = (int16_t)slot;
        }
        __syncthreads();
        return true;
    }
    __device__ int before(int expert, int q) const   // listed samples below sample q
    {
        const uint64_t m0 = mask[expert][0];
        return q < 64 ? __popcll(m0 & ((1ull << q) - 1)) : __popcll(m0) + __popcll(mask[expert][1] & ((1ull << (q - 64)) - 1));
    }
};

// Weight gradients of the backward passes, as split contractions over the tokens with fp32 partial
// tiles.  A launch covers up to four gradient tensors ("sets") of the same shape [n][M][N] at once, in parts that
// hold as much of an expert's list each (WgradPlan, WgradOrder); a reduction kernel adds an expert's
// parts in order.  Both factors are read as the other kernels wrote them, token-major (engine flag GEMM_A_KM):
// a transposed copy of the left one cost its writer 2-byte scattered LDS or memory stores and a third of its traffic.
//
// Expert-selection UoME: for expert i,
//   dW[M, N] = sum over the (sample b, slot s) pairs with expert_idx[b,s] == i of  L_{b,s}^T R_b
// contracted over the l tokens of the sample.  K segments = ranges of a pair's tokens, l / items each, found by the workgroup
// itself (prepare), in sample order, which fixes the summation order.
//   set 0: dA^O_i   [d_e, d]:  left = H  [b][l][k*d_e] (columns s*d_e + e of the pair), right = d_out [b][l][d]
//   set 1: dA^I_i^T [d_e, d]:  left = dZ [b][l][k*d_e] (the same columns),              right = u     [b][l][d]
template <typename T> struct WgradProblem {
    const T *left[2], *right[2];
    const int32_t *expert_idx;
    float *partial;        // [sets*parts, M, N]
    int b, l, n, kact, range;   // range: tokens of an item
    WgradOrder<false, false> parts;   // b <= 128
    int M, N;              // rows and columns of one expert's gradient (d_e and d)

    static constexpr bool kF32Out = true;
    __device__ int rows(int) const { return M; }
    __device__ int ncols() const { return N; }
    __host__ __device__ int kseg(int) const { return range; }
    __device__ long a_stride(int) const { return (long)kact * M; }
    __device__ long b_stride() const { return N; }
    __device__ int kdim(int) const { return 0; }  // prepare() supplies K
    static constexpr bool kPrepare = true;
    // context of a segment: slot in bits 0-4, sample in bits 5-11, range above
    __device__ int decode(int g) const { return parts.decode(g); }
    __device__ int prepare(int &g, uint32_t *segtab, void *scratch, int tid, int) const
    {
        PartList &list = *static_cast<PartList *>(scratch);
        int expert, first, last;
        if (!list.fill(expert_idx, b, kact, n, parts, g, tid, expert, first, last)) return -1;
        if (tid < b && list.slot_of[tid] >= 0) {
            const int at = list.before(expert, tid) * parts.w.items - first;
            for (int r = 0; r < parts.w.items; ++r)
                if (at + r >= 0 && at + r < last - first) segtab[at + r] = ((uint32_t)r << 12) | ((uint32_t)tid << 5) | (uint32_t)list.slot_of[tid];
        }
        __syncthreads();
        return (last - first) * range;
    }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ size_t token(uint32_t ctx) const { return (size_t)(ctx >> 5 & 0x7Fu) * l + (size_t)(ctx >> 12) * range; }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t ctx) const
    {
        return (parts.set(g) == 0 ? left[0] : left[1]) + (token(ctx) * kact + (ctx & 0x1Fu)) * M + r;
    }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t ctx) const { return (parts.set(g) == 0 ? right[0] : right[1]) + token(ctx) * N + nn; }
    static constexpr bool kRowScale = false;
    static constexpr bool kColScale = false;
    __device__ float col_scale(int, int) const { return 1.0f; }
    __device__ float epi(float val, float) const { return val; }
    __device__ bool has_residual() const { return false; }
    __device__ uint4 res8(int, int, int) const { return make_uint4(0, 0, 0, 0); }
    __device__ void put8(int, int, int, uint4) const {}
    __device__ void put4_f32(int g, int r, int nn, float4 v) const
    {
        *reinterpret_cast<float4 *>(partial + (parts.tile(g) * M + r) * N + nn) = v;
    }
};

// Blocks with patch-wise data selection (SMHA; the data-selected UoME): for expert i,
//   dW[M, d] = sum over the units (b, slot s) of expert i and their c picks t of
//              L^T[unit][M columns][tokens of pick t]  x  R[b][tokens of the picked patch][d]
// i.e. the left factor is a per-unit tensor [unit][l_a][columns] (the set's M columns start at col0)
// and the right factor is a [b, l, d] tensor (x, u or the
// upstream gradient) whose rows are gathered patch by patch (Eq. 18), never copied.  K segments =
// (unit, pick) of l_p tokens, in (sample, pick) order.
//   SMHA, M = d_h:  sets 0-2: dW^{q,k,v}_i^T, left = [dq|dk|dv] [unit][l_a][3d_h] columns set*d_h.., right = x
//                   set 3:    dW^O_i,         left = gated o    [unit][l_a][d_h],                    right = d_out
//   UoME, M = d_e:  set 0: dA^O_i, left = H [unit][l_a][d_e], right = d_out;  set 1: dA^I_i^T, left = dZ, right = u
template <typename T> struct SmhaWgradProblem {
    const T *left[4], *right[4];
    int row_len[4], col0[4];    // elements of a row of left[set]; first column of the set's M
    const int32_t *expert_idx, *patch_idx;
    float *partial;             // [sets*parts, M, d]
    int b, l, d, n, kact, m, c, l_p, l_a;
    WgradOrder<false, true> parts;   // b <= 128
    int M;

    static constexpr bool kF32Out = true;
    __device__ int rows(int) const { return M; }
    __device__ int ncols() const { return d; }
    __host__ __device__ int kseg(int) const { return l_p; }
    __device__ long a_stride(int g) const { return row_len[parts.set(g)]; }
    __device__ long b_stride() const { return d; }
    __device__ int kdim(int) const { return 0; }
    static constexpr bool kPrepare = true;
    // context of a segment: sample in bits 0-6, slot in bits 7-11, pick in bits 12-21, patch in bits 22-31
    __device__ int decode(int g) const { return parts.decode(g); }
    __device__ int prepare(int &g, uint32_t *segtab, void *scratch, int tid, int nthreads) const
    {
        PartList &list = *static_cast<PartList *>(scratch);
        int expert, first, last;
        if (!list.fill(expert_idx, b, kact, n, parts, g, tid, expert, first, last)) return -1;
        // thread (sample bb, pick t): its position in the expert's list is (listed samples before bb) * c + t
        for (int idx = tid; idx < b * c; idx += nthreads) {
            const int bb = idx / c, t = idx - bb * c;
            if (list.slot_of[bb] < 0) continue;
            const int pos = list.before(expert, bb) * c + t;
            if (pos < first || pos >= last) continue;
            const int p = clampi(patch_idx[((size_t)bb * n + expert) * c + t], m);
            segtab[pos - first] = (uint32_t)bb | ((uint32_t)list.slot_of[bb] << 7) | ((uint32_t)t << 12) | ((uint32_t)p << 22);
        }
        __syncthreads();
        return (last - first) * l_p;
    }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t ctx) const
    {
        const int bb = (int)(ctx & 0x7Fu), s = (int)((ctx >> 7) & 0x1Fu), t = (int)((ctx >> 12) & 0x3FFu);
        const int set = parts.set(g);
        return left[set] + (((size_t)bb * kact + s) * l_a + (size_t)t * l_p) * row_len[set] + col0[set] + r;
    }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t ctx) const
    {
        const int bb = (int)(ctx & 0x7Fu), p = (int)(ctx >> 22);
        return right[parts.set(g)] + ((size_t)bb * l + (size_t)p * l_p) * d + nn;
    }
    static constexpr bool kRowScale = false;
    static constexpr bool kColScale = false;
    __device__ float col_scale(int, int) const { return 1.0f; }
    __device__ float epi(float val, float) const { return val; }
    __device__ bool has_residual() const { return false; }
    __device__ uint4 res8(int, int, int) const { return make_uint4(0, 0, 0, 0); }
    __device__ void put8(int, int, int, uint4) const {}
    __device__ void put4_f32(int g, int r, int nn, float4 v) const
    {
        *reinterpret_cast<float4 *>(partial + (parts.tile(g) * M + r) * d + nn) = v;
    }
};

}  // namespace uoe
