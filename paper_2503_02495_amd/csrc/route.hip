// Routing of one block (Sec. III-B): expert-selection router (Eq. 21-22) and patch-wise
// data-selection router (Eq. 13, 14, 17).
//
// Kernels:
//   route_expert_mfma : expert router, bf16.  Eq. 21 is a [b, l*d] x [l*d, n] product with a huge
//                       inner dimension: a workgroup owns a chunk of the flat l*d axis for up to
//                       64 samples and all experts, its waves stream x and W_E straight from
//                       global memory into v_mfma_f32_16x16x32_bf16 fragments (rows = samples,
//                       columns = experts).  Every byte of x and of W_E is requested once.
//   route_partial<E>  : expert router on the vector ALU (fp32 storage).  A workgroup owns (chunk
//                       of tokens, sample); each wave streams token rows of x and the matching rows
//                       of the n W_E slices and keeps n running dot products per lane (a W_E chunk
//                       is shared by the b samples through L2).
//   route_data_mfma   : data router, bf16.  t1 = x W_B for 16 tokens per wave as
//                       v_mfma_f32_16x16x32_bf16 (A fragments straight from global, W_B staged in
//                       LDS), then the tokens' rows of W_A fold t1, still in the accumulators, into a partial
//                       [n,m] logit tile as v_mfma_f32_16x16x4_f32.
//   route_partial<D>  : the same data router on the vector ALU (fp32 storage, or W_B too large
//                       for LDS next to the MFMA staging).
//   route_reduce      : sums the data router's per-chunk partials in a fixed order (deterministic).
//   route_select      : per (expert row, sample): + noise, softmax over experts (Eq. 14 / 21), then
//                       top-c per expert and top-k per sample by rank counting: rank(j) = #{j' :
//                       g_j' > g_j or (g_j' == g_j and j' < j)}; keep rank < c.  The output slot of
//                       a kept index is the number of kept lower indices, so the list comes out
//                       ascending with no sort and ties go to the lower index by construction.
#include "common.h"
#include "select.h"
#include <cstdlib>

namespace uoe {

// LDS row pitch in dwords for a [k][cols] bf16 tile read with the transposing LDS read: the four
// 64-byte row pieces a half-wave touches must fall into different banks (pitch % 64 dwords = 16 or 48)
__host__ __device__ constexpr int b_pitch16(int cols)
{
    int p = cols / 2;
    while ((p % 64) != 16 && (p % 64) != 48) p += 4;
    return p;
}

// Chunks of fewer than 16 tokens only where route_select still adds up the data router's partials
static int route_data_short(int l, int n, int m, int tc)
{
    while (tc < 16 && tc < l && (n * m > 512 || (long)n * m * ((l + tc - 1) / tc) > 16384)) tc = 2 * tc < l ? 2 * tc : l;
    return tc > 16 ? 16 : tc;
}

// Tokens per chunk of fp32 routers with fewer than 8192 tokens: 4, 8, 12 or 16.  16 leave compute units idle and a chunk is a chain of its own, but it has
// its fixed work too, some four tokens', and route_partial deals chunks to the XCDs whole, all samples' of one to the same.  Counted in tokens of the
// XCD with the most: the work, or the longest chain in three quarters of the workgroups that fit, whichever is more; whole rounds of the long
// workgroups of more than 16 experts.  Less than 16 only if that gains a tenth.  The data router takes the expert router's chunks unless its partial sums
// are many.  Forward, us, 16 tokens / all that are idle otherwise, from 4 on / these: 2 x 64 x 64 46.8 / 41.7 / 41.7; 8 x 512 x 512, 8 experts 147.1 / 143.7 /
// 143.7; 28 x 217 x 184, 14 experts 104.2 / 110.3 / 104.1; 61 x 72 x 280, 6 and 16 79.2 / 83.5 / 75.7; 15 x 288 x 360, 32 and 2 112.0 / 115.2 / 110.9;
// 1 x 2006 x 784, 12 (W_E 75 MB, more than 1024 tokens a sample: longer runs of it stream better) 112.3 / 125.7 / 111.4; 2 x 530 x 992, 12 119 / 102 / 101;
// 1 x 3913 x 576, 16 154 / 167 / 150.
static int route_short_tokens_per_chunk(int b, int l, int d, int n, int m)
{
    const int regs = n <= 4 ? 7 : (n <= 8 || (n > 16 && n <= 24) ? 5 : (n <= 12 || n > 16 ? 4 : 3));   // workgroups a compute unit's registers hold
    const int lds = m > 1 ? 160 * 1024 / (n * d * 4 + 2048) : regs;                                    // and its LDS, with W_B
    const long fit = 32L * (lds < regs ? lds : regs);
    const auto load = [&](int tc) { return (long)(((l + tc - 1) / tc + 7) / 8) * b; };
    const auto cost = [&](int tc) {
        const int tc_d = m > 1 ? route_data_short(l, n, m, tc) : 0, longest = tc_d > tc ? tc_d : tc;
        const long data = m > 1 ? load(tc_d) : 0, work = load(tc) * (tc + 4) + data * (tc_d + 4), chain = fit * 3 / 4 * (longest + 4);
        if (n > 16) return (load(tc) + data + fit - 1) / fit * (tc + 4);
        return work > chain ? work : chain;
    };
    int best = 16;
    for (int tc = n > 16 ? 8 : 12; tc >= 4; tc -= 4)
        if (cost(tc) < cost(best) && cost(tc) * 10 < cost(16) * 9 && (n <= 16 || tc > 4 || cost(tc) == tc + 4)) best = tc;
    return best;
}

int route_tokens_per_chunk(int b, int l, int d, int n, int m, bool bf16)
{
    // aim for >= ~512 workgroups but keep a chunk within [16, 64] tokens (longer chunks stream
    // better: measured 3.3 / 3.6 / 3.9 TB/s at 16 / 32 / 64 tokens on the largest shape)
    long tc = ((long)b * l) / 512;
    if (tc > l / 8) tc = l / 8;  // at least ~8 chunks per sample so the last, short chunk does not dominate
    tc = (tc / 4) * 4;
    if (tc < 16) tc = !bf16 && (long)b * l < 8192 && (n > 16 || l <= 1024 || (double)n * l * d * sizeof(float) <= 16e6) ? route_short_tokens_per_chunk(b, l, d, n, m) : 16;
    if (tc > 64) tc = 64;
    if (tc > l) tc = l;
    return (int)tc;
}

// Expert router, MFMA kernel: tokens per chunk.  The chunk count does not depend on b (a workgroup
// takes all samples of its chunk), so aim for ~512 chunks.
int route_expert_mfma_tokens_per_chunk(int b, int l, int d, int n)
{
    (void)b; (void)d; (void)n;  // ~512 chunks whatever the shape: measured best from `lm` to `large`
    const int tc = l / 512;
    return tc < 1 ? 1 : tc;
}

constexpr int DATA_TOKENS = 64;    // tokens the data router's MFMA kernel takes at a time,
constexpr int DATA_FOLD_TILES = 4; // and 16-patch tiles it folds them onto at a time
// Whether the data router's MFMA kernel applies: W_B, 64 tokens' t1 and the fold's partial sums side by side within 60 KiB (what
// the kernel holds at a time is less).
bool route_data_uses_mfma(int b, int l, int d, int n, bool bf16)
{
    (void)b; (void)l;
    const int np = (n + 15) & ~15;
    const size_t wb = (size_t)((d + 7) / 8) * (8 * np * 2 + (np == 16 ? 128 : 32));
    return bf16 && wb + (size_t)64 * np * sizeof(float) + 256 * 8 * sizeof(float) <= 60 * 1024;
}
// Plan of the streaming router kernel (route_stream_kernel): one workgroup per compute unit, each
// owning a contiguous run of whole tokens.
RouteStreamPlan route_stream_plan(int b, int l, int d, int n, bool bf16, bool has_d)
{
    RouteStreamPlan p{};
    if (!bf16 || d % 128 != 0) return p;   // every wave takes d/128 of the 32-element steps of each token
    p.rt = b > 32 ? 4 : (b > 16 ? 2 : 1);
    p.ct = n <= 16 ? 1 : 2;
    p.rb = p.rt == 1 ? 1024 : 512;
    const int bg = b < p.rt * 16 ? b : p.rt * 16;           // samples of one workgroup
    const int rows = bg + n, rpi = 1024 / p.rb;             // rows per stage; rows per load instruction
    p.ipw = ((rows + rpi - 1) / rpi + 3) / 4;
    p.tpc = (l + ROUTE_STREAM_CHUNKS - 1) / ROUTE_STREAM_CHUNKS;
    p.nchunks = (l + p.tpc - 1) / p.tpc;
    const int np = p.ct * 16;
    p.lds = (size_t)3 * p.ipw * 4 * 1024 + sizeof(float) * 4 * p.rt * 16 * (np + 1);
    if (has_d) p.lds += (size_t)(d / 8) * (8 * np * 2 + (np == 16 ? 128 : 32)) + (size_t)4 * p.tpc * bg * n * sizeof(float);
    p.ok = p.lds <= 150 * 1024 && p.ipw <= 16;
    return p;
}
// Token ranges of route_fold_mfma: whole 128-token blocks (32 per wave and step), at most 512 tokens,
// about 256 workgroups when the batch allows.  Up to 16 ranges per sample route_select adds the
// partial tiles up itself; beyond that route_reduce does.
RouteFoldPlan route_fold_plan(int b, int l)
{
    int want = 256 / b;
    want = want < 1 ? 1 : (want > 16 ? 16 : want);
    RouteFoldPlan p;
    p.tr = ((l + want - 1) / want + 127) / 128 * 128;
    if (p.tr > 512) p.tr = 512;   // 4 steps of 32 tokens per wave: every load of a wave is in flight at once
    p.ranges = (l + p.tr - 1) / p.tr;
    return p;
}

// Whether the streaming kernel is used when it applies: from about 100 MB of x and W_E.  Below that the
// register-staged kernels are as fast or faster (their workgroups are many and short, which suits
// inputs that a single round of 256 long-lived workgroups does not keep busy), measured per shape:
// 50 MB (b16 l4096 d256 n8) runs at 29-30 us either way, 335 MB (b4 l8192 d1024 n16) at 95 vs 113 us.
// UOE_ROUTE_STREAM_MIN_BYTES in the environment overrides the threshold (0: whenever the kernel applies).
bool route_stream_pays(int b, int l, int d, int n)
{
    const char *env = getenv("UOE_ROUTE_STREAM_MIN_BYTES");
    const double min_bytes = env ? atof(env) : 100e6;
    return ((double)b + n) * l * d * 2 >= min_bytes;
}
// Tokens per chunk of the data router: the MFMA kernel's workgroup, also the chunks of route_fold_kernel.  16 (the waves split the
// columns) up to 256 workgroups, where rows of x are long and the partial tiles, which route_select adds up, few for them: 64 workgroups of 64 keep a
// quarter of the compute units on x (both routers and the selection, us, with 16 and with 64: 8 x 512 x 512, 8 x 16 logits, 10.3 and 11.8; 1 x 912 x 512, 11 x 12,
// 12.7 and 13.2; 4 x 900 x 256, 6 x 30, 11.5 and 10.6; 4 x 1000 x 128, 8 x 20, 11.1 and 10.0).  Two times 64 where that saves route_reduce's launch, from
// 128 workgroups on (16 x 4096 x 256, 8 x 64 logits: 21.2 and 25.9; 5 x 4096 x 128, 8 x 64: 13.0 and 13.6); otherwise it gains nothing (60 x 1000 x 128 16.8 and
// 16.7, 64 x 1024 x 256 24.5 and 24.4) or loses (32 x 1024 x 512 20.5 and 18.9).
int route_data_tokens_per_chunk(int b, int l, int d, int n, int m, bool bf16)
{
    if (route_data_uses_mfma(b, l, d, n, bf16)) {
        const long tokens = (long)b * l;
        const long sums = (long)n * m * ((l + 15) / 16);
        if (tokens <= 4096 && n * m <= 512 && d >= 192 && sums <= 24L * d && sums <= 16384) return DATA_TOKENS / 4;
        const auto selected = [&](int tc) { return n * m <= 512 && (long)n * m * ((l + tc - 1) / tc) <= 16384; };   // (route_select adds them up)
        return tokens > 16 * 1024 && m <= DATA_FOLD_TILES * 16 && !selected(DATA_TOKENS) && selected(2 * DATA_TOKENS) ? 2 * DATA_TOKENS : DATA_TOKENS;
    }
    if (route_stream_plan(b, l, d, n, bf16, true).ok) return 64;
    const int tc = route_tokens_per_chunk(b, l, d, n, m, bf16);
    return tc < 16 ? route_data_short(l, n, m, tc) : tc;
}

constexpr int ROUTE_THREADS = 256;
constexpr int ROUTE_WAVES = ROUTE_THREADS / 64;

template <typename T, int NMAX, bool HAS_E, bool HAS_D>
__device__ __forceinline__ void route_partial(const RouteArgs &a, unsigned char *smem, const int lin)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Workgroup order: the b samples of one chunk are neighbours in time and sit on the same XCD
    // (workgroup ids are dealt round-robin over the 8 XCDs), so a chunk of W_E is fetched from HBM
    // once and found in that XCD's L2 by the other samples.
    const int tc = HAS_D ? a.tc_d : a.tc, nchunks = HAS_D ? a.nchunks_d : a.nchunks;
    const int chunk = ((lin >> 3) / a.b) * 8 + (lin & 7), bb = (lin >> 3) % a.b;
    if (chunk >= nchunks) return;
    const int n = a.n, d = a.d, l = a.l, m = a.m;
    const int t0 = chunk * tc;
    const int tcur = min(tc, l - t0);

    // LDS carve-up: W_B transposed [n][d] (storage type), t1 [tc][NMAX], zred [waves][NMAX]
    T *wb_t = reinterpret_cast<T *>(smem);
    size_t off = HAS_D ? (((size_t)n * d * sizeof(T) + 15) & ~(size_t)15) : 0;
    float *t1s = reinterpret_cast<float *>(smem + off);
    float *zsh = t1s + (HAS_D ? tc * NMAX : 0);

    const T *x = static_cast<const T *>(a.x);
    const T *w_e = static_cast<const T *>(a.w_e);
    if (HAS_D) {
        const T *w_b = static_cast<const T *>(a.w_b);
        for (int idx0 = tid; idx0 < n * d; idx0 += 8 * ROUTE_THREADS) {
            T v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = w_b[min(idx0 + q * ROUTE_THREADS, n * d - 1)];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int idx = idx0 + q * ROUTE_THREADS, e = idx / n, i = idx - e * n;  // W_B is [d, n]
                if (idx < n * d) wb_t[i * d + e] = v[q];
            }
        }
        __syncthreads();
    }

    float zacc[NMAX];
#pragma unroll
    for (int i = 0; i < NMAX; ++i) zacc[i] = 0.f;

    // Rows i >= n of the unrolled NMAX loops re-read row n-1 and accumulate into slots that are
    // never written out: the hot loop has no branches, so all NMAX+1 loads of an iteration are in
    // flight together.
    const size_t ld = (size_t)l * d;
    size_t wrow[NMAX];
#pragma unroll
    for (int i = 0; i < NMAX; ++i) wrow[i] = (size_t)min(i, n - 1) * ld;
    for (int tl = wave; tl < tcur; tl += ROUTE_WAVES) {
        const int t = t0 + tl;
        const T *xr = x + ((size_t)bb * l + t) * d;
        float tacc[NMAX];
#pragma unroll
        for (int i = 0; i < NMAX; ++i) tacc[i] = 0.f;
        for (int e = lane * 8; e < d; e += 64 * 8) {
            float xv[8];
            load8(xr + e, xv);
            if (HAS_E) {
                const T *wp = w_e + (size_t)t * d + e;
                float wv[NMAX][8];
#pragma unroll
                for (int i = 0; i < NMAX; ++i) load8(wp + wrow[i], wv[i]);
#pragma unroll
                for (int i = 0; i < NMAX; ++i)
#pragma unroll
                    for (int q = 0; q < 8; ++q) zacc[i] = fmaf(xv[q], wv[i][q], zacc[i]);
            }
            if (HAS_D) {
#pragma unroll
                for (int i = 0; i < NMAX; ++i) {
                    float wv[8];
                    load8(wb_t + min(i, n - 1) * d + e, wv);
#pragma unroll
                    for (int q = 0; q < 8; ++q) tacc[i] = fmaf(xv[q], wv[q], tacc[i]);
                }
            }
        }
        if (HAS_D) {
#pragma unroll
            for (int i = 0; i < NMAX; ++i) {
                const float s = wave_sum(tacc[i]);
                if (lane == 0) t1s[tl * NMAX + i] = s;
            }
        }
    }
    if (HAS_E) {
#pragma unroll
        for (int i = 0; i < NMAX; ++i) {
            const float s = wave_sum(zacc[i]);
            if (lane == 0) zsh[wave * NMAX + i] = s;
        }
    }
    __syncthreads();
    if (HAS_E && tid < n) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < ROUTE_WAVES; ++w) s += zsh[w * NMAX + tid];
        a.zpart[zpart_at(a, chunk, bb, tid)] = s;
    }
    if (HAS_D) {
        const T *w_a = static_cast<const T *>(a.w_a);
        const int nm = n * m;
        for (int o = tid; o < nm; o += ROUTE_THREADS) {
            const int i = o / m, j = o - i * m;
            float s = 0.f;
            for (int tl0 = 0; tl0 < tcur; tl0 += 8) {
                T v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = w_a[(size_t)(t0 + min(tl0 + q, tcur - 1)) * m + j];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (tl0 + q < tcur) s = fmaf(t1s[(tl0 + q) * NMAX + i], to_f32(v[q]), s);
            }
            a.gpart[((size_t)chunk * a.b + bb) * nm + o] = s;
        }
    }
}

// blocks below data_blocks: the data router (the longer chains); the others: the expert router.  Either part may be empty.
template <typename T, int NMAX> __global__ __launch_bounds__(ROUTE_THREADS) void route_partial_kernel(RouteArgs a, int data_blocks)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int id = blockIdx.x;
    if (id < data_blocks) route_partial<T, NMAX, false, true>(a, smem, id);
    else route_partial<T, NMAX, true, false>(a, smem, id - data_blocks);
}

typedef __bf16 rt_bf16x8 __attribute__((ext_vector_type(8)));
typedef float rt_f32x4 __attribute__((ext_vector_type(4)));

typedef short rt_s16x4 __attribute__((ext_vector_type(4)));
typedef rt_s16x4 __attribute__((address_space(3))) * rt_lds_s16x4_ptr;

// Second half of the data router (Eq. 13) behind the streaming kernel, any m: fold per-token expert scores with the chunk's rows of W_A,
// g[i][j] = sum_t t1[t][i] * W_A[t][j], for the tcur tokens of the chunk, into sample bb's
// partial logit tile gpart[chunk][bb][n*m].  t1s: LDS, [token][np] fp32.  A thread owns
// (token group tg, output group og): one expert i and VEC consecutive patches, for the tokens
// tg, tg + TG, ...; the TG partial sums of an output are then added in group order.  (With few
// outputs per sample, one thread per output would leave most of the workgroup idle behind a
// serial walk over all the chunk's tokens.)  part: LDS scratch of NTHREADS * 8 floats.
// w_a: LDS copy of the chunk's rows.
template <int NTHREADS>
__device__ __forceinline__ void route_fold(const RouteArgs &a, int chunk, int bb, int tcur, const float *t1s, int np,
                                           float *part, const uint16_t *w_a)
{
    const int tid = threadIdx.x;
    const int n = a.n, m = a.m;
    const int nm = n * m;
    float *gout = a.gpart + ((size_t)chunk * a.b + bb) * nm;
    const int vec = (m & 7) == 0 ? 8 : 1, mv = m / vec, og_n = n * mv;
    const int tg_n = og_n >= NTHREADS ? 1 : NTHREADS / og_n;
    auto fold = [&](int og, int tl0, int tstep, float *dst) {
        const int i = og / mv, j0 = (og - i * mv) * vec;
        float sacc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) sacc[q] = 0.f;
        if (vec == 8) {
#pragma unroll 4
            for (int tl = tl0; tl < tcur; tl += tstep) {
                float wv[8];
                load8(reinterpret_cast<const bf16_t *>(w_a) + (size_t)tl * m + j0, wv);
                const float t1 = t1s[tl * np + i];
#pragma unroll
                for (int q = 0; q < 8; ++q) sacc[q] = fmaf(t1, wv[q], sacc[q]);
            }
        } else {
#pragma unroll 4
            for (int tl = tl0; tl < tcur; tl += tstep)
                sacc[0] = fmaf(t1s[tl * np + i], __uint_as_float((uint32_t)w_a[(size_t)tl * m + j0] << 16), sacc[0]);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (q < vec) dst[i * m + j0 + q] = sacc[q];
    };
    if (tg_n > 1) {
        const int og = tid % og_n, tg = tid / og_n;
        if (tg < tg_n) fold(og, tg, tg_n, part + (size_t)tg * nm);
        __syncthreads();
        for (int o = tid; o < nm; o += NTHREADS) {
            float t = 0.f;
            for (int q = 0; q < tg_n; ++q) t += part[(size_t)q * nm + o];
            gout[o] = t;
        }
    } else {
        for (int og = tid; og < og_n; og += NTHREADS) fold(og, 0, 1, gout);
    }
}

// W_B [d, n] copied to LDS as it is: rows of NP = 16 or 32 columns (columns >= n are left as they are:
// they only feed output columns that are never read), in blocks of 8 rows with a pad after each block
// (128 bytes for 32-byte rows, 32 bytes for 64-byte rows) so that the row groups of the four k-slices
// of a transposing read fall into different banks.  Row e starts at (e/8)*BLK + (e%8)*ROWB.
template <int NP, int NTHREADS>
__device__ __forceinline__ void stage_w_b(const RouteArgs &a, unsigned char *wb)
{
    constexpr int ROWB = NP * 2, BLK = 8 * ROWB + (NP == 16 ? 128 : 32);
    const int tid = threadIdx.x, n = a.n, d = a.d;
    const uint16_t *w_b = static_cast<const uint16_t *>(a.w_b);
    // the widest piece that never straddles a row; several of them a thread in flight together (a loop's remainder, one at a time, waits
    // out a memory round trip each)
    auto stage = [&](auto piece, int pr) __attribute__((always_inline)) {   // pr pieces a row
        typedef decltype(piece) P;
        constexpr int BATCH = sizeof(P) == 16 ? 4 : 8;
        const int pieces = d * pr;
        // piece / pr by the reciprocal rounded up: exact below 2^16 pieces (d * n <= 24576)
        const uint32_t inv = pr > 1 ? 0xFFFFFFFFu / (uint32_t)pr + 1u : 0u;
        for (int i0 = tid; i0 < pieces; i0 += BATCH * NTHREADS) {
            P v[BATCH];
#pragma unroll
            for (int q = 0; q < BATCH; ++q) v[q] = reinterpret_cast<const P *>(w_b)[min(i0 + q * NTHREADS, pieces - 1)];
#pragma unroll
            for (int q = 0; q < BATCH; ++q) {
                const int idx = i0 + q * NTHREADS, e = pr > 1 ? (int)__umulhi((uint32_t)idx, inv) : idx;
                if (idx < pieces) *reinterpret_cast<P *>(wb + (e >> 3) * BLK + (e & 7) * ROWB + (idx - e * pr) * (int)sizeof(P)) = v[q];
            }
        }
    };
    if ((n & 7) == 0) stage(once_u32x4{}, n >> 3);
    else if ((n & 1) == 0) stage(uint32_t{}, n >> 1);
    else stage(uint16_t{}, n);
}

// The same for the streaming kernel, once in a long workgroup and behind its first transfers to LDS, where batches gain nothing.  Two other forms
// of these loops, a few instructions shorter, cost that kernel 2 % (4 x 8192 x 1024, n 16, m 128: 94.3 us for the whole routing, 96.2;
// 8 x 8192 x 512 49.5 and 50.3): its main loop has the same instructions then, but lies otherwise across the lines of the instruction cache.
template <int NP, int NTHREADS>
__device__ __forceinline__ void stage_w_b_loop(const RouteArgs &a, unsigned char *wb)
{
    constexpr int ROWB = NP * 2, BLK = 8 * ROWB + (NP == 16 ? 128 : 32);
    const int tid = threadIdx.x, n = a.n, d = a.d;
    const uint16_t *w_b = static_cast<const uint16_t *>(a.w_b);
    auto row_at = [&](int e) { return wb + (size_t)(e >> 3) * BLK + (e & 7) * ROWB; };
    if ((n & 7) == 0) {  // 16-byte pieces never straddle a row
        const int pr = n >> 3;
#pragma unroll 4
        for (int idx = tid; idx < d * pr; idx += NTHREADS) {
            const int e = idx / pr, pc = idx - e * pr;
            *reinterpret_cast<uint4 *>(row_at(e) + pc * 16) = *reinterpret_cast<const uint4 *>(w_b + (size_t)idx * 8);
        }
    } else if ((n & 1) == 0) {
        const int pr = n >> 1;
#pragma unroll 4
        for (int idx = tid; idx < d * pr; idx += NTHREADS) {
            const int e = idx / pr, pc = idx - e * pr;
            *reinterpret_cast<uint32_t *>(row_at(e) + pc * 4) = *reinterpret_cast<const uint32_t *>(w_b + (size_t)idx * 2);
        }
    } else {
#pragma unroll 4
        for (int idx = tid; idx < d * n; idx += NTHREADS) {
            const int e = idx / n, i = idx - e * n;
            *reinterpret_cast<uint16_t *>(row_at(e) + i * 2) = w_b[idx];
        }
    }
}

// Data router (Eq. 13), bf16, MFMA.  Workgroup = four waves = a.tc_d tokens of one sample, 64 at a time (16 per wave), or KS = 4: 16
// tokens, of which each wave takes a quarter of the columns.
// MFMA 16x16x32 operand layout: lane = (row r = lane%16, k-slice 8*(lane/16)); accumulator register q
// of a lane is output row 4*(lane/16)+q, column lane%16.
// t1 = x W_B: rows = tokens, columns = experts.  W_B [d, n] is copied to LDS as it is (rows of np = 16 or 32 columns; columns >= n are
// left as they are: they only feed output columns that are never read) and the B fragments (8 consecutive k
// of one expert column) are taken with the transposing LDS read: in a group of 16 lanes, lane j
// points at row k0 + j/4, columns 4*(j%4)..+3, and lane i receives column i, rows k0..k0+3.  Rows are
// stored in blocks of 8 with a pad after each block (128 bytes for 32-byte rows, 32 bytes for
// 64-byte rows) so that the row groups of the four k-slices fall into different banks.
// The fold g = t1^T W_A takes t1 where it is: register j of a lane is token 4*(lane/16)+j of expert lane%16, which is the A operand of
// v_mfma_f32_16x16x4_f32 for the four tokens j, 4+j, 8+j, 12+j, so that four of them, exact fp32 products, fold 16 tokens onto 16
// patches; their W_A values are one 2-byte load each, for any m.  The waves' tiles are added in wave order.
// What bounds it is the chain of dependent steps, on 64 to 512 workgroups: a memory round trip costs 2 us at the start of a launch, so
// 256 columns of x, W_B and the first 64 columns of W_A are in flight together, and the k-steps' fragments are read four steps ahead of their products.
// (512 columns take 142 registers, three waves a SIMD instead of four, also for the expert router's workgroups of the same launch: 13 x 2048 x 384,
// n 12, 20.2 us for both routers and the selection against 17.5, 32 x 1024 x 512 20.1 and 18.9; they gain 0.3 of 13 us on 12 x 1024 x 512.)
// Both routers' launch, us, against W_A fetched for a fold on the vector ALU behind the products and one set of 128 columns in flight:
// 8 x 512 x 512, n 8, m 16: 10.2 -> 6.5; 6 x 1000 x 360, n 6, m 25: 12.2 -> 6.7; 128 x 196 x 384, n 6, m 14: 13.7 -> 11.3.
// LDS: W_B, and in its place at the end the four waves' tiles of n x 64 sums
static size_t data_lds(int n, int d)
{
    const int np = (n + 15) & ~15;
    const size_t wb = (size_t)((d + 7) / 8) * (8 * np * 2 + (np == 16 ? 128 : 32));
    const size_t sums = (size_t)4 * np * (DATA_FOLD_TILES * 16 + 4) * sizeof(float);
    return wb > sums ? wb : sums;
}

template <int NTILE, int KS>
__device__ __forceinline__ void route_data_mfma_body(const RouteArgs &a, int chunk, int bb, unsigned char *smem)
{
    constexpr int NP = NTILE * 16, ROWB = NP * 2, BLK = 8 * ROWB + (NP == 16 ? 128 : 32);
    constexpr int UN = 4, SPAN = UN * 32, UB = 4;           // k-steps of one register set (two sets are in flight); fragments read ahead
    constexpr int TOK = DATA_TOKENS / KS;                   // tokens at a time
    constexpr int FT = DATA_FOLD_TILES, RP = FT * 16 + 4;   // row pitch of the sums in LDS
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int d = a.d, l = a.l, n = a.n, m = a.m, nm = n * m;
    unsigned char *wb = smem;
    float *sums = reinterpret_cast<float *>(smem);               // [wave][NP][RP], once W_B is done with
    const int begin = chunk * a.tc_d, end = min(l, begin + a.tc_d);
    // this wave's columns of x and the first of its 16 tokens
    const int kq = KS == 1 ? d : ((d + 31) / 32 + KS - 1) / KS * 32, kb = KS == 1 ? 0 : min(wave * kq, d), ke = min(d, kb + kq);
    const int tw = KS == 1 ? wave * 16 : 0;
    const int reps = (end - begin + TOK - 1) / TOK, spans = (kq + SPAN - 1) / SPAN, sets = reps * spans;
    const int tiles = (m + 15) / 16;                             // reps > 1 only with at most FT of them

    const int r = lane & 15, q4 = lane >> 4, ksl = q4 * 8;
    const uint16_t *xb = static_cast<const uint16_t *>(a.x) + (size_t)bb * l * d;
    struct Set {
        uint4 v[UN];
    } set0, set1;
    int lrep = 0, lspan = 0;   // the set to load next
    auto load_set = [&](Set &t) __attribute__((always_inline)) {
        const int trow = min(begin + lrep * TOK + tw + r, l - 1);  // rows past the end repeat the last token; never used
        const uint16_t *xr = xb + (size_t)trow * d;
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int kk = kb + lspan * SPAN + u * 32 + ksl;
            t.v[u] = *reinterpret_cast<const uint4 *>(xr + (kk < ke ? kk : 0));   // slices past the wave's: any piece, zeroed below
        }
        if (++lspan == spans) {
            lspan = 0;
            ++lrep;
        }
    };
    // W_A of this lane's tokens 4 q4 + j and patch tile * 16 + r (past m or the tokens: any value, never used)
    uint16_t wa[FT][4] = {};
    auto load_wa = [&](int rep, int tile0) __attribute__((always_inline)) {
        const int t0 = begin + rep * TOK + tw + q4 * 4;
#pragma unroll
        for (int t = 0; t < FT; ++t) {
            if (tile0 + t >= tiles) break;   // uniform
#pragma unroll
            for (int j = 0; j < 4; ++j)
                wa[t][j] = static_cast<const uint16_t *>(a.w_a)[(size_t)min(t0 + j, l - 1) * m + min((tile0 + t) * 16 + r, m - 1)];
        }
    };
    load_set(set0);
    if (sets > 1) load_set(set1);
    load_wa(0, 0);
    stage_w_b<NP, ROUTE_THREADS>(a, wb);
    __syncthreads();

    rt_f32x4 acc[NTILE], g[NTILE][FT];
#pragma unroll
    for (int c = 0; c < NTILE; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc[c][q] = 0.f;
#pragma unroll
            for (int t = 0; t < FT; ++t) g[c][t][q] = 0.f;
        }
    // transposing-read lane roles: k-slice group lane/16, row (lane%16)/4 of the group's 4, 4 columns
    const int tr_row = ksl + ((lane & 15) >> 2), tr_col = (lane & 3) * 4;
    auto fragment = [&](int row, int c) __attribute__((always_inline)) -> rt_bf16x8 {   // rows row..+3 and row+4..+7: one block of 8
        const unsigned char *src = wb + (row >> 3) * BLK + (row & 7) * ROWB + (c * 16 + tr_col) * 2;
        const rt_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rt_lds_s16x4_ptr)(src));
        const rt_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rt_lds_s16x4_ptr)(src + 4 * ROWB));
        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
        return __builtin_bit_cast(rt_bf16x8, make_uint4(l2.x, l2.y, h2.x, h2.y));
    };
    auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < FT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float w = __uint_as_float((uint32_t)wa[t][j] << 16);
#pragma unroll
                for (int c = 0; c < NTILE; ++c) g[c][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(acc[c][j], w, g[c][t], 0, 0, 0);
            }
    };
    int rep = 0, span = 0;   // of the set to multiply next
    auto use_set = [&](Set &t, bool next) __attribute__((always_inline)) {   // next: a set to load into these registers
        const int k0 = kb + span * SPAN;
#pragma unroll
        for (int u0 = 0; u0 < UN; u0 += UB) {
            if (k0 + u0 * 32 >= ke) break;   // uniform
            rt_bf16x8 f[UB][NTILE];
#pragma unroll
            for (int u = 0; u < UB; ++u)
#pragma unroll
                for (int c = 0; c < NTILE; ++c)   // slices past the wave's: W_B at a valid row, so that the product with zero stays zero
                    f[u][c] = fragment(min(k0 + (u0 + u) * 32 + tr_row, d - 8 + ((lane & 15) >> 2)), c);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                if (k0 + (u0 + u) * 32 >= ke) break;   // uniform
                const uint4 xv = k0 + (u0 + u) * 32 + ksl < ke ? t.v[u0 + u] : make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int c = 0; c < NTILE; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(rt_bf16x8, xv), f[u][c], acc[c], 0, 0, 0);
            }
        }
        if (next) load_set(t);
        if (++span < spans) return;
        span = 0;
        const int left = end - begin - rep * TOK - tw - q4 * 4;   // of this lane's four tokens
#pragma unroll
        for (int c = 0; c < NTILE; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[c][j] = j < left ? acc[c][j] : 0.f;
        if (++rep < reps) {
            fold();
            load_wa(rep, 0);
#pragma unroll
            for (int c = 0; c < NTILE; ++c)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[c][j] = 0.f;
        }
    };
    for (int s = 0; s < sets; s += 2) {
        use_set(set0, s + 2 < sets);
        if (s + 1 < sets) use_set(set1, s + 3 < sets);
    }
    // the last tokens' fold, tile group by tile group
    float *gout = a.gpart + ((size_t)chunk * a.b + bb) * nm;
    for (int tile0 = 0; tile0 < tiles; tile0 += FT) {
        if (tile0) {
            load_wa(reps - 1, tile0);
#pragma unroll
            for (int c = 0; c < NTILE; ++c)
#pragma unroll
                for (int t = 0; t < FT; ++t)
#pragma unroll
                    for (int q = 0; q < 4; ++q) g[c][t][q] = 0.f;
        }
        fold();
        __syncthreads();   // W_B, or the sums of the group before, are done with
#pragma unroll
        for (int c = 0; c < NTILE; ++c)
#pragma unroll
            for (int t = 0; t < FT; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) sums[(wave * NP + c * 16 + q4 * 4 + q) * RP + t * 16 + r] = g[c][t][q];
        __syncthreads();
        const int cols = min(FT * 16, m - tile0 * 16);
        for (int o = tid; o < n * FT * 16; o += ROUTE_THREADS) {
            const int i = o / (FT * 16), j = o % (FT * 16);
            const float *at = sums + i * RP + j;
            if (j < cols) gout[i * m + tile0 * 16 + j] = (at[0] + at[NP * RP]) + (at[2 * NP * RP] + at[3 * NP * RP]);
        }
    }
}

template <int NTILE, int KS>
__global__ __launch_bounds__(ROUTE_THREADS, NTILE == 1 ? 4 : 2) void route_data_mfma_kernel(RouteArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    route_data_mfma_body<NTILE, KS>(a, blockIdx.x, blockIdx.y, smem);
}

// Expert router (Eq. 21), bf16, MFMA.  Workgroup = 4 waves = (chunk of a.tc tokens, i.e. a.tc*d
// consecutive elements of the flat l*d axis; group of RT*16 samples).  The chunk is cut into steps of
// 32 elements; wave w takes a contiguous quarter of the steps.  In one step lane (r = lane%16,
// q = lane/16) loads elements [32*step + 8*q, +8) of sample row r (one A fragment per 16 samples)
// and of expert row r (one B fragment per 16 experts); rows past b or n repeat the last valid row
// (they only produce output rows / columns that are never stored).  The last step of a chunk may
// be partial (multiples of 8 elements): its missing slices are zeroed.  Accumulator register v of
// a lane is Z[sample 4*q + v][expert r].  The four waves' tiles are summed in wave order.
template <int RT, int CT> constexpr size_t route_expert_mfma_lds() { return sizeof(float) * 4 * RT * 16 * (CT * 16 + 1); }

template <int RT, int CT>
__device__ __forceinline__ void route_expert_mfma_body(const RouteArgs &a, int chunk, int b0, unsigned char *smem)
{
    float(*zsh)[RT * 16][CT * 16 + 1] = reinterpret_cast<float(*)[RT * 16][CT * 16 + 1]>(smem);  // [4 waves]
    constexpr int U = RT == 4 ? 2 : 4;  // steps whose loads are in flight together (four: no third wave a SIMD beside 64 samples' rows)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int b = a.b, n = a.n;
    const long ld = (long)a.l * a.d;
    const long c0 = (long)chunk * a.tc * a.d;
    const long c1 = min(ld, c0 + (long)a.tc * a.d);
    const int steps = (int)((c1 - c0 + 31) / 32);
    const int per = (steps + 3) / 4;
    const int s0 = wave * per, s1 = min(steps, s0 + per);

    const uint16_t *xp[RT], *wp[CT];
#pragma unroll
    for (int t = 0; t < RT; ++t) xp[t] = static_cast<const uint16_t *>(a.x) + (size_t)min(b0 + t * 16 + r, b - 1) * ld;
#pragma unroll
    for (int t = 0; t < CT; ++t) wp[t] = static_cast<const uint16_t *>(a.w_e) + (size_t)min(t * 16 + r, n - 1) * ld;
    rt_f32x4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int u = 0; u < CT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[t][u][v] = 0.f;

    // Two register sets: the loads of the next U steps are issued before the MFMAs of the current
    // ones, so a wave always has loads in flight (the kernel is a pure stream: bytes in flight are
    // its throughput).
    uint4 xa[2][U][RT], wb[2][U][CT];
    auto load_steps = [&](int s, int set) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long e = c0 + (long)(s + u) * 32 + q * 8;
            const bool ok = s + u < s1 && e < c1;
            const long ec = ok ? e : c0;  // any valid address
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                xa[set][u][t] = *reinterpret_cast<const uint4 *>(xp[t] + ec);
                if (!ok) xa[set][u][t] = make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < CT; ++t) wb[set][u][t] = *reinterpret_cast<const uint4 *>(wp[t] + ec);
        }
    };
    auto mfma_steps = [&](int set) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int v = 0; v < CT; ++v)
                    acc[t][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(rt_bf16x8, xa[set][u][t]),
                                                                        __builtin_bit_cast(rt_bf16x8, wb[set][u][v]), acc[t][v], 0, 0, 0);
    };
    if (s0 < s1) load_steps(s0, 0);
    for (int s = s0; s < s1; s += 2 * U) {
        if (s + U < s1) load_steps(s + U, 1);
        mfma_steps(0);
        if (s + U < s1) {
            if (s + 2 * U < s1) load_steps(s + 2 * U, 0);
            mfma_steps(1);
        }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int u = 0; u < CT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) zsh[wave][t * 16 + q * 4 + v][u * 16 + r] = acc[t][u][v];
    __syncthreads();
    for (int o = tid; o < RT * 16 * CT * 16; o += 256) {
        const int row = o / (CT * 16), col = o - row * (CT * 16);
        if (b0 + row < b && col < n)
            a.zpart[zpart_at(a, chunk, b0 + row, col)] = (zsh[0][row][col] + zsh[1][row][col]) + (zsh[2][row][col] + zsh[3][row][col]);
    }
}

// Workgroups are dealt round the eight XCDs: consecutive chunks go to the workgroups of one, whose L2 then completes the 128-byte lines
// that 32 chunks' partials of one (sample, expert) share; with the chunk as the block index a line is written from eight L2s.
__device__ __forceinline__ int chunk_of(int id, int nchunks)
{
    const int x = id & 7;
    return x * (nchunks / 8) + min(x, nchunks % 8) + (id >> 3);
}

template <int RT, int CT>
__global__ __launch_bounds__(256) void route_expert_mfma_kernel(RouteArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    route_expert_mfma_body<RT, CT>(a, chunk_of(blockIdx.x, a.nchunks), blockIdx.y * RT * 16, smem);
}

// Both routers of a block in one launch (they are independent and both stream x): workgroups
// [0, n_data) run the data router with four waves (chunk = id % nchunks_d, sample = id / nchunks_d) -
// first, because each is a longer chain of dependent steps - and the rest the expert router
// (chunk = id' % nchunks, sample group = id' / nchunks).
template <int RT, int CT, int KS>
__global__ __launch_bounds__(256, CT == 1 ? 4 : 2) void route_expert_data_kernel(RouteArgs a, int n_data)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int id = blockIdx.x;
    if (id < n_data) {
        route_data_mfma_body<CT, KS>(a, id % a.nchunks_d, id / a.nchunks_d, smem);
    } else {
        const int f = id - n_data;
        route_expert_mfma_body<RT, CT>(a, chunk_of(f % a.nchunks, a.nchunks), (f / a.nchunks) * RT * 16, smem);
    }
}

// ---------------------------------------------------------------------------------------------
// Streaming router kernel (bf16, d % 128 == 0): the expert router (Eq. 21) and, optionally, the first
// map of the data router (Eq. 13, t1 = x W_B) in one pass over x.
//
// Eq. 21 is a [b, l*d] x [l*d, n] product with a huge inner dimension and almost no arithmetic: what
// counts is how the bytes are requested.  One workgroup per compute unit owns a contiguous run of
// whole tokens (chunk) for up to RT*16 samples and all experts.  The chunk moves through LDS in
// stages of RB bytes per row (rows = the samples' rows of x, then the experts' rows of W_E), fetched
// by global_load_lds (16 bytes per lane, 1 KiB of consecutive LDS per instruction: whole 0.5-1 KiB
// runs of one row per request, no registers held by loads in flight), three stages deep.  Measured
// against register-staged fragment loads of 64 bytes per row the same stream runs 20 % faster.
// Within a row the 16-byte chunks are permuted (slot = chunk ^ (row & 15), applied on the global
// side where every lane supplies its own address) so that the fragment reads of 16 rows hit 64
// distinct banks.
// MFMA v_mfma_f32_16x16x32_bf16, rows = samples, columns = experts.  A stage holds RB/64 steps of 32
// elements; wave w takes steps w, w+4, ....  For the data router the same x fragment is multiplied a
// second time, with the matching W_B fragment (transposing LDS read of a copy of W_B, as in
// route_data_mfma): since d % 128 == 0 every wave owns d/128 steps of every token, so each wave
// carries one partial row of t1 per token, parks it in LDS when the token ends, and after the stream
// the four partial rows are added in wave order and go to t1 [b][l][n] (fp32) for route_fold_kernel.  Nothing but the stage loads touches vector memory
// inside the loop, whose completion is tracked by hand (s_waitcnt vmcnt) as in the GEMM engine.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void rs_dma16(const void *gptr, uint32_t lds_byte)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_byte), "v"(gptr) : "memory", "m0");
}
// The same with the non-temporal hint, for the rows of W_E: they are read once per call and are larger
// than the memory-side cache, where they would push out x, u and the hidden activations that the
// kernels after the router read again.
__device__ __forceinline__ void rs_dma16_once(const void *gptr, uint32_t lds_byte)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds_byte), "v"(gptr) : "memory", "m0");
}
#pragma clang diagnostic pop
// wait until at most n (0..16) of this wave's vector-memory operations are outstanding
__device__ __forceinline__ void rs_wait(int n)
{
#define UOE_W(N) case N: asm volatile("s_waitcnt vmcnt(" #N ")" ::: "memory"); break;
    switch (n) {
        UOE_W(1) UOE_W(2) UOE_W(3) UOE_W(4) UOE_W(5) UOE_W(6) UOE_W(7) UOE_W(8) UOE_W(9) UOE_W(10) UOE_W(11) UOE_W(12)
        UOE_W(13) UOE_W(14) UOE_W(15) UOE_W(16)
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
#undef UOE_W
}

template <int RT, int CT, int RB, bool HAS_D>
__global__ __launch_bounds__(256) void route_stream_kernel(RouteArgs a, int ipw, int once)
{
    constexpr int STAGES = 3, SE = RB / 2, SPS = SE / 32, LPR = RB / 16, RPI = 64 / LPR;
    constexpr int NP = CT * 16, ROWB = NP * 2, BLK = 8 * ROWB + (NP == 16 ? 128 : 32);
    extern __shared__ __align__(1024) unsigned char smem[];
    const int chunk = blockIdx.x, b0 = blockIdx.y * RT * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q4 = lane >> 4;
    const int b = a.b, n = a.n, d = a.d, l = a.l;
    const long ld = (long)l * d;
    const int bg = min(RT * 16, b - b0), rows = bg + n;
    const int t0 = chunk * a.tc, tcur = min(a.tc, l - t0);
    const long c0 = (long)t0 * d;
    const int spt = d / 32;                       // steps per token
    const int gsteps = tcur * spt;                // steps of this chunk
    const int nst = (gsteps + SPS - 1) / SPS;
    const int SB = ipw * 4 * 1024;                // bytes of one stage buffer

    unsigned char *stage0 = smem;
    float(*zsh)[RT * 16][NP + 1] = reinterpret_cast<float(*)[RT * 16][NP + 1]>(smem + (size_t)STAGES * SB);
    unsigned char *wb = reinterpret_cast<unsigned char *>(&zsh[4][0][0]);
    float *t1w = reinterpret_cast<float *>(wb + (size_t)(d / 8) * BLK);   // [4 waves][tc][bg][n]
    auto row_at = [&](int e) { return wb + (size_t)(e >> 3) * BLK + (e & 7) * ROWB; };
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;

    // stage st -> buffer buf: instruction I = wave + 4 i fills LDS rows I*RPI .. of the stage
    auto issue = [&](int st, int buf) {
        for (int i = 0; i < ipw; ++i) {
            const int ins = wave + 4 * i;
            const int row = ins * RPI + lane / LPR, rc = min(row, rows - 1);
            const uint16_t *base = rc < bg ? static_cast<const uint16_t *>(a.x) + (size_t)(b0 + rc) * ld
                                           : static_cast<const uint16_t *>(a.w_e) + (size_t)(rc - bg) * ld;
            long e = c0 + (long)st * SE + (((lane % LPR) ^ (row & 15)) * 8);
            e = e < ld - 8 ? e : ld - 8;           // past the end of the row: any valid address (never used)
            if (once && ins * RPI >= bg) rs_dma16_once(base + e, lds_base + buf * SB + ins * 1024);   // all rows of the instruction are W_E's (wave-uniform)
            else rs_dma16(base + e, lds_base + buf * SB + ins * 1024);
        }
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
        if (s < nst) issue(s, s);
    if (HAS_D) stage_w_b_loop<NP, 256>(a, wb);

    rt_f32x4 accz[RT][CT], acct[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int u = 0; u < CT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) accz[t][u][v] = acct[t][u][v] = 0.f;
    int xoff[RT], woff[CT];   // byte offsets of this lane's fragment rows inside a stage, chunk XOR term separate
    int xsw[RT], wsw[CT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int row = min(t * 16 + r, bg - 1);
        xoff[t] = row * RB;
        xsw[t] = row & 15;
    }
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int row = bg + min(t * 16 + r, n - 1);
        woff[t] = row * RB;
        wsw[t] = row & 15;
    }
    const int tr_row = q4 * 8 + ((lane & 15) >> 2), tr_col = (lane & 3) * 4;

    int tk = 0, sq = wave;   // token and step-in-token of this wave's next step (its steps are wave, wave + 4, ...)
    int buf = 0, nbuf = STAGES - 1;
    for (int st = 0; st < nst; ++st) {
        if (st + STAGES - 1 < nst) rs_wait(ipw); else rs_wait(0);
        __syncthreads();   // stage st has landed for every wave; the buffer of stage st-1 is free
        if (st + STAGES - 1 < nst) issue(st + STAGES - 1, nbuf);
        const unsigned char *sb = stage0 + (size_t)buf * SB;
        // steps wave, wave + 4, ... of the stage: the x fragment feeds both products
#pragma unroll
        for (int u = 0; u < SPS / 4; ++u) {
            const int sl = u * 4 + wave;
            if (st * SPS + sl < gsteps) {
                const int c = sl * 4 + q4;
                rt_bf16x8 wf[CT], bfr[CT], xf[RT];
#pragma unroll
                for (int v = 0; v < CT; ++v) wf[v] = *reinterpret_cast<const rt_bf16x8 *>(sb + woff[v] + ((c ^ wsw[v]) * 16));
#pragma unroll
                for (int t = 0; t < RT; ++t) xf[t] = *reinterpret_cast<const rt_bf16x8 *>(sb + xoff[t] + ((c ^ xsw[t]) * 16));
                if (HAS_D) {
                    const int kr = sq * 32 + tr_row;   // W_B row = feature index of the step
#pragma unroll
                    for (int v = 0; v < CT; ++v) {
                        const rt_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rt_lds_s16x4_ptr)(row_at(kr) + (v * 16 + tr_col) * 2));
                        const rt_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rt_lds_s16x4_ptr)(row_at(kr + 4) + (v * 16 + tr_col) * 2));
                        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
                        bfr[v] = __builtin_bit_cast(rt_bf16x8, make_uint4(l2.x, l2.y, h2.x, h2.y));
                    }
                }
#pragma unroll
                for (int t = 0; t < RT; ++t)
#pragma unroll
                    for (int v = 0; v < CT; ++v) {
                        accz[t][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[t], wf[v], accz[t][v], 0, 0, 0);
                        if (HAS_D) acct[t][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[t], bfr[v], acct[t][v], 0, 0, 0);
                    }
                if (HAS_D) {
                    sq += 4;
                    if (sq >= spt) {   // this wave's share of token tk is complete
#pragma unroll
                        for (int t = 0; t < RT; ++t)
#pragma unroll
                            for (int v = 0; v < CT; ++v)
#pragma unroll
                                for (int w = 0; w < 4; ++w) {
                                    const int row = t * 16 + q4 * 4 + w, col = v * 16 + r;
                                    if (row < bg && col < n) t1w[(((size_t)wave * a.tc + tk) * bg + row) * n + col] = acct[t][v][w];
                                    acct[t][v][w] = 0.f;
                                }
                        sq -= spt;
                        ++tk;
                    }
                }
            }
        }
        buf = buf + 1 == STAGES ? 0 : buf + 1;
        nbuf = nbuf + 1 == STAGES ? 0 : nbuf + 1;
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int u = 0; u < CT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) zsh[wave][t * 16 + q4 * 4 + v][u * 16 + r] = accz[t][u][v];
    __syncthreads();
    for (int o = tid; o < RT * 16 * NP; o += 256) {
        const int row = o / NP, col = o - row * NP;
        if (row < bg && col < n)
            a.zpart[zpart_at(a, chunk, b0 + row, col)] = (zsh[0][row][col] + zsh[1][row][col]) + (zsh[2][row][col] + zsh[3][row][col]);
    }
    if (HAS_D) {
        for (int o = tid; o < tcur * bg * n; o += 256) {
            const int i = o % n, bb = (o / n) % bg, tl = o / (n * bg);
            const size_t at = ((size_t)tl * bg + bb) * n + i, ws = (size_t)a.tc * bg * n;
            a.t1[((size_t)(b0 + bb) * l + t0 + tl) * n + i] = (t1w[at] + t1w[ws + at]) + (t1w[2 * ws + at] + t1w[3 * ws + at]);
        }
    }
}

// Second kernel of the one-pass routing: workgroup = (chunk of a.tc_d tokens, sample).  The chunk's
// rows of t1 and of W_A go to LDS with every load of the workgroup in flight at once (the fold
// itself is a short loop per thread; fed from global memory it is a chain of load latencies), then
// the fold writes the chunk's partial logit tile (summed by route_reduce or route_select, exactly
// as the partial tiles of route_data_mfma are).
__global__ __launch_bounds__(256) void route_fold_kernel(RouteArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int chunk = blockIdx.x, bb = blockIdx.y, n = a.n, m = a.m;
    const int t0 = chunk * a.tc_d, tcur = min(a.tc_d, a.l - t0);
    uint16_t *wa_s = reinterpret_cast<uint16_t *>(smem);                                            // [tc_d][m]
    float *t1s = reinterpret_cast<float *>(smem + (((size_t)a.tc_d * m * 2 + 15) & ~(size_t)15));   // [tc_d][n]
    const uint16_t *wa_g = static_cast<const uint16_t *>(a.w_a) + (size_t)t0 * m;
    const int wa_elems = tcur * m;
    if ((m & 7) == 0) {
        for (int o = threadIdx.x * 8; o < wa_elems; o += 256 * 8)
            *reinterpret_cast<uint4 *>(wa_s + o) = *reinterpret_cast<const uint4 *>(wa_g + o);
    } else {
        for (int o = threadIdx.x; o < wa_elems; o += 256) wa_s[o] = wa_g[o];
    }
    const float *src = a.t1 + ((size_t)bb * a.l + t0) * n;
    for (int o = threadIdx.x; o < tcur * n; o += 256) t1s[o] = src[o];
    __syncthreads();
    route_fold<256>(a, chunk, bb, tcur, t1s, n, t1s + (size_t)a.tc_d * n, wa_s);
}

// The fold of the one-pass routing on the matrix cores (n*m outputs per sample, l products each: 67 M
// multiply-adds on the largest shape, a latency chain on the vector ALU).  Workgroup = (token range,
// sample); g[i][j] += sum_t t1[t][i] * W_A[t][j] as v_mfma_f32_16x16x32_bf16 with rows = experts,
// columns = patches, k = 32 tokens.  t1 is fp32 and selection has to agree with an fp64 reference to
// 1e-5 relative, so it enters as three bf16 terms, t1 = hi + mid + lo (each the rounded remainder of
// the ones before: 24 significant bits, exact to fp32), three MFMAs against the same W_A fragment.
// Wave w takes the 32-token steps w, w+4, ... of the range (at most 4): A fragments straight from global memory
// (lane (i, q) holds tokens 8q..8q+7 of expert i), the step's rows of W_A through a wave-private LDS
// tile and the transposing LDS read.  The four waves' tiles are added in wave order.
constexpr int FOLD_MAX_M = 128;   // accumulators: (m/16) x (n/16) tiles of 4 registers; LDS within 64 KiB
static bool route_fold_mfma_ok(int n, int m)
{
    if ((m & 7) != 0 && m > 16) return false;   // the W_A rows of a step: at most 8 loads per lane
    return n <= 16 ? m <= FOLD_MAX_M : m <= FOLD_MAX_M / 2;
}
// MT = column tiles computed (>= ceil(m/16); tiles past m work on zero-filled LDS columns and are not stored),
// STEPS = 32-token steps per wave (steps past the range work on zeros): straight-line code, no
// accumulator ever crosses a branch.
template <int CT, int MT, int STEPS>
__global__ __launch_bounds__(256) void route_fold_mfma_kernel(RouteArgs a, int tr)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i16 = lane & 15, q4 = lane >> 4;
    const int n = a.n, m = a.m, l = a.l, nm = n * m;
    const int rg = blockIdx.x, bb = blockIdx.y;
    const int t_begin = rg * tr, t_end = min(l, t_begin + tr);
    constexpr int pitch = 2 * b_pitch16(MT * 16);                  // elements per LDS row of W_A
    uint16_t *wa_s = reinterpret_cast<uint16_t *>(smem) + (size_t)wave * 32 * pitch;   // [32 tokens][pitch], this wave's
    float *red = reinterpret_cast<float *>(smem);   // [4 waves][CT*16][MT*16], over the W_A tiles once every wave is done with them

    rt_f32x4 acc[CT][MT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[c][j][v] = 0.f;
    const float *t1 = a.t1 + (size_t)bb * l * n;
    const uint16_t *w_a = static_cast<const uint16_t *>(a.w_a);
    const int tr_row = q4 * 8 + ((lane & 15) >> 2), tr_col = (lane & 3) * 4;

    // A dependent memory round trip costs microseconds here, so ALL loads of the wave (8 values of t1 and
    // PC pieces of W_A per lane and step, none depending on another) are issued before anything else.
    // W_A rows: 16-byte pieces when m % 8 == 0 (a row of the LDS tile = MT*2 pieces, columns past m come
    // from the next row and are never used), single elements otherwise (m <= 16).
    const bool vec = (m & 7) == 0;
    // pieces per lane and step: 32 rows * (m/8 <= 2 MT) / 64 lanes; up to 32 * 16 / 64 single elements when m <= 16
    constexpr int PC = MT == 1 ? 8 : (MT <= 4 ? MT : 8);
    const int pr = vec ? m >> 3 : m;                // pieces per row
    int prow[PC], goff[PC], loff[PC];
#pragma unroll
    for (int u = 0; u < PC; ++u) {
        const int idx = lane + 64 * u, row = idx / pr, within = idx - row * pr;
        prow[u] = row;                              // rows >= 32 are never loaded or stored
        goff[u] = vec ? row * m + within * 8 : idx;
        loff[u] = row * pitch + (vec ? within * 8 : within);
    }
    float tv[STEPS][CT][8];
    uint4 wv[STEPS][PC];
    uint16_t we[STEPS][PC];
#pragma unroll
    for (int sidx = 0; sidx < STEPS; ++sidx) {
        const int k0 = t_begin + (wave + 4 * sidx) * 32;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int t = k0 + q4 * 8 + e, i = c * 16 + i16;
                const bool ok = t < t_end && i < n;       // tokens past the range contribute zero
                tv[sidx][c][e] = t1[ok ? (size_t)t * n + i : (size_t)t_begin * n];
                if (!ok) tv[sidx][c][e] = 0.f;
            }
#pragma unroll
        for (int u = 0; u < PC; ++u) {
            const bool ok = prow[u] < 32 && k0 + prow[u] < t_end;
            const size_t at = ok ? (size_t)k0 * m + goff[u] : (size_t)0;
            if (vec) {
                wv[sidx][u] = *reinterpret_cast<const uint4 *>(w_a + (at & ~(size_t)7));
                if (!ok) wv[sidx][u] = make_uint4(0, 0, 0, 0);
            } else {
                we[sidx][u] = w_a[at];
                if (!ok) we[sidx][u] = 0;
            }
        }
    }
#pragma unroll
    for (int sidx = 0; sidx < STEPS; ++sidx) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < PC; ++u) {
            if (prow[u] < 32) {
                if (vec) *reinterpret_cast<uint4 *>(wa_s + loff[u]) = wv[sidx][u];
                else wa_s[loff[u]] = we[sidx][u];
            }
        }
        __builtin_amdgcn_wave_barrier();   // a wave reads back only what it wrote itself; LDS runs one wave's instructions in order
        rt_bf16x8 af[CT][3];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            uint32_t w3[3][4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float r0 = tv[sidx][c][2 * e], r1 = tv[sidx][c][2 * e + 1];
#pragma unroll
                for (int term = 0; term < 3; ++term) {
                    w3[term][e] = pack2_bf16(r0, r1);
                    r0 -= __uint_as_float(w3[term][e] << 16);
                    r1 -= __uint_as_float(w3[term][e] & 0xFFFF0000u);
                }
            }
#pragma unroll
            for (int term = 0; term < 3; ++term)
                af[c][term] = __builtin_bit_cast(rt_bf16x8, make_uint4(w3[term][0], w3[term][1], w3[term][2], w3[term][3]));
        }
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            const uint16_t *src = wa_s + tr_row * pitch + j * 16 + tr_col;
            const rt_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rt_lds_s16x4_ptr)(src));
            const rt_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rt_lds_s16x4_ptr)(src + 4 * pitch));
            const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
            const rt_bf16x8 bfr = __builtin_bit_cast(rt_bf16x8, make_uint4(l2.x, l2.y, h2.x, h2.y));
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int term = 2; term >= 0; --term)   // small terms first
                    acc[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[c][term], bfr, acc[c][j], 0, 0, 0);
        }
    }
    // accumulator register v of lane (i16, q4) in tile (c, j) is expert c*16 + 4*q4 + v, patch j*16 + i16
    constexpr int mp = MT * 16;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[((size_t)wave * CT * 16 + c * 16 + q4 * 4 + v) * mp + j * 16 + i16] = acc[c][j][v];
    __syncthreads();
    float *gout = a.gpart + ((size_t)rg * a.b + bb) * nm;
    constexpr size_t ws = (size_t)CT * 16 * mp;
    for (int o = tid; o < nm; o += 256) {
        const int i = o / m, j = o - i * m;
        const size_t at = (size_t)i * mp + j;
        gout[o] = (red[at] + red[ws + at]) + (red[2 * ws + at] + red[3 * ws + at]);
    }
}

// Sums the data router's per-chunk partials in a fixed order (deterministic).  A block owns 16
// reduced values of one sample; thread (value, chunk group) adds every 16th chunk, then the 16
// group sums are added in group order.  (The expert router's n values per sample are summed by
// route_select itself.)
__global__ __launch_bounds__(256) void route_reduce_kernel(RouteArgs a)
{
    __shared__ float part[16][17];
    const int bb = blockIdx.y, vi = threadIdx.x & 15, cg = threadIdx.x >> 4;
    const int nm = a.n * a.m;
    const int v = blockIdx.x * 16 + vi;
    float s = 0.f;
    if (v < nm) {
        const float *src = a.gpart + (size_t)bb * nm + v;
        const size_t stride = (size_t)a.b * nm;
        for (int ch = cg; ch < a.nchunks_d; ch += 16) s += src[(size_t)ch * stride];
    }
    part[cg][vi] = s;
    __syncthreads();
    if (threadIdx.x < 16 && v < nm) {
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < 16; ++q) t += part[q][vi];
        a.gred[(size_t)bb * nm + v] = t;
    }
}

// One workgroup per (expert row, sample), or for all rows of a sample (launch_route): top-c of each row of the patch gate; one more
// per sample for its top-k over experts.  LDS: ranking keys of the rows + the sample's n*m noisy logits.  The kernel is a chain of small
// dependent steps on at most 8192 numbers, bound by latency alone: everything from global memory is fetched up front
// by loads that do not depend on each other, loops over experts or patches read LDS eight values at a time (one
// value per iteration waits out the LDS latency every time), ranks and positions are counted by groups of lanes and
// by ballots, and the expert selection runs beside the patch selections instead of behind one of them.
// Against one chain per workgroup with a value per loop iteration: 16 experts x 128 patches 17.7 -> 9.8 us, 8 x 16
// 7.6 -> 5.5 us, experts alone 6.0 -> 5.1 us.

// max and sum of exp over the experts of one patch, from the staged logits (column j of [n][m])
__device__ __forceinline__ void column_softmax(const float *col, int n, int m, float &mx, float &den)
{
    mx = -INFINITY;
    for (int i0 = 0; i0 < n; i0 += 8) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = col[min(i0 + q, n - 1) * m];
#pragma unroll
        for (int q = 0; q < 8; ++q) mx = fmaxf(mx, v[q]);
    }
    den = 0.f;
    for (int i0 = 0; i0 < n; i0 += 8) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = col[min(i0 + q, n - 1) * m];
#pragma unroll
        for (int q = 0; q < 8; ++q) den += i0 + q < n ? expf(v[q] - mx) : 0.f;
    }
}

// Expert selection of one sample, by a workgroup of its own.
__device__ __forceinline__ void select_experts(const RouteArgs &a, int bb, int has_e)
{
    __shared__ float sums[SELECT_THREADS], ge[32];
    const int tid = threadIdx.x;
    const float noise = expert_noise(a, bb, tid);
    if (has_e) {
        expert_logits<SELECT_THREADS>(a, bb, sums, ge, tid);
        __syncthreads();
    }
    if (tid < 64) rank_experts(a, bb, has_e, ge, noise, true, nullptr, tid);
}

// fuse_reduce: the data router's per-chunk partials are summed here (each of the n workgroups of
// a sample repeats the sum: worth it only while n*m*chunks is small) instead of by route_reduce.
// The last workgroup of a sample selects experts, the others patches.
// ALL: every expert row of the sample in one workgroup (launch_route).
template <bool ALL> __device__ __forceinline__ void route_select(const RouteArgs &a, int has_e, int has_d, int fuse_reduce, int rows)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, i0 = ALL ? 0 : blockIdx.x, bb = blockIdx.y;
    if ((int)blockIdx.x == (ALL ? 1 : rows)) {
        select_experts(a, bb, has_e);
        return;
    }
    const int n = a.n, m = a.m, c = a.c, nm = n * m, pm = ALL ? nm : m;   // pm: (expert row, patch) pairs of this workgroup
    float *key = reinterpret_cast<float *>(smem);
    float *glog = reinterpret_cast<float *>(smem + (((size_t)pm * sizeof(float) + 15) & ~(size_t)15));  // [n*m]
    __shared__ float dpart[SELECT_THREADS];
    __shared__ uint64_t kept_bits[ALL ? 64 : 16];   // [rows of the workgroup][words of a row]: one row of m <= 1024, or at most 32 rows with 512 pairs
    const int words = ALL ? (m + 63) / 64 : 0;
    const float *gsrc = a.gred + (size_t)bb * nm;
    if (has_d) {
        const float *nzs = a.noise_p ? a.noise_p + (size_t)bb * nm : nullptr;
        if (fuse_reduce == 2) {  // few partial tiles of any size: every thread adds up its values in tile order
            const float *src = a.gpart + (size_t)bb * nm;
            const size_t stride = (size_t)a.b * nm;
            // four values per thread and pass, at most 16 tiles each (route_fold_plan): all loads of a pass in
            // flight together, tiles added in order
            for (int base = 0; base < nm; base += 4 * SELECT_THREADS) {
                float pv[4][16], nv[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int idx = min(base + q * SELECT_THREADS + tid, nm - 1);
                    nv[q] = nzs ? nzs[idx] : 0.f;
#pragma unroll
                    for (int ch = 0; ch < 16; ++ch) pv[q][ch] = src[(size_t)min(ch, a.nchunks_d - 1) * stride + idx];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int idx = base + q * SELECT_THREADS + tid;
                    if (idx < nm) {
                        float t = nv[q];
#pragma unroll
                        for (int ch = 0; ch < 16; ++ch) t += ch < a.nchunks_d ? pv[q][ch] : 0.f;
                        glog[idx] = t;
                    }
                }
            }
        } else if (fuse_reduce) {  // nm <= SELECT_THREADS: thread = (chunk group, value), groups summed in order
            const float *src = a.gpart + (size_t)bb * nm;
            const size_t stride = (size_t)a.b * nm;
            const int dgroups = SELECT_THREADS / nm, v = tid % nm, cg = tid / nm;
            const float nz = nzs && tid < nm ? nzs[tid] : 0.f;
            if (cg < dgroups) {
                float s = 0.f;
                for (int c0 = cg; c0 < a.nchunks_d; c0 += 8 * dgroups) {
                    float pv[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) pv[q] = src[(size_t)min(c0 + q * dgroups, a.nchunks_d - 1) * stride + v];
#pragma unroll
                    for (int q = 0; q < 8; ++q) s += c0 + q * dgroups < a.nchunks_d ? pv[q] : 0.f;
                }
                dpart[tid] = s;
            }
            __syncthreads();
            if (tid < nm) {
                float t = nz;
#pragma unroll 8
                for (int q = 0; q < dgroups; ++q) t += dpart[q * nm + tid];
                glog[tid] = t;
            }
        } else {
#pragma unroll 8
            for (int idx = tid; idx < nm; idx += SELECT_THREADS) glog[idx] = gsrc[idx] + (nzs ? nzs[idx] : 0.f);
        }
        __syncthreads();
    }

    // ---- data selection: Eq. 13 logits (+noise) -> Eq. 14 gate -> Eq. 17 top-c of each row
    for (int p = tid; p < pm; p += SELECT_THREADS) {
        const int r = ALL ? p / m : 0, j = p - r * m;
        float kv = 0.f, gate = 1.f;
        if (has_d) {  // softmax over the n experts of patch j
            float mx, den;
            column_softmax(glog + j, n, m, mx, den);
            const float own = glog[i0 * m + p];
            gate = expf(own - mx) / den;
            // ranking key: the log of the gate.  Same order as the gate itself, but a gate too
            // small for fp32 keeps its rank instead of collapsing into a tie at zero.
            kv = (own - mx) - logf(den);
        }
        key[p] = kv;
        if (a.patch_gate) a.patch_gate[(size_t)bb * nm + (size_t)i0 * m + p] = gate;
    }
    if (tid < (ALL ? 64 : 16)) kept_bits[tid] = 0;
    __syncthreads();
    // rank of a pair's patch in its row: G neighbouring lanes share its comparisons
    int G = 1;
    while (G < 64 && 2 * G * pm <= SELECT_THREADS) G *= 2;
    for (int p0 = 0; p0 < pm; p0 += SELECT_THREADS / G) {
        const int p = p0 + tid / G, g = tid % G, r = ALL ? p / m : 0, j = p - r * m;
        int rank = 0;
        if (p < pm) {
            const float *row = key + r * m;
            const float v = row[j];
            for (int q0 = g; q0 < m; q0 += 8 * G) {
                float w[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) w[q] = row[min(q0 + q * G, m - 1)];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int jj = q0 + q * G;
                    rank += jj < m && (w[q] > v || (w[q] == v && jj < j)) ? 1 : 0;
                }
            }
        }
        for (int off = 1; off < G; off <<= 1) rank += __shfl_xor(rank, off, 64);
        if (p < pm && g == 0 && rank < c) atomicOr(reinterpret_cast<unsigned int *>(kept_bits + r * words) + j / 32, 1u << (j % 32));
    }
    __syncthreads();
    if (a.patch_idx)
        for (int p = tid; p < pm; p += SELECT_THREADS) {
            const int r = ALL ? p / m : 0, j = p - r * m;
            const uint64_t *kept = kept_bits + r * words;
            if (!((kept[j / 64] >> (j % 64)) & 1)) continue;
            int pos = __popcll(kept[j / 64] & ((1ull << (j % 64)) - 1));
            for (int w = 0; w < j / 64; ++w) pos += __popcll(kept[w]);
            if (pos < c) a.patch_idx[((size_t)bb * n + i0 + r) * c + pos] = j;
        }
    if (i0 != 0 || !a.capacity || !has_d) return;  // uniform per workgroup

    // ---- dynamic capacity (Eq. 15-16) and balance statistics (Eq. 43-44), from the staged logits.
    // Stage 1: patch j names its patch_k best experts (rank counting on the logits, which order the
    // experts of one patch exactly as the gates do; ties to the lower index); count_i = number of
    // patches that named expert i (integer LDS adds: order-independent); c = max_i count_i.
    __shared__ int ccount[32];
    if (tid < n) ccount[tid] = 0;
    __syncthreads();  // also: every thread is past its last read of glog as logits of row 0
    for (int j = tid; j < m; j += SELECT_THREADS) {
        float mx = -INFINITY;
        for (int ii = 0; ii < n; ++ii) mx = fmaxf(mx, glog[ii * m + j]);
        float den = 0.f;
        for (int ii = 0; ii < n; ++ii) den += expf(glog[ii * m + j] - mx);
        for (int ii = 0; ii < n; ++ii) {
            const float v = glog[ii * m + j];
            int rank = 0;
            for (int t = 0; t < n; ++t) {
                const float w = glog[t * m + j];
                rank += (w > v || (w == v && t < ii)) ? 1 : 0;
            }
            if (rank < a.patch_k) atomicAdd(&ccount[ii], 1);
        }
        // this thread alone owns column j: the logits can now be replaced by the gates
        for (int ii = 0; ii < n; ++ii) glog[ii * m + j] = expf(glog[ii * m + j] - mx) / den;
    }
    __syncthreads();
    if (tid < n) {
        if (a.load_f) a.load_f[(size_t)bb * n + tid] = (float)n * (float)ccount[tid] / ((float)a.patch_k * (float)m);
        if (a.load_p) {
            float sum = 0.f;
            for (int j = 0; j < m; ++j) sum += glog[tid * m + j];  // fixed order
            a.load_p[(size_t)bb * n + tid] = sum / (float)m;
        }
    }
    if (tid == 0) {
        int cmax = 0;
        for (int ii = 0; ii < n; ++ii) cmax = max(cmax, ccount[ii]);
        a.capacity[bb] = cmax;
    }
}

__global__ __launch_bounds__(SELECT_THREADS) void route_select_kernel(RouteArgs a, int has_e, int has_d, int fuse_reduce, int rows)
{
    route_select<false>(a, has_e, has_d, fuse_reduce, rows);
}

// Eq. 42 per sample and its gradient through P_i = mean_j g_{i,j} (Eq. 44); f_i (Eq. 43) is a count.
// One workgroup per sample; the n products are added in expert order.
__global__ __launch_bounds__(256) void balance_loss_kernel(const float *load_f, const float *load_p, float alpha, float *loss,
                                                           float *d_patch_gate, int n, int m)
{
    const int bb = blockIdx.x, tid = threadIdx.x;
    const float *f = load_f + (size_t)bb * n;
    if (loss && tid == 0) {
        const float *pr = load_p + (size_t)bb * n;
        float s = 0.f;
        for (int i = 0; i < n; ++i) s += f[i] * pr[i];
        loss[bb] = alpha * s;
    }
    if (d_patch_gate) {
        float *dg = d_patch_gate + (size_t)bb * n * m;
        const float scale = alpha / (float)m;
        for (int idx = tid; idx < n * m; idx += 256) dg[idx] += scale * f[idx / m];
    }
}

hipError_t launch_balance_loss(const float *load_f, const float *load_p, float alpha, float *loss, float *d_patch_gate,
                               int b, int n, int m, hipStream_t st)
{
    hipLaunchKernelGGL(balance_loss_kernel, dim3(b), dim3(256), 0, st, load_f, load_p, alpha, loss, d_patch_gate, n, m);
    return hipGetLastError();
}

// Both routers side by side in one launch (one after the other on fp32 storage: 8 x 512 x 512 14.4 + 15.7 us, 2 x 64 x 64
// 4.6 + 8.7 us)
template <typename T, int NMAX>
static hipError_t launch_partial(const RouteArgs &a, bool has_e, bool has_d, hipStream_t st)
{
    const int data_blocks = has_d ? (a.nchunks_d + 7) / 8 * 8 * a.b : 0, expert_blocks = has_e ? (a.nchunks + 7) / 8 * 8 * a.b : 0;
    size_t sh = (size_t)ROUTE_WAVES * NMAX * sizeof(float);
    if (has_d) sh += (((size_t)a.n * a.d * sizeof(T) + 15) & ~(size_t)15) + (size_t)a.tc_d * NMAX * sizeof(float);
    hipLaunchKernelGGL((route_partial_kernel<T, NMAX>), dim3(data_blocks + expert_blocks), dim3(ROUTE_THREADS), sh, st, a, data_blocks);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_partial_n(const RouteArgs &a, bool has_e, bool has_d, hipStream_t st)
{
    if (a.n <= 2) return launch_partial<T, 2>(a, has_e, has_d, st);
    if (a.n <= 4) return launch_partial<T, 4>(a, has_e, has_d, st);
    if (a.n <= 6) return launch_partial<T, 6>(a, has_e, has_d, st);
    if (a.n <= 8) return launch_partial<T, 8>(a, has_e, has_d, st);
    if (a.n <= 12) return launch_partial<T, 12>(a, has_e, has_d, st);
    if (a.n <= 16) return launch_partial<T, 16>(a, has_e, has_d, st);
    if (a.n <= 24) return launch_partial<T, 24>(a, has_e, has_d, st);
    return launch_partial<T, 32>(a, has_e, has_d, st);
}

// dynamic LDS above 64 KiB has to be allowed per kernel (once per device is enough)
template <int RT, int CT, int RB, bool HAS_D>
static hipError_t launch_stream(const RouteArgs &a, const RouteStreamPlan &sp, dim3 grid, hipStream_t st)
{
    static bool allowed[64] = {};
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev >= 0 && dev < 64 && !allowed[dev]) {
        err = hipFuncSetAttribute(reinterpret_cast<const void *>(&route_stream_kernel<RT, CT, RB, HAS_D>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (err != hipSuccess) return err;
        allowed[dev] = true;
    }
    // W_E is read once per call: non-temporal from the size on that stream_once names (always, at the sizes this kernel is chosen for)
    const int once = stream_once((size_t)a.n * a.l * a.d * 2) ? 1 : 0;
    hipLaunchKernelGGL((route_stream_kernel<RT, CT, RB, HAS_D>), grid, dim3(256), sp.lds, st, a, sp.ipw, once);
    return hipGetLastError();
}

// a kernel of its own, behind the others: as two instances of one template where route_select_kernel stands the lm forward took 0.5
// to 1 percent more with the same instructions in each kernel (measured; why was not found, and other changes of the code's size move
// single calls by up to 1.5 percent either way)
__global__ __launch_bounds__(SELECT_THREADS) void route_select_all_kernel(RouteArgs a, int has_e, int has_d, int fuse_reduce, int rows)
{
    route_select<true>(a, has_e, has_d, fuse_reduce, rows);
}

hipError_t launch_route(const RouteArgs &a_in, bool bf16, hipStream_t st, RouteSelect *beside)
{
    const int most = beside ? beside->most : 0;
    if (beside) beside->on = 0;
    RouteArgs a = a_in;
    a.zgroups = SELECT_THREADS / a.n;
    const bool has_e = a.w_e != nullptr, has_d = a.w_b != nullptr;
    hipError_t err = hipSuccess;
    const bool data_mfma = has_d && route_data_uses_mfma(a.b, a.l, a.d, a.n, bf16);
    const bool split = a.tc_d < DATA_TOKENS;   // the data router's waves split the columns of x
    const int rt = a.b > 32 ? 4 : (a.b > 16 ? 2 : 1);
    const int groups_e = (a.b + rt * 16 - 1) / (rt * 16);
    int fold_ranges = 0;   // > 0: partial tiles of route_fold_mfma, few enough for route_select to add up
    const RouteStreamPlan sp = route_stream_plan(a.b, a.l, a.d, a.n, bf16, has_d);
    if (has_e && sp.ok && route_stream_pays(a.b, a.l, a.d, a.n)) {
        // streaming kernel: expert router and the data router's first map in one pass over x, then the fold
        a.tc = sp.tpc;
        a.nchunks = sp.nchunks;
        const dim3 grid(sp.nchunks, (a.b + sp.rt * 16 - 1) / (sp.rt * 16));
#define UOE_STREAM(RT, CT, RB)                                                                                              \
    do {                                                                                                                    \
        if (has_d) err = launch_stream<RT, CT, RB, true>(a, sp, grid, st);                                                   \
        else err = launch_stream<RT, CT, RB, false>(a, sp, grid, st);                                                        \
    } while (0)
        if (sp.ct == 1) {
            if (sp.rt == 4) UOE_STREAM(4, 1, 512);
            else if (sp.rt == 2) UOE_STREAM(2, 1, 512);
            else UOE_STREAM(1, 1, 1024);
        } else {
            if (sp.rt == 4) UOE_STREAM(4, 2, 512);
            else if (sp.rt == 2) UOE_STREAM(2, 2, 512);
            else UOE_STREAM(1, 2, 1024);
        }
#undef UOE_STREAM
        if (err != hipSuccess) return err;
        if (has_d && route_fold_mfma_ok(a.n, a.m)) {
            // fold on the matrix cores: a few token ranges per sample, summed by route_select itself
            const RouteFoldPlan fp = route_fold_plan(a.b, a.l);
            a.tc_d = fp.tr;
            a.nchunks_d = fp.ranges;
            const int mt = (a.m + 15) / 16, ct = a.n <= 16 ? 1 : 2;
            const int mtt = mt <= 1 ? 1 : (mt <= 2 ? 2 : (mt <= 4 ? 4 : 8)), steps = fp.tr <= 128 ? 1 : (fp.tr <= 256 ? 2 : 4);
            const size_t sh_wa = (size_t)4 * 32 * 2 * b_pitch16(mtt * 16) * 2, sh_red = (size_t)4 * ct * 16 * mtt * 16 * sizeof(float);
            const size_t shf = sh_wa > sh_red ? sh_wa : sh_red;
            const dim3 grid(fp.ranges, a.b);
#define UOE_FOLD3(CT, MT, ST) hipLaunchKernelGGL((route_fold_mfma_kernel<CT, MT, ST>), grid, dim3(256), shf, st, a, fp.tr)
#define UOE_FOLD2(CT, MT) do { if (steps == 1) UOE_FOLD3(CT, MT, 1); else if (steps == 2) UOE_FOLD3(CT, MT, 2); else UOE_FOLD3(CT, MT, 4); } while (0)
#define UOE_FOLD1(CT) do { if (mtt == 1) UOE_FOLD2(CT, 1); else if (mtt == 2) UOE_FOLD2(CT, 2); else if (mtt == 4) UOE_FOLD2(CT, 4); else UOE_FOLD2(CT, 8); } while (0)
            if (ct == 1) UOE_FOLD1(1);
            else if (mtt == 1) UOE_FOLD2(2, 1);
            else if (mtt == 2) UOE_FOLD2(2, 2);
            else UOE_FOLD2(2, 4);
#undef UOE_FOLD1
#undef UOE_FOLD2
#undef UOE_FOLD3
            if ((err = hipGetLastError()) != hipSuccess) return err;
            fold_ranges = fp.ranges;
        } else if (has_d) {
            const size_t shf = (((size_t)a.tc_d * a.m * 2 + 15) & ~(size_t)15) + (size_t)a.tc_d * a.n * sizeof(float) + 256 * 8 * sizeof(float);
            hipLaunchKernelGGL(route_fold_kernel, dim3(a.nchunks_d, a.b), dim3(256), shf, st, a);
            if ((err = hipGetLastError()) != hipSuccess) return err;
        }
    } else
    // one launch for both routers while x is small enough that the two do not simply queue up on HBM
    if (has_e && bf16 && data_mfma && (double)a.b * a.l * a.d * 2 <= 48e6) {
        const int n_data = a.nchunks_d * a.b;
        const dim3 grid(n_data + a.nchunks * groups_e);
        const size_t shd = data_lds(a.n, a.d);
#define UOE_FUSED(RT, CT)                                                                                         \
    do {                                                                                                          \
        const size_t she = route_expert_mfma_lds<RT, CT>();                                                       \
        if (split) hipLaunchKernelGGL((route_expert_data_kernel<RT, CT, 4>), grid, dim3(256), she > shd ? she : shd, st, a, n_data);   \
        else hipLaunchKernelGGL((route_expert_data_kernel<RT, CT, 1>), grid, dim3(256), she > shd ? she : shd, st, a, n_data);   \
    } while (0)
        if (a.n <= 16) {
            if (rt == 4) UOE_FUSED(4, 1);
            else if (rt == 2) UOE_FUSED(2, 1);
            else UOE_FUSED(1, 1);
        } else {
            if (rt == 4) UOE_FUSED(4, 2);
            else if (rt == 2) UOE_FUSED(2, 2);
            else UOE_FUSED(1, 2);
        }
#undef UOE_FUSED
        if ((err = hipGetLastError()) != hipSuccess) return err;
    } else {
        if (has_e && bf16) {  // a.tc / a.nchunks follow route_expert_mfma_tokens_per_chunk
            const dim3 grid(a.nchunks, groups_e);
#define UOE_EXPERT(RT, CT) hipLaunchKernelGGL((route_expert_mfma_kernel<RT, CT>), grid, dim3(256), (route_expert_mfma_lds<RT, CT>()), st, a)
            if (a.n <= 16) {
                if (rt == 4) UOE_EXPERT(4, 1);
                else if (rt == 2) UOE_EXPERT(2, 1);
                else UOE_EXPERT(1, 1);
            } else {
                if (rt == 4) UOE_EXPERT(4, 2);
                else if (rt == 2) UOE_EXPERT(2, 2);
                else UOE_EXPERT(1, 2);
            }
#undef UOE_EXPERT
            if ((err = hipGetLastError()) != hipSuccess) return err;
        } else if (has_e) {
            if ((err = launch_partial_n<float>(a, true, has_d, st)) != hipSuccess) return err;
        }
        if (data_mfma) {
            const size_t sh = data_lds(a.n, a.d);
            const dim3 grid(a.nchunks_d, a.b);
            if (a.n <= 16 && split) hipLaunchKernelGGL((route_data_mfma_kernel<1, 4>), grid, dim3(256), sh, st, a);
            else if (a.n <= 16) hipLaunchKernelGGL((route_data_mfma_kernel<1, 1>), grid, dim3(256), sh, st, a);
            else if (split) hipLaunchKernelGGL((route_data_mfma_kernel<2, 4>), grid, dim3(256), sh, st, a);
            else hipLaunchKernelGGL((route_data_mfma_kernel<2, 1>), grid, dim3(256), sh, st, a);
            if ((err = hipGetLastError()) != hipSuccess) return err;
        } else if (has_d && (bf16 || !has_e)) {
            err = bf16 ? launch_partial_n<bf16_t>(a, false, true, st) : launch_partial_n<float>(a, false, true, st);
            if (err != hipSuccess) return err;
        }
    }
    if (beside && !has_d && !a.capacity && a.nchunks * a.n <= most) {
        *beside = {a, 1, (int)has_e, most};
        return hipSuccess;
    }
    // patch lists and gates: none when neither is asked for (a capacity call needs row 0)
    const int rows = (a.patch_idx || a.patch_gate) ? a.n : (a.capacity && has_d ? 1 : 0);
    // all rows of a sample in one workgroup where a workgroup per row would be more than two a compute unit and every thread still
    // has at most one (row, patch) pair: the sample's logits are summed and staged once instead of once per row (128 samples of
    // 6 x 14: 10.0 -> 5.1 us).  With fewer the rows are better off side by side (16 samples of 8 x 64: the layer's forward 122.0
    // against 125.8 us, 8 of 8 x 16 60.4 against 61.2).
    const bool all = rows == a.n && (long)rows * a.b > 512 && rows * a.m <= SELECT_THREADS;
    // n * m <= 8192: the sample's logits always fit LDS
    const size_t sh = (((size_t)(all ? rows : 1) * a.m * sizeof(float) + 15) & ~(size_t)15) + (has_d ? (size_t)a.n * a.m * sizeof(float) : 0);
    int fuse_reduce = has_d && a.n * a.m <= SELECT_THREADS && (long)a.n * a.m * a.nchunks_d <= 16384;
    if (has_d && fold_ranges > 0 && fold_ranges <= 16) fuse_reduce = 2;
    if (has_d && !fuse_reduce) {
        hipLaunchKernelGGL(route_reduce_kernel, dim3((a.n * a.m + 15) / 16, a.b), dim3(256), 0, st, a);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    if (all) hipLaunchKernelGGL(route_select_all_kernel, dim3(2, a.b), dim3(SELECT_THREADS), sh, st, a, (int)has_e, (int)has_d, fuse_reduce, rows);
    else hipLaunchKernelGGL(route_select_kernel, dim3(rows + 1, a.b), dim3(SELECT_THREADS), sh, st, a, (int)has_e, (int)has_d, fuse_reduce, rows);
    return hipGetLastError();
}

}  // namespace uoe
