// The first step of the data router's backward pass (dL, U and W_B^T): a launch of its own (route_bwd.hip), or workgroups beside the last
// contractions of the SMHA block's backward pass.
#pragma once
#include "common.h"

namespace uoe {

typedef float rb_f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rb_f32x4 mfma_f32(float x, float y, rb_f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0);  // lane: row / column lane & 15, k lane >> 4
}

// Softmax backward of one logit, dz_i = g_i (dg_i - sum_j g_j dg_j) for any gates, evaluated as
// g_i (sum_j g_j (dg_i - dg_j) + (1 - sum_j g_j) dg_i): with one gate close to 1 the first form subtracts two nearly equal
// numbers, the second adds small terms of mixed sign only.  Gates of a softmax sum to one up to their rounding, (n + 1) 2^-23 at
// most (a division, and the sums in the forward pass and here); that much of the last term is rounding, not gate, and left out.
__device__ __forceinline__ float softmax_bwd(const float *g, const float *dg, int n, int stride, int i)
{
    const float mine = dg[i * stride];
    float s = 0.f, rest = 1.f;
    for (int q = 0; q < n; ++q) {
        s = fmaf(g[q * stride], mine - dg[q * stride], s);
        rest -= g[q * stride];
    }
    if (fabsf(rest) > (float)(n + 1) * 1.1920929e-7f) s = fmaf(mine, rest, s);
    return g[i * stride] * s;
}

constexpr int PREP_TOK = 64, PREP_J = 64, PREP_ST = PREP_J + 4;  // row stride = 4 mod 64 banks: 16 rows x 4 k, no conflict
// Block (token tile, sample): the sample's dL (Eq. 14 backwards) and U = W_A dL^T for 64 tokens, 64 patches at a
// time.  Blocks behind the last token tile write W_B^T (the d_x workgroups read 8 of its columns per 16 bytes).
struct RoutePrepLds {
    float gs[2][32][PREP_J], dls[32][PREP_ST], was[PREP_TOK][PREP_ST];
};
// bx, bb: of nx blocks a sample
template <typename T> __device__ __forceinline__ void route_prep_block(const RouteBwdArgs &a, int bx, int bb, int nx, RoutePrepLds &lds)
{
    auto &gs = lds.gs; auto &dls = lds.dls; auto &was = lds.was;
    const int tid = threadIdx.x, tiles = (a.l + PREP_TOK - 1) / PREP_TOK;
    if (bx >= tiles) {
        const int step = (nx - tiles) * a.b * 256;
        for (int idx = ((bx - tiles) * a.b + bb) * 256 + tid; idx < a.d * a.n; idx += step) {
            const int i = idx / a.d, e = idx - i * a.d;
            static_cast<T *>(a.wbt)[idx] = static_cast<const T *>(a.w_b)[(size_t)e * a.n + i];
        }
        return;
    }
    const int t0 = bx * PREP_TOK, wave = tid >> 6, r = tid & 15, q = (tid & 63) >> 4;
    const float *g = a.g_p + (size_t)bb * a.n * a.m, *dg = a.d_g_p + (size_t)bb * a.n * a.m;
    const int rows = (a.n + 15) & ~15;
    rb_f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    for (int j0 = 0; j0 < a.m; j0 += PREP_J) {
        const int nj = min(PREP_J, a.m - j0);
        const int jj = tid % PREP_J, row = tid / PREP_J;
        const size_t j = j0 + min(jj, nj - 1);  // clamped, unconditional loads: all of them in flight at once
        T wv[16];
        float gv[8], dgv[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int i = min(row + 4 * v, a.n - 1);
            gv[v] = g[i * a.m + j];
            dgv[v] = dg[i * a.m + j];
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) wv[v] = static_cast<const T *>(a.w_a)[(size_t)min(t0 + row + 4 * v, a.l - 1) * a.m + j];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            gs[0][row + 4 * v][jj] = gv[v];
            gs[1][row + 4 * v][jj] = dgv[v];
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) was[row + 4 * v][jj] = jj < nj ? to_f32(wv[v]) : 0.f;
        __syncthreads();
        for (int i = row; i < rows; i += 4) {
            float v = 0.f;
            if (i < a.n && jj < nj) {
                v = softmax_bwd(&gs[0][0][jj], &gs[1][0][jj], a.n, PREP_J, i);
                if (bx == 0) a.dl[((size_t)bb * a.n + i) * a.m + j0 + jj] = v;
            }
            dls[i][jj] = v;
        }
        __syncthreads();
        for (int s = 0; s < (nj + 3) / 4; ++s) {
            const float av = was[16 * wave + r][4 * s + q];
            acc[0] = mfma_f32(av, dls[r][4 * s + q], acc[0]);
            if (a.n > 16) acc[1] = mfma_f32(av, dls[16 + r][4 * s + q], acc[1]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = t0 + 16 * wave + 4 * q + e, i = 16 * nt + r;
            if (t < a.l && i < a.n) a.u[((size_t)bb * a.l + t) * a.n + i] = acc[nt][e];
        }
}

template <typename T> struct RoutePrep {
    static constexpr int THREADS = 256;
    static constexpr bool OPTIONAL = true;   // (BwdTail::prep_done)
    static constexpr size_t LDS = sizeof(RoutePrepLds);
    RouteBwdArgs a;
    int nx;
    RoutePrep() = default;
    // (8 elements of W_B^T per thread)
    explicit RoutePrep(const RouteBwdArgs &args) : a(args), nx((args.l + PREP_TOK - 1) / PREP_TOK + (args.d * args.n + 2048 * args.b - 1) / (2048 * args.b)) {}
    __host__ int blocks() const { return nx * a.b; }
    template <int NT> __device__ __forceinline__ void run(int block, void *lds) const
    {
        static_assert(NT == 256, "256 threads");
        route_prep_block<T>(a, block % nx, block / nx, nx, *static_cast<RoutePrepLds *>(lds));
    }
};

}  // namespace uoe
