// Backward pass of the UoME block, bf16 storage.  Expert-selection mode first (Eq. 38-40 with
// Eq. 24-26); the data-selection mode (Eq. 37 with Eq. 12-18) follows at the end of the file.
// Forward, per sample b with active experts i(s), s < k, gate w_s (1 without the gate flag):
//   Z = u W1_b           W1_b = [A^I_i(0) | ... | A^I_i(k-1)]            [l, k*d_e]
//   H = SiLU(Z) * w      (column block s scaled by w_s)
//   h = (u) + H W2_b     W2_b = [A^O_i(0); ...; A^O_i(k-1)]              [l, d]
// Backward for an upstream gradient d_out = dL/dh:
//   dH  = d_out W2_b^T                                   GEMM, A^O_i read as [n][k]
//   dZ  = dH * w * SiLU'(Z),  H as above,  d_gate[b,i(s)] = sum over block s of dH * SiLU(Z)
//   d_u = (d_out) + dZ W1_b^T                            GEMM
//   dA^O_i = sum_{(b,s): i(s) = i} H_{b,s}^T d_out_b     GEMM over the tokens of those samples
//   dA^I_i = sum_{(b,s): i(s) = i} u_b^T dZ_{b,s}        GEMM over the tokens of those samples
// All five contractions run on the pipelined MFMA engine, on operands as they lie in memory: the products with a
// transposed weight read it as [n][k], the weight gradients read H, dZ, u and d_out token-major ([k][m], [k][n]); dA^I
// is formed as its transpose (dZ^T u) and turned back by the reduction that adds the split-K partials.  The
// elementwise middle (dZ, H and the gate gradient from Z and dH) is the epilogue of the dH contraction, and dH never
// reaches memory.  Where the tiles leave room (gemm_dma_dual_fits) Z is formed by the same workgroup and does not
// either; otherwise (256-column tiles, data selection) it is written in the storage dtype and read there and nowhere else.
// dZ and H are kept in the storage dtype between the kernels.
// Against separate dH, middle and weight-transposing launches with token-minor copies of dZ and H (b 4, l 8192,
// d 1024, 8 of 16 experts of 256): 15.7 + 144.5 + 131.8 us -> 212 us, and the weight gradients 317 -> 285 us.
#include "common.h"
#include "problems.h"
#include "gemm_mfma.h"
#include "gemm_dma.h"
#include "wgrad_reduce.h"

namespace uoe {

int uome_backward_gate_chunks(int l, int d_e) { return (l / 32) * (d_e / 32); }

// Elementwise middle for 8 elements: dZ, H and the sum of dH * SiLU(Z), an fp32 output.
__device__ __forceinline__ float uome_mid8(uint4 z8, uint4 dh8, float w, uint4 &dz8, uint4 &h8)
{
    const uint32_t z[4] = {z8.x, z8.y, z8.z, z8.w}, dh[4] = {dh8.x, dh8.y, dh8.z, dh8.w};
    uint32_t oz[4], oh[4];
    float part = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float dzv[2], hv[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float zv = __uint_as_float(e ? z[q] & 0xFFFF0000u : z[q] << 16);
            const float dv = __uint_as_float(e ? dh[q] & 0xFFFF0000u : dh[q] << 16);
            const float sig = sigmoid(zv);
            const float v = zv * sig;
            part = fmaf(dv, v, part);
            hv[e] = v * w;
            dzv[e] = dv * w * (sig * (1.0f + zv * (1.0f - sig)));
        }
        oz[q] = pack2_bf16(dzv[0], dzv[1]);
        oh[q] = pack2_bf16(hv[0], hv[1]);
    }
    dz8 = make_uint4(oz[0], oz[1], oz[2], oz[3]);
    h8 = make_uint4(oh[0], oh[1], oh[2], oh[3]);
    return part;
}

// dH = d_out W2_b^T (A^O_i [d_e, d] read as [n][k]) with the middle as its epilogue: the wave's tile of dH is staged in
// LDS in bf16 as for a plain store; each lane then walks its 16-byte pieces, with the matching pieces of Z a batch
// ahead, and stores pieces of dZ and H.  A lane's pieces lie in one 8-column group, four neighbouring lanes in one
// 32-column block of one expert: the block's sum for the gate gradient goes to gpart, one entry per 32 rows of the
// sample (tiles of 64 and 128 rows leave zeros in the entries behind their first).
template <typename T> struct UomeDhProblem {
    typedef typename storage_elem<T>::type Elem;
    const T *d_out, *a_out, *z;
    const int32_t *expert_idx;
    const float *expert_gate;   // NULL: weight 1
    T *dz, *h;                  // [b, l, k*d_e]
    float *gpart;               // [b, k, gchunks]
    int l, d, n, kact, d_e, gchunks;
    int once;                   // Z, dZ and H are larger than the caches: Z (its last use) is read past them
    static constexpr bool kWriteOut = true, kPrepare = false, kRowScale = false, kColScale = true;
    __device__ int rows(int) const { return l; }
    __device__ int kdim(int) const { return d; }
    __device__ int ncols() const { return kact * d_e; }
    __host__ __device__ int kseg(int) const { return d; }
    __device__ long b_stride() const { return 0; }
    __device__ uint32_t seg_ctx(int, int) const { return 0; }
    __device__ int expert(int g, int nn) const { return clampi(expert_idx[g * kact + nn / d_e], n); }
    __device__ const T *a_ptr_ctx(int g, int r, int, uint32_t) const { return d_out + ((size_t)g * l + r) * d; }
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t) const
    {
        return a_out + ((size_t)expert(g, nn) * d_e + nn % d_e) * d;
    }
    __device__ float col_scale(int g, int nn) const { return expert_gate ? expert_gate[(size_t)g * n + expert(g, nn)] : 1.0f; }
    __device__ float epi(float v, float) const { return v; }
    __device__ bool has_early() const { return true; }
    template <bool ONCE> __device__ uint4 early8(int g, int r, int nn) const { return load16<ONCE>(z + ((size_t)g * l + r) * ((size_t)kact * d_e) + nn); }
    template <int TM, int TN, int SPITCH, typename EARLY>
    __device__ void write_out(uint16_t (*stage)[SPITCH], const float *colw, const float (&)[TM], int g, int grow0, int gcol0, int M, int N, int lane,
                              const EARLY &early) const
    {
        constexpr int WM = TM * 32, WC = TN * 4, NPIECE = WM * WC / 64, BATCH = largest_divisor_upto(NPIECE, 8);
        static_assert(64 % WC == 0, "a lane keeps its 8-column group");
        const int pc = lane % WC, gcol = gcol0 + pc * 8;
        const bool col_ok = gcol < N;
        const float w = colw[pc];
        const size_t width = (size_t)kact * d_e;
        float part = 0.f;
#pragma unroll
        for (int t0 = 0; t0 < NPIECE; t0 += BATCH) {
            uint4 zp[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int grow = min(grow0 + (lane + (t0 + u) * 64) / WC, M - 1);
                if constexpr (!std::is_same<EARLY, NoEarlyPieces>::value) zp[u] = early.piece[t0 + u];
                else zp[u] = once ? early8<true>(g, grow, col_ok ? gcol : 0) : early8<false>(g, grow, col_ok ? gcol : 0);
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int row = (lane + (t0 + u) * 64) / WC, grow = grow0 + row;
                uint4 dz8, h8;
                const float s = uome_mid8(zp[u], *reinterpret_cast<const uint4 *>(&stage[row][pc * 8]), w, dz8, h8);
                if (grow < M && col_ok) {
                    part += s;
                    const size_t at = ((size_t)g * l + grow) * width + gcol;
                    store16<false>(dz + at, dz8);
                    store16<false>(h + at, h8);
                }
            }
        }
        part += __shfl_xor(part, 1, 64);
        part += __shfl_xor(part, 2, 64);
#pragma unroll
        for (int off = WC; off < 64; off <<= 1) part += __shfl_xor(part, off, 64);
        if (lane < WC && lane % 4 == 0 && col_ok) {
            const int s = gcol / d_e, blocks = d_e / 32;
            float *dst = gpart + ((size_t)g * kact + s) * gchunks + (gcol - s * d_e) / 32;
#pragma unroll
            for (int i = 0; i < TM; ++i)
                if (grow0 + i * 32 < M) dst[(grow0 / 32 + i) * blocks] = i == 0 ? part : 0.f;
        }
    }
};

// The same from the accumulators, with the tile of Z beside that of dH: neither reaches memory, and a launch goes (4096 x
// 512 x 1024, lm shape: 11.2 + 14.0 -> 19.4 us; its forward + backward 227 -> 223 us).  The 32-column blocks' sums go to
// gpart as above.
template <typename T> struct UomeDhPairProblem : UomeDhProblem<T> {
    static constexpr bool kPairOut = true;
    template <int TM, int TN, int SPITCH>
    __device__ void pair_out(f32x16_t (&acc)[TM][TN], f32x16_t *z, uint16_t (*stage)[SPITCH], const float *colw, int g, int grow0, int gcol0, int M, int N,
                             int lane) const
    {
        const int lr = lane & 31, blocks = this->d_e / 32;
        // in place: z becomes H, the accumulators dZ
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int c32 = gcol0 + j * 32;   // uniform over the wave, one expert's
            if (c32 >= N) continue;
            const float w = colw[j * 4];
            float part = 0.f;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                float ps = 0.f;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float zv = z[i * TN + j][e], dv = acc[i][j][e];
                    const float sig = sigmoid(zv), v = zv * sig;
                    ps = fmaf(dv, v, ps);
                    z[i * TN + j][e] = v * w;
                    acc[i][j][e] = dv * w * (sig * (1.0f + zv * (1.0f - sig)));
                }
                if (grow0 + i * 32 + lr < M) part += ps;
            }
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) part += __shfl_xor(part, off, 64);
            const int s = c32 / this->d_e;
            if (lane == 0) {
                float *dst = this->gpart + ((size_t)g * this->kact + s) * this->gchunks + (c32 - s * this->d_e) / 32;
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    if (grow0 + i * 32 < M) dst[(grow0 / 32 + i) * blocks] = i == 0 ? part : 0.f;
            }
        }
        auto plane = [&](T *dst, auto value) {
            stage_plane<TM, TN, SPITCH>(
                stage, lane, M - grow0,
                [&](int i, int j, int q) {
                    const f32x16_t &v = value(i, j);
                    return make_uint2(pack2_bf16(v[q * 4], v[q * 4 + 1]), pack2_bf16(v[q * 4 + 2], v[q * 4 + 3]));
                },
                [&](int row, int col, uint4 piece) {
                    if (grow0 + row < M && gcol0 + col < N)
                        store16<false>(dst + ((size_t)g * this->l + grow0 + row) * ((size_t)this->kact * this->d_e) + gcol0 + col, piece);
                });
        };
        plane(this->h, [&](int i, int j) -> const f32x16_t & { return z[i * TN + j]; });
        plane(this->dz, [&](int i, int j) -> const f32x16_t & { return acc[i][j]; });
    }
};

// the last launch of the expert-selection pass where the gates did not fit beside another: the gate gradient's blocks and the
// weight-gradient tiles
__global__ __launch_bounds__(256) void uome_bwd_finish_kernel(WgradReduceArgs ra, UomeBwdArgs a, int nx, int ny, int gates)
{
    __shared__ __align__(16) unsigned char lds[RED_LDS];
    const int id = (int)blockIdx.x - gates;
    if (id >= 0) wgrad_reduce_tile<bf16_t, false>(ra, reinterpret_cast<RedTile>(lds), id % nx, id / nx % ny, id / (nx * ny));
    else uome_bwd_gate_block<256>(a, blockIdx.x % a.k, blockIdx.x / a.k, reinterpret_cast<float *>(lds));
}

hipError_t launch_uome_ds_backward(const UomeBwdArgs &a, hipStream_t st, BwdTail *tail);

hipError_t launch_uome_backward(const UomeBwdArgs &a, hipStream_t st, BwdTail *tail)
{
    typedef bf16_t T;
    if (a.wgrad.parts > WGRAD_MAX_PARTS) return hipErrorInvalidValue;
    if (a.patch_idx) return launch_uome_ds_backward(a, st, tail);
    hipError_t err;
    const int width = a.k * a.d_e;
    UomeUpProblem<T, true> zp;  // Z = u W1_b (plain product)
    zp.u = static_cast<const T *>(a.u); zp.a_in = static_cast<const T *>(a.a_in);
    zp.expert_idx = a.expert_idx; zp.expert_gate = nullptr; zp.hidden = static_cast<T *>(a.z);
    zp.l = a.l; zp.d = a.d; zp.n = a.n; zp.kact = a.k; zp.d_e = a.d_e;
    zp.once = stream_once((size_t)a.b * a.l * width * sizeof(T));   // Z: written here, read once by the next kernel

    UomeDhPairProblem<T> hp;    // dH = d_out W2_b^T, and dZ, H and the gate gradient's partial sums from Z and it
    hp.d_out = static_cast<const T *>(a.d_out); hp.a_out = static_cast<const T *>(a.a_out); hp.z = static_cast<const T *>(a.z);
    hp.expert_idx = a.expert_idx; hp.expert_gate = (a.flags & F_GATE_EXPERT) ? a.expert_gate : nullptr;
    hp.dz = static_cast<T *>(a.dz); hp.h = static_cast<T *>(a.h); hp.gpart = a.gpart; hp.gchunks = a.gchunks;
    hp.l = a.l; hp.d = a.d; hp.n = a.n; hp.kact = a.k; hp.d_e = a.d_e; hp.once = zp.once;
    if (gemm_dma_dual_fits(a.b, a.l, width, a.d, a.d))
        err = launch_gemm_dma_dual_auto<0, GEMM_B_NK>(zp, hp, a.b, a.l, width, a.d, st);
    else if ((err = launch_gemm_dma_auto(zp, a.b, a.l, width, a.d, a.d, st)) == hipSuccess)
        err = launch_gemm_dma_auto<GEMM_B_NK>(static_cast<const UomeDhProblem<T> &>(hp), a.b, a.l, width, a.d, a.d, st);
    if (err != hipSuccess) return err;

    UomeDownProblem<T> up;  // d_u = (d_out) + dZ W1_b^T: the second-layer contraction with A^I_i [d, d_e] as [n][k]
    up.hidden = static_cast<const T *>(a.dz); up.a_out = static_cast<const T *>(a.a_in); up.w_nk = 1;
    up.u = static_cast<const T *>(a.d_out); up.expert_idx = a.expert_idx; up.out = static_cast<T *>(a.d_u);
    up.l = a.l; up.d = a.d; up.n = a.n; up.kact = a.k; up.d_e = a.d_e; up.flags = a.flags;

    // weight gradients, both in one launch: [d_e, d] tiles per part of an expert's tokens; (dA^I_i)^T = sum dZ_{b,s}^T u_b is stored back as [d, d_e] by the reduction
    WgradProblem<T> wp;
    wp.left[0] = static_cast<const T *>(a.h); wp.right[0] = static_cast<const T *>(a.d_out);  // dA^O_i
    wp.left[1] = static_cast<const T *>(a.dz); wp.right[1] = static_cast<const T *>(a.u);     // (dA^I_i)^T
    wp.expert_idx = a.expert_idx; wp.partial = a.partial;
    wp.b = a.b; wp.l = a.l; wp.n = a.n; wp.kact = a.k; wp.parts = {2, BY_SAMPLE, a.wgrad, a.part_end};
    wp.M = a.d_e; wp.N = a.d; wp.range = a.l / a.wgrad.items;
    // one launch for d_u and the weight gradients while neither fills the chip's slots (two per compute unit) by itself
    const int groups = wp.parts.groups(), kseg = wp.range;
    int gates = a.d_gate ? a.b * a.k : 0;
    const long du64 = (long)a.b * ((a.l + 63) / 64) * ((a.d + 127) / 128), wg128 = (long)groups * ((a.d_e + 127) / 128) * ((a.d + 127) / 128);
    if (a.d_e % 64 == 0 && kseg % 64 == 0 && a.d_e > 64 && du64 <= 512 && wg128 <= 512) {
        typedef GemmTile<UomeDownProblem<T>, 64, 128, 64, 2, 2, 3, GEMM_B_NK> Du;
        typedef GemmTile<WgradProblem<T>, 128, 128, 64, 2, 2, 2, GEMM_A_KM> Wg;
        // (and the gate gradient, which the routers' pass waits for: the reduction can then run beside that pass)
        err = launch_gemm_dma_pair<Wg, Du, 2>(wp, groups, a.d_e, a.d, up, a.b, a.l, a.d, st, UomeGates{a}, gates);
        gates = 0;
    } else if ((err = launch_gemm_dma_auto<GEMM_B_NK>(up, a.b, a.l, a.d, width, a.d_e, st)) == hipSuccess)
        err = launch_gemm_dma_auto<GEMM_A_KM>(wp, groups, a.d_e, a.d, 0, kseg, st);
    if (err != hipSuccess) return err;
    WgradReduceArgs ra{};
    ra.partial = a.partial; ra.n = a.n; ra.M = a.d_e; ra.N = a.d;
    ra.w = a.wgrad; ra.part_end = a.part_end;
    ra.dst[0] = a.d_a_out; ra.transposed[0] = 0;
    ra.dst[1] = a.d_a_in; ra.transposed[1] = 1;
    if (!gates) return launch_wgrad_reduce<T>(ra, 2, st, tail);
    const RedGrid g(ra, 2);
    hipLaunchKernelGGL(uome_bwd_finish_kernel, dim3(g.tiles + gates), dim3(256), 0, st, ra, a, g.nx, g.ny, gates);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Data-selection mode (Eq. 37-40 with Eq. 12-18): expert i of an active unit sees only the l_a
// gathered rows of its c patches.  Same chain as above per unit, with the gathers folded into
// operand addressing (the forward's gathered projection for Z and dH, the output-stationary
// per-patch contraction for d_u, patch-gathered right operands for the weight gradients) and the
// row weight w_t = expert gate and/or the gate of the row's patch.

// dH_raw = d_out[T] A^O_i^T with the middle as its epilogue (see UomeDhProblem): the row weight arrives per row
// (fetched before the K loop, one row per lane, handed round by a shuffle), and a row's dL/dw_t = sum_j dH_raw * SiLU(Z)
// leaves one part per wave tile's columns.
template <typename T> struct UomeDsDhProblem : UomeDsUpProblem<T> {   // u = d_out, a_in = A^O, hidden unused
    const T *z;
    T *dz, *h;                  // [units, l_a, d_e]
    float *rt;                  // [parts][units*l_a]
    size_t rt_stride;
    static constexpr bool kWriteOut = true;
    __device__ const T *b_ptr_ctx(int g, int, int nn, uint32_t) const { return this->a_in + ((size_t)this->expert(g) * this->d_e + nn) * this->d; }
    __device__ float epi(float v, float) const { return v; }
    template <int TM, int TN, int SPITCH>
    __device__ void write_out(uint16_t (*stage)[SPITCH], const float *, const float (&rs)[TM], int g, int grow0, int gcol0, int M, int N, int lane) const
    {
        constexpr int WM = TM * 32, WC = TN * 4, NPIECE = WM * WC / 64, BATCH = largest_divisor_upto(NPIECE, 8);
        static_assert(64 % WC == 0, "a row lies in WC neighbouring lanes");
        const int pc = lane % WC, gcol = gcol0 + pc * 8;
        const bool col_ok = gcol < N;
        if (gcol0 >= N) return;
#pragma unroll
        for (int t0 = 0; t0 < NPIECE; t0 += BATCH) {
            uint4 zp[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int grow = min(grow0 + (lane + (t0 + u) * 64) / WC, M - 1);
                zp[u] = load16<false>(z + ((size_t)g * M + grow) * N + (col_ok ? gcol : 0));
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int row = (lane + (t0 + u) * 64) / WC, grow = grow0 + row;   // 64 / WC rows at a time: row / 32 is uniform
                const float w = __shfl(rs[(t0 + u) * (64 / WC) / 32], row & 31, 64);
                uint4 dz8, h8;
                float s = uome_mid8(zp[u], *reinterpret_cast<const uint4 *>(&stage[row][pc * 8]), w, dz8, h8);
                if (!col_ok) s = 0.f;
#pragma unroll
                for (int off = 1; off < WC; off <<= 1) s += __shfl_xor(s, off, 64);
                if (grow < M && col_ok) {
                    const size_t at = ((size_t)g * M + grow) * N + gcol;
                    store16<false>(dz + at, dz8);
                    store16<false>(h + at, h8);
                    if (pc == 0) rt[gcol0 / (TN * 32) * rt_stride + (size_t)g * M + grow] = s;
                }
            }
        }
    }
};

hipError_t launch_uome_ds_backward(const UomeBwdArgs &a, hipStream_t st, BwdTail *tail)
{
    typedef bf16_t T;
    hipError_t err;
    const int l_p = a.l / a.m, l_a = a.c * l_p, units = a.b * a.k;
    // Z = u[T] A^I_i: the gathered projection with one output block
    QkvProblem<T> zp;
    zp.x = static_cast<const T *>(a.u);
    zp.wq = zp.wk = zp.wv = static_cast<const T *>(a.a_in);
    zp.expert_idx = a.expert_idx; zp.patch_idx = a.patch_idx;
    zp.q = zp.k = zp.v = static_cast<T *>(a.z); zp.q32 = nullptr;
    zp.l = a.l; zp.d = a.d; zp.n = a.n; zp.kact = a.k; zp.m = a.m; zp.c = a.c;
    zp.l_p = l_p; zp.l_a = l_a; zp.d_h = a.d_e; zp.q_scale = 1.0f; zp.nout = 1;
    if ((err = launch_gemm_dma_auto(zp, units, l_a, a.d_e, a.d, a.d, st)) != hipSuccess) return err;

    UomeDsDhProblem<T> hp;      // dH_raw, and dZ, H and the row terms from Z and it
    hp.u = static_cast<const T *>(a.d_out); hp.a_in = static_cast<const T *>(a.a_out); hp.hidden = nullptr;
    hp.expert_idx = a.expert_idx; hp.patch_idx = a.patch_idx;
    hp.expert_gate = (a.flags & F_GATE_EXPERT) ? a.expert_gate : nullptr;
    hp.patch_gate = (a.flags & F_GATE_PATCH) ? a.patch_gate : nullptr;
    hp.l = a.l; hp.d = a.d; hp.n = a.n; hp.kact = a.k; hp.m = a.m; hp.c = a.c; hp.l_p = l_p; hp.l_a = l_a; hp.d_e = a.d_e;
    hp.z = static_cast<const T *>(a.z); hp.dz = static_cast<T *>(a.dz); hp.h = static_cast<T *>(a.h);
    hp.rt = a.rt; hp.rt_stride = (size_t)units * l_a;
    int wave_cols;
    if ((err = launch_gemm_dma_auto<GEMM_B_NK>(hp, units, l_a, a.d_e, a.d, a.d, st, &wave_cols)) != hipSuccess) return err;

    SmhaBwdArgs ga{};  // the gate gradients' blocks read its routing fields, the row terms and the gates
    ga.f.expert_idx = a.expert_idx; ga.f.patch_idx = a.patch_idx;
    ga.f.b = a.b; ga.f.l = a.l; ga.f.d = a.d; ga.f.n = a.n; ga.f.k = a.k; ga.f.m = a.m; ga.f.c = a.c;
    ga.expert_gate = a.expert_gate; ga.patch_gate = a.patch_gate; ga.flags = a.flags;
    ga.d_expert_gate = a.d_gate; ga.d_patch_gate = a.d_patch_gate; ga.rt = a.rt;
    ga.rt_parts = (a.d_e + wave_cols - 1) / wave_cols;

    // d_u = (d_out) + scatter-add of dZ A^I_i^T: the output-stationary per-patch contraction
    OutProjProblem<T> xp;
    xp.o = static_cast<const T *>(a.dz); xp.o_lo = nullptr; xp.parts = 1;
    xp.wo = static_cast<const T *>(a.a_in); xp.w_nk = 1; xp.x = static_cast<const T *>(a.d_out);
    xp.expert_idx = a.expert_idx; xp.patch_idx = a.patch_idx;
    xp.out = static_cast<T *>(a.d_u);
    xp.l = a.l; xp.d = a.d; xp.n = a.n; xp.kact = a.k; xp.m = a.m; xp.c = a.c;
    xp.l_p = l_p; xp.l_a = l_a; xp.d_h = xp.o_row = a.d_e; xp.flags = a.flags & F_RESIDUAL;

    SmhaWgradProblem<T> wp;  // both weight gradients in one launch
    wp.left[0] = static_cast<const T *>(a.h); wp.right[0] = static_cast<const T *>(a.d_out);  // dA^O_i
    wp.left[1] = static_cast<const T *>(a.dz); wp.right[1] = static_cast<const T *>(a.u);     // (dA^I_i)^T
    wp.left[2] = wp.left[3] = wp.right[2] = wp.right[3] = nullptr;
    for (int q = 0; q < 4; ++q) { wp.row_len[q] = a.d_e; wp.col0[q] = 0; }
    wp.expert_idx = a.expert_idx; wp.patch_idx = a.patch_idx; wp.partial = a.partial;
    wp.b = a.b; wp.l = a.l; wp.d = a.d; wp.n = a.n; wp.kact = a.k; wp.m = a.m; wp.c = a.c;
    wp.l_p = l_p; wp.l_a = l_a; wp.parts = {2, DEALT, a.wgrad, a.part_end}; wp.M = a.d_e;
    // one launch with d_u while the weight gradients do not fill the chip's slots (two per compute unit)
    const int groups = wp.parts.groups();
    typedef GemmTile<OutProjProblem<T>, 32, 128, 32, 1, 4, 4, GEMM_B_NK> Du32;
    typedef GemmTile<OutProjProblem<T>, 64, 128, 32, 2, 2, 4, GEMM_B_NK> Du64;
    typedef GemmTile<SmhaWgradProblem<T>, 128, 128, 32, 2, 2, 4, GEMM_A_KM> Wg;
    const bool pair = a.d_e > 64 && (long)groups * ((a.d_e + 127) / 128) * ((a.d + 127) / 128) <= 512;
    if (pair) {   // (and with the gate gradients)
        const UnitGates gates{ga, UnitGates::count(ga)};
        err = l_p <= 32 ? launch_gemm_dma_pair<Wg, Du32, 2>(wp, groups, a.d_e, a.d, xp, a.b * a.m, l_p, a.d, st, gates, gates.units)
                        : launch_gemm_dma_pair<Wg, Du64, 2>(wp, groups, a.d_e, a.d, xp, a.b * a.m, l_p, a.d, st, gates, gates.units);
    } else {
        if (l_p <= 32) err = launch_gemm_dma<OutProjProblem<T>, 32, 128, 32, 1, 4, 4, 2, GEMM_B_NK>(xp, a.b * a.m, l_p, a.d, st);
        else err = launch_gemm_dma<OutProjProblem<T>, 64, 128, 32, 2, 2, 4, 2, GEMM_B_NK>(xp, a.b * a.m, l_p, a.d, st);
        if (err == hipSuccess) err = launch_gemm_dma_auto<GEMM_A_KM>(wp, groups, a.d_e, a.d, 0, l_p, st);
    }
    if (err != hipSuccess) return err;
    WgradReduceArgs ra{};
    ra.partial = a.partial; ra.n = a.n; ra.M = a.d_e; ra.N = a.d;
    ra.w = a.wgrad; ra.part_end = a.part_end;
    ra.dst[0] = a.d_a_out; ra.transposed[0] = 0;
    ra.dst[1] = a.d_a_in; ra.transposed[1] = 1;
    return pair ? launch_wgrad_reduce<T>(ra, 2, st, tail) : launch_wgrad_reduce_gates<T>(ra, 2, ga, st);
}

}  // namespace uoe
