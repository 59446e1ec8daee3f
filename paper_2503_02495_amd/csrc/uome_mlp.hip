// Both layers of the expert-selection UoME block (Eq. 38-40) in one launch, for narrow tokens: bf16, d <= 256, widths that are multiples of 32.
//
// Apart they write and read the hidden activations, and at d = 256 an output element of the second layer has so few products that both are
// bound by that traffic and by their epilogues.  Here a wave owns 32 tokens from u to out, as the attention kernel owns queries: its rows of u
// stay in registers as the second operand of (u W1)^T = W1^T u^T, whose accumulators, through SiLU and packed in place, are the second operand
// of out^T = W2^T h^T, which stays in accumulators over all hidden columns (16 registers per 32 columns of d: what bounds d).  Only the weights go
// through LDS: 64 hidden columns of the sample's experts a stage, both layers' slices, copied by all waves two stages deep,
// one barrier a stage; every fragment read feeds one product, so LDS and matrix pipes are about equally busy, and the two waves of a SIMD run
// their SiLU under each other's products.
// 16 x 4096 x 256, 2 of 8 experts of 128: 41.8 -> 30.9 us (u and out 67 MB, 12.4; with 16 x 256 hidden columns 1.05 PFLOP/s); 16 x 4096 x 64, 4 of 256,
// 71 -> 32 (uome_mlp_waves has more).  Four waves of 32 tokens, one a SIMD, where eight would leave compute units without work.
#include "common.h"
#include "problems.h"
#include "gemm_mfma.h"
#include "gemm_dma.h"

namespace uoe {

constexpr int MLP_HC = 64;

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// dma_load16 at a byte offset of the lane's from a base that all lanes share
__device__ __forceinline__ void dma_load16_at(const void *base, uint32_t offset, uint32_t lds_byte)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_byte), "v"(offset), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int DT, int NW, bool SEL>
__global__ __launch_bounds__(NW * 64, NW / 4) void uome_mlp_kernel(UomeUpProblem<bf16_t, false, false, SEL> up, UomeDownProblem<bf16_t> dn, TileGrid tg)
{
    constexpr int D = DT * 32, HC = MLP_HC, CD = D / 8;      // CD: 16-byte chunks of a row of W2
    constexpr int W_BYTES = D * HC * 2, STAGE = 2 * W_BYTES; // a stage: W1 [D][HC], then W2 [HC][D]
    constexpr int INSTR = D / 8;                             // load instructions of either
    constexpr int SPITCH = D + 8;                            // of the epilogue's staging tiles
    constexpr int EPI = NW * 32 * SPITCH * 2, ROWS = NW * 32;
    __shared__ __align__(1024) unsigned char lds[2 * STAGE > EPI ? 2 * STAGE : EPI];
    __shared__ int expert[32];
    __shared__ float gate[32];

    const int tile = ((int)blockIdx.x & 7) * tg.per_xcd + ((int)blockIdx.x >> 3);
    if (tile >= tg.total) return;
    const int g = tile / tg.m_tiles, m0 = (tile - g * tg.m_tiles) * ROWS, M = up.l, W = up.kact * up.d_e, d_e = up.d_e;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lr = lane & 31, lh = lane >> 5;
    const int row0 = m0 + wave * 32;

    // the wave's tokens: k = ks*16 + lh*8 .. +7 of row lr
    bf16x8_t uf[DT * 2];
    {
        const bf16_t *src = up.u + ((size_t)g * M + min(row0 + lr, M - 1)) * D + lh * 8;
#pragma unroll
        for (int ks = 0; ks < DT * 2; ++ks) uf[ks] = __builtin_bit_cast(bf16x8_t, load16<false>(src + ks * 16));
    }
    if constexpr (SEL) up.template select<NW * 64>(g, tile - g * tg.m_tiles, lds, tid);
    if (tid < up.kact) {
        expert[tid] = up.expert(g, tid);
        gate[tid] = up.col_scale(g, tid * d_e);
    }
    __syncthreads();

    // Loads of a stage.  W1: slot (r, pos) <- chunk pos ^ (((r >> 1) & 1) << 2) of row r (rows of 128 bytes); W2: as the engine's [k][n] tiles, and
    // as they lie where rows are an odd number of 64 bytes (four of them are in different banks by themselves).  Either half of the stage's columns is
    // one expert's: a lane's address is its place in a tile plus its half's offset (32 bits, uome_mlp_waves).
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    auto swz = [](int row) { return D % 128 == 0 ? (row & 3) << 2 : (D % 64 == 0 ? ((row >> 1) & 1) << 2 : 0); };
    auto issue = [&](int stage) {
        int ln = lane;   // (see the fragment offsets)
        asm volatile("" : "+v"(ln));
        const int h0 = stage * HC, h1 = h0 + 32 < W ? h0 + 32 : h0;   // (a last stage of 32 columns: the same twice)
        const int s0 = h0 / d_e, s1 = h1 / d_e;
        const uint32_t e0 = __builtin_amdgcn_readfirstlane(expert[s0]), e1 = __builtin_amdgcn_readfirstlane(expert[s1]);
        const uint32_t at = base + (stage & 1) * STAGE;
        const int chunk = (ln & 7) ^ (((ln >> 4) & 1) << 2);
        const uint32_t w1_half = chunk < 4 ? e0 * (uint32_t)(D * d_e) + (h0 - s0 * d_e) : e1 * (uint32_t)(D * d_e) + (h1 - s1 * d_e);
        const uint32_t w1 = (w1_half + (ln >> 3) * d_e + (chunk & 3) * 8) * 2;
        const uint32_t w2_0 = (e0 * (uint32_t)d_e + (h0 - s0 * d_e)) * (D * 2), w2_1 = (e1 * (uint32_t)d_e + (h1 - s1 * d_e) - 32) * (D * 2);
#pragma unroll
        for (int i = 0; i < (INSTR + NW - 1) / NW; ++i) {
            const int q = i * NW + wave;
            if (INSTR % NW == 0 || q < INSTR) dma_load16_at(up.a_in, w1 + (uint32_t)(q * 16 * d_e), at + q * 1024);
        }
#pragma unroll
        for (int i = 0; i < (INSTR + NW - 1) / NW; ++i) {
            const int q = i * NW + wave, slot = q * 64 + ln, row = slot / CD, pos = slot - row * CD;
            if (INSTR % NW == 0 || q < INSTR)
                dma_load16_at(dn.a_out, (row < 32 ? w2_0 : w2_1) + row * (D * 2) + (pos ^ swz(row)) * 16, at + W_BYTES + q * 1024);
        }
    };

    f32x16_t acc[DT];
#pragma unroll
    for (int j = 0; j < DT; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;

    const int stages = (W + HC - 1) / HC;
    issue(0);
    // u has to be here before the loop: the compiler's own wait for it would stand at its first use and drain the copies at every turn
#pragma unroll
    for (int ks = 0; ks < DT * 2; ++ks) asm volatile("" : "+v"(uf[ks]));
    // A tile of 32 hidden columns takes 2*DT fragments of W1, then 2*DT of W2.  They are read RING products ahead, also across the SiLU and into the
    // next tile of the stage (16 x 4096 x 256, each read waited for in front of its product: 36 us traced, 31 so; eight ahead no faster).
    constexpr int N = DT * 2, TILES = HC / 32, RING = NW == 4 || DT <= 4 ? 8 : 4;
    bf16x8_t ring[RING];
    const bool live = row0 < M;
    for (int s = 0; s < stages; ++s) {
        dma_wait<0>();
        __syncthreads();   // the stage has landed, and the other buffer's readers are done
        if (s + 1 < stages) issue(s + 1);
        if (!live) continue;
        // Fragment offsets: 32 columns from a tile's first; rows k0.. as the first product takes them (lh*8 + 0..7) and as the second one finds
        // them in the first one's accumulators (lh*4 + 0..3, 8 + lh*4 + 0..3).  Formed at every turn, from a lane number that the compiler cannot
        // see through: kept over the loop they took registers there are none of, and a reload waits for the copies in flight.
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int x = (ln & 15) >> 2, part = ((ln >> 4) & 1) * 2 + ((ln & 3) >> 1), h2 = ln >> 5;
        const uint32_t st = (uint32_t)((s & 1) * STAGE + (ln & 1) * 8), w1_off = st + (h2 * 8 + x) * (HC * 2), w2_off = st + W_BYTES + (h2 * 4 + x) * (D * 2);
        const uint32_t w1_swz = ((x >> 1) & 1) << 2, w2_swz = swz(x);
        auto w1_frag = [&](int t, int ks) {
            const uint16_t *p = reinterpret_cast<const uint16_t *>(lds + w1_off + ((t * 4 + part) ^ w1_swz) * 16 + ks * 16 * (HC * 2));
            const uint2 a = lds_read_tr4(p), b = lds_read_tr4(p + 4 * HC);
            return __builtin_bit_cast(bf16x8_t, make_uint4(a.x, a.y, b.x, b.y));
        };
        auto w2_frag = [&](int k0, int j) {
            const uint16_t *p = reinterpret_cast<const uint16_t *>(lds + w2_off + ((j * 4 + part) ^ w2_swz) * 16 + k0 * (D * 2));
            const uint2 a = lds_read_tr4(p), b = lds_read_tr4(p + 8 * D);
            return __builtin_bit_cast(bf16x8_t, make_uint4(a.x, a.y, b.x, b.y));
        };
        // fragment f of the stage; behind a last stage's only tile they are read all the same (finite: a clamped copy of its columns)
        auto frag = [&](int f) {
            const int t = f / (2 * N), i = f % (2 * N);
            return i < N ? w1_frag(t, i) : w2_frag(t * 32 + (i - N) / DT * 16, (i - N) % DT);
        };
#pragma unroll
        for (int i = 0; i < RING; ++i) ring[i] = frag(i);
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            if (s * HC + t * 32 >= W) break;
            const float w = gate[(s * HC + t * 32) / d_e];
            f32x16_t z;
#pragma unroll
            for (int q = 0; q < 16; ++q) z[q] = 0.f;
            auto next = [&](int f) {   // the slot of fragment f is free
                if (f + RING < TILES * 2 * N) ring[f % RING] = frag(f + RING);
                __builtin_amdgcn_sched_barrier(0);
            };
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int f = t * 2 * N + i;
                z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[f % RING], uf[i], z, 0, 0, 0);
                next(f);
            }
            // the second half's SiLU between the first half's products
            bf16x8_t h;
            auto pack = [&](int k) {
                uint32_t p[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = pack2_bf16(z[k * 8 + 2 * e], z[k * 8 + 2 * e + 1]);
                h = __builtin_bit_cast(bf16x8_t, make_uint4(p[0], p[1], p[2], p[3]));
            };
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = up.epi(z[e], w);
            pack(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int f = t * 2 * N + N + i;
                acc[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[f % RING], h, acc[i % DT], 0, 0, 0);
                if (i < DT) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (e * DT / 8 == i) z[8 + e] = up.epi(z[8 + e], w);
                }
                if (i == DT - 1) pack(1);
                next(f);
            }
        }
    }
    __syncthreads();   // LDS is free for the epilogue
    if (!live) return;
    // The residual's pieces are under way while the tile is staged (u's registers hold them), 16 bytes a lane, neighbouring lanes in a row; rounded as in
    // the second layer's own launch: the product first.
    constexpr int PIECES = D / 16;
    const bool res = dn.has_residual();
    uint4 piece[PIECES];
    const size_t at0 = ((size_t)g * M + row0) * D;
    const int rows = M - row0;
#pragma unroll
    for (int t = 0; t < PIECES; ++t) {
        const int c = lane + t * 64, r = c / CD;
        if (res) piece[t] = dn.once ? load16<true>(dn.u + at0 + (size_t)min(r, rows - 1) * D + (c - r * CD) * 8)
                                    : load16<false>(dn.u + at0 + (size_t)min(r, rows - 1) * D + (c - r * CD) * 8);
    }
    uint16_t(*tile_out)[SPITCH] = reinterpret_cast<uint16_t(*)[SPITCH]>(lds) + wave * 32;
#pragma unroll
    for (int j = 0; j < DT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<uint2 *>(&tile_out[lr][j * 32 + q * 8 + lh * 4]) = make_uint2(pack2_bf16(acc[j][q * 4], acc[j][q * 4 + 1]), pack2_bf16(acc[j][q * 4 + 2], acc[j][q * 4 + 3]));
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < PIECES; ++t) {
        const int c = lane + t * 64, r = c / CD, col = (c - r * CD) * 8;
        uint4 v = *reinterpret_cast<const uint4 *>(&tile_out[r][col]);
        if (res) v = add8_bf16(v, piece[t]);
        if (r < rows) {
            if (dn.once) store16<true>(dn.out + at0 + (size_t)r * D + col, v);
            else store16<false>(dn.out + at0 + (size_t)r * D + col, v);
        }
    }
}

// Waves of a workgroup: 8, 4, or 0 where the two launches are better.  What counts is how full the last round of one workgroup a compute unit is, of
// tokens: a wave's 32, whatever the sample leaves of them, go through all hidden columns one after the other.  us, two launches / eight / four waves:
//   16 x 4096 x 256, W (hidden columns) 256       41.8  30.9  42.2      12 x 4096 x 256, W 1024 (0.75 full)      86.3  62.6  99.0
//   16 x 4096 x 128, W 1024                       85.2  48.1  53.1      20 x 4096 x 256, W 256 (0.63)            58.5  48.9  56.1
//   16 x 4096 x 64, W 1024                        71.1  32.2  36.8       8 x 4096 x 256, W 1024 (0.5; four: 1)   56.6  62.5  52.8
//   128 x 196 x 192, W 768 (0.38; four: 0.77)     41.5  39.6  34.4      24 x 1024 x 128, W 1024 (0.38; 0.75)     37.6  39.7  34.3
//   128 x 196 x 256, W 384 (0.38; 0.77)           26.1  30.6  25.9      20 x 1024 x 128, W 1024 (0.31; 0.63)     33.8  40.0  34.1
//   8 x 2048 x 256, W 1024 (0.25; 0.5)            33.6  58.8  50.1      128 x 100 x 192, W 768 (0.2; 0.39)       25.5  27.5  32.5
// Four waves are alone on their SIMDs and not for d = 256, where they gain 7 % at the most, nor for more than two rounds of d > 128 unless the rounds are full
// (forward, two launches and four waves: 10 x 7556 x 224, W 576, 600 workgroups, 180 and 192; 23 x 3244 x 192, W 96, 598, 101 and 106; 54 x 1132 x 192,
// W 448, 486, 122 and 116; 89 x 1300 x 224, W 32, 979, 159 and 146; 12 x 6472 x 128, W 800, 612, 163 and 137).
int uome_mlp_waves(const UomeArgs &a)
{
    if (a.d > 256 || a.d % 32 || a.d_e % 32 || (double)a.n * a.d * a.d_e * sizeof(bf16_t) > 4.0e9) return 0;   // (32-bit offsets into a weight)
    const auto wgs = [&](int rows) { return (long)a.b * ((a.l + rows - 1) / rows); };
    const auto full = [&](int rows) { return (double)a.b * a.l / ((double)((wgs(rows) + 255) / 256) * 256 * rows); };
    if (full(256) >= 0.6) return 8;
    return a.d <= 224 && full(128) >= (a.d > 128 && wgs(128) > 512 ? 0.85 : 0.75) ? 4 : 0;
}

template <int DT, int NW, bool SEL> static hipError_t launch_mlp_as(const UomeUpProblem<bf16_t, false, false, SEL> &up, const UomeDownProblem<bf16_t> &dn, int b, hipStream_t st)
{
    TileGrid tg;
    const hipError_t err = make_tile_grid<NW * 32, 64>(tg, b, up.l, 1);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL((uome_mlp_kernel<DT, NW, SEL>), dim3(tg.per_xcd * 8), dim3(NW * 64), 0, st, up, dn, tg);
    return hipGetLastError();
}
template <int DT, bool SEL> static hipError_t launch_mlp(const UomeUpProblem<bf16_t, false, false, SEL> &up, const UomeDownProblem<bf16_t> &dn, int b, bool four, hipStream_t st)
{
    if constexpr (DT < 8)   // (uome_mlp_waves)
        if (four) return launch_mlp_as<DT, 4, SEL>(up, dn, b, st);
    return launch_mlp_as<DT, 8, SEL>(up, dn, b, st);
}

template <bool SEL> static hipError_t launch_uome_mlp_as(const UomeArgs &a, hipStream_t st)
{
    UomeUpProblem<bf16_t, false, false, SEL> up;
    if constexpr (SEL) up.sel = *a.select;
    up.u = static_cast<const bf16_t *>(a.u);
    up.a_in = static_cast<const bf16_t *>(a.a_in);
    up.expert_idx = a.expert_idx;
    up.expert_gate = (a.flags & F_GATE_EXPERT) ? a.expert_gate : nullptr;
    up.hidden = nullptr;
    up.l = a.l; up.d = a.d; up.n = a.n; up.kact = a.k; up.d_e = a.d_e;
    UomeDownProblem<bf16_t> dn;
    dn.hidden = nullptr;
    dn.a_out = static_cast<const bf16_t *>(a.a_out);
    dn.u = static_cast<const bf16_t *>(a.u);
    dn.expert_idx = a.expert_idx;
    dn.out = static_cast<bf16_t *>(a.out);
    dn.l = a.l; dn.d = a.d; dn.n = a.n; dn.kact = a.k; dn.d_e = a.d_e; dn.flags = a.flags;
    dn.once = stream_once((size_t)a.b * a.l * a.d * sizeof(bf16_t));
    const bool four = uome_mlp_waves(a) == 4;
    switch (a.d / 32) {
        case 1: return launch_mlp<1, SEL>(up, dn, a.b, four, st);
        case 2: return launch_mlp<2, SEL>(up, dn, a.b, four, st);
        case 3: return launch_mlp<3, SEL>(up, dn, a.b, four, st);
        case 4: return launch_mlp<4, SEL>(up, dn, a.b, four, st);
        case 5: return launch_mlp<5, SEL>(up, dn, a.b, four, st);
        case 6: return launch_mlp<6, SEL>(up, dn, a.b, four, st);
        case 7: return launch_mlp<7, SEL>(up, dn, a.b, four, st);
        default: return launch_mlp<8, SEL>(up, dn, a.b, four, st);
    }
}

hipError_t launch_uome_mlp(const UomeArgs &a, hipStream_t st) { return a.select ? launch_uome_mlp_as<true>(a, st) : launch_uome_mlp_as<false>(a, st); }

}  // namespace uoe
