// What the grouped GEMMs (gemm_dma.h) and the attention kernels share on the matrix cores (gfx950): fragment reads, the
// epilogue of a wave tile, the workgroup order.
//
// Operand layout.  The MFMA wants, per lane, 8 K-consecutive values of one row of its first operand and of one column
// of its second.  Activations A are [M,K] with K contiguous: a 16-byte LDS read of a row is already a fragment.
// Weights B are [K,N] with N contiguous (the paper's [n,d,width] layout); they are copied to LDS as they are, [k][n], and
// the fragments are taken with the gfx950 transposing LDS read (ds_read_b64_tr_b16): in a group of 16 lanes, lane j points
// at row k0 + j/4, columns c0 + 4*(j%4)..+3, and lane i receives column c0 + i, rows k0..k0+3.
// The product is computed transposed, D = B^T A^T (weights as the first MFMA operand), so that an accumulator lane is one
// output ROW and its registers run along N in groups of four: the epilogue can then hand 8-byte row pieces to LDS and
// write 16-byte row pieces to memory.
#pragma once
#include <type_traits>
#include <utility>
#include "common.h"

namespace uoe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;

// 4 K-consecutive values of one column from a [k][n] LDS tile (see the header comment)
__device__ __forceinline__ uint2 lds_read_tr4(const uint16_t *p)
{
    const s16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
    return __builtin_bit_cast(uint2, v);
}

__host__ __device__ constexpr int largest_divisor_upto(int n, int cap)
{
    int b = cap < n ? cap : n;
    while (n % b) --b;
    return b;
}

// Epilogue of one wave.  acc is the transposed-product accumulator of a TM x TN grid of 32x32
// tiles: register q of lane (lr, lh) in tile (i, j) is output row i*32 + lr, column
// j*32 + (q/4)*8 + lh*4 + q%4 of the wave tile.  The wave stages its tile in LDS (stage: WM rows
// of SPITCH elements, private to the wave) and then moves 16-byte pieces of rows to memory,
// residual pieces loaded a batch ahead of the stores.  wcol0 = first column of the wave tile
// inside the workgroup tile (indexes coltab); (grow0, gcol0) = its global position.
// Per-row factors of the rows this lane owns in the epilogue (rows i*32 + lane%32 of the wave tile),
// fetched before the K loop like the column factors.
template <typename P, int TM>
__device__ __forceinline__ void load_row_scale(const P &p, float (&rs)[TM], int g, int grow0, int M, int lane)
{
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        rs[i] = 1.0f;
        if constexpr (P::kRowScale) {
            const int row = grow0 + i * 32 + (lane & 31);
            rs[i] = p.row_scale(g, row < M ? row : M - 1);
        }
    }
}

// problems that store fp32 tiles straight from the accumulators declare kF32Out and put4_f32
template <typename P, typename = void> struct writes_f32 {
    static constexpr bool value = false;
};
template <typename P> struct writes_f32<P, std::void_t<decltype(P::kF32Out)>> {
    static constexpr bool value = P::kF32Out;
};

// problems that store some column blocks as fp16 instead of bf16 declare f16_col(column)
template <typename P, typename = void> struct has_f16_cols {
    static constexpr bool value = false;
};
template <typename P> struct has_f16_cols<P, std::void_t<decltype(&P::f16_col)>> {
    static constexpr bool value = true;
};
// problems that rotate pairs of columns on the way out: kRotates, rotates(first column of 8), rotate(row, column, 4 values)
template <typename P, typename = void> struct has_rotation : std::false_type {};
template <typename P> struct has_rotation<P, std::void_t<decltype(P::kRotates)>> : std::bool_constant<P::kRotates> {};
// two fp32 -> packed fp16, round to nearest even
__device__ __forceinline__ uint32_t pack2_f16_rn(float a, float b)
{
    const _Float16 ha = (_Float16)a, hb = (_Float16)b;
    return (uint32_t)__builtin_bit_cast(uint16_t, ha) | ((uint32_t)__builtin_bit_cast(uint16_t, hb) << 16);
}

template <typename P, typename = void> struct streams_once : std::false_type {};
template <typename P> struct streams_once<P, std::void_t<decltype(std::declval<P>().once)>> : std::true_type {};

// problems that take the accumulators themselves: acc_out<TM, TN>(acc, rs, g, first row, first column, M, N, lane)
template <typename P, typename = void> struct takes_acc : std::false_type {};
template <typename P> struct takes_acc<P, std::void_t<decltype(P::kAccOut)>> : std::true_type {};
// problems that take the tile of another contraction beside their own: pair_out<TM, TN, SPITCH>(acc, first, stage, column factors, g, ...)
template <typename P, typename = void> struct takes_pair : std::false_type {};
template <typename P> struct takes_pair<P, std::void_t<decltype(P::kPairOut)>> : std::true_type {};
// problems with a second half of their own: write_out<TM, TN, SPITCH>(stage, coltab + first 8-column group, rs, ...)
template <typename P, typename = void> struct writes_itself : std::false_type {};
template <typename P> struct writes_itself<P, std::void_t<decltype(P::kWriteOut)>> : std::true_type {};

// problems whose epilogue reads a tensor of the output's shape: has_early(), early8<ONCE>(g, row, column).  EarlyPieces holds a wave
// tile's pieces of it where the engine fetches them ahead: the first eight under the last K-step, the others while the tile is staged.
template <typename P, typename = void> struct has_early_pieces : std::false_type {};
template <typename P> struct has_early_pieces<P, std::void_t<decltype(&P::has_early)>> : std::true_type {};
template <int TM, int TN> struct EarlyPieces {
    static constexpr int N = TM * TN * 2, BATCH = largest_divisor_upto(N, 8);
    uint4 piece[N];
    template <bool ONCE, typename P>
    __device__ __forceinline__ void fetch_as(const P &p, int from, int to, int g, int grow0, int gcol0, int M, int N_, int lane)
    {
#pragma unroll
        for (int t = 0; t < N; ++t) {
            if (t < from || t >= to) continue;
            const int c = lane + t * 64, col = gcol0 + c % (TN * 4) * 8;
            piece[t] = p.template early8<ONCE>(g, min(grow0 + c / (TN * 4), M - 1), col < N_ ? col : 0);   // (unconditional: all in flight together)
        }
    }
    template <typename P> __device__ __forceinline__ void fetch(const P &p, int from, int to, int g, int grow0, int gcol0, int M, int N_, int lane)
    {
        if (!p.has_early()) return;
        if (p.once) fetch_as<true>(p, from, to, g, grow0, gcol0, M, N_, lane);
        else fetch_as<false>(p, from, to, g, grow0, gcol0, M, N_, lane);
    }
};
struct NoEarlyPieces {};

// second half of the epilogue: the staged wave tile back out of LDS in 16-byte pieces, the residual
// added, the pieces stored (ONCE: through the problem's non-temporal accessors)
template <typename P, int TM, int TN, int SPITCH, bool ONCE, typename EARLY>
__device__ __forceinline__ void wave_write_out(const P &p, uint16_t (*stage)[SPITCH], int g, int grow0, int gcol0, int M, int N, int lane,
                                               const EARLY &early)
{
    constexpr bool FETCHED = !std::is_same<EARLY, NoEarlyPieces>::value;
    constexpr int WM = TM * 32, WN = TN * 32;
    constexpr int WC = WN / 8;           // 16-byte pieces per staged row
    constexpr int NPIECE = (WM * WC) / 64;
    constexpr int BATCH = largest_divisor_upto(NPIECE, 8);
    const bool res = p.has_residual();
#pragma unroll
    for (int t0 = 0; t0 < NPIECE; t0 += BATCH) {
        uint4 r[BATCH];
        if constexpr (FETCHED) {
#pragma unroll
            for (int u = 0; u < BATCH; ++u) r[u] = early.piece[t0 + u];
        } else if (res) {
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int c = lane + (t0 + u) * 64;
                const int grow = grow0 + c / WC, gcol = gcol0 + (c % WC) * 8;
                if constexpr (streams_once<P>::value)
                    r[u] = (grow < M && gcol < N) ? p.template res8_as<ONCE>(g, grow, gcol) : make_uint4(0, 0, 0, 0);
                else r[u] = (grow < M && gcol < N) ? p.res8(g, grow, gcol) : make_uint4(0, 0, 0, 0);
            }
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int c = lane + (t0 + u) * 64;
            const int row = c / WC, pc = c % WC;
            const int grow = grow0 + row, gcol = gcol0 + pc * 8;
            uint4 piece = *reinterpret_cast<const uint4 *>(&stage[row][pc * 8]);
            if (res) piece = add8_bf16(piece, r[u]);
            if (grow < M && gcol < N) {
                if constexpr (streams_once<P>::value) p.template put8_as<ONCE>(g, grow, gcol, piece);
                else p.put8(g, grow, gcol, piece);
            }
        }
    }
}

// One 16-bit plane of a wave tile from the accumulators' layout to rows, through the wave's staging tile: words(i, j, q) are
// the lane's 4 values of row i*32 + lr, columns j*32 + q*8 + lh*4; put(row, first column, 8 values) takes 16-byte pieces, whose
// neighbouring lanes complete 64 bytes and more of a row (straight from the accumulators two lanes complete 16).  A lane's pieces are all of
// the same columns.  rows: of the tile, that are any; blocks of 32 behind them are left out.
template <int TM, int TN, int SPITCH, typename Words, typename Put>
__device__ __forceinline__ void stage_plane(uint16_t (*stage)[SPITCH], int lane, int rows, Words words, Put put)
{
    constexpr int WC = TN * 4, NPIECE = TM * 32 * WC / 64;
    const int lr = lane & 31, lh = lane >> 5;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (i && i * 32 >= rows) break;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2 *>(&stage[i * 32 + lr][j * 32 + q * 8 + lh * 4]) = words(i, j, q);
    }
    __builtin_amdgcn_wave_barrier();
    static_assert(64 % WC == 0, "a lane keeps its columns");
#pragma unroll
    for (int t = 0; t < NPIECE; ++t) {
        const int c = lane + t * 64, row = c / WC, col = c % WC * 8;
        if (t * 64 / WC % 32 == 0 && t && t * 64 / WC >= rows) break;
        put(row, col, *reinterpret_cast<const uint4 *>(&stage[row][col]));
    }
    __builtin_amdgcn_wave_barrier();
}

template <typename P, int TM, int TN, int SPITCH, typename EARLY = NoEarlyPieces>
__device__ __forceinline__ void wave_epilogue(const P &p, f32x16_t (&acc)[TM][TN], uint16_t (*stage)[SPITCH], const float *coltab,
                                              const float (&rs)[TM], int g, int grow0, int gcol0, int wcol0, int M, int N,
                                              int lane, const EARLY &early = EARLY())
{
    const int lr = lane & 31, lh = lane >> 5;
    if constexpr (writes_f32<P>::value) {
        // a lane holds 4 consecutive columns of one row per register quad: 16-byte stores; the two
        // half-waves and the four quads of a row complete its 128-byte line in L2
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int grow = grow0 + i * 32 + lr;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int qg = 0; qg < 4; ++qg) {
                    const int gcol = gcol0 + j * 32 + qg * 8 + lh * 4;
                    if (grow < M && gcol < N)
                        p.put4_f32(g, grow, gcol, make_float4(acc[i][j][qg * 4 + 0], acc[i][j][qg * 4 + 1],
                                                              acc[i][j][qg * 4 + 2], acc[i][j][qg * 4 + 3]));
                }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int qg = 0; qg < 4; ++qg) {
            const int cl = j * 32 + qg * 8 + lh * 4;  // first of 4 consecutive columns, wave-local
            float sc = 1.0f;
            if constexpr (P::kColScale) sc = coltab[(wcol0 + cl) >> 3];
            bool half = false;   // uniform over the wave: a column block's format
            if constexpr (has_f16_cols<P>::value) half = p.f16_col(gcol0 + j * 32 + qg * 8);
            bool rot = false;    // uniform as well
            if constexpr (has_rotation<P>::value) rot = p.rotates(gcol0 + j * 32 + qg * 8);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const float s2 = P::kRowScale ? sc * rs[i] : sc;
                float e0 = p.epi(acc[i][j][qg * 4 + 0], s2), e1 = p.epi(acc[i][j][qg * 4 + 1], s2);
                float e2 = p.epi(acc[i][j][qg * 4 + 2], s2), e3 = p.epi(acc[i][j][qg * 4 + 3], s2);
                if constexpr (has_rotation<P>::value) {
                    if (rot) p.rotate(grow0 + i * 32 + lr, gcol0 + cl, e0, e1, e2, e3);
                }
                const uint32_t w0 = half ? pack2_f16_rn(e0, e1) : pack2_bf16(e0, e1);
                const uint32_t w1 = half ? pack2_f16_rn(e2, e3) : pack2_bf16(e2, e3);
                *reinterpret_cast<uint2 *>(&stage[i * 32 + lr][cl]) = make_uint2(w0, w1);
                if constexpr (has_f16_cols<P>::value) {
                    const int grow = grow0 + i * 32 + lr;
                    if (half && p.v_copy && grow < M && gcol0 + cl < N) p.put4_copy(g, grow, gcol0 + cl, make_uint2(pack2_bf16(e0, e1), pack2_bf16(e2, e3)));
                }
            }
        }
    // no workgroup barrier: a wave reads back only what it staged itself, and the LDS executes one
    // wave's instructions in order
    __builtin_amdgcn_wave_barrier();
    // Problems with a `once` member choose per launch whether the residual read and the output store carry
    // the non-temporal hint; the choice is made here, once per wave, so that each version keeps its
    // batch of residual loads in flight (a test per access would put a branch between them).
    if constexpr (writes_itself<P>::value) {
        if constexpr (has_early_pieces<P>::value) p.template write_out<TM, TN, SPITCH>(stage, coltab + (wcol0 >> 3), rs, g, grow0, gcol0, M, N, lane, early);
        else p.template write_out<TM, TN, SPITCH>(stage, coltab + (wcol0 >> 3), rs, g, grow0, gcol0, M, N, lane);
    } else if constexpr (streams_once<P>::value) {
        if (p.once) wave_write_out<P, TM, TN, SPITCH, true>(p, stage, g, grow0, gcol0, M, N, lane, early);
        else wave_write_out<P, TM, TN, SPITCH, false>(p, stage, g, grow0, gcol0, M, N, lane, early);
    } else {
        wave_write_out<P, TM, TN, SPITCH, false>(p, stage, g, grow0, gcol0, M, N, lane, early);
    }
}

// smallest pad (in dwords) that makes (cols/2 + pad) % 64 equal to 16 or 48
__host__ __device__ constexpr int b_pitch_dwords(int cols)
{
    int p = cols / 2;
    while ((p % 64) != 16 && (p % 64) != 48) p += 4;
    return p;
}

// Workgroup order.  The grid is one-dimensional; hardware deals consecutive workgroup ids
// round-robin over the 8 XCDs (each with its own L2).  Id L therefore maps to tile
// (L % 8) * ceil(tiles / 8) + L / 8, with tiles numbered n-tile fastest, then m-tile, then group:
// every XCD works on one contiguous run of tiles, i.e. a few row-tiles of A times all column
// tiles, so an A row-tile and the group's weight slices are fetched into one L2 only.
struct TileGrid {
    int n_tiles, m_tiles, total, per_xcd;
};

}  // namespace uoe
