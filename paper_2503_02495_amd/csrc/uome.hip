// Union-of-MLP-Experts, expert-selection mode (Eq. 38-40 with Eq. 24-26), sample-major:
// a sample's k active experts are column slices of A^I and row slices of A^O, so together they
// are ONE two-layer MLP of hidden width k*d_e for that sample.  GEMM-1 writes the gated
// SiLU hidden activations [l, k*d_e]; GEMM-2 contracts over the stacked K = k*d_e and writes every
// output row once with the residual added: no per-expert partial outputs, no atomics.
#include "common.h"
#include "problems.h"
#include "gemm_mfma.h"
#include "gemm_dma.h"

namespace uoe {

// any width, either storage type (SiLU by a division: the reciprocal of silu_fast is zero where the sigmoid is no normal
// number, z <= -87.4; 6 x 1000 tokens, d 360, 3 x 232 hidden columns: 2 us of 89 for the layer's forward)
template <typename T, bool SEL> static hipError_t uome_up_tail(const UomeArgs &a, hipStream_t st)
{
    UomeUpProblem<T, false, true, SEL> up;
    if constexpr (SEL) up.sel = *a.select;
    up.u = static_cast<const T *>(a.u);
    up.a_in = static_cast<const T *>(a.a_in);
    up.expert_idx = a.expert_idx;
    up.expert_gate = (a.flags & F_GATE_EXPERT) ? a.expert_gate : nullptr;
    up.hidden = static_cast<T *>(a.hidden);
    up.l = a.l; up.d = a.d; up.n = a.n; up.kact = a.k; up.d_e = a.d_e;
    return launch_gemm_tail<0>(up, a.b, a.l, a.k * a.d_e, st);
}

template <typename T> static hipError_t uome_down_tail(const UomeArgs &a, hipStream_t st)
{
    UomeDownProblem<T> dn;
    dn.hidden = static_cast<const T *>(a.hidden);
    dn.a_out = static_cast<const T *>(a.a_out);
    dn.u = static_cast<const T *>(a.u);
    dn.expert_idx = a.expert_idx;
    dn.out = static_cast<T *>(a.out);
    dn.l = a.l; dn.d = a.d; dn.n = a.n; dn.kact = a.k; dn.d_e = a.d_e; dn.flags = a.flags;
    return launch_gemm_tail<0>(dn, a.b, a.l, a.d, st);
}

// MFMA path: bf16 storage, and every K segment (d for GEMM-1, d_e for GEMM-2) a multiple of 32
static bool uome_mfma_ok(const UomeArgs &a, bool bf16) { return bf16 && a.d % 32 == 0 && a.d_e % 32 == 0; }

template <bool SEL> static hipError_t uome_up_mfma(const UomeArgs &a, hipStream_t st)
{
    UomeUpProblem<bf16_t, false, false, SEL> up;
    if constexpr (SEL) up.sel = *a.select;
    up.u = static_cast<const bf16_t *>(a.u);
    up.a_in = static_cast<const bf16_t *>(a.a_in);
    up.expert_idx = a.expert_idx;
    up.expert_gate = (a.flags & F_GATE_EXPERT) ? a.expert_gate : nullptr;
    up.hidden = static_cast<bf16_t *>(a.hidden);
    up.l = a.l; up.d = a.d; up.n = a.n; up.kact = a.k; up.d_e = a.d_e;
    up.once = stream_once((size_t)a.b * a.l * a.k * a.d_e * sizeof(bf16_t));
    return launch_gemm_dma_auto(up, a.b, a.l, a.k * a.d_e, a.d, a.d, st);  // K segment = d
}

static hipError_t uome_down_mfma(const UomeArgs &a, hipStream_t st)
{
    UomeDownProblem<bf16_t> dn;
    dn.hidden = static_cast<const bf16_t *>(a.hidden);
    dn.a_out = static_cast<const bf16_t *>(a.a_out);
    dn.u = static_cast<const bf16_t *>(a.u);
    dn.expert_idx = a.expert_idx;
    dn.out = static_cast<bf16_t *>(a.out);
    dn.l = a.l; dn.d = a.d; dn.n = a.n; dn.kact = a.k; dn.d_e = a.d_e; dn.flags = a.flags;
    dn.once = stream_once((size_t)a.b * a.l * a.d * sizeof(bf16_t));
    return launch_gemm_dma_auto(dn, a.b, a.l, a.d, (long)a.k * a.d_e, a.d_e, st);  // K segments = the active experts' d_e rows
}

// Selecting beside the first layer saves 1 to 2 us of a launch's 4 to 5; the rest goes with every workgroup's own sums.  It does while the workgroups start
// at about the same time (counted in 128 x 128 tiles, 64 x 64 in fp32, or in those of both layers' launch) and have few partials to add up.  Forward,
// us, with a launch and beside (tiles, partials): 19 x 628 x 704, W (hidden columns) 960 (760, 7536) 114.8 and 113.7; 32 x 944 x 72, W 480 (1024, 7552)
// 74.9 and 76.2; 13 x 680 x 160, W 320 (234, 16320) 59.8 and 62.6; 2 x 572 x 224, W 2304 (180, 13728) 60.8 and 61.8; 5 x 700 x 208, W 1568 (546, 11200)
// 68.1 and 67.0; fp32 26 x 1132 x 128, W 88 (936, 252) 138.7 and 140.5, 23 x 156 x 248, W 672 (759, 468) 92.5 and 91.1; both layers in one launch, 16 x
// 4096 x 256, W 256 and 1024 (256, 4096) 89.7 and 88.6, 133.7 and 132.2.
int uome_select_values(const UomeArgs &a, bool bf16)
{
    const int waves = bf16 ? uome_mlp_waves(a) : 0, tile = bf16 ? 128 : 64;
    const long wgs = waves ? (long)a.b * ((a.l + waves * 32 - 1) / (waves * 32)) : (long)a.b * ((a.l + tile - 1) / tile) * ((a.k * a.d_e + tile - 1) / tile);
    return wgs <= 768 ? 12 * 1024 : 0;
}

hipError_t launch_uome_up(const UomeArgs &a, bool bf16, hipStream_t st)
{
    if (uome_mfma_ok(a, bf16)) return a.select ? uome_up_mfma<true>(a, st) : uome_up_mfma<false>(a, st);
    if (bf16) return a.select ? uome_up_tail<bf16_t, true>(a, st) : uome_up_tail<bf16_t, false>(a, st);
    return a.select ? uome_up_tail<float, true>(a, st) : uome_up_tail<float, false>(a, st);
}

hipError_t launch_uome_down(const UomeArgs &a, bool bf16, hipStream_t st)
{
    if (uome_mfma_ok(a, bf16)) return uome_down_mfma(a, st);
    return bf16 ? uome_down_tail<bf16_t>(a, st) : uome_down_tail<float>(a, st);
}

hipError_t launch_uome(const UomeArgs &a, bool bf16, hipStream_t st)
{
    if (bf16 && uome_mlp_waves(a)) return launch_uome_mlp(a, st);
    const hipError_t err = launch_uome_up(a, bf16, st);
    return err != hipSuccess ? err : launch_uome_down(a, bf16, st);
}

}  // namespace uoe
