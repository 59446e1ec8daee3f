// How the weight gradients of the backward passes are cut into parts (host side; plain C++).
#pragma once

namespace uoe {

// How the sums of the weight gradients over an expert's tokens are cut into parts, one fp32 partial tile (or grid of them) each.  The
// samples go in chunks of 128 (a workgroup's tables); within a chunk an expert has `items` items for each (sample, slot) pair that
// selected it (picked patches, or ranges of the token axis), in sample order, and its list is cut evenly into parts of at most `per`.
// Experts are not selected equally often: with the same number of parts for each the launch took as long as the most popular one
// (4 x 8192 tokens, 8 of 16 experts of 1024 x 256: 352 us, 255 to 268 with equal parts).
// Finding them takes 1 to 2 us, so experts keep one number of parts (`each`) where that is one, where a part is short (less than 256 tokens
// on the average, 512 in fp32: 6 x 120 x 608, 6 of 12 experts of 64, 242 us for the layer's forward + backward, 249 with equal parts), and with 20
// pairs and more an expert (128 samples, 3 of 6 experts: within 10 % of each other; 96 us became 112 and 99 in the two orders there
// are for unequal parts; 57 x 128 x 96, 4 of 11: 168.6 -> 174.0 for forward + backward; fp32 8 x 512 x 512, 4 of 8: 559 -> 535 with one selection, 547 -> 556 with
// another that was nearly even).
// `per` is the least for which no more than `parts` parts come of it, found by every workgroup from the selection (PartScan).
struct WgradPlan {
    int chunks, items, parts;
    int lo, hi;        // bounds of `per`: all parts full; feasible for any selection
    int each;          // not 0: an expert has so many parts, whatever its list (experts with many pairs: their lists hardly differ)
};
// `splits`: parts of an expert with the average number of pairs; `cap`: entries of a workgroup's segment table; item_k: tokens of an item, half of them in fp32
inline WgradPlan wgrad_plan(int b, int n, int k, int splits, int items, int cap, int item_k)
{
    const int nb = b < 128 ? b : 128, most = nb * items;   // most: an expert every sample selected
    const int need = (most + cap - 1) / cap;
    splits = splits > need ? splits : need;                // (with `cap` items a part an expert has at most `splits` of them)
    const long total = (long)nb * k * items, parts = (long)n * splits;
    const long lo = (total + parts - 1) / parts;
    // sum over experts of ceil(items of the expert / per) <= total / per + n
    long hi = splits > 1 ? (total + parts - n - 1) / (parts - n) : most;
    hi = hi < most ? hi : most;
    hi = hi < cap ? hi : cap;
    WgradPlan w;
    w.chunks = (b + 127) / 128;
    w.items = items;
    w.parts = (int)parts;
    w.each = splits == 1 || total * item_k < 256 * parts || (long)nb * k >= 20L * n ? splits : 0;
    w.lo = (int)(lo < hi ? lo : hi);
    w.hi = (int)hi;
    return w;
}

// Expert-selection UoME on the 32-grid
inline WgradPlan uome_backward_wgrad(int b, int l, int d, int n, int k, int d_e)
{
    // parts until the launch of both gradients has 512 tiles of 256 x 128, while one keeps on average >= 1024 of K; two of them also
    // where one would do, for experts with longer lists.  (Until one gradient has 512: 4 x 8192 tokens, 16 experts of 1024 x 256, 128
    // instead of 64 MB of fp32 tiles written and read again: 1974 against 1944 us for the layer's forward + backward.)  Pairs are cut
    // into ranges of tokens, a multiple of 64, until a part has two items (for lists that do not divide evenly) and there are as many as
    // parts: no part can then be longer than with the token axis cut so often (8 x 512, 4 of 8 experts, whole pairs: the longest part longer
    // than that for 20 % of random selections).
    int s = 1, ranges = 1;
    const long pairs = (long)b * k, k_avg = pairs * l / n, tiles = (long)n * ((d_e + 255) / 256) * ((d + 127) / 128);
    while (s < 8 && tiles * s < (s == 1 ? 512 : 256) && k_avg / (2 * s) >= 1024) s *= 2;
    while ((pairs * ranges < 2L * n * s || ranges < s) && l % (2 * ranges * 64) == 0) ranges *= 2;
    return wgrad_plan(b, n, k, s, ranges, 128, l / ranges);
}

// Lists of picked patches on the 32-grid: SMHA (4 sets), UoME with data selection (2)
inline WgradPlan smha_backward_wgrad(int b, int n, int k, int c, int l_p, int sets, int rows, int cols)
{
    // parts of an average expert's (unit, pick) list: about 8 segments each, and at most 8 parts; not more than two where 256 tiles
    // of 128 x 128 come of it, a part's fp32 tiles being written and read again (4 x 8192 tokens, 16 experts of 64 x 1024: 4 parts
    // 66 us and 16 for the reduction, 2 parts 54 and 12; 8 x 512, 8 of 256 x 512: 27 and 23)
    const int avg = (int)(((long)b * k * c + n - 1) / n);
    const long tiles = (long)sets * n * ((rows + 127) / 128) * ((cols + 127) / 128), most = tiles >= 128 ? 2 : (256 + tiles - 1) / tiles;
    long s = avg / 8;
    s = s < 1 ? 1 : (s > 8 ? 8 : s);
    return wgrad_plan(b, n, k, (int)(s < most ? s : most), c, 128, l_p);
}

// Expert-selection UoME of any shape or in fp32, `splits` parts an average expert; tokens of an item, pairs cut into `items`
inline int uome_any_range(int l, int items) { return items == 1 ? l : ((l + items - 1) / items + 31) / 32 * 32; }
inline WgradPlan uome_any_wgrad(int b, int l, int n, int k, int splits, bool f32)
{
    // as many ranges a pair as parts, whole pairs from four pairs a part on: no part can be longer than with the token axis (the list of
    // pairs) cut so often.  (Two items a part: ranges of 128 tokens instead of 64 for 8 x 512, 4 of 8 experts, and the longest part
    // longer for 43 % of random selections, with parts of as many items and of equal length alike.)
    int items = (long)b * k >= 4L * n * splits ? 1 : splits;
    if (items > 1) items = (l + uome_any_range(l, items) - 1) / uome_any_range(l, items);   // (as many as there are)
    const int range = uome_any_range(l, items);
    return wgrad_plan(b, n, k, splits, items, 128, f32 ? range / 2 : range);
}

}  // namespace uoe
