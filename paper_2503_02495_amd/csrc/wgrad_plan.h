// How the weight gradients of the backward passes are cut into parts (host side; plain C++).
#pragma once

namespace uoe {

// How the sums of the weight gradients over an expert's tokens are cut into parts, one fp32 partial tile (or grid of them) each.  The
// samples go in chunks of 128 (a workgroup's tables); within a chunk an expert has `items` items for each (sample, slot) pair that
// selected it (picked patches, or ranges of the token axis), in sample order, and its list is cut evenly into parts of at most `per`.
// Experts are not selected equally often: with the same number of parts for each the launch took as long as the most popular one
// (4 x 8192 tokens, 8 of 16 experts of 1024 x 256: 352 us, 255 to 268 with equal parts).
// Finding them takes 1 to 2 us (more off the 32-grid, where the order by samples goes with it and pairs are cut finer), so experts keep one number of
// parts (`each`) unless equal ones are shorter by 256 tokens (384 off the grid; lists of patches 192, off the grid 128) than those of an expert with a standard
// deviation more pairs than the average (68 x 200 x 352, one of 7 experts of 56, 250 and 350 tokens: 52.1 us for the MLP's backward, 49.2 with one
// number; 18 x 1680 x 288, one of 10 of 144, 378 and 840: 97.9 and 112; patches 8 x 512 x 512, 4 of 8 of 256, 544 and 768: 47.7 and 48.4).  With 20 pairs
// and more an expert lists hardly differ (128 samples, 3 of 6 experts: within 10 %; 96 us became 112 and 99 in the two orders there are for
// unequal parts), with half a one and less a few experts have all parts, which the reduction adds one after the other (1 x 5040 x 120, one of 6 of 200:
// 50.6 and 54.7).  Several experts that share the rows of a large tensor have equal parts, whose order brings those rows together, from 256 tokens a
// part on (13 x 3712 x 768, 3 of 9 experts of 32: 130 and 151; 21 x 1664 x 800, 6 of 13 of 64: 211 and 220).
// `per` is the least, of up to 64 values evenly between `lo` and `hi`, for which no more than `parts` parts come of it: every workgroup finds it
// from the selection (PartScan).
constexpr int WGRAD_MAX_PARTS = 8192;   // of a chunk: what a launch's groups are coded for
struct WgradPlan {
    int chunks, items, parts;
    int lo, hi;        // bounds of `per`: all parts full; feasible for any selection
    int each;          // not 0: an expert has so many parts, whatever its list
};
// the average number of pairs an expert, and a standard deviation more (each rounded up)
inline long wgrad_pairs(long pairs, int n) { return (pairs + n - 1) / n; }
inline long wgrad_more_pairs(long pairs, int n)
{
    long more = wgrad_pairs(pairs, n);
    while ((more * n - pairs) * (more * n - pairs) < pairs * n) ++more;
    return more;
}
// items of a part of an expert with that many pairs, one number of parts
inline long wgrad_one(long pairs, int n, int items, int splits) { return (wgrad_more_pairs(pairs, n) * items + splits - 1) / splits; }
// items of equal parts, in as many as `parts`: lists do not end on whole parts unless a pair does, half a part an expert on the average
inline long wgrad_fair(long pairs, int items, int n, long parts)
{
    const long lo = (pairs * items + parts - 1) / parts;
    return items % lo == 0 || 2 * pairs * items + n * (lo - 1) <= 2 * lo * parts ? lo : lo + 1;
}
// `splits`: parts of an expert with the average number of pairs; `cap`: entries of a workgroup's segment table; `tokens` of a pair; `elems` of the
// tensor whose rows the experts share (0: each has patches of its own); `one`: tokens of a part of wgrad_one, with other items (0: these)
inline WgradPlan wgrad_plan(int b, int n, int k, int splits, int items, int cap, long tokens, double elems, long one = 0, int gain = 256)
{
    const int nb = b < 128 ? b : 128, most = nb * items;   // most: an expert every sample selected
    const int need = (most + cap - 1) / cap;
    splits = splits > need ? splits : need;                // (with `cap` items a part an expert has at most `splits` of them)
    const long pairs = (long)nb * k, total = pairs * items, parts = (long)n * splits;
    const long lo = (total + parts - 1) / parts;
    // sum over experts of ceil(items of the expert / per) <= total / per + n
    long hi = splits > 1 ? (total + parts - n - 1) / (parts - n) : most;
    hi = hi < most ? hi : most;
    hi = hi < cap ? hi : cap;
    WgradPlan w;
    w.chunks = (b + 127) / 128;
    w.items = items;
    w.parts = (int)parts;
    w.lo = (int)(lo < hi ? lo : hi);
    w.hi = (int)hi;
    if (!one) one = wgrad_one(pairs, n, items, splits) * tokens / items;
    const bool pays = one - wgrad_fair(pairs, items, n, parts) * tokens / items >= gain || (k > 1 && elems >= 16e6 && pairs * tokens >= 256 * parts);
    w.each = splits > 1 && pairs < 20L * n && 2 * pairs > n && pays ? 0 : splits;
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
    return wgrad_plan(b, n, k, s, ranges, 128, l, (double)b * l * d);
}

// Lists of picked patches on the 32-grid: SMHA (4 sets), UoME with data selection (2)
inline WgradPlan smha_backward_wgrad(int b, int n, int k, int c, int l_p, int sets, int rows, int cols)
{
    // parts of an average expert's (unit, pick) list: about 8 segments each, and at most 8 parts; not more than two where 256 tiles
    // of 128 x 128 come of it, a part's fp32 tiles being written and read again (4 x 8192 tokens, 16 experts of 64 x 1024: 4 parts
    // 66 us and 16 for the reduction, 2 parts 54 and 12; 8 x 512, 8 of 256 x 512: 27 and 23); fewer tiles: SMHA's heads of 128, whose launch is then one of
    // its own, until the compute units' last round is three quarters full (14 x 2688, 12 of 128 x 160, 96 tiles: three parts, 32 tiles in a second round, 37 us
    // and 8; eight 28 and 9).  The others share the launch with d_x's tiles or have tiles of 64 rows, four to a unit (10 x 1568, 11 of 32 x 64, 44 tiles:
    // six parts 14.5 us, eight 16.0)
    const int avg = (int)(((long)b * k * c + n - 1) / n);
    const long tiles = (long)sets * n * ((rows + 127) / 128) * ((cols + 127) / 128);
    long s = avg / 8, most = tiles >= 128 ? 2 : (256 + tiles - 1) / tiles;
    s = s < 1 ? 1 : (s > 8 ? 8 : s);
    while (sets == 4 && rows > 64 && tiles < 128 && most < s && (tiles * most - 1) % 256 < 191) ++most;
    return wgrad_plan(b, n, k, (int)(s < most ? s : most), c, 128, (long)c * l_p, 0, 0, 192);
}

// SMHA of any shape or in fp32, `splits` parts an average expert of at most `cap` (unit, pick) entries.  A token of (hi, lo) pairs or of split
// products takes twice as long (57 x 840 x 352, one of 12 experts of 32 x 24 patches, three selections: contraction 28.8 us with equal parts and 34 to 36
// without, the backward pass 136 to 137 and 139 to 145; 10 x 817 x 72 207 to 211 and 213 to 219; threshold 96: 273 random calls 0.02 % faster)
inline WgradPlan smha_any_wgrad(int b, int n, int k, int c, int l_p, int splits, int cap) { return wgrad_plan(b, n, k, splits, c, cap, (long)c * l_p, 0, 0, 128); }

// Expert-selection UoME of any shape or in fp32, `splits` parts an average expert.  Tokens of an item, a pair being cut into `items`
inline int uome_any_range(int l, int items) { return items == 1 ? l : ((l + items - 1) / items + 31) / 32 * 32; }
inline int uome_any_items(int l, int items) { return (l + uome_any_range(l, items) - 1) / uome_any_range(l, items); }   // (as many as there are)
inline WgradPlan uome_any_wgrad(int b, int l, int d, int n, int k, int splits, bool f32)
{
    // One number of parts: the number of ranges, at most as many as parts, whose longest part is least for experts with the average number of
    // pairs to a standard deviation more, a segment's lookups counted as 16 tokens, 4 in fp32, whose products take longer.  (49 x 102 x 312, 2 of 7
    // experts in 8 parts: ranges of 32 tokens leave half of the parts without work, 30.6 us, whole pairs 21.4.  8 x 512, 4 of 8 experts in 8 parts, fp32: with
    // two items a part, 128 tokens, the longest part was longer than with ranges of 64 for 43 % of random selections.)
    const long pairs = (long)(b < 128 ? b : 128) * k;
    const long lookup = f32 ? 4 : 16, parts = (long)n * splits;
    const auto least = [&](int upto, auto in_a_part) {
        int best = 1;
        long best_cost = 0;
        for (int i = 1; i <= upto; ++i) {
            const int range = (uome_any_range(l, i) + 31) / 32 * 32;
            const long cost = in_a_part(i) * (range + lookup);
            if ((i == 1 || cost < best_cost) && uome_any_items(l, i) == i) best = i, best_cost = cost;
        }
        return best;
    };
    const int whole = least(splits, [&](int i) {
        long sum = 0;
        for (long c = wgrad_pairs(pairs, n); c <= wgrad_more_pairs(pairs, n); ++c) sum += (c * i + splits - 1) / splits;
        return sum;
    });
    // parts of equal length: finer where whole pairs or few ranges leave parts without work (fp32 3 x 4400, 2 of 4 experts, as many ranges as parts: 24
    // of 32 had some), as far as the table holds them
    if (splits > 1) {
        const int most = 128 * splits / (b < 128 ? b : 128);
        const int items = least(most < 8 * splits ? most : 8 * splits, [&](int i) { return wgrad_fair(pairs, i, n, parts); });
        const long one = wgrad_one(pairs, n, whole, splits) * uome_any_range(l, whole);
        const WgradPlan w = wgrad_plan(b, n, k, splits, items, 128, l, (double)b * l * d, one, 384);
        if (!w.each) return w;
    }
    WgradPlan w = wgrad_plan(b, n, k, splits, whole, 128, l, (double)b * l * d);
    w.each = w.parts / n;
    return w;
}

}  // namespace uoe
