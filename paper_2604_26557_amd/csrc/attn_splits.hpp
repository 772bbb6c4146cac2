// How decode attention cuts the tokens of a batch into splits and the query heads of a KV head into workgroups: host arithmetic
// without a GPU call, so that it can be tested on its own.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace kvb {

constexpr int kTile = 16;             // tokens per MFMA tile
constexpr int tiles_per_step(int D) { return D >= 128 ? 1 : 2; }  // 8 KiB of K and V in flight per wavefront
constexpr int kMaxHeads = 16;         // query heads one workgroup takes: the columns of an MFMA
constexpr int kPlanTableSeqs = 64;    // the plan gives ragged batches up to this size per-sequence split counts
constexpr int kMaxTableSeqs = 128;    // the launch does so up to this size

// Ragged batch: sequence b is cut into first[b + 1] - first[b] splits, each of tokens[b] token rows (the last one shorter).
struct SplitTable {
    int first[kMaxTableSeqs + 1];
    int tokens[kMaxTableSeqs];
};

constexpr int kMaxSplits = 1024;
constexpr int kXcds = 8;              // dies with an L2 of their own

// cus: compute units of the GPU.  The plan aims at one workgroup for each (a workgroup is eight wavefronts, six at
// head_dim 256; with one per compute unit every one of them starts at once and none waits for a second round).  What is launched may have
// more: see cut_tokens.
struct AttnShape {
    int B, H, Hq, D, cus;
};

// Workgroups that share a KV head: as few as the columns of an MFMA allow, so that K and V are read once.
inline int group_parts(int G) { return (G + kMaxHeads - 1) / kMaxHeads; }
// What kv_decode_attn_splits plans with, and so what the workspace has to hold: parts of 4, 2 or 1 query heads.
inline int planned_parts(int G) { return G % 4 == 0 ? G / 4 : (G % 2 == 0 ? G / 2 : G); }

// Tokens per split are a multiple of this: four steps.
inline int split_quantum(int D) { return 4 * kTile * tiles_per_step(D); }

// Splits of `st` tokens that hold a sequence of `len` (both up to 2^31 - 1: their sum only fits unsigned).
constexpr int splits_of(int len, int st) { return (int)(((unsigned)len + (unsigned)st - 1u) / (unsigned)st); }

// The same for a batch, and their sum.  A product with the reciprocal in double takes a fraction of an integer division, and is exact: the
// numerator, below 2^32 and with a half, puts the quotient at least 0.5 / st from a whole number, which is far more than it is off.
inline void splits_of_all(const int32_t *lens, int B, int st, int *n)
{
    const double up = st - 0.5, per = 1.0 / st;
    for (int b = 0; b < B; ++b) n[b] = (int)((lens[b] + up) * per);
}
inline int splits_in_all(const int32_t *lens, int B, int st)
{
    const double up = st - 0.5, per = 1.0 / st;
    int n = 0;
    for (int b = 0; b < B; ++b) n += (int)((lens[b] + up) * per);
    return n;
}

// Most splits the automatic choice can make for sequences of up to max_len tokens (sizes the workspace).
inline int max_auto_splits(const AttnShape &s, int max_len)
{
    const int q = split_quantum(s.D);
    return (int)std::min<long long>(kMaxSplits, std::max<long long>(1, ((long long)max_len + q - 1) / q));
}

// Uniform batch: split length from the total token count, so that about one workgroup per compute unit has
// tokens to read; never shorter than the quantum.
inline int choose_splits(const AttnShape &s, int parts, long long total_tokens, int max_len)
{
    if (max_len <= 0) return 1;
    const int q = split_quantum(s.D);
    const long long groups_per_seq = (long long)s.H * parts;
    const long long wgs = s.cus;
    long long st = (total_tokens * groups_per_seq + wgs - 1) / wgs;
    st = std::max<long long>(q, (st + q - 1) / q * q);
    const long long ns = ((long long)max_len + st - 1) / st;
    return (int)std::min<long long>(std::max<long long>(1, ns), max_auto_splits(s, max_len));
}

inline int split_tokens_for(const AttnShape &s, int n_splits, int max_len)
{
    const int q = split_quantum(s.D);
    long long st = ((long long)max_len + n_splits - 1) / n_splits;
    st = (st + q - 1) / q * q;
    return (int)std::max<long long>(st, q);
}

// Cuts sequence b into nb[b] equal splits, rounded up to whole steps, which may leave fewer.  Returns the largest split count.
inline int even_table(const AttnShape &s, const int32_t *lens, const int *nb, SplitTable *t)
{
    const unsigned step = kTile * tiles_per_step(s.D);   // a power of two
    const int q = split_quantum(s.D), B = s.B;
    int tokens[kMaxTableSeqs], n[kMaxTableSeqs];   // apart from the table, which for the compiler could be the lengths' memory
    for (int b = 0; b < B; ++b) {   // quotients as above; no tokens: 0 of 0
        const double len = lens[b];
        const int even = (int)((len + nb[b] - 0.5) / std::max(nb[b], 1));
        tokens[b] = std::max(q, (int)(((unsigned)even + step - 1) & ~(step - 1)));
        n[b] = (int)((len + (tokens[b] - 0.5)) / tokens[b]);
    }
    int first = 0, most = 1;
    for (int b = 0; b < B; ++b) {
        t->first[b] = first;
        t->tokens[b] = tokens[b];
        first += n[b];
        most = std::max(most, n[b]);
    }
    for (int b = B; b <= kMaxTableSeqs; ++b) t->first[b] = first;
    return most;
}

// Ragged batch of up to kPlanTableSeqs sequences: every sequence with tokens gets one split; the remaining
// workgroups of the budget (one per compute unit, shared by the query-head groups) go, one at a time, to the
// sequence whose splits are longest; no sequence gets more than cap splits or splits shorter than the quantum.
// A sequence's split length is then rounded up to whole steps only, not to the quantum: steps are handed out
// on demand, so nothing is gained by a whole number of rounds, and the longest split gets shorter.
// Returns the largest split count.
inline int apportion_splits(const AttnShape &s, int parts, const int32_t *lens, int cap, SplitTable *t)
{
    const int q = split_quantum(s.D);
    const long long groups_per_seq = (long long)s.H * parts;
    int nb[kMaxTableSeqs], top[kMaxTableSeqs];   // top: no more splits than these
    double cur[kMaxTableSeqs];                   // split length of a sequence that may get another one
    long long used = 0, total = 0;
    for (int b = 0; b < s.B; ++b) {
        nb[b] = lens[b] > 0 ? 1 : 0;
        top[b] = std::min(cap, splits_of(lens[b], q));
        used += nb[b];
        total += lens[b];
    }
    const long long budget = std::max<long long>(used, s.cus / groups_per_seq);
    if (used > 0 && used < budget) {
        // Every step that starts from a split longer than `share` comes before any other, and there are no more of those than workgroups to
        // give out: they are taken at once, and few are left for the search.  (One by one: 64 sequences, 1 KV head 27 us of host time, now 1.2.)
        const int extra = (int)(budget - used);
        double share = (double)total / extra, low = (double)total / (double)budget;
        for (int i = 0; i < 6; ++i) {
            const double mid = 0.5 * (low + share), per = (1 + 1e-12) / mid;   // no step is missed by rounding
            int steps = 0;
            for (int b = 0; b < s.B; ++b) steps += std::max(0, std::min((int)(lens[b] * per), top[b] - 1));
            (steps <= extra ? share : low) = mid;
        }
        for (int b = 0; b < s.B; ++b) {
            int k = (int)(lens[b] / share) + 1;   // the last step that starts from more than a share
            while (k > 0 && (double)lens[b] / k <= share) --k;
            const int n = std::max(nb[b], std::min(nb[b] + k, top[b]));
            used += n - nb[b];
            nb[b] = n;
            cur[b] = n > 0 && n < top[b] ? (double)lens[b] / n : 0.0;
        }
        for (; used < budget; ++used) {
            int best = 0;
            for (int b = 1; b < s.B; ++b)
                if (cur[b] > cur[best]) best = b;
            if (cur[best] <= 0.0) break;
            ++nb[best];
            cur[best] = nb[best] < top[best] ? (double)lens[best] / nb[best] : 0.0;
        }
    }
    return even_table(s, lens, nb, t);
}

// One split length for all sequences.
inline void common_table(const AttnShape &s, const int32_t *lens, int split_tokens, SplitTable *t)
{
    const int B = s.B;
    int nb[kMaxTableSeqs], first = 0;
    splits_of_all(lens, B, split_tokens, nb);
    for (int b = 0; b < B; ++b) {
        t->first[b] = first;
        t->tokens[b] = split_tokens;
        first += nb[b];
    }
    for (int b = B; b <= kMaxTableSeqs; ++b) t->first[b] = first;
}

// Split choice for the given lengths: fills the table (ragged batches of up to kPlanTableSeqs sequences) or the
// common split length; returns the split count the partials are laid out for, at most `cap` unless the caller gave it.
inline int plan_splits(const AttnShape &s, int parts, const int32_t *lens, int n_splits, int cap, bool *use_table, SplitTable *tab,
                int *split_tokens)
{
    int max_len = 0;
    long long total_len = 0;
    bool uniform = true;
    for (int b = 0; b < s.B; ++b) {
        max_len = std::max(max_len, lens[b]);
        total_len += lens[b];
        if (lens[b] != lens[0]) uniform = false;
    }
    *use_table = !uniform && s.B <= kPlanTableSeqs;
    if (*use_table && n_splits == 0) {
        *split_tokens = split_quantum(s.D);  // not used by the kernels in table mode
        return apportion_splits(s, parts, lens, std::min(cap, max_auto_splits(s, max_len)), tab);
    }
    const int ns = n_splits > 0 ? n_splits : std::min(cap, choose_splits(s, parts, total_len, max_len));
    *split_tokens = split_tokens_for(s, ns, max_len);
    if (*use_table) common_table(s, lens, *split_tokens, tab);
    return ns;
}

// Sequences whose K and V are this short per KV head are not split: the second launch and the partials cost more than one
// workgroup needs for two rounds of its wavefronts.  Replayed from a graph, one split against the automatic choice, us per layer
// (1 and 8 KV heads, 1 and 8 sequences, 1 to 16 query heads each): head_dim 64, 256 tokens 4.5-5.7 / 6.2-8.2, 512 tokens 5.8-7.7 / 6.3-9.0 (the worst
// pair 7.00 / 6.95); 128, 128 tokens 4.1-6.0 / 6.0-9.2, 256 tokens 5.1-8.0 / 6.1-10.3; 256, 128 tokens 5.3-9.5 / 6.6-12.7.  The line lies where
// the worst pair is level; launched call by call a launch that is left out saves another 2.2 us of host time.
constexpr long long kWholeBytes = 128 * 1024;

// Where the launch cuts more finely than the plan, splits beyond 64 of a sequence hold at least 256 tokens: below that the partials cost
// the combine kernel more than the shorter splits save (2 KV heads of 128, bf16, us per layer from a graph: 8K tokens 64 / 128 splits 9.8 / 10.9,
// 32K 15.7 / 14.3; 1 KV head: 16K tokens 64 / 128 / 256 splits 11.3 / 11.3 / 14.4, 32K 128 / 256 13.2 / 15.5).
inline int replan_cap(int max_len) { return std::min(kMaxSplits, std::max(64, max_len / 256)); }

// The cut of one launch.
struct AttnCut {
    int ns;             // splits the partials are laid out for
    bool use_table;     // the grid walks `tab`; otherwise every sequence is cut into splits of split_tokens
    int split_tokens;
    int subs;           // workgroups that share a KV head
    SplitTable tab;
    // Table: the workgroups of all KV heads for one split lie side by side, and the sequences with the longest splits come first.
    bool longest_first;
    unsigned char order[kMaxTableSeqs];   // sequences in the order of the grid
};

// What a cut costs, as bytes that one compute unit reads in that time.  The plan has one workgroup per compute unit, which is the best cut where
// it is an even one: every further workgroup costs its start and its merge.  But whole sequences, or few splits of each, are rarely
// even, and where they are not, several smaller workgroups for every compute unit, dealt out as compute units become free, end together.
//  * A compute unit reads no more than 1 / kAlone of its share of HBM when others are idle.
//  * item_bytes for every workgroup after the first (1.2 us at 25 GB/s and compute unit; 4.4 us at head_dim 256 with several query heads per KV head:
//    5 sequences of 4000 tokens, 8 x 8 x 256, one / two / three workgroups for each 30.6 / 33.4 / 36.8, where 8 x 1 x 256, 4 of 4000 takes 24.9 / 25.1 / 26.7.  The geometric mean over
//    22 shapes in two types and layouts whose cut depends on it is 32.2 us with 110e3, 32.4 with 60e3, 33.9 with 30e3, over ten 34.4, with 85e3 34.8, with 160e3 34.9:
//    profiles/attn_cut_width256.md), kCombineBytes for the second launch (3.4 us on the GPU).
//  * kFinerBytes (1 us) is what a finer cut has to save: about its own host time, and what the model is off by for batches of 10 us.  128 sequences of
//    260-400 tokens, 2 x 4 x 128, called one by one: without it 16.4 us a layer, with it 15.6.
//  * Costs are compared with a margin of 1 % (uniform) or 3 %, within which the plan stays.
// us per layer from a graph, one workgroup per compute unit (or sequence) / this cut: paged batch of 48 sequences of 200-4000 tokens, 4 KV heads
// x 7 x 128 51.7 / 42.9, 8 x 4 x 128 113 / 76.6; 20 of 1K-8K, 8 x 4 x 128 74.9 / 65.1; 30 of 200-8000, 5 x 4 x 64 39.7 / 33.2.  Where the plan is
// even it stays: 8 of 1K-8K 31.0 / 31.8, 3 of 2.5K-20K 26.3 / 29.5.
constexpr double kAlone = 0.85, kCombineBytes = 84e3, kFinerBytes = 25e3;
inline double item_bytes(const AttnShape &s) { return s.D >= 256 && s.Hq > s.H ? 110e3 : 30e3; }

// per_cu: workgroups per compute unit; longest: token rows of the compute unit that has most.
inline double cut_cost(const AttnShape &s, double total_tokens, double per_cu, double longest, bool split)
{
    const double row = 4.0 * s.D;   // bytes of K and V
    double c = std::max(total_tokens * s.H / s.cus, kAlone * longest) * row + item_bytes(s) * std::max(0.0, per_cu - 1);
    if (split) c += kCombineBytes + per_cu * (s.Hq / s.H) * (s.D + 2) * 8;   // partials are written and read
    return c;
}

// Uniform batch: the split count, of the plan's and of those that make just one, two, three or four workgroups for a compute unit.
// us per layer from a graph: 48 sequences of 2000 tokens, 8 x 4 x 128: not split 74.2, in 2 67.2.
inline int even_splits(const AttnShape &s, int parts, int len, int plan, int cap)
{
    const long long units = (long long)s.B * s.H * parts;
    double best_cost = 0.0;
    int best = 0;
    for (int k = 0; k <= 4; ++k) {
        int ns = k == 0 ? plan : (int)std::min<long long>(cap, k * (long long)s.cus / units);
        if (ns < 1) continue;
        const int st = split_tokens_for(s, ns, len);
        if (k > 0) ns = splits_of(len, st);
        const double per_cu = (double)splits_of(len, st) * units / s.cus, rounds = (double)(long long)(per_cu + 0.999999);
        const double cost = cut_cost(s, (double)len * s.B * parts, per_cu, rounds * std::min(st, len), ns > 1);
        if (best == 0 || cost < 0.99 * best_cost) { best = ns; best_cost = cost; }
    }
    return best;
}

// Sequences by descending split length, equal ones in the order of the batch: a counting sort of up to 7 bits per pass (128 sequences of 200-4000 tokens:
// 0.43 us of host time; a comparison sort whose branches are predicted 0.75).
inline void order_splits(const AttnShape &s, const int32_t *lens, const SplitTable &t, unsigned char *order)
{
    static_assert(kMaxTableSeqs < 256, "a sequence, and a number of them, is a byte");
    const int B = s.B;
    int size[kMaxTableSeqs], top = 0;
    unsigned char from[kMaxTableSeqs], to[kMaxTableSeqs];
    for (int b = 0; b < B; ++b) {
        size[b] = std::min(t.tokens[b], (int)lens[b]);
        top = std::max(top, size[b]);
        to[b] = (unsigned char)b;
    }
    const int bits = top > 0 ? 32 - __builtin_clz((unsigned)top) : 0, passes = (bits + 6) / 7;
    const int width = passes > 0 ? (bits + passes - 1) / passes : 0, mask = (1 << width) - 1;
    for (int pass = 0, shift = 0; pass < passes; ++pass, shift += width) {
        unsigned char at[128] = {};
        for (int b = 0; b < B; ++b) ++at[(top - size[b]) >> shift & mask];
        for (int i = 0, n = 0; n < B; ++i) {
            const unsigned char k = at[i];
            at[i] = (unsigned char)n;
            n += k;
        }
        std::copy(to, to + B, from);
        for (int r = 0; r < B; ++r) to[at[(top - size[from[r]]) >> shift & mask]++] = from[r];
    }
    std::copy(to, to + B, order);
}

// *ordered: whether `order` is the table's; it is made where the cost depends on it.
inline double table_cost(const AttnShape &s, int parts, const int32_t *lens, const SplitTable &t, int most, unsigned char *order, bool *ordered)
{
    const double m = (double)s.cus / (s.H * parts);   // compute units for each of the heads
    const int n = t.first[s.B];
    long long sum = 0;
    int size0 = 0;
    for (int b = 0; b < s.B; ++b) {
        sum += lens[b];
        size0 = std::max(size0, std::min(t.tokens[b], (int)lens[b]));
    }
    // The grid deals the longest out first, then the next to the same compute units; the third round goes to whichever is free, and where it
    // is not a whole one (whole sequences) part of a split is left at the end.
    const double total = (double)sum;
    double longest = size0;
    if (n > 2 * m && most > 1 && 2.0 * size0 <= total / m / kAlone) {
        longest = total / m / kAlone;   // whatever the second one is
    } else if (n > m) {
        int full = 0;   // items as long as the longest
        for (int b = 0; b < s.B; ++b) full += std::min(t.tokens[b], (int)lens[b]) == size0 ? t.first[b + 1] - t.first[b] : 0;
        auto size_at = [&](int item) {
            if (item < full) return size0;
            if (!*ordered) order_splits(s, lens, t, order);
            *ordered = true;
            for (int r = 0, f = 0; r < s.B; ++r) {
                const int b = order[r];
                f += t.first[b + 1] - t.first[b];
                if (f > item) return std::min(t.tokens[b], (int)lens[b]);
            }
            return 0;
        };
        longest += size_at((int)m);
        if (n > 2 * m) longest = std::max(longest, (total / m + (most > 1 ? 0 : size_at(n - (int)m) / 4.0)) / kAlone);
    }
    return cut_cost(s, total * parts, n / m, longest, most > 1);
}

// Whether the sequences, not split, are worth a table.  Its order, the longest first, saves up to what those take beyond the mean, but each workgroup of
// a compute unit in turn waits for the lookup, `lookup` in bytes that it would read meanwhile: more beyond 64 sequences, which take a second round of
// loads, and at head_dim 256, of whose larger instances a compute unit holds one workgroup or two.  us per layer of eager calls, table / none: up to 128 KiB, 40 of 20-250 tokens,
// 32 x 1 x 128 17.4 / 19.5, of 10-60 9.3 / 8.9; 128 of 20-180, 8 x 4 x 128 15.0 / 15.7, of 20-96 12.1 / 11.4; 128 of 20-250, 32 x 4 x 128 61.3 / 58.0, 64 of those
// 30.1 / 31.0.  Longer, 80 of 300-2000, 8 x 4 x 128 65.8 / 77.3; 128 of 400-700, 32 x 1 x 64 99.2 / 91.1; 66 of 130-300, 16 x 4 x 256 49.7 / 45.2.
inline bool table_pays(const AttnShape &s, int parts, const int32_t *lens, const SplitTable &t, double lookup)
{
    long long sum = 0;
    int longest = 0, used = 0;
    for (int b = 0; b < s.B; ++b) {
        const int size = std::min(t.tokens[b], (int)lens[b]);
        sum += size;
        used += size > 0;
        longest = std::max(longest, size);
    }
    return kAlone * (longest - (double)sum / used) * 4.0 * s.D > lookup * t.first[s.B] * s.H * parts / s.cus;
}

// Cuts every sequence into equal splits, of at most as many tokens as make three workgroups for a compute unit, or one more for each than there are
// sequences; but no more splits than the sequence has eights of steps, a step for each of eight wavefronts.  Returns the largest split count, or 0
// (and no table) where the cut cannot cost less than `worth`.
// us per layer from a graph, geometric mean of 36 batches of 9-108 sequences, 1-32 KV heads and all three widths: 2 workgroups for a compute unit 43.5, 2.5
// 44.2, 3 41.7, 3.5 44.1, 4 42.3 (profiles/attn_cut_targets.md).  A number that is not whole leaves a round half empty.  The plan / a split per four
// steps / per eight: 96 sequences of 260-600, 1 x 4 x 128 11.8 / 13.1 / 10.6; 80 of 600-900, 2 x 2 x 64 14.0 / 13.1 / 12.7; 66 of 130-500, 2 x 4 x 256 17.95 /
// 17.9 / 17.2.
inline int finer_splits(const AttnShape &s, int parts, const int32_t *lens, int cap, double worth, SplitTable *t)
{
    const int q = split_quantum(s.D);
    long long total = 0;
    int used = 0, max_len = 0;
    for (int b = 0; b < s.B; ++b) { total += lens[b]; used += lens[b] > 0; max_len = std::max(max_len, (int)lens[b]); }
    const double m = (double)s.cus / (s.H * parts);
    const int target = std::max((int)(3 * m), used + (int)m);
    long long lo = std::max<long long>(2 * q, std::max<long long>(total / target, splits_of(max_len, cap))), hi = std::max<long long>(lo, max_len);
    // a workgroup for each sequence at least, an even share for every compute unit at best; that it splits is often known beforehand
    const double mean = (double)total * parts;
    if (lo < hi && used + (double)total / ((lo + hi) / 2) <= target && cut_cost(s, mean, used / m, 0, true) >= worth) return 0;
    for (int i = 0; i < 7 && lo < hi; ++i) {   // hi holds the target; lo may not
        const int st = (int)((lo + hi) / 2);
        if (used + (double)total / st <= target || splits_in_all(lens, s.B, st) <= target) hi = st; else lo = st + 1;
    }
    if (cut_cost(s, mean, used / m, 0, hi < max_len) >= worth) return 0;
    int nb[kMaxTableSeqs];
    splits_of_all(lens, s.B, (int)hi, nb);
    return even_table(s, lens, nb, t);
}

// False: the workspace is too small for the plan.
inline bool cut_tokens(const AttnShape &s, const int32_t *lens, int n_splits, size_t ws_bytes, AttnCut *c)
{
    int max_len = 0;
    for (int b = 0; b < s.B; ++b) max_len = std::max(max_len, lens[b]);
    const int G = s.Hq / s.H;
    const size_t per_split = (size_t)s.B * s.Hq * (s.D + 2) * sizeof(float);
    // The plan counts a workgroup per 4, 2 or 1 query heads; where one workgroup takes more, the same number of
    // workgroups makes more splits, as far as the workspace holds them.  (A workspace for the most splits any plan makes
    // holds the plan, and it need not be made: it costs about 1 us for 4 sequences.)
    const bool whole = n_splits == 0 && (long long)max_len * s.D * 4 <= kWholeBytes;
    const bool replan = n_splits == 0 && !whole && planned_parts(G) != group_parts(G);
    bool limited = n_splits > 0;
    c->subs = group_parts(G);
    c->use_table = false;
    c->longest_first = false;
    c->ns = 0;
    if (!(whole || replan) || ws_bytes < per_split * max_auto_splits(s, max_len)) {
        c->ns = plan_splits(s, planned_parts(G), lens, n_splits, kMaxSplits, &c->use_table, &c->tab, &c->split_tokens);
        if (ws_bytes < per_split * c->ns) return false;
    }
    bool uniform = true, empty = false;
    for (int b = 0; b < s.B; ++b) { uniform = uniform && lens[b] == max_len; empty = empty || lens[b] == 0; }
    if (whole) {
        c->ns = 1;
        c->split_tokens = split_tokens_for(s, 1, max_len);
        c->use_table = !uniform && !empty && s.B <= kMaxTableSeqs && (long long)s.B * s.H * c->subs > s.cus;
        if (c->use_table) {
            for (int b = 0; b <= kMaxTableSeqs; ++b) {
                c->tab.first[b] = std::min(b, s.B);
                if (b < s.B) c->tab.tokens[b] = c->split_tokens;
            }
            c->use_table = table_pays(s, c->subs, lens, c->tab, s.B > 64 ? 7e3 : 3.5e3);
        }
    } else if (replan) {
        const int cap = (int)std::min<size_t>(replan_cap(max_len), ws_bytes / per_split);
        c->ns = plan_splits(s, group_parts(G), lens, 0, cap, &c->use_table, &c->tab, &c->split_tokens);
        limited = cap < replan_cap(max_len);
    }
    // The plan, or a finer cut where that is the cheaper one.  All of it is made again by each layer's call, from the lengths alone: us of host time, 48
    // sequences of 200-4000 tokens, 4 x 7 x 128 1.6; 64, 1 x 4 x 128 1.2; 128, 8 x 4 x 128 1.6; 8 of 1K-8K, 8 x 4 x 128 0.25.
    bool ordered = false;   // c->order is the table's
    const int cap = (int)std::min<size_t>(replan_cap(max_len), ws_bytes / per_split);
    if (n_splits == 0 && !whole && max_len > 0 && cap > 0) {
        if (uniform) {
            c->ns = even_splits(s, c->subs, max_len, c->ns, cap);
            c->split_tokens = split_tokens_for(s, c->ns, max_len);
        } else if (s.B <= kMaxTableSeqs) {
            if (!c->use_table) {   // more sequences than the plan tables: as it is launched without a table
                c->use_table = true;
                common_table(s, lens, c->split_tokens, &c->tab);
            }
            const double cost = table_cost(s, c->subs, lens, c->tab, c->ns, c->order, &ordered), worth = std::min(0.97 * cost, cost - kFinerBytes);
            SplitTable fine;
            unsigned char order[kMaxTableSeqs];
            bool fine_ordered = false;
            const int most = finer_splits(s, c->subs, lens, cap, worth, &fine);
            if (most > 0 && table_cost(s, c->subs, lens, fine, most, order, &fine_ordered) < worth) {
                c->tab = fine;
                c->ns = most;
                ordered = fine_ordered;
                if (ordered) std::copy(order, order + s.B, c->order);
            } else if (s.B > kPlanTableSeqs) {
                // Without a table where few workgroups of the whole grid would have no tokens, and either its order does not pay or there is none.  With several
                // splits each, the remainders of all sequences would fall to the same XCDs (70 of 300-700 tokens, 4 x 4 x 128: table 20.4, none 24.3).
                const long long n = c->tab.first[s.B];
                if (4LL * c->ns * s.B <= 5 * n)
                    c->use_table = c->ns == 1 ? table_pays(s, c->subs, lens, c->tab, s.D >= 256 ? 20e3 : 8e3) : n * s.H * c->subs > s.cus;
            }
        }
    }
    // A split count from the caller, or from a workspace for the plan alone, was made for a workgroup per 4, 2 or 1 heads and
    // leaves compute units idle where one takes all.  As long as there are idle ones the heads are shared out, provided that the workgroups of
    // a KV head meet in one L2 (workgroups go round the XCDs in turn, and these are `apart` apart), so that K and V still come from memory
    // once.  us per layer from a graph, one / shared: 8 KV heads x 16, 32K tokens in 8 splits 65.8 / 61.5, x 8 in 16 splits 39.1 / 38.0,
    // 2 x 7, 4K in 16 splits 10.6 / 9.8.  Without a common L2 the same costs: 8 x 16, 4 sequences of 8K in 2 splits 66.8 / 91.8, 8 x 7, 32K in 5
    // splits 99.9 / 229.8.
    if (limited && !whole) {
        const int items = c->use_table ? c->tab.first[s.B] : c->ns * s.B, apart = c->use_table ? items : c->ns;
        if (items > 0 && apart % kXcds == 0)
            c->subs = std::max(c->subs, std::min(planned_parts(G), (int)(s.cus / ((long long)items * s.H))));
    }
    if (c->use_table) {
        // More workgroups than compute units: those with most to do start first, whichever KV head they belong to.  us per layer from a graph, in the order
        // of the batch / longest first: 32 sequences of 200-1000 tokens, 32 KV heads x 1 x 128 66.0 / 53.9, 60 of 100-600, 8 x 4 x 128 23.2 / 20.6.
        c->longest_first = c->subs == 1 && (long long)c->tab.first[s.B] * s.H > s.cus && c->tab.first[s.B] <= 65535;   // a grid's y dimension
        if (!c->longest_first) for (int b = 0; b < s.B; ++b) c->order[b] = (unsigned char)b;
        else if (!ordered) order_splits(s, lens, c->tab, c->order);
    }
    return true;
}

}  // namespace kvb
