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
constexpr int kMaxTableSeqs = 64;     // ragged batches up to this size get per-sequence split counts

// Ragged batch: sequence b owns work items [first[b], first[b+1]) of the grid's x dimension, each of
// tokens[b] token rows (the last one shorter).
struct SplitTable {
    int first[kMaxTableSeqs + 1];
    int tokens[kMaxTableSeqs];
};

constexpr int kMaxSplits = 1024;
constexpr int kXcds = 8;              // dies with an L2 of their own

// cus: compute units of the GPU.  The automatic choice aims at one workgroup for each (a workgroup is eight wavefronts, six at
// head_dim 256; with one per compute unit every one of them starts at once and none waits for a second round).
struct AttnShape {
    int B, H, Hq, D, cus;
};

// Workgroups that share a KV head: as few as the columns of an MFMA allow, so that K and V are read once.
inline int group_parts(int G) { return (G + kMaxHeads - 1) / kMaxHeads; }
// What kv_decode_attn_splits plans with, and so what the workspace has to hold: parts of 4, 2 or 1 query heads.
inline int planned_parts(int G) { return G % 4 == 0 ? G / 4 : (G % 2 == 0 ? G / 2 : G); }

// Tokens per split are a multiple of this: four steps.
inline int split_quantum(int D) { return 4 * kTile * tiles_per_step(D); }

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

// Ragged batch of up to kMaxTableSeqs sequences: every sequence with tokens gets one split; the remaining
// workgroups of the budget (one per compute unit, shared by the query-head groups) go, one at a time, to the
// sequence whose splits are longest; no sequence gets more than cap splits or splits shorter than the quantum.
// A sequence's split length is then rounded up to whole steps only, not to the quantum: steps are handed out
// on demand, so nothing is gained by a whole number of rounds, and the longest split gets shorter.
// Returns the largest split count.
inline int apportion_splits(const AttnShape &s, int parts, const int32_t *lens, int cap, SplitTable *t)
{
    const int q = split_quantum(s.D);
    const long long groups_per_seq = (long long)s.H * parts;
    int nb[kMaxTableSeqs];
    long long used = 0;
    for (int b = 0; b < s.B; ++b) { nb[b] = lens[b] > 0 ? 1 : 0; used += nb[b]; }
    const long long budget = std::max<long long>(used, s.cus / groups_per_seq);
    while (used < budget) {
        int best = -1;
        double longest = 0.0;
        for (int b = 0; b < s.B; ++b) {
            if (nb[b] == 0 || nb[b] >= cap || (long long)(nb[b] + 1) * q > (long long)lens[b] + q - 1) continue;
            const double cur = (double)lens[b] / nb[b];
            if (cur > longest) { longest = cur; best = b; }
        }
        if (best < 0) break;
        ++nb[best];
        ++used;
    }
    const int step = kTile * tiles_per_step(s.D);
    int most = 1, first = 0;
    for (int b = 0; b < s.B; ++b) {
        t->first[b] = first;
        int st = q;
        if (nb[b] > 0) {
            st = std::max(q, (int)((((long long)lens[b] + nb[b] - 1) / nb[b] + step - 1) / step * step));
            nb[b] = (lens[b] + st - 1) / st;   // rounding the split length up may leave fewer splits
        }
        t->tokens[b] = st;
        first += nb[b];
        most = std::max(most, nb[b]);
    }
    for (int b = s.B; b <= kMaxTableSeqs; ++b) t->first[b] = first;
    return most;
}

// Split choice for the given lengths: fills the table (ragged batches of up to kMaxTableSeqs sequences) or the
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
    *use_table = !uniform && s.B <= kMaxTableSeqs;
    if (*use_table && n_splits == 0) {
        *split_tokens = split_quantum(s.D);  // not used by the kernels in table mode
        return apportion_splits(s, parts, lens, std::min(cap, max_auto_splits(s, max_len)), tab);
    }
    const int ns = n_splits > 0 ? n_splits : std::min(cap, choose_splits(s, parts, total_len, max_len));
    *split_tokens = split_tokens_for(s, ns, max_len);
    if (*use_table) {
        int first = 0;
        for (int b = 0; b < s.B; ++b) {
            tab->first[b] = first;
            tab->tokens[b] = *split_tokens;
            first += (lens[b] + *split_tokens - 1) / *split_tokens;
        }
        for (int b = s.B; b <= kMaxTableSeqs; ++b) tab->first[b] = first;
    }
    return ns;
}

// Sequences whose K and V are this short per KV head are not split: the second launch and the partials cost more than one
// workgroup needs for two rounds of its wavefronts.  Replayed from a graph, one split against the automatic choice, us per layer
// (1 and 8 KV heads, 1 and 8 sequences, 1 to 16 query heads each): head_dim 64, 256 tokens 4.5-5.7 / 6.2-8.2, 512 tokens 5.8-7.7 / 6.3-9.0 (the worst
// pair 7.00 / 6.95); 128, 128 tokens 4.1-6.0 / 6.0-9.2, 256 tokens 5.1-8.0 / 6.1-10.3; 256, 128 tokens 5.3-9.5 / 6.6-12.7.  The line lies where
// the worst pair is level; launched call by call a launch that is left out saves another 3.4 us of host time.
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
};

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
    c->ns = 0;
    if (!(whole || replan) || ws_bytes < per_split * max_auto_splits(s, max_len)) {
        c->ns = plan_splits(s, planned_parts(G), lens, n_splits, kMaxSplits, &c->use_table, &c->tab, &c->split_tokens);
        if (ws_bytes < per_split * c->ns) return false;
    }
    if (whole) {
        c->use_table = false;
        c->ns = 1;
        c->split_tokens = split_tokens_for(s, 1, max_len);
    } else if (replan) {
        const int cap = (int)std::min<size_t>(replan_cap(max_len), ws_bytes / per_split);
        c->ns = plan_splits(s, group_parts(G), lens, 0, cap, &c->use_table, &c->tab, &c->split_tokens);
        limited = cap < replan_cap(max_len);
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
    return true;
}

}  // namespace kvb
