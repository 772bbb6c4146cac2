// Drives the split choice of decode attention without a GPU.  One call per line of the input:
//   B H Hq D cus n_splits ws_splits len_0 .. len_{B-1}
// ws_splits: the workspace holds that many splits (-1: as many as any plan makes).  One line of the output each:
//   ok ns use_table split_tokens subs, then per sequence: splits that hold tokens, tokens per split
#include <cstdio>
#include <vector>

#include "attn_splits.hpp"

int main()
{
    kvb::AttnShape s{};
    int n_splits = 0, ws_splits = 0;
    while (std::scanf("%d %d %d %d %d %d %d", &s.B, &s.H, &s.Hq, &s.D, &s.cus, &n_splits, &ws_splits) == 7) {
        std::vector<int32_t> lens((size_t)s.B);
        int max_len = 0;
        for (auto &n : lens) {
            if (std::scanf("%d", &n) != 1) return 1;
            max_len = n > max_len ? n : max_len;
        }
        const size_t per_split = (size_t)s.B * s.Hq * (s.D + 2) * sizeof(float);
        const size_t ws = per_split * (size_t)(ws_splits >= 0 ? ws_splits : kvb::max_auto_splits(s, max_len));
        kvb::AttnCut c{};
        const bool ok = kvb::cut_tokens(s, lens.data(), n_splits, ws, &c);
        std::printf("%d %d %d %d %d", ok, c.ns, c.use_table, c.split_tokens, c.subs);
        for (int b = 0; ok && b < s.B; ++b) {
            const int st = c.use_table ? c.tab.tokens[b] : c.split_tokens;
            std::printf(" %d %d", c.use_table ? c.tab.first[b + 1] - c.tab.first[b] : (lens[b] + st - 1) / st, st);
        }
        std::printf("\n");
    }
    return 0;
}
