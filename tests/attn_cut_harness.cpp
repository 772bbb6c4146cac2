// The cut of ragged batches against the same rules written plainly (integer divisions, comparison sorts, one compute unit handed out at a time),
// and what it costs the host.
//   attn_cut_harness            compares; returns a number that says what differs
//   attn_cut_harness time       one line per batch: time of a cut over the time of std::sort on 128 keys
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "attn_splits.hpp"

namespace plain {
using namespace kvb;

int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }

int table(const AttnShape &s, const int32_t *lens, const std::vector<int> &nb, SplitTable *t)
{
    const int step = kTile * tiles_per_step(s.D), q = split_quantum(s.D);
    int most = 1;
    t->first[0] = 0;
    for (int b = 0; b < s.B; ++b) {
        t->tokens[b] = nb[b] > 0 ? std::max(q, ceil_div(ceil_div(lens[b], nb[b]), step) * step) : q;
        const int n = nb[b] > 0 ? ceil_div(lens[b], t->tokens[b]) : 0;
        t->first[b + 1] = t->first[b] + n;
        most = std::max(most, n);
    }
    return most;
}

int apportion(const AttnShape &s, int parts, const int32_t *lens, int cap, SplitTable *t)
{
    const int q = split_quantum(s.D);
    std::vector<int> nb(s.B);
    int used = 0;
    for (int b = 0; b < s.B; ++b) used += nb[b] = lens[b] > 0;
    for (const int budget = s.cus / (s.H * parts); used < budget; ++used) {
        int best = -1;
        double longest = 0;
        for (int b = 0; b < s.B; ++b) {
            if (nb[b] == 0 || nb[b] >= cap || nb[b] + 1 > ceil_div(lens[b], q)) continue;
            if ((double)lens[b] / nb[b] > longest) { longest = (double)lens[b] / nb[b]; best = b; }
        }
        if (best < 0) break;
        ++nb[best];
    }
    return table(s, lens, nb, t);
}

int finer(const AttnShape &s, int parts, const int32_t *lens, int cap, SplitTable *t)
{
    long long total = 0;
    int used = 0, max_len = 0;
    for (int b = 0; b < s.B; ++b) { total += lens[b]; used += lens[b] > 0; max_len = std::max(max_len, (int)lens[b]); }
    const double m = (double)s.cus / (s.H * parts);
    const int target = std::max((int)(3 * m), used + (int)m);
    long long lo = std::max<long long>({2 * split_quantum(s.D), total / target, ceil_div(max_len, cap)}), hi = std::max<long long>(lo, max_len);
    for (int i = 0; i < 7 && lo < hi; ++i) {
        const long long st = (lo + hi) / 2;
        long long n = 0;
        for (int b = 0; b < s.B; ++b) n += ceil_div(lens[b], st);
        if (n <= target) hi = st; else lo = st + 1;
    }
    std::vector<int> nb(s.B);
    for (int b = 0; b < s.B; ++b) nb[b] = ceil_div(lens[b], hi);
    return table(s, lens, nb, t);
}

std::vector<int> order(const AttnShape &s, const int32_t *lens, const SplitTable &t)
{
    std::vector<int> o(s.B);
    for (int b = 0; b < s.B; ++b) o[b] = b;
    std::stable_sort(o.begin(), o.end(), [&](int x, int y) { return std::min(t.tokens[x], (int)lens[x]) > std::min(t.tokens[y], (int)lens[y]); });
    return o;
}

double cost(const AttnShape &s, int parts, const int32_t *lens, const SplitTable &t, int most)
{
    std::vector<int> size;   // of every workgroup, in the grid's order
    double total = 0;
    for (int b : order(s, lens, t)) {
        size.insert(size.end(), t.first[b + 1] - t.first[b], std::min(t.tokens[b], (int)lens[b]));
        total += lens[b];
    }
    const double m = (double)s.cus / (s.H * parts);
    const int n = (int)size.size();
    double longest = size[0];
    if (n > m) longest += size[(int)m];
    if (n > 2 * m) longest = std::max(longest, (total / m + (most > 1 || (int)m == 0 ? 0 : size[n - (int)m] / 4.0)) / kAlone);
    return cut_cost(s, total * parts, n / m, longest, most > 1);
}
}  // namespace plain

static int compare()
{
    std::srand(23);
    auto below = [](int n) { return std::rand() % n; };
    int skipped = 0, even = 0;
    for (int it = 0; it < 20000; ++it) {
        const int G = 1 + below(20), H = 1 + below(below(2) ? 4 : 32), D = 64 << below(3), B = 1 + below(below(2) ? kvb::kMaxTableSeqs : 12), parts = kvb::group_parts(G);
        const int hi = (int)(48 * std::pow(32768 / 48., below(1000) / 999.)), lo = 1 + below(hi), kind = below(5);
        int32_t lens[kvb::kMaxTableSeqs], max_len = 0;
        for (int b = 0; b < B; ++b) {
            lens[b] = lo + below(hi - lo + 1);
            if (kind == 1 && below(4) == 0) lens[b] = 0;
            if (kind == 2) lens[b] = below(8) ? 1 + below(200) : hi;
            if (kind == 3) lens[b] = (lens[b] + 63) / 64 * 64;   // whole quanta, many ties
            max_len = std::max(max_len, lens[b]);
        }
        if (max_len == 0) continue;
        const kvb::AttnShape s{B, H, H * G, D, below(4) ? 256 : 60};
        const int cap = below(3) ? kvb::replan_cap(max_len) : 1 + below(64);
        kvb::SplitTable a, b;
        auto same = [&] { return std::equal(a.first, a.first + B + 1, b.first) && std::equal(a.tokens, a.tokens + B, b.tokens); };
        if (B <= kvb::kPlanTableSeqs) {
            if (kvb::apportion_splits(s, parts, lens, cap, &a) != plain::apportion(s, parts, lens, cap, &b) || !same()) return 1;
        } else {
            const int st = kvb::split_tokens_for(s, 1 + below(cap), max_len);
            kvb::common_table(s, lens, st, &a);
            for (int i = 0; i < B; ++i)
                if (a.tokens[i] != st || a.first[i + 1] - a.first[i] != plain::ceil_div(lens[i], st)) return 2;
        }
        int most = 1;
        for (int i = 0; i < B; ++i) most = std::max(most, a.first[i + 1] - a.first[i]);
        for (int turn = 0; turn < 2; ++turn) {   // the plan's table, then the finer one
            unsigned char order[kvb::kMaxTableSeqs];
            bool ordered = false;
            const double cost = kvb::table_cost(s, parts, lens, a, most, order, &ordered);
            if (cost != plain::cost(s, parts, lens, a, most)) return 3;
            even += !ordered;
            kvb::order_splits(s, lens, a, order);
            const std::vector<int> want = plain::order(s, lens, a);
            if (!std::equal(want.begin(), want.end(), order)) return 4;
            if (turn) break;
            most = kvb::finer_splits(s, parts, lens, cap, 1e300, &a);
            const int fine = plain::finer(s, parts, lens, cap, &b);
            if (most != fine || !same()) return 5;
            if (kvb::finer_splits(s, parts, lens, cap, cost, &a) == 0) {   // only what is no cheaper is left out
                if (plain::cost(s, parts, lens, b, fine) < cost) return 6;
                ++skipped;
            }
            a = b;
        }
    }
    return skipped > 1000 && even > 1000 ? 0 : 7;
}

template <class F> static double best_of(F f)
{
    double best = 1e9;
    for (int r = 0; r < 40; ++r) {
        const auto t0 = std::chrono::steady_clock::now();
        for (int i = 0; i < 50; ++i) f();
        best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 50);
    }
    return best;
}

static int time_cuts()
{
    static const int cases[][6] = {   // B, H, G, D, shortest, longest
        {96, 1, 4, 128, 260, 600}, {128, 2, 4, 128, 260, 400}, {128, 1, 4, 64, 513, 700}, {128, 8, 4, 128, 200, 4000}, {96, 4, 7, 128, 200, 4000},
        {128, 8, 4, 256, 100, 3000}, {64, 1, 4, 128, 200, 4000}, {32, 1, 4, 128, 200, 4000}, {48, 4, 7, 128, 200, 4000}};
    for (const auto &c : cases) {
        const int B = c[0];
        int32_t lens[128], max_len = 0;
        std::srand(3);
        for (int b = 0; b < B; ++b) {
            lens[b] = c[4] + std::rand() % (c[5] - c[4]);
            max_len = std::max(max_len, lens[b] + 1);
        }
        const kvb::AttnShape s{B, c[1], c[1] * c[2], c[3], 256};
        const size_t ws = (size_t)B * s.Hq * (s.D + 2) * 4 * kvb::max_auto_splits(s, max_len);
        uint64_t keys[16][128];
        for (auto &row : keys)
            for (auto &k : row) k = (uint64_t)std::rand();
        int turn = 0;
        volatile uint64_t sink = 0;
        kvb::AttnCut cut{};
        double ratio = 1e9;
        for (int r = 0; r < 5; ++r) {
            const double sort = best_of([&] { uint64_t k[128]; std::copy(keys[turn & 15], keys[turn & 15] + 128, k); ++turn; std::sort(k, k + 128); sink = k[5]; });
            const double t = best_of([&] { lens[turn++ % B] ^= 1; kvb::cut_tokens(s, lens, 0, ws, &cut); sink = (uint64_t)cut.ns; });
            ratio = std::min(ratio, t / sort);
        }
        std::printf("%d %d %d %d %.2f\n", B, c[1], c[2], c[3], ratio);
    }
    return 0;
}

int main(int argc, char **) { return argc > 1 ? time_cuts() : compare(); }
