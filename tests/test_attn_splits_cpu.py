"""How a decode attention launch cuts its tokens and shares out its query heads (host arithmetic, no GPU): the cut that is
launched, which with an automatic split count differs from the plan that sizes the workspace."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("splits") / "attn_splits_harness")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2604_26557_amd", "csrc"),
                           os.path.join(ROOT, "tests", "attn_splits_harness.cpp"), "-o", exe])
    return exe


def _cut(exe, cases):
    """cases: (H, G, D, lens, n_splits, ws_splits) -> dicts"""
    text = "".join(f"{len(lens)} {H} {H * G} {D} {CUS} {ns} {ws} {' '.join(map(str, lens))}\n" for H, G, D, lens, ns, ws in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(cases)
    res = []
    for line in out:
        v = list(map(int, line.split()))
        res.append({"ok": v[0], "ns": v[1], "table": v[2], "subs": v[4], "splits": v[5::2], "tokens": v[6::2]})
    return res


def _planned(G):
    return G // 4 if G % 4 == 0 else G // 2 if G % 2 == 0 else G


def test_every_cut_tiles_its_tokens_within_the_workspace(harness):
    rnd = random.Random(11)
    cases = []
    for _ in range(600):
        H, G, D = rnd.choice([1, 2, 3, 4, 8, 32]), rnd.choice([1, 2, 3, 4, 5, 7, 8, 12, 16, 17, 40]), rnd.choice([64, 128, 256])
        n = rnd.choice([1, 63, 200, 1000, 5000, 40000])
        B = rnd.choice([1, 2, 5, 64, 70])
        lens = [n] * B if rnd.random() < 0.4 else [rnd.choice([0, 1, rnd.randint(1, n)]) for _ in range(B)]
        cases.append((H, G, D, lens, rnd.choice([0, 0, 0, 1, 5, 16]), rnd.choice([-1, -1, 1, 3, 40])))
    for (H, G, D, lens, n_splits, ws), c in zip(cases, _cut(harness, cases)):
        q, step = (128, 32) if D == 64 else (64, 16)
        most = min(1024, max(1, -(-max(lens) // q)))
        if not c["ok"]:
            assert ws >= 0 or n_splits > most                     # a workspace for any plan is always enough for one
            continue
        assert c["ns"] <= (ws if ws >= 0 else max(most, n_splits)) and (n_splits == 0 or c["ns"] == n_splits)
        assert -(-G // 16) <= c["subs"] <= max(-(-G // 16), _planned(G))
        for n, nb, st in zip(lens, c["splits"], c["tokens"]):
            assert nb <= c["ns"] and st >= q and st % (step if c["table"] else q) == 0
            assert nb == -(-n // st)


def test_short_sequences_are_whole_and_wide_groups_fill_the_compute_units(harness):
    r = _cut(harness, [(8, 4, 128, [256], 0, -1), (8, 4, 128, [257], 0, -1), (8, 4, 64, [512, 3], 0, -1), (1, 4, 256, [129], 0, -1),
                       (8, 7, 128, [32768], 0, -1), (8, 8, 128, [32768], 0, -1), (8, 4, 128, [32768], 0, -1),
                       (4, 7, 128, [200, 4000, 3000, 1000], 0, -1)])
    assert [c["ns"] for c in r[:4]] == [1, 5, 1, 3]
    # one workgroup takes all query heads of a KV head, and the tokens are cut for the compute units that leaves
    assert [c["ns"] for c in r[4:7]] == [32, 32, 32] and all(c["subs"] == 1 for c in r[4:])
    assert r[7]["table"] == 1 and 56 <= sum(r[7]["splits"]) <= CUS // 4   # split lengths are rounded up to steps


def test_a_workspace_for_the_plan_alone_bounds_the_cut(harness):
    """The plan of 7 heads (7 workgroups for each KV head) makes 5 splits of 32K tokens; a workspace for those is accepted and not
    exceeded, one less is refused."""
    r = _cut(harness, [(8, 7, 128, [32768], 0, 5), (8, 7, 128, [32768], 0, 4), (8, 7, 128, [32768], 0, 12)])
    assert r[0]["ok"] and r[0]["ns"] == 5 and not r[1]["ok"] and r[2]["ns"] == 12


def test_finer_cuts_than_the_plan_keep_256_tokens_beyond_64_splits(harness):
    r = _cut(harness, [(2, 16, 128, [8192], 0, -1), (1, 7, 128, [16384], 0, -1), (1, 7, 128, [65536], 0, -1), (4, 8, 128, [8192], 0, -1),
                       (1, 7, 128, [16384, 100], 0, -1)])
    assert [c["ns"] for c in r[:4]] == [64, 64, 256, 64] and r[4]["splits"][0] == 64
    # where the plan is launched as it is, it is not touched
    assert _cut(harness, [(1, 4, 128, [16384], 0, -1)])[0]["ns"] == 256


def test_a_given_split_count_shares_out_the_heads_within_one_l2(harness):
    """Split counts made for a workgroup per 4, 2 or 1 query heads: idle compute units take a share of the heads where the workgroups of
    a KV head lie a multiple of 8 apart, and never more than the plan has."""
    r = _cut(harness, [(8, 16, 128, [32768], 8, -1), (8, 8, 128, [32768], 16, -1), (8, 8, 128, [32768], 32, -1), (8, 7, 128, [32768], 5, -1),
                       (2, 7, 128, [4096], 16, -1), (8, 16, 128, [32768], 0, 8), (8, 16, 128, [32768], 0, -1), (8, 4, 128, [32768], 8, -1),
                       (8, 16, 128, [8192] * 4, 2, -1), (2, 16, 128, [8192] * 2, 16, -1)])
    assert [c["subs"] for c in r] == [4, 2, 1, 1, 7, 4, 1, 1, 1, 4]


def test_batches_that_fill_the_compute_units_unevenly_are_cut_more_finely(harness):
    """Where one workgroup for each compute unit, or a whole sequence for each, leaves some with far more tokens than the mean, there are several
    workgroups for every compute unit instead; an even plan stays."""
    rnd = random.Random(5)
    ragged = [rnd.randint(200, 4000) for _ in range(48)]
    r = _cut(harness, [(4, 7, 128, ragged, 0, -1), (8, 4, 128, ragged, 0, -1), (8, 4, 128, [2000] * 48, 0, -1), (3, 4, 128, [6000] * 8, 0, -1),
                       (8, 4, 128, [4000] * 32, 0, -1), (32, 1, 128, [544] * 32, 0, -1), (8, 4, 128, [5000, 5100, 5200, 5300], 0, -1),
                       (4, 7, 128, ragged, 0, 2)])
    for c, H in ((r[0], 4), (r[1], 8)):
        assert c["table"] and 2.6 * CUS <= H * sum(c["splits"]) <= 3 * CUS
        size = [min(n, st) for n, st in zip(ragged, c["tokens"])]
        assert max(size) * H * 2 <= sum(ragged) * H * H / CUS       # no split is longer than half of a compute unit's share
    assert r[2]["splits"] == [2] * 48                               # 768 workgroups, three for each of 256; 384 would be one and a half
    assert 8 * 3 * r[3]["splits"][0] <= CUS                         # not a few more than there are compute units
    assert r[4]["ns"] == 1 and r[5]["ns"] == 1                      # one, or four, for each as it is
    assert 0.9 * CUS <= 8 * sum(r[6]["splits"]) <= CUS              # ragged, but even with one for each
    assert r[7]["ok"] and r[7]["ns"] <= 2                           # within the workspace


def test_a_finer_cut_has_to_save_more_than_it_costs(harness):
    """Two workgroups for each compute unit as planned, of at most 256 tokens: three would save less than 1 us by the model, and take more."""
    rnd = random.Random(5)
    r = _cut(harness, [(2, 4, 128, [rnd.randint(260, 400) for _ in range(128)], 0, -1)])[0]
    assert r["ns"] == 2 and set(r["splits"]) <= {1, 2}


def test_a_finer_cut_has_a_step_for_every_wavefront(harness):
    """One split for every eight steps of a sequence at most: 128 tokens, 256 at head_dim 64."""
    rnd = random.Random(9)
    cases = [(1, 4, 128, [rnd.randint(260, 600) for _ in range(96)], 0, -1), (2, 2, 64, [rnd.randint(600, 900) for _ in range(80)], 0, -1),
             (2, 4, 256, [rnd.randint(130, 500) for _ in range(66)], 0, -1)]
    for (H, G, D, lens, _, _), c in zip(cases, _cut(harness, cases)):
        assert c["table"] and max(c["splits"]) > 1
        assert all(nb <= -(-n // (256 if D == 64 else 128)) for n, nb in zip(lens, c["splits"]))


def test_a_table_is_made_where_its_order_saves_more_than_its_lookups(harness):
    """The cuts that need none (whole sequences, and one split length for more than 64) have one where lengths differ by much, or where there are several splits
    each and more than compute units; none where a compute unit has many workgroups for that or all are about as long, nor where sequences are fewer
    than compute units, equal, or empty ones are to be written."""
    rnd = random.Random(3)
    ragged = lambda B, lo, hi: [rnd.randint(lo, hi) for _ in range(B)]
    whole = _cut(harness, [(32, 1, 128, ragged(40, 20, 250), 0, -1), (8, 4, 128, ragged(128, 20, 250), 0, -1), (32, 1, 128, ragged(64, 20, 250), 0, -1),
                           (32, 1, 128, ragged(40, 10, 60), 0, -1), (3, 4, 64, ragged(128, 20, 100), 0, -1), (32, 4, 128, ragged(128, 20, 250), 0, -1),
                           (32, 1, 128, ragged(7, 20, 250), 0, -1), (32, 1, 128, [200] * 40, 0, -1), (32, 1, 128, ragged(40, 20, 250) + [0], 0, -1)])
    assert all(c["ns"] == 1 for c in whole)
    assert [c["table"] for c in whole] == [1, 1, 1, 0, 0, 0, 0, 0, 0]
    cut = _cut(harness, [(8, 4, 128, ragged(80, 300, 2000), 0, -1), (16, 2, 128, ragged(80, 130, 400), 0, -1), (1, 4, 128, [200] * 99 + [30000], 0, -1),
                         (4, 4, 128, ragged(70, 300, 700), 0, -1), (32, 1, 64, ragged(128, 400, 700), 0, -1), (1, 4, 64, ragged(65, 513, 600), 0, -1),
                         (16, 4, 256, ragged(66, 130, 300), 0, -1)])
    assert [c["table"] for c in cut] == [1, 1, 1, 1, 0, 0, 0]


def test_the_order_of_the_grid_holds_every_sequence(tmp_path):
    """Every sequence is in the order once; where the longest come first, the splits' sizes fall along it."""
    src = tmp_path / "order.cpp"
    src.write_text(r"""
#include <cstdio>
#include <cstdlib>
#include "attn_splits.hpp"
int main()
{
    std::srand(7);
    int sorted = 0;
    for (int it = 0; it < 3000; ++it) {
        const int G = 1 + std::rand() % 20, H = 1 + std::rand() % 32, D = 64 << (std::rand() % 3), B = 1 + std::rand() % 140, top = 1 + std::rand() % (it % 2 ? 6000 : 300);
        int32_t lens[140];
        for (int b = 0; b < B; ++b) lens[b] = std::rand() % 9 ? std::rand() % top + 1 : it % 3 ? 1 : 0;
        const kvb::AttnShape s{B, H, H * G, D, 256};
        int max_len = 0;
        for (int b = 0; b < B; ++b) max_len = lens[b] > max_len ? lens[b] : max_len;
        kvb::AttnCut c{};
        const size_t ws = (size_t)B * H * G * (D + 2) * 4 * kvb::max_auto_splits(s, max_len);
        if (!kvb::cut_tokens(s, lens, it % 5 ? 0 : 1 + std::rand() % 3, ws, &c)) continue;
        if (!c.use_table) { if (c.longest_first) return 1; continue; }
        bool seen[140] = {};
        int last = 1 << 30, items = 0;
        for (int r = 0; r < B; ++r) {
            const int b = c.order[r], n = c.tab.first[b + 1] - c.tab.first[b], size = lens[b] < c.tab.tokens[b] ? lens[b] : c.tab.tokens[b];
            if (b >= B || seen[b]) return 2;
            seen[b] = true;
            if (n < 0 || n > c.ns || (long long)n * c.tab.tokens[b] < lens[b]) return 3;
            if (c.longest_first && size > last) return 4;
            last = size;
            items += n;
        }
        if (items != c.tab.first[B] || (c.longest_first && (items > 65535 || c.subs != 1))) return 5;
        sorted += c.longest_first;
    }
    std::printf("%d\n", sorted);
    return sorted > 100 ? 0 : 6;
}
""")
    exe = str(tmp_path / "order")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined", "-I", os.path.join(ROOT, "paper_2604_26557_amd", "csrc"), str(src), "-o", exe])
    subprocess.check_call([exe])


def test_cuts_of_very_long_sequences(tmp_path):
    """Lengths whose sum with a split length does not fit 32 signed bits: every cut holds its tokens, within the workspace, and no
    arithmetic overflows."""
    src = tmp_path / "long.cpp"
    src.write_text(r"""
#include <cstdlib>
#include "attn_splits.hpp"
int main()
{
    std::srand(17);
    for (int it = 0; it < 4000; ++it) {
        const int G = 1 + std::rand() % 20, H = 1 + std::rand() % 32, D = 64 << (std::rand() % 3), B = 1 + std::rand() % 140;
        const int32_t top = (1 << 29) + std::rand() % (3 << 29);
        int32_t lens[140];
        for (int b = 0; b < B; ++b) lens[b] = it % 2 ? top : std::rand() % 3 ? top - std::rand() % (1 << 29) : std::rand() % 1000;
        const kvb::AttnShape s{B, H, H * G, D, 256};
        const size_t per_split = (size_t)B * H * G * (D + 2) * 4;
        const int max_ws = it % 5 ? 1024 : 1 + std::rand() % 64;
        kvb::AttnCut c{};
        if (!kvb::cut_tokens(s, lens, it % 7 ? 0 : 1 + std::rand() % 40, per_split * max_ws, &c)) continue;
        if (c.ns < 1 || c.ns > max_ws) return 1;
        for (int b = 0; b < B; ++b) {
            const long long st = c.use_table ? c.tab.tokens[b] : c.split_tokens, n = c.use_table ? c.tab.first[b + 1] - c.tab.first[b] : c.ns;
            if (st < 1 || n < 0 || n > c.ns || n * st < lens[b]) return 2;
            if (kvb::splits_of(lens[b], (int)st) != (lens[b] + st - 1) / st) return 3;
        }
    }
    return 0;
}
""")
    exe = str(tmp_path / "long")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                           "-I", os.path.join(ROOT, "paper_2604_26557_amd", "csrc"), str(src), "-o", exe])
    subprocess.check_call([exe])


def _cut_harness(tmp_path, *flags):
    exe = str(tmp_path / "attn_cut")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", *flags, "-I", os.path.join(ROOT, "paper_2604_26557_amd", "csrc"),
                           os.path.join(ROOT, "tests", "attn_cut_harness.cpp"), "-o", exe])
    return exe


def test_the_cut_of_a_ragged_batch_is_the_plainly_written_one(tmp_path):
    """Tables, costs and orders of 20000 batches, every number equal; a cut that is left out unseen is not the cheaper one."""
    subprocess.check_call([_cut_harness(tmp_path, "-O1", "-fsanitize=address,undefined")])


def test_the_cut_of_a_ragged_batch_costs_the_host_little(tmp_path):
    """Every layer's call makes the cut, so it must not weigh beside a launch.  The yardstick is a comparison sort of 128 keys in the same process
    (0.8 us where these cuts take 0.5-2.8); a cut that sorts its tables each time takes six to eight of those, one that gives out
    256 workgroups one by one over 64 sequences more than twenty."""
    out = subprocess.run([_cut_harness(tmp_path, "-O3"), "time"], capture_output=True, text=True, check=True).stdout.splitlines()
    ratios = {line.rsplit(" ", 1)[0]: float(line.rsplit(" ", 1)[1]) for line in out}
    assert len(ratios) == 9
    assert all(r < 4.5 for r in ratios.values()), ratios
