"""The rules that choose a GEMM's kernel and the heights of its row tiles (csrc/ffn_rules.hpp), compiled for the host: what the GPU
tests' shapes reach, so that a change of a rule cannot empty those tests, and that tiles cover the rows and fit the lists."""
import random
import subprocess

import pytest

import test_gpu_dispatch as dispatch
import test_gpu_edges as edges
from paper_2512_07710_amd.build import CSRC, HIPCC, ROOT

PROGRAM = r"""
#include "ffn_rules.hpp"
#include <cstdio>
#include <vector>
using namespace moe355;
static int height(const ListShape& s, const std::vector<int>& c, long& units) {
    int tiles[HEIGHTS] = {}, groups = 0;
    for (int n : c) {
        groups += (n + 31) / 32;
        for (int j = 0; j < HEIGHTS; ++j) tiles[j] += (n + tile_height(j) - 1) / tile_height(j);
    }
    const int h = list_height(s, tiles, groups);
    units = 0;
    for (int j = 0; j < HEIGHTS; ++j) if (tile_height(j) == h) units = (long)tiles[j] * s.n_ft;
    return h;
}
int main() {
    char what;
    while (scanf(" %c", &what) == 1) {
        if (what == 'L') {                                     // rows K NOUT -> form, rows of the tiles
            int rows, K, NOUT;
            if (scanf("%d %d %d", &rows, &K, &NOUT) != 3) return 1;
            if (few_linear_groups(rows, NOUT)) printf("few %d\n", few_linear_groups(rows, NOUT));
            else if (linear_streams(rows, NOUT)) printf("stream\n");
            else {
                printf("big");
                const int nt = linear_tiles(rows, (NOUT + 255) / 256, K / QBLOCK);
                for (int i = 0; i < nt; ++i) { Work w; split_rows(rows, nt, i, w); printf(" %d", w.nrows); }
                printf("\n");
            }
        } else {                                               // d F E k counts -> forms; height, units, room, then rows:tiles:narrow of each
            moe_dims D{};
            if (scanf("%d %d %d %d", &D.d, &D.F, &D.E, &D.k) != 4) return 1;
            std::vector<int> c(D.E);
            int N = 0;
            for (int& n : c) { if (scanf("%d", &n) != 1) return 1; N += n; }
            D.T = N / D.k;
            printf("%s %s\n", gate_up_flows(&D) ? "flow" : gate_up_few(&D) ? "few" : gate_up_streams(&D) ? "stream" : "big",
                   down_flows(&D) ? "flow" : down_few(&D) ? "few" : down_form(&D) == Down::STREAM ? "stream" : down_form(&D) == Down::BIG ? "big" : "either");
            for (int list = 0; list < 2; ++list) {
                const ListShape s = list ? down_shape(&D) : gate_up_shape(&D);
                long units;
                const int h = height(s, c, units);
                printf("%d %ld %d", h, units, s.capacity);
                for (int n : c)
                    for (int i = 0, nt = (n + h - 1) / h, at = 0; i < nt; ++i) {
                        Work w;
                        split_rows(n, nt, i, w);
                        if (w.row0 != at) return 2;
                        at += w.nrows;
                        if (i == nt - 1 && at != n) return 3;
                        printf(" %d:%d:%d", w.nrows, w.tiles, narrow_tile(w));
                    }
                printf("\n");
            }
        }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text(PROGRAM)
    subprocess.run([HIPCC, "--cuda-host-only", "-O2", "-std=c++17", "-I", CSRC, "-I", ROOT + "/include", str(d / "rules.hip"), "-o",
                    str(d / "rules")], check=True, capture_output=True)

    def ask(text):
        return subprocess.run([str(d / "rules")], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
    return ask


def _layer(rules, counts, d, F, k=1):
    """((form, height, units, room, [(rows, tiles of the expert, narrow)]) of the gate/up projection, of the down projection)"""
    forms, *lists = rules(f"G {d} {F} {len(counts)} {k} " + " ".join(map(str, counts)))
    out = []
    for form, line in zip(forms.split(), lists):
        h, units, room, *tiles = line.split()
        out.append((form, int(h), int(units), int(room), [tuple(map(int, t.split(":"))) for t in tiles]))
    return out


def test_tile_height_layers_reach_every_height_and_group_count(rules):
    heights, groups = [set(), set()], [set(), set()]
    shapes = [(edges.HEIGHT_COUNTS, d, F) for d, F in edges.HEIGHT_SHAPES] + edges.HEIGHT_LAYERS
    for counts, d, F in shapes:
        for p, (form, h, _, _, tiles) in enumerate(_layer(rules, counts, d, F)):
            assert form == "big"
            heights[p].add(h)
            groups[p] |= {((n + 31) // 32, nt > 1, narrow, "one K block" if (d, F)[p] == 128 else "more", p == 1 and d // 128 % 2 == 1)
                          for n, nt, narrow in tiles}
    for p in range(2):
        assert heights[p] == {256, 224, 192, 160, 128}
        for want in ("one K block", "more"):
            met = {(g, shared, narrow) for g, shared, narrow, k_blocks, _ in groups[p] if k_blocks == want}
            # narrow tiles alone, two groups beside a taller tile, full tiles alone and as one of several
            assert met >= {(g, False, 1) for g in (1, 2, 3)} | {(2, True, 1)} | {(g, False, 0) for g in range(4, 9)} | {(g, True, 0) for g in range(3, 8)}
            assert {(g, shared) for g, shared, narrow in met if narrow} == {(1, False), (2, False), (3, False), (2, True)}
    half_empty = {(g, narrow) for g, _, narrow, _, empty in groups[1] if empty}
    assert half_empty >= {(1, 1), (2, 1), (3, 1)} | {(g, 0) for g in range(3, 9)}


def test_layers_of_one_round_stream(rules):
    forms = lambda d, F: [p[0] for p in _layer(rules, edges.ROUND_COUNTS, d, F)]
    assert [forms(*s) for s in edges.ROUND_SHAPES] == [["stream", "stream"], ["stream", "stream"], ["big", "stream"]]


def test_linear_shapes_reach_what_they_are_for(rules):
    form = lambda r, K, n: rules(f"L {r} {K} {n}")[0].split()
    met = set()
    for shape in dispatch.BIG_LINEARS:
        kind, *rows = form(*shape)
        assert kind == "big" and sum(map(int, rows)) == shape[0]
        met |= {(int(n) + 31) // 32 for n in rows}
    assert met >= set(range(2, 9))
    assert {form(*s)[0] for s in edges.SMALL_LINEARS} == {"few", "stream"}


def test_lists_have_room_for_their_units(rules):
    """Random loads, even to concentrated: whatever height is taken, its units fit the list (and the launch) made for it."""
    rng = random.Random(1)
    for _ in range(300):
        E, k = rng.randint(1, 256), 1
        mean = 2 ** rng.uniform(0, 10)
        p = [rng.random() ** rng.choice([0, 1, 4, 30]) for _ in range(E)]
        counts = [int(mean * E * v / sum(p)) for v in p]
        if sum(counts) == 0 or max(counts) > 60000:
            continue
        for form, _, units, room, _ in _layer(rules, counts, 128 * rng.randint(1, 56), 128 * rng.randint(1, 16)):
            if form == "big":
                assert units <= room


DEAL = r"""
#include "ffn_rules.hpp"
#include <algorithm>
#include <array>
#include <cstdio>
#include <random>
#include <vector>
using namespace moe355;
struct Xcds {                                                  // what the lanes of a wave are to deal() on the device
    template <class T> using Each = std::array<T, NXCD + 1>;
    template <class F, class... A>
    auto each(F f, const A&... a) const {
        Each<decltype(f(0, a[0]...))> r;
        for (int x = 0; x <= NXCD; ++x) r[x] = f(x, a[x]...);
        return r;
    }
    Each<int> next(const Each<int>& v) const { return each([&](int x) { return v[std::min(x + 1, NXCD)]; }); }
    int last(const Each<int>& v) const { return v[NXCD]; }
    float most(const Each<float>& v) const { return *std::max_element(v.begin(), v.end() - 1); }
    int sum(const Each<int>& v) const { int s = 0; for (int x = 0; x < NXCD; ++x) s += v[x]; return s; }
    bool any(const Each<bool>& v) const { return std::any_of(v.begin(), v.end() - 1, [](bool b) { return b; }); }
    void put(int32_t* to, const Each<int>& v, int n) const { std::copy_n(v.begin(), n, to); }
};
struct Launch {                                                // its blocks, in an order as mixed as can be: one that looks may be overtaken
    const Queue& q;
    std::mt19937& rng;
    std::vector<int> blocks, times;
    size_t started = 0;
    int lost = 0;
    Rest rest[NXCD] = {};
    struct Counts {
        Launch& l;
        int take(int x) const { return l.rest[x].taken++; }
        int taken(int y) const {
            const int t = l.rest[y].taken;
            while (y == NXCD - 1 && l.rng() % 4 != 0 && l.block()) {}
            return t;
        }
    };
    bool block() {
        if (started == blocks.size()) return false;
        const int b = blocks[started++];
        int u = own_unit(q.begin[b % NXCD], q.fixed[b % NXCD], q.helpers, b / NXCD);
        if (u == LOOK) u = take_rest(q, Counts{*this}, b % NXCD);
        if (u >= (int)times.size()) ++lost;
        else if (u >= 0) ++times[u];
        return true;
    }
};
int main() {                       // height, feature tiles, slots, experts, their rows -> the queue, the cuts; how often each unit is taken
    int h, n_ft, slots, E;
    std::mt19937 rng(1);
    while (scanf("%d %d %d %d", &h, &n_ft, &slots, &E) == 4) {
        std::vector<int> rows(E);
        int tiles = 0, cost_all = 0, tiles_to = 0, cost_to = 0;
        for (int& r : rows) {
            if (scanf("%d", &r) != 1) return 1;
            tiles += (r + h - 1) / h;
            cost_all += tiles_share((r + h - 1) / h, (r + 31) / 32);
        }
        const int units = tiles * n_ft;
        Cuts cuts;
        for (int x = 0; x <= NXCD; ++x) cuts.begin[x] = 1000 * x, cuts.cost_to[x] = 1000 * x * x;   // not read in one round
        if (units > CUS) for (int x = 0; x <= NXCD; ++x) no_cut(cuts, x, units);
        if (units > CUS) for (int r : rows) {
            const int nt = (r + h - 1) / h, cost = tiles_share(nt, (r + 31) / 32);
            tiles_to += nt;
            cost_to += cost;
            if (nt > 0) cut_expert(cuts, nt, tiles_to, cost, cost_to, cost_all, n_ft, units);
        }
        Queue q;
        deal(Xcds{}, cuts, units, slots, q);
        printf("%d %d", q.total, q.helpers);
        for (int b : q.begin) printf(" %d", b);
        for (int f : q.fixed) printf(" %d", f);
        for (int b : cuts.begin) printf(" %d", b);
        for (int c : cuts.cost_to) printf(" %d", c);
        Launch l{q, rng, std::vector<int>(NXCD * slots), std::vector<int>(units)};
        for (int i = 0; i < NXCD * slots; ++i) l.blocks[i] = i;
        std::shuffle(l.blocks.begin(), l.blocks.end(), rng);
        while (l.block()) {}
        for (int t : l.times) l.lost += t != 1;
        printf(" %d\n", l.lost);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    """(list height, feature tiles, blocks of an XCD, rows of the experts), ... -> (helpers, begin, fixed, cuts, cost up to the even cuts) of each,
    after every block of the launch has taken its unit."""
    d = tmp_path_factory.mktemp("deal")
    (d / "deal.hip").write_text(DEAL)
    subprocess.run([HIPCC, "--cuda-host-only", "-O2", "-std=c++17", "-I", CSRC, "-I", ROOT + "/include", str(d / "deal.hip"), "-o",
                    str(d / "deal")], check=True, capture_output=True)

    def ask(lists):
        text = "\n".join(" ".join(map(str, [h, n_ft, slots, len(rows), *rows])) for h, n_ft, slots, rows in lists)
        out = subprocess.run([str(d / "deal")], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
        assert len(out) == len(lists)
        answers = []
        for (h, n_ft, slots, rows), line in zip(lists, out):
            total, helpers, *v, lost = map(int, line.split())
            begin, fixed, cuts, cost_to = v[:9], v[9:17], v[17:26], v[26:]
            assert total == n_ft * sum(-(-r // h) for r in rows) and lost == 0
            assert begin[0] == 0 and begin[8] == total and begin == sorted(begin)
            assert all(0 <= f <= min(b - a, slots) for f, a, b in zip(fixed, begin, begin[1:]))
            answers.append((helpers, begin, fixed, cuts, cost_to))
        return answers
    return ask


def _random_list(rng):
    h, n_ft, E = rng.choice([256, 224, 192, 160, 128]), rng.choice([1, 2, 3, 9, 16, 28, 56]), rng.randint(1, 256)
    mean, skew = 2 ** rng.uniform(0, 10), rng.choice([0.0, 0.5, 2.0])
    rows = [int(mean * rng.lognormvariate(0, skew)) if rng.random() > 0.1 else 0 for _ in range(E)]
    units = n_ft * sum(-(-r // h) for r in rows)
    if units > 60000:
        return _random_list(rng)
    return h, n_ft, (units + 7) // 8 + rng.choice([0, 0, 1, units // 32, units // 8]), rows


def test_every_unit_of_a_dealt_list_has_a_block(deal):
    """Random lists, even to all on one XCD, with barely enough blocks to many more: every unit is taken once, whoever comes first; the cuts of
    equal cost lie on the feature tile in which that cost is reached, and are taken where the slowest XCD gains by them and only there."""
    rng = random.Random(2)
    lists = [_random_list(rng) for _ in range(1500)] + [(256, 8, 6, [1300]), (128, 1, 0, [0, 0])]
    branches = set()
    for (h, n_ft, slots, rows), (helpers, begin, fixed, cuts, cost_to) in zip(lists, deal(lists)):
        tiles = [-(-r // h) for r in rows]
        cost = [8 * t + -(-r // 32) for t, r in zip(tiles, rows)]
        units, chunk = begin[8], -(-begin[8] // 8)
        even = [min(x * chunk, units) for x in range(9)]
        if units <= 256:
            assert begin == even and cuts == [1000 * x for x in range(9)]
            branches.add("one round")
            continue
        for x in range(1, 8):                                  # feature tile by feature tile, an expert's cost is spread evenly
            before = base = 0
            for t, c in zip(tiles, cost):
                if t and before + c > sum(cost) * x // 8:
                    reached = (sum(cost) * x // 8 - before) * n_ft / c
                    assert (cuts[x] - base) % t == 0 and abs((cuts[x] - base) // t - reached) < 1 + 1e-3
                    break
                before, base = before + c, base + t * n_ft
        for x in range(9):
            left, want = even[x], 0.0
            for t, c in zip(tiles, cost):
                if t:
                    want += c / t * min(left, t * n_ft)
                    left -= min(left, t * n_ft)
            assert abs(cost_to[x] - want) <= 1 + 1e-6 * want
        slowest = lambda cut, part: max([-(-(b - a) // 32) * c / (b - a) for a, b, c in zip(cut, cut[1:], part) if b > a], default=0)
        by_cost, by_number = slowest(cuts, [cost_to[8] / 8] * 8), slowest(even, [b - a for a, b in zip(cost_to, cost_to[1:])])
        gains = by_cost < by_number and any(abs(c - e) > chunk // 8 for c, e in zip(cuts[:8], even))
        if abs(by_cost - by_number) > 1e-5 * by_number:
            assert begin == (cuts if gains else even)
        shared = sum(b - a - f for a, b, f in zip(begin, begin[1:], fixed))
        branches.add(("cost" if begin != even else "numbers", shared > 0, helpers == slots and shared > 0))
    assert branches == {"one round", ("numbers", False, False), ("numbers", True, False), ("cost", False, False), ("cost", True, False), ("cost", True, True)}


def test_dealt_layers_reach_what_they_are_for(rules, deal):
    def branch(counts, d, F, projection):
        form, h, units, room, _ = _layer(rules, counts, d, F)[projection]
        assert form == "big"
        slots = -(-room // 8)
        (helpers, begin, fixed, *_), = deal([(h, (F // 128, (d + 255) // 256)[projection], slots, counts)])
        shared = sum(begin[1:]) - sum(begin[:8]) - sum(fixed)
        return "numbers" if begin == [min(x * -(-units // 8), units) for x in range(9)] else "cost", shared > 0, helpers == slots
    assert [branch(*layer, p) for layer, p in zip(edges.DEALT_LAYERS, (0, 0, 0, 1))] == [
        ("numbers", True, False), ("cost", True, True), ("cost", False, False), ("cost", True, False)]
