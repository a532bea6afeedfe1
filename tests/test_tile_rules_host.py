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
        } else {                                               // d F E k counts -> forms; height, units, room, then rows:tiles of each
            moe_dims D{};
            if (scanf("%d %d %d %d", &D.d, &D.F, &D.E, &D.k) != 4) return 1;
            std::vector<int> c(D.E);
            int N = 0;
            for (int& n : c) { if (scanf("%d", &n) != 1) return 1; N += n; }
            D.T = N / D.k;
            printf("%s %s\n", gate_up_few(&D) ? "few" : gate_up_streams(&D) ? "stream" : "big",
                   down_few(&D) ? "few" : down_form(&D) == Down::STREAM ? "stream" : down_form(&D) == Down::BIG ? "big" : "either");
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
                        printf(" %d:%d", w.nrows, w.tiles);
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
    """((form, height, units, room, [(rows, tiles of the expert)]) of the gate/up projection, of the down projection)"""
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
            groups[p] |= {((n + 31) // 32, nt > 1, "one K block" if (d, F)[p] == 128 else "more", p == 1 and d // 128 % 2 == 1)
                          for n, nt in tiles}
    for p in range(2):
        assert heights[p] == {256, 224, 192, 160, 128}
        for want in ("one K block", "more"):
            met = {(g, shared) for g, shared, k_blocks, _ in groups[p] if k_blocks == want}
            # narrow tiles alone, two groups beside a taller tile, full tiles alone and as one of several
            assert met >= {(1, False), (2, False), (2, True)} | {(g, False) for g in range(3, 9)} | {(g, True) for g in range(3, 8)}
    assert {g for g, _, _, half_empty in groups[1] if half_empty} == set(range(1, 9))


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
#include <cstdio>
using namespace moe355;
int main() {                                                   // slots, nine boundaries -> helpers, begin and fixed of each XCD
    int slots, begin[NXCD + 1];
    while (scanf("%d", &slots) == 1) {
        for (int& b : begin) if (scanf("%d", &b) != 1) return 1;
        const int units = begin[NXCD], chunk = (units + NXCD - 1) / NXCD;
        bool uneven = false;                                   // as the wave of the kernel that makes the lists does, lane by lane
        int at[NXCD + 1], fixed[NXCD], left = 0, room = 0;
        for (int x = 0; x < NXCD; ++x) uneven |= far_off(begin[x], min(x * chunk, units), chunk);
        for (int x = 0; x <= NXCD; ++x) at[x] = uneven ? begin[x] : min(x * chunk, units);
        for (int x = 0; x < NXCD; ++x) left += at[x + 1] - at[x] - (fixed[x] = fixed_units(at[x + 1] - at[x], slots));
        const int helpers = helpers_for(left);
        for (int x = 0; x < NXCD; ++x) room += min(helpers, slots - fixed[x]);
        printf("%d", room >= left ? helpers : slots);
        for (int b : at) printf(" %d", b);
        for (int f : fixed) printf(" %d", f);
        printf("\n");
    }
    return 0;
}
"""


def test_every_unit_of_a_dealt_list_has_a_block(tmp_path):
    """Random lists, even to all on one XCD, with barely enough blocks to twice as many: the parts cover the list in order, and the
    blocks that look for a unit of the rest are at least as many as it has units."""
    (tmp_path / "deal.hip").write_text(DEAL)
    subprocess.run([HIPCC, "--cuda-host-only", "-O2", "-std=c++17", "-I", CSRC, "-I", ROOT + "/include", str(tmp_path / "deal.hip"), "-o",
                    str(tmp_path / "deal")], check=True, capture_output=True)
    rng, cases = random.Random(2), []
    for _ in range(2000):
        units = int(2 ** rng.uniform(0, 15)) - 1
        even = [units * x // 8 for x in range(9)]
        cuts = [0, *sorted(rng.randint(0, units) for _ in range(7)), units]
        mix = rng.choice([0.0, 0.02, 0.3, 1.0])
        slots = (units + 7) // 8 + rng.choice([0, 0, 1, units // 32, units // 8])
        cases.append((slots, [0, *sorted(round(a + mix * (b - a)) for a, b in zip(even, cuts))[1:-1], units]))
    cases.append((5, [0] * 8 + [40]))
    out = subprocess.run([str(tmp_path / "deal")], input="\n".join(f"{s} " + " ".join(map(str, b)) for s, b in cases), check=True,
                         capture_output=True, text=True).stdout.splitlines()
    assert len(out) == len(cases)
    for (slots, cuts), line in zip(cases, out):
        helpers, *rest = map(int, line.split())
        begin, fixed = rest[:9], rest[9:]
        count = [b - a for a, b in zip(begin, begin[1:])]
        assert begin[0] == 0 and begin[8] == cuts[8] and min(count) >= 0
        assert all(0 <= f <= min(c, slots) for f, c in zip(fixed, count))
        assert sum(min(helpers, slots - f) for f in fixed) >= sum(count) - sum(fixed)
