// Which kernel takes which GEMM, and how its rows are cut into tiles: arithmetic on sizes only, for the host and the device.
#pragma once
#include "moe_internal.hpp"

#include <cmath>

namespace moe355 {

// Row tiles of an expert up to which its weights are read past the caches (us, through / past them; gate/up | down): 64 experts x 4096
// x 1408 at 80 rows 141.6 / 133.8 | 102 / 89, 112 148 / 141 | 112 / 98, 224 200 / 197 | 153 / 140, 258 (two tiles) 234 / 236 | 164 /
// 157, 420 337 / 340 | 232 / 235; 128 x 2048 x 768 at 112 88 / 83 | 76 / 69, 258 142 / 143 | 126 / 119; 16 x 3072 x 2048 at 80 42.1 /
// 38.3 | 26.3 / 25.7.  With four tiles (1030 rows) the gate/up projection is 2 % slower past them, 4 % at 7168 x 2048.
constexpr int GATE_UP_ONCE_TILES = 1, DOWN_ONCE_TILES = 2;
// Tiles that take the narrow path of ffn_gemm: up to so many rows if they are all of their expert's, up to so many if another tile shares
// the weights.  (16 experts of 130 rows x 7168 x 512, tiles of 64 and 66, gate/up, us: both narrow 62.2, one 51.4: two and three groups
// do not keep in step.)
constexpr int NARROW_ROWS = 96, NARROW_SHARED_ROWS = 64;

// one work unit: rows [row0, row0 + nrows) of an expert x feature tile ft (128 features gate/up, 256 down); tiles: row tiles of the
// expert, as far as MANY_TILES
struct Work { int32_t expert; int32_t row0; int32_t ft; int16_t nrows, tiles; };
constexpr int MANY_TILES = 3;
__host__ __device__ inline bool narrow_tile(const Work& w) { return w.nrows <= (w.tiles == 1 ? NARROW_ROWS : NARROW_SHARED_ROWS); }

// Rows [row0, row0 + nrows) of tile i when `rows` rows make nt tiles.
// The expert's G = ceil(cnt/32) groups of 32 rows are dealt out evenly: tile i covers groups [i*G/nt, (i+1)*G/nt).
// The tiles that share a weight tile are then within one group of each other: they advance nearly in step and
// fetch it once, only the expert's last group is partly filled, and a tile's matrix time follows its height.
// With the groups of 64 of a layout whose short tiles left whole waves idle (so that every tile cost the time
// of a full one) the gate/up projection took 1.98 ms at 1030 rows per expert and takes 1.82, at 258 rows
// 0.81 -> 0.71 ms, at 896..1152 rows 1.94 -> 1.87 ms (d = 7168, F = 2048, 64 experts; 258: d = 5120, F = 1536,
// 128 experts); at full tiles nothing changes.  The down projection is 6 % faster at 258 rows, 3 % at 960, and
// 3..5 % slower at 1030..1152; cutting its remainder off as one short tile measures the same as dealing evenly.
// A remainder of at most 64 rows as a narrow tile that reads past the caches does not pay in the gate/up projection: it runs ahead
// of the tiles it shares the weight tile with, and the weight tile is fetched twice (8 % slower at 248..264 rows).
// An expert of 129..160 rows in tiles of at most 128 has 64 rows in a narrow tile and the others in a full one.  Both read the
// weights the same way (GATE_UP_ONCE_TILES): with the narrow one past the caches each of the two fetched them, and the gate/up
// projection of such experts took (us, that / this / both on the full tile's loop / one tile of 160): 32 x 7168 x 512 113 / 80 / 85 /
// 78, 16 x 7168 x 1024 91 / 69 / 76 / 77, 8 x 7168 x 2048 79 / 64 / 72 / 73, 8 x 5120 x 1536 53 / 48 / 51 / 57, 16 x 2048 x 768 24.3 /
// 22.9 / 25.1 / 27.7.
__host__ __device__ inline void split_rows(int rows, int nt, int i, Work& w) {
    const int64_t G = (rows + 31) / 32;
    const int lo = min(rows, 32 * (int)(i * G / nt)), hi = min(rows, 32 * (int)((i + 1) * G / nt));
    w.row0 = lo;
    w.nrows = (int16_t)(hi - lo);
    w.tiles = (int16_t)min(nt, MANY_TILES);
}

// ------------------------------------------------------------------ tile heights
// 256 rows are the most a tile can have, but not always the best: units come in rounds of one a CU, and a round that is a
// quarter full takes nearly as long as a full one.  16 experts of 750 rows x 3072 x 2048 make 3.25 rounds of tiles of up to 256 rows,
// 178 us, and 4 full ones of shorter tiles, 160.  The cost of `units` units in K steps of a tile of eight groups of 32 rows (a step costs
// 0.2 + 0.1 n at n groups, what lies between two tiles 4 steps, a started round 0.7 of a full one) was fitted to 27 layers of 130 to 1100
// rows per expert, both projections, heights 96 to 256: the height it picks is 0.2 % above the best of them on average, always
// taking 256 5.7 %.
constexpr int CUS = 256, NXCD = 8;
constexpr int HEIGHTS = 5;                          // 256, 224, 192, 160, 128
__host__ __device__ constexpr int tile_height(int j) { return TOK_TILE - 32 * j; }
__host__ __device__ inline float tiles_cost(int64_t units, float groups_per_tile, int nkb) {
    const int64_t full = units / 256, rest = units % 256;
    const float rounds = (float)full + (rest ? 0.7f + 0.3f / 256.0f * (float)rest : 0.0f);
    return rounds * (4.0f + (float)nkb * (0.2f + 0.1f * groups_per_tile));
}
// the best of the heights that need at most `capacity` units (256 needs no asking)
__host__ __device__ inline int pick_height(const int (&tiles)[HEIGHTS], int groups, int n_ft, int nkb, int64_t capacity) {
    int best = 0;
    float least = 0.0f;
    for (int j = 0; j < HEIGHTS && tiles[0] > 0; ++j) {
        const int64_t units = (int64_t)tiles[j] * n_ft;
        if (j > 0 && units > capacity) break;
        const float c = tiles_cost(units, (float)groups / (float)tiles[j], nkb);
        if (j == 0 || c < least) {
            least = c;
            best = j;
        }
    }
    return tile_height(best);
}

// ------------------------------------------------------------------ dealing a list to the XCDs
// Every XCD gets a contiguous part of its list, so that tiles which share weights stay behind one L2.  Parts of equal numbers are of
// unequal cost where loads are skewed (4096 tokens x 8 of 128 Zipf experts, gate/up: XCDs done between 474 and 692 us), and XCDs are not
// equally fast (256 experts of about 1024 rows: 6.66 to 7.10 ms with the same work).  Hence parts of equal cost where the slowest XCD
// gains by them, and of a part of six rounds and more the last sixteenth is nobody's: a block that finds no unit of its own takes the next of
// its XCD, then of the XCD with the most left.  us, equal numbers / this: the Zipf layer 1245 / 1175, the 256 experts 13505 / 13305, 128
// experts of 257..261 rows 1116 / 1100.
// What an expert's tiles cost, for each feature tile: a tile of 8 groups 1.6 times one of 2 (Zipf gate/up 68 and 46 us).
__host__ __device__ inline int tiles_share(int tiles, int groups) { return 8 * tiles + groups; }
// Units run one to a CU in rounds, and with few rounds it is their number that counts: a list that makes one full round in parts of equal
// numbers may make two where an XCD with cheap units gets more of them than it has CUs.  So parts of equal cost are taken only where the
// slowest XCD, by its rounds and its mean unit, is the faster for it (us, equal numbers / equal cost always / this: 8 experts of 2372 x 5
// tokens, 2816 x 640 148.8 / 181.1 / 148.7, 17 Zipf experts of 2920 x 2, 4096 x 1792 204.6 / 230.9 / 201.5, 43 of 1179 x 8, 3328 x 1152
// 215.9 / 241.4 / 216.7, 60 of 777 x 5, 2176 x 896 130.4 / 117.1 / 122.7).
__host__ __device__ inline float rounds_time(int units, float cost) {
    return units > 0 ? (float)((units + CUS / NXCD - 1) / (CUS / NXCD)) * cost / (float)units : 0.0f;
}
struct alignas(128) Queue {
    int32_t total;                                   // units of the list
    int32_t helpers;                                 // blocks of each XCD that look for a unit of the rest
    int32_t begin[NXCD + 1];                         // XCD x has [begin[x], begin[x+1])
    int32_t fixed[NXCD];                             // of which the first so many go to its blocks in turn, and the rest to whoever is free
};
struct alignas(128) Rest { int32_t taken; };         // how many of an XCD's rest are gone
__host__ __device__ inline int list_blocks(int units) { return (units + NXCD - 1) / NXCD * NXCD; }
// A unit of the rest waits for an atomic, 1..2 us, and so does a block that finds none: with six rounds of units or more to an XCD it is
// not felt, with four (64 experts of 150..200 rows x 4096 x 1408, down, 117 us) it took 7 us.  For the same reason only twice as many blocks
// look for one as there are, or every block where those would be too few.
constexpr int REST_UNITS = 192;
// Parts of equal cost are not taken either where no XCD would be off by more than an eighth of its part (whole rounds stay whole).
__host__ __device__ inline bool far_off(int begin, int even, int chunk) { return begin - even > chunk / 8 || even - begin > chunk / 8; }
// slots: blocks that each XCD will have.  Any unit of the rest finds a block: 8 * slots are at least as many as all units.
__host__ __device__ inline int fixed_units(int count, int slots) { return min(count >= REST_UNITS ? count - count / 16 : count, slots); }
__host__ __device__ inline int helpers_for(int left) { return (left + NXCD - 1) / NXCD * 2; }

// Where a list of `units` would be cut, at equal costs (begin) and at equal numbers (what lies before those cuts costs cost_to).
struct Cuts { int32_t begin[NXCD + 1], cost_to[NXCD + 1]; };
__host__ __device__ inline void no_cut(Cuts& c, int x, int units) {
    c.begin[x] = x == 0 ? 0 : units;
    c.cost_to[x] = 0;
}
// The cuts that fall into one expert of nt > 0 tiles and cost `cost`; the list up to and with it has tiles_to tiles that cost cost_to.
__host__ __device__ inline void cut_expert(Cuts& c, int nt, int tiles_to, int cost, int cost_to, int cost_all, int n_ft, int units) {
    const float per_cost = (float)n_ft / (float)cost, per_unit = (float)cost / (float)nt;
    const int first = (tiles_to - nt) * n_ft, chunk = (units + NXCD - 1) / NXCD;
#pragma unroll
    for (int x = 1; x < NXCD; ++x) {                           // on whole feature tiles: their row tiles share the weights
        const int in = cost_all * x / NXCD - (cost_to - cost);
        if (in >= 0 && in < cost) c.begin[x] = first + min((int)((float)in * per_cost), n_ft - 1) * nt;
    }
#pragma unroll
    for (int x = 1; x <= NXCD; ++x) {
        const int in = min(x * chunk, units) - first;
        if (in > 0 && in <= nt * n_ft) c.cost_to[x] = (cost_to - cost) * n_ft + (int)((float)in * per_unit);
    }
}
// Which of the two cuts a list gets, and what of it is left to whoever is free.  V holds a number for every XCD and one more: a lane
// each in a wave of the kernel (by one thread, one XCD after another, 1.5 us), an array on the host.
template <class V>
__host__ __device__ inline void deal(const V& v, const Cuts& cuts, int units, int slots, Queue& q) {
    const int chunk = (units + NXCD - 1) / NXCD;
    const auto even = v.each([&](int x) { return min(x * chunk, units); });
    auto at = even;
    if (units > CUS) {                                         // (a round or less: by numbers)
        const auto begin = v.each([&](int x) { return cuts.begin[x]; });
        const auto cost_to = v.each([&](int x) { return cuts.cost_to[x]; });
        const float part = (float)v.last(cost_to) / NXCD;
        const float by_cost = v.most(v.each([&](int, int b, int next) { return rounds_time(next - b, part); }, begin, v.next(begin)));
        const float by_number = v.most(v.each([&](int, int e, int next, int c, int c_next) { return rounds_time(next - e, (float)(c_next - c)); },
                                              even, v.next(even), cost_to, v.next(cost_to)));
        if (by_cost < by_number && v.any(v.each([&](int, int b, int e) { return far_off(b, e, chunk); }, begin, even))) at = begin;
    }
    const auto count = v.each([&](int, int b, int next) { return next - b; }, at, v.next(at));
    const auto fixed = v.each([&](int, int n) { return fixed_units(n, slots); }, count);
    const int left = v.sum(v.each([&](int, int n, int f) { return n - f; }, count, fixed)), helpers = helpers_for(left);
    const int room = v.sum(v.each([&](int, int f) { return min(helpers, slots - f); }, fixed));
    v.put(q.begin, at, NXCD + 1);
    v.put(q.fixed, fixed, NXCD);
    q.total = units;
    q.helpers = room >= left ? helpers : slots;
}

// The unit of block `slot` of an XCD, or whether it looks for one of the rest.
constexpr int LOOK = -1, NO_UNIT = -2;
__host__ __device__ inline int own_unit(int begin, int fixed, int helpers, int slot) {
    return slot < fixed ? begin + slot : slot < fixed + helpers ? LOOK : NO_UNIT;
}
// A unit of what the XCDs have left over, for a block of XCD x with no unit of its own: of its own XCD while there are any, then of the
// one with the most.  NO_UNIT: none anywhere.  R counts what is gone of each XCD's rest: take(y) one more, of how many before; taken(y).
template <class R>
__host__ __device__ inline int take_rest(const Queue& q, R rest, int x) {
    for (int tries = 0; tries <= NXCD; ++tries) {              // (a try that fails has found one more XCD's rest used up, for good)
        const int own = q.begin[x + 1] - q.begin[x] - q.fixed[x];
        if (own > 0) {
            const int t = rest.take(x);
            if (t < own) return q.begin[x] + q.fixed[x] + t;
        }
        int taken[NXCD], most = 0;
#pragma unroll
        for (int y = 0; y < NXCD; ++y) taken[y] = rest.taken(y);
#pragma unroll
        for (int y = 0; y < NXCD; ++y) {
            const int left = q.begin[y + 1] - q.begin[y] - q.fixed[y] - taken[y];
            x = left > most ? y : x;
            most = max(most, left);
        }
        if (most == 0) return NO_UNIT;
    }
    return NO_UNIT;
}

// One list for each projection: its feature tiles, K blocks and room.
struct ListShape { int n_ft, nkb, capacity; bool one_height; };
__host__ __device__ inline int list_height(const ListShape& s, const int (&tiles)[HEIGHTS], int groups) {
    return s.one_height ? TOK_TILE : pick_height(tiles, groups, s.n_ft, s.nkb, s.capacity);
}

// ------------------------------------------------------------------ which kernel takes which GEMM
// The streaming kernels (ffn_stream.hip) where the weights are the bound, the big tiles where matrix work or the L2 reuse of
// weights between row tiles counts.  The lines were measured with both sides on the same buffers (us, big tiles / streaming;
// the big-tile side already reads the weights of narrow tiles past the caches):
//   gate/up  rows per expert 2: 1026 / 1006 (256 experts), 3: 163 / 142, 6: 136 / 133, 12: 129.5 / 133, 16: 251..287 / 274..287
//            and, where the tiles leave compute units idle: 96 units, 4 rows 35 / 23, 32 rows 33 / 28; 384 units, 8 rows 79 / 68
//   down     even loads, rows per expert: 64 experts x 4096 x 1408 12: 72 / 67, 24: 77 / 72, 40: 82 / 80; 128 x 5120 x 1536 24: 199 /
//            193, 40: 211 / 209, 64 level to 7 % slower; 128 x 2048 x 768 24: 51 / 48, 40: 55 / 52; 16 x 3072 x 2048 40: 24.8 / 25.4;
//            256 x 7168 x 2048 12: 668 / 639, 24: 709 / 697, 30: 705 / 715, 40: 736 / 762.  The widest layers cross at 27 rows, but
//            only with even loads: Zipf loads at a mean of 12..48 rows 638 / 624 to 931 / 887 there
//   linear   by streaming units, big tiles of the chosen height / streaming (more than 64 rows; K = 1024 and 7168 cross at the same
//            place): 128 units 512 x 4096 x 4096 27.4 / 17.4, 256 512 x 8192 35.0 / 31.5, 1000 x 4096 29.2 / 24.3, 2000 x 2048 29.2 / 24.7;
//            320 320 x 16384 35.9 / 44.8, 352 1400 x 4096 30.7 / 36.2, 512 1000 x 8192 39.6 / 57.1, 704 700 x 16384 47.9 / 78.6
constexpr int64_t GATE_UP_STREAM_ROWS = 8, GATE_UP_STREAM_ROWS_IDLE = 32, DOWN_STREAM_ROWS = 48;
// Rows per expert are a mean.  A skewed load is no reason against streaming (down projection, Zipf loads at a mean of 6..48: 0.73..0.99
// of the big tiles' time; nine tokens in ten on the same k experts: 0.70..0.97), but a concentrated one is: with every token on the same
// k experts nothing but their weights is read, once for each tile of 64 rows, matrix work counts, and streaming takes 1.1..1.8 times as
// long.  The host cannot see the load.  Where the streaming units of such a batch, k experts of T rows, are at most the figures
// below it still costs a layer nothing to speak of (448 units: 145 us before there was a streaming kernel, 145 with it; 384: 98 and 86; 512: 74.3
// and 74.0; above: 672 units 160 and 178, 3584 units 424 and 553).  Beyond them the gate/up projection takes the big tiles, which
// are level there, and for the down projection the kernel that makes the lists counts: more than twice as many 64-row tiles as big ones
// (an ordinary load has 1.0..1.55 times as many, a concentrated one of that size 2.5..4) fill the big tiles' list, otherwise it
// stays empty; both kernels are launched and the one that has nothing to do returns.
constexpr int64_t GATE_UP_SKEW_UNITS = 256, DOWN_SKEW_UNITS = 512;
constexpr int LINEAR_STREAM_UNITS = 256;

// upper bound on row tiles: every full tile, and one more for each expert that has rows
inline int64_t max_row_tiles(const moe_dims* D, int rows) {
    const int64_t N = (int64_t)D->T * D->k;
    return N / rows + (N < D->E ? N : D->E);
}
// A small layer streams whatever its rows per expert: at most one gate/up unit to a CU, and at most four of the shorter down units (the big
// tiles' units are half as many and leave more than half of the chip idle; neither list nor sorted scales are needed).  The down projection
// alone, beside big gate/up tiles that need their list anyway: one unit to a CU.  The units at most: no load
// makes more.  Layers, us, big tiles / streaming, and units of the gate/up | down projection: 350 tokens x 4 of 16 experts, 2048 x 512
// 46.0 / 34.5, 148 | 296; 400 x 2 of 8, 4096 x 1024 66.0 / 43.2, 160 | 320; 60 x 6 of 8, 7168 x 2048 88.5 / 73.4, 208 | 364; 640 x 1 of 8,
// 7168 x 1536 96.9 / 91.8, 216 | 504; 200 x 8 of 9, 7168 x 512 83.3 / 68.2, 136 | 952; 700 x 4 of 16, 2048 x 512 49.0 / 48.1, 236 | 472;
// Zipf loads 500 x 4 of 8, 2048 x 512 48.1 / 42.1, 156 | 312; and beyond: 1024 x 1 of 16, 4096 x 1024 72.0 / 75.2, 256 | 512, 1000 x 2 of 8,
// 1024 x 1024 39.4 / 40.6, 312 | 156.  The down projection alone: 92 units 23.2 / 13.6, 156 16.2 / 13.7, 180 13.7 / 11.4, 216 13.7 / 12.9,
// 252 15.8 / 17.5.
// Layers narrower than 512 do not cross at these units: with one to three K blocks a unit, many units are mostly ends (7000 x 1 of 4,
// 2048 x 256 65.0 / 69.7, 226 | 904; 700 x 5 of 64, 2048 x 256 58.6 / 63.2, 236 | 944; 500 x 5 of 40, 3072 x 384 70.2 / 73.5, 237 | 948;
// 2500 x 4 of 16, 1024 x 128 51.4 / 52.9, 172 | 688), while few units or narrow inputs gain (400 x 2 of 8, 7168 x 384 86.4 / 54.4, 60 | 560;
// 300 x 4 of 8, 256 x 1536 34.7 / 30.0, 312 | 26).
constexpr int64_t SMALL_GATE_UP_UNITS = 240, SMALL_DOWN_UNITS = 1000, SMALL_DOWN_ALONE_UNITS = 200, SMALL_WIDTH = 512;
inline bool few_units(const moe_dims* D, int feature_tiles, int64_t most) {
    return D->d >= SMALL_WIDTH && D->F >= SMALL_WIDTH && max_row_tiles(D, STREAM_ROWS) * feature_tiles <= most;
}
inline bool small_layer(const moe_dims* D) {
    return few_units(D, D->F / 128, SMALL_GATE_UP_UNITS) && few_units(D, (D->d + 255) / 256, SMALL_DOWN_UNITS);
}

inline bool skew_is_harmless(const moe_dims* D, int feature_tiles, int64_t most_units) {
    const int64_t tiles = (D->T + STREAM_ROWS - 1) / STREAM_ROWS;
    return tiles <= 1 || D->k * tiles * feature_tiles <= most_units;    // one tile: no weight passes twice
}
enum class Down { BIG, STREAM, EITHER };
inline Down down_form(const moe_dims* D) {
    if (small_layer(D) || few_units(D, (D->d + 255) / 256, SMALL_DOWN_ALONE_UNITS)) return Down::STREAM;
    if ((int64_t)D->T * D->k > DOWN_STREAM_ROWS * D->E) return Down::BIG;
    return skew_is_harmless(D, (D->d + 255) / 256, DOWN_SKEW_UNITS) ? Down::STREAM : Down::EITHER;
}
inline double experts_met(const moe_dims* D) {                 // with at least one row when the router favours none
    return D->E * (1.0 - pow(1.0 - (double)D->k / D->E, (double)D->T));
}
// (only where the down projection streams for certain: then no lists are needed)
inline bool gate_up_streams(const moe_dims* D) {
    const int64_t N = (int64_t)D->T * D->k;
    if (N > 0 && small_layer(D)) return true;
    if (N == 0 || down_form(D) != Down::STREAM || !skew_is_harmless(D, D->F / 128, GATE_UP_SKEW_UNITS)) return false;
    if (N <= GATE_UP_STREAM_ROWS * D->E) return true;
    return N <= GATE_UP_STREAM_ROWS_IDLE * D->E && experts_met(D) * (D->F / 128) < CUS;
}
// One token to a few, so that a tile of 16 rows holds every expert's rows: the kernels of ffn_few.hip (streaming = 1).
// Gate/up while the streaming blocks leave the chip half empty or in an uneven second round.  By units of 128 features, d = 4096:
// 66 units 0.81, 132 0.79, 198 0.98, 308 0.91; d = 5120: 96 0.88, 192 0.90, 264 0.89, 336 level; shorter rows pay for the ends of a
// block (d = 2048: 48 units 0.82, 132 0.94, 168 level, 234 1.17), longer ones keep a streaming block busy (d = 7168: 20 0.46, 64 0.73,
// 128 1.10, 256 1.10).
// Down, six blocks of 25 KB to a CU: whatever their number where K = F is long enough for the ends of a block not
// to count.  F = 1280, 6144 features, 1152..14054 blocks: 0.85..0.96; 1408, 768..6496: 0.94..1.00; 1536, 1280..13188: 0.86..1.00; 2048,
// 4096 features, 1024..10550: 0.98..1.03, 2048 features, 512..6526: 0.81..1.04, 7168 features, 1792..22840: 0.96..1.03, level.
// Shorter ones up to 1400 blocks: F = 768 0.93..1.00, beyond them 1464..6496 0.97..1.15; F = 1024, 2796..7913 1.02, 1.01, 0.95.
inline bool gate_up_few(const moe_dims* D) {
    if (D->T > FEW_ROWS || !gate_up_streams(D)) return false;
    const double units = experts_met(D) * (D->F / 128);
    return units < (D->d >= 6144 ? 112 : D->d >= 3072 ? 320 : 200);
}
inline bool down_few(const moe_dims* D) {
    return D->T <= FEW_ROWS && down_form(D) == Down::STREAM && (D->F >= 1280 || experts_met(D) * (D->d / 32) <= 1400);
}
// Persistent blocks (ffn_flow.hip), one to a CU: gate/up projections bound by their weights, with enough units to keep most CUs busy.  Whole layers,
// us, big tiles or streaming / this, by units of 128 features: 108..120 units 55 / 68, 41 / 46, 39 / 43; 155 (34 rows per expert) 42.2 / 39.4, 180
// 79.0 / 72.5, 204 102.5 / 94.4, 245 123.6 / 115.0, 315 130 / 124, 376 143 / 137, 533 272 / 263, 704 (256 x 6 of 64, 4096 x 1408) 247 / 237, 1120
// (112 experts of 13 rows, 1152 x 1280) 113 / 97, 1632 (16 x 8 of 256, 7168 x 2048) 687 / 682.  Up to eight rows per expert the streaming kernel is
// the other one, whose blocks are half a unit, two to a CU: this one has to fill its rounds of units (as even loads make them; skewed ones make
// fewer), and more than one: a single round gains with even loads, 190 units 49.4 / 45.1, and loses as much where a log meets fewer experts than
// that, 207 expected of a Zipf load (63 x 1 of 69, 4480 x 640) 52.3 / 57.7.  By the share of the last round's blocks that have a unit and those
// before it: 0.52 137 / 150, 0.66 165 / 179 and 63.4 / 65.8, 0.70 81.1 / 84.2, 0.74 94.8 / 98.9, 0.81 (Zipf) 245 / 258, 0.82 496 / 503; 0.91 687 /
// 682, 0.97 189 / 178, 0.98 105 / 97; in between either way, 0.78 104 / 100, 0.79 166 / 158.
// Tiles are of up to 96 rows, so a concentrated log's weights pass more often than in tiles of 256 (GATE_UP_SKEW_UNITS).  Where its
// units make one round of blocks at most this is still the faster form, 210 units 86.6 / 70.9, 200 109.6 / 97.9, 208 75.4 / 62.4 and 45.0 /
// 35.8; beyond one round not: 294 117.5 / 142.5, 315 64.9 / 73.9, 396 102.8 / 110.5, 672 127.6 / 155.9, and neither is it with Zipf loads of
// that size (1.02 to 1.07).  (Even loads would gain 0 to 3 % there.)
// Down: level with the streaming kernel (0.97 to 1.1), so taken where that one is not: with more rows, or where a list would be needed to choose
// (48..96 rows and more, us, big tiles / this, behind gate/up in persistent blocks: 62.3 / 58.2, 56.2 / 50.5, 56.6 / 52.4).
constexpr int FLOW_ROWS = 96, FLOW_MAX_KB = 128;  // expert-sorted rows per tile; K blocks
constexpr int64_t FLOW_UNITS = 140, FLOW_SKEW_UNITS = 256;
constexpr double FLOW_FILL_FEW_ROWS = 0.85;
inline bool gate_up_flows(const moe_dims* D) {
    const int64_t N = (int64_t)D->T * D->k;
    if (N == 0 || N > FLOW_ROWS * D->E || gate_up_few(D)) return false;
    for (int K : {D->d, D->F})
        if (K < 4 * QBLOCK || K > FLOW_MAX_KB * QBLOCK) return false;
    if ((D->T + FLOW_ROWS - 1) / FLOW_ROWS * D->k * (D->F / 128) > FLOW_SKEW_UNITS) return false;
    const double units = experts_met(D) * (D->F / 128);
    if (N > GATE_UP_STREAM_ROWS * D->E) return units >= FLOW_UNITS;
    return units > CUS && units >= FLOW_FILL_FEW_ROWS * CUS * ceil(units / CUS);
}
inline bool down_flows(const moe_dims* D) {
    return gate_up_flows(D) && ((int64_t)D->T * D->k > DOWN_STREAM_ROWS * D->E || down_form(D) != Down::STREAM);
}
inline bool linear_streams(int32_t rows, int32_t NOUT) {
    return rows <= STREAM_ROWS || ((int64_t)rows + STREAM_ROWS - 1) / STREAM_ROWS * ((NOUT + 255) / 256) <= LINEAR_STREAM_UNITS;
}

// Output rows of the big tiles go past the caches where nobody will find them there: stored through them, each XCD's L2 is full of dirty
// lines that wait to be written while the next kernel loads, and the last-level cache keeps outputs instead of inputs (us, through / past).
// Linear with its quantisation, calls one behind another, nine states in turn (nothing is found in a cache): 268 MB of y 8192 x 7168 x 8192
// 486 / 476, K = 4096 309 / 305, K = 2048 191 / 193, 302 MB 9216 x 7168 x 8192 562 / 552, 537 MB 16384 x 7168 x 8192 939 / 928, K = 2048
// 366 / 367, 724 MB 12727 x 4864 x 14208 858 / 847; the same weights again 476 / 450, 305 / 285, 189 / 179, 557 / 528, 942 / 928, 354 /
// 344, 851 / 842; everything again 481 / 445 and, K = 2048, 190 / 179.  One call alone on new inputs and buffers ends later, 470 / 481 and
// 483 / 489, K = 2048 177 / 201, 9216 rows 552 / 552, 12727 rows 814 / 810: what the caches would have written behind its end has been
// written in it.  256 MB is the last-level cache's size.  Below it the same buffers gain as well, 210 MB 3200 x 2048 x 16384 126 / 123,
// K = 7168 356 / 347, 235 MB 7168 x 7168 x 8192 419 / 391, but 197 MB 3000 x 2048 x 16384 114.5 / 116.1; so do some with K = 1024, 393 MB 6000
// x 1024 x 16384 153 / 147, 268 MB 16384 x 1024 x 4096 120 / 121.
// Layers, whose combine comes at once and finds the last part, three states in turn: 805 MB 8192 x 6 of 64, 4096 x 1408 1133 / 1116, 1.3 GB
// 8192 x 8 of 128, 5120 x 1536 2037 / 2007, 1.6 GB 16000 x 6 of 64, 4096 x 1024 1692 / 1659, 7.5 GB 32768 x 8 of 256, 7168 x 2048 13040 /
// 12943, a call alone on new inputs and buffers 1 to 2 % shorter as well; 720 MB 5500 x 8 of 64, 4096 x 1024 817 / 812 (alone 843 / 847),
// 671 MB 4096 x 8 of 128, 5120 x 1536 1150 / 1157, 402 MB 4096 x 6 of 64, 4096 x 1408 633 / 643.
constexpr int64_t LINEAR_Y_PAST_BYTES = 256ll << 20, LAYER_Y_PAST_BYTES = 768ll << 20;
constexpr int LINEAR_Y_PAST_MIN_K = 2048;
inline bool y_bytes_at_least(int64_t rows, int32_t cols, int64_t bytes) { return rows * cols * (int64_t)sizeof(float) >= bytes; }
inline bool down_goes_past(const moe_dims* D) { return y_bytes_at_least((int64_t)D->T * D->k, D->d, LAYER_Y_PAST_BYTES); }
inline bool linear_goes_past(int32_t rows, int32_t K, int32_t NOUT) {
    return K >= LINEAR_Y_PAST_MIN_K && y_bytes_at_least(rows, NOUT, LINEAR_Y_PAST_BYTES);
}

// 129..160 rows can make two tiles, one of them of 64 rows (us, as chosen / one tile: 130 x 1024 x 22016 12.1 / 13.4, 150 x 4096 x
// 24576 39.0 / 41.3, 160 x 7168 x 32768 65.2 / 70.3)
inline int linear_tiles(int32_t rows, int nft, int nkb) {
    int tiles[HEIGHTS];
    for (int j = 0; j < HEIGHTS; ++j) tiles[j] = (int)(((int64_t)rows + tile_height(j) - 1) / tile_height(j));
    const int h = pick_height(tiles, (int)(((int64_t)rows + 31) / 32), nft, nkb, (int64_t)1 << 30);
    return (int)(((int64_t)rows + h - 1) / h);
}

// Room of a big-tile list, and blocks of its launch: the least height that can be the better one has to fit.  A first round that is
// not full may gain from half the height; the more rounds, the less there is to gain.  us, this room / room for half the height
// everywhere / for 256 alone, gate/up | down: 16 x 3072 x 2048 at 750 rows (992 | 744 units) 172 / 172 / 184 | 99 / 100 / 112, 32 x 3072 x
// 2048 at 260 (1008 | 756) 150 / 150 / 150 | 82 / 82 / 99, 64 x 2048 x 768 at 400 109 / 109 / 108 | 100 / 89 / 94, 32 x 7168 x 2048 at
// 520 (1552 | 2716) 501 / 513 / 507 | 308 / 311 / 310, 128 x 5120 x 1536 at 300 (3324 | 5540) 755 / 762 / 759 | 477 / 478 / 480: beyond a
// few rounds level, and the longer list would be room and blocks for nothing.
// The choice itself is not free (777 tokens x 5 of 60 experts 1.3 us, 256 x 6 of 64 0.8): experts with a mean of up to 96 rows are one
// tile each whatever the height, but for a few of a skewed load.
constexpr int64_t ONE_HEIGHT_ROWS = 96;
inline bool one_height(const moe_dims* D) { return (int64_t)D->T * D->k <= ONE_HEIGHT_ROWS * D->E; }
inline int64_t big_units(const moe_dims* D, int nft) {
    const int64_t units = max_row_tiles(D, TOK_TILE) * nft, half = max_row_tiles(D, TOK_TILE / 2) * nft;
    if (one_height(D)) return units;
    if (half <= 2 * CUS) return half;
    return units <= 8 * CUS ? max_row_tiles(D, 192) * nft : units <= 16 * CUS ? max_row_tiles(D, 224) * nft : units;
}
inline int64_t gate_up_units(const moe_dims* D) {
    if (!gate_up_streams(D)) return big_units(D, D->F / 128);
    return max_row_tiles(D, gate_up_few(D) ? FEW_ROWS : STREAM_ROWS) * (D->F / 128);
}
inline int64_t down_stream_units(const moe_dims* D) { return max_row_tiles(D, STREAM_ROWS) * ((D->d + 255) / 256); }
// EITHER: S > 2B tiles of 64 / of 256 rows over m experts with rows (B >= m, S <= (N + 63m)/64) leave m <= N/65
inline int64_t down_big_units(const moe_dims* D) {
    const int64_t N = (int64_t)D->T * D->k;
    const int nft = (D->d + 255) / 256;
    return down_form(D) == Down::EITHER ? (N / TOK_TILE + N / 65) * nft : big_units(D, nft);
}

inline ListShape gate_up_shape(const moe_dims* D) { return {D->F / 128, D->d / QBLOCK, (int)gate_up_units(D), one_height(D)}; }
inline ListShape down_shape(const moe_dims* D) { return {(D->d + 255) / 256, D->F / QBLOCK, (int)down_big_units(D), one_height(D)}; }

// Dense linear, up to how many blocks of 32 features ffn_few.hip is the better kernel, one to a CU (streaming kernel = 1): 256 blocks,
// 16-row tiles 16 x 4096 x 8192 0.71, 32-row 32 x 4096 x 8192 0.76, 64-row 40 x 4096 x 8192 0.85, 64 x 4096 x 8192 0.97, 128 x 7168 x 4096
// 0.94, 256 x 4096 x 2048 0.83; 384 blocks of 16-row tiles (75 KB, two to a CU) 0.91..1.02, of 32-row tiles 1.2, 512 of 64-row tiles 1.5.
// Tiles of 32 rows while they fit too (128 x 4096 x 2048 0.62 against 0.83 in tiles of 64).
constexpr int FEW_BLOCKS = 256, FEW_BLOCKS_16 = 320;
inline int few_linear_groups(int32_t rows, int32_t NOUT) {           // 16-row groups per tile; 0: another kernel is the better one
    const int64_t cols = NOUT / 32;
    if (rows <= 16) return cols <= FEW_BLOCKS_16 ? 1 : 0;
    if (((int64_t)rows + 31) / 32 * cols <= FEW_BLOCKS) return 2;
    return ((int64_t)rows + 63) / 64 * cols <= FEW_BLOCKS ? 4 : 0;
}

}  // namespace moe355
