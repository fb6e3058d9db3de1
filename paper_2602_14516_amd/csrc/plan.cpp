// Host-side work planner (see plan.h).  Pure integer host code: no HIP calls.
#include "plan.h"

#include <algorithm>
#include <utility>

namespace ampd {

namespace {

constexpr int KV_TILE = 64;          // keys per LDS tile of a wide item; split points are multiples of it
constexpr int MIN_NARROW_CHUNK = 256;
constexpr int NARROW_ITEM_KEYS = 512;  // fixed cost of a narrow item (item, Q, page ids, first block, merge), in keys streamed
constexpr int MIN_WIDE_CHUNK = 512;          // tiles of a launch without decode rows
constexpr int MIN_WIDE_CHUNK_MIXED = 1024;   // ... of a mixed launch
constexpr int WIDE_STAGE_KEYS = 128;   // a tile works through its keys in stages of 128: part of a stage costs a whole one
constexpr int WIDE_ITEM_KEYS = 128;    // fixed cost of a tile (item, Q, first stage, output), in keys of a tile
constexpr int WIDE_SPLIT_KEYS = 1408;  // a piece of a cut tile also writes a partial result of up to 256 rows that the
                                       // combine pass reads again (fitted to single-request latencies, like the others)
constexpr int NUM_XCD = NUM_QUEUES;   // accelerator dies; workgroup i is dispatched to die i % NUM_XCD

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct Cost { int64_t cost; int32_t idx, piece; };      // of an item: its index (or its block's, and which piece of it)

// Longest first, equal ones in the order they have (a library sort with a comparison took a third of planning a launch of 500 items).
void longest_first(std::vector<Cost>& v) {
    if (v.size() <= 32) {
        for (size_t i = 1; i < v.size(); ++i) {
            const Cost c = v[i];
            size_t j = i;
            for (; j > 0 && v[j - 1].cost < c.cost; --j) v[j] = v[j - 1];
            v[j] = c;
        }
        return;
    }
    int64_t most = 0;
    for (const Cost& c : v) most = std::max(most, c.cost);
    std::vector<Cost> to(v.size());
    for (int shift = 0; most >> shift; shift += 8) {               // by the digits of what a cost lacks to the largest one
        int32_t at[257] = {0};
        for (const Cost& c : v) ++at[((most - c.cost) >> shift & 255) + 1];
        for (int i = 1; i < 256; ++i) at[i] += at[i - 1];
        for (const Cost& c : v) to[at[(most - c.cost) >> shift & 255]++] = c;
        v.swap(to);
    }
}

}  // namespace

namespace {

// Whether a small launch with prefill rows goes as blocks of at most 32 query rows throughout (narrow items, whose 8 waves share
// the keys) instead of tiles of 256, and the chunk that their key ranges are cut to.
// Blocks are eight times as many workgroups, each of them 256 keys further in 1.75 us where a tile takes 3 us for 128: while they fit
// one round of the CUs they take half of the tiles' time, and shorter ranges need no cut and no combine pass; but eight of them read
// the keys that one tile reads, and together they do only a third of its work per time.  Both ways are priced in ns, from launches of
// 1 and 4 rows of 16 to 512 new tokens over 0 to 16 k, five head geometries and both caches (us, tiles -> blocks, 8-bit and bf16: 32 tokens
// over 256, 8 heads of 64 15.9 -> 12.6 and 11.0 -> 9.8; 64 over 1 024, 8 KV heads, groups of 4 27.0 -> 17.7 and 22.6 -> 14.6; 256 over
// 2 048, the same 39.6 -> 28.8 and 34.2 -> 25.8; four times 64 over 4 096 46.7 -> 42.9 and 42.8 -> 42.7, 16 k 82 -> 133 and 88 -> 170; 512
// over 1 024 44.1 -> 37.3 and, with more items than the table in the arguments holds, 38.4 -> 43.0).
bool take_blocks(const Shape& s, const std::vector<ReqInfo>& reqs, const PlanOptions& opt, int64_t* chunk_out) {
    const int tq = 32 / (s.Hq / s.Hkv), tile = ATTN_WAVES * tq;
    const bool d64 = s.D == 64, fp8 = opt.kv_bytes == 1;
    const int64_t slots = opt.wg_slots;
    int64_t n_blocks = 0;
    bool any = false;
    for (const ReqInfo& r : reqs) {
        if (r.L <= 0) continue;
        n_blocks += r.L <= tq ? s.Hkv : ceil_div(r.L, tq) * s.Hkv;
        if (n_blocks > (fp8 ? 2 : 1) * slots) return false;
        any |= r.L > tq;
    }
    if (!any) return false;
    struct Run { int32_t keys; uint32_t units; int32_t n; };   // n blocks or tiles of about that many keys: units of 256 or 128 keys
    std::vector<Run> list;                                     // rows of more than one block, as blocks; the others (few); tiles
    list.reserve(3 * reqs.size());
    auto add = [&](int32_t keys, int32_t unit, int64_t n) { list.push_back(Run{keys, (uint32_t)ceil_div(keys, unit), (int32_t)n}); };
    for (const ReqInfo& r : reqs)
        if (r.L > tq) add(r.C + r.L, 256, ceil_div(r.L, tq) * s.Hkv);
    const size_t n_runs = list.size();
    for (const ReqInfo& r : reqs)                              // cut by the rule for decode
        if (r.L > 0 && r.L <= tq) add(r.C + r.L, 256, s.Hkv);
    const size_t n_few = list.size();
    int64_t n_tiles[2] = {0, 0}, tile_units = 0;               // full tiles; tiles of at most 128 query rows, half the work a stage
    uint32_t longest[2] = {0, 0};                              // in stages
    for (const ReqInfo& r : reqs) {
        if (r.L <= tq) continue;
        const int32_t nt = (int32_t)ceil_div(r.L, tile), rest = r.L - (nt - 1) * tile, half = 2 * rest <= tile;
        for (int h = 0; h < 2; ++h) {
            const int32_t n = (h ? half : nt - half) * s.Hkv;
            if (n == 0) continue;
            add(h && nt > 1 ? r.C + r.L % tile : r.C + r.L, WIDE_STAGE_KEYS, h ? -n : n);
            n_tiles[h] += n;
            tile_units += (int64_t)list.back().units * n;
            longest[h] = std::max(longest[h], list.back().units);
        }
    }
    const Run *runs = list.data(), *few = runs + n_runs, *tiles = runs + n_few, *end = runs + list.size();
    auto pieces = [](const Run* i, const Run* e, uint32_t units) {      // of `units` units each
        int64_t n = 0;
        for (; i != e; ++i) n += (int64_t)((i->units + units - 1) / units) * i->n;
        return n;
    };
    // Both searches start from the uncut launch and end where the longest piece alone is no better than the best so far.
    // blocks: rounds of 256 keys, whole or in pieces that fit one round, cut only while a table in the arguments holds the cut blocks (the
    // rule the prices were fitted with, over lists in the workspace too); the pieces of a row's blocks read its
    // keys from the memory-side cache, at 8 TB/s
    const int64_t round_ns = d64 ? 1030 : 1750, start_ns = d64 ? 4700 : 6500;
    auto price = [&](const Run* v, const Run* e, int64_t* chunk) {
        int64_t blocks = 0, bytes = 0, units = 0;
        uint32_t longest = 0;
        for (const Run* i = v; i != e; ++i) {
            longest = std::max(longest, i->units);
            blocks += i->n;
            units += (int64_t)i->units * i->n;
            bytes += (int64_t)i->keys * i->n * 2 * s.D * opt.kv_bytes;
        }
        // Between one block a CU and two: the second ones start late, and the fewer they are the less evenly the launch ends.  (80 launches of
        // 257 to 512 blocks, 8-bit: with a fixed tenth on top, 10 were slower than as tiles, 7 rows of 40 tokens over 3 000 41.4 -> 46.4 the most.)
        const int64_t all = blocks > slots ? units * round_ns * (10 * slots + 3 * std::max<int64_t>(0, 2 * slots - blocks)) / (10 * slots * slots) +
                                                 (d64 ? 800 : 3500)
                                           : 0;
        int64_t best = start_ns + 5 * blocks + std::max<int64_t>(longest * round_ns, all);
        *chunk = 1 << 30;
        if (blocks > TILE_TABLE_COMBS) return best;
        for (uint32_t rounds = 1; rounds < longest; rounds += 1 + rounds / 8) {
            if (start_ns + rounds * round_ns + 4000 + 13 * blocks > best) break;
            if (units > slots * rounds) continue;
            const int64_t n = pieces(v, e, rounds);
            if (n > slots) continue;
            const int64_t cost = start_ns + std::max(rounds * round_ns, bytes / 8000) + 4000 + 13 * n;
            if (cost < best || (cost == best && *chunk == 1 << 30)) {
                best = cost;
                *chunk = 256 * (int64_t)rounds;
            }
        }
        return best;
    };
    int64_t best = price(runs, few, chunk_out);
    // tiles: stages of 128 keys, whole or in pieces of four stages or more that fit one round
    const int64_t full_ns = d64 ? 1950 : 3000, half_ns = d64 ? 1050 : 1650, extra_ns = d64 ? 50 : 200, piece_ns = d64 ? 12 : 22;
    auto tile_cost = [&](uint32_t stages, int64_t nf, int64_t nh) {
        const int64_t work = std::max(std::min(stages, longest[0]) * (full_ns + (2 * nf + nh) * extra_ns / slots), std::min(stages, longest[1]) * half_ns);
        return (d64 ? 5200 : 6600) + work * (fp8 ? 23 : 20) / 20 + (fp8 ? 1200 : 0);
    };
    const uint32_t longest_tile = std::max(longest[0], longest[1]);
    int64_t best_tiles = tile_cost(longest_tile, n_tiles[0], n_tiles[1]);
    for (uint32_t stages = 4; stages < longest_tile; stages += 1 + stages / 8) {
        if (tile_cost(stages, n_tiles[0], n_tiles[1]) >= best_tiles) break;
        if (tile_units > slots * stages) continue;
        int64_t nf = 0, nh = 0;
        for (const Run* i = tiles; i != end; ++i) {
            const int64_t n = (int64_t)((i->units + stages - 1) / stages) * i->n;
            (n > 0 ? nf : nh) += n > 0 ? n : -n;
        }
        if (nf + nh <= slots) best_tiles = std::min(best_tiles, tile_cost(stages, nf, nh) + 4000 + (2 * nf + nh) * piece_ns);
    }
    if (few != tiles) {
        // Next to decode rows: only where the tiles last longer than those would alone (otherwise the launch is a matter of cutting
        // the decode rows well: 76 rows of 2.5-6 k tokens next to two of up to 30 34.5 -> 43.6).  Over a bf16 cache tiles cost 4 us more there:
        // their list needs an upload launch, which most blocks do without (see build_blocks), and where the blocks' list does not fit the
        // arguments either, tiles are still dearer than priced above: 70 such drawn batches, which go as blocks for those
        // 4 us alone, take 1.17 times as long sent as tiles (37 short rows next to two prefills 23.1 -> 37.9, the most; the least 0.84).
        int64_t chunk;
        const int64_t others = price(few, tiles, &chunk);
        if (others > best_tiles) return false;
        best = std::max(std::max(best, others), start_ns + pieces(runs, tiles, 1) * round_ns * 11 / (10 * slots) + 1000);
        best_tiles += fp8 ? 0 : 4000;
    }
    // The prices were fitted where this matters most, on launches of up to 40 us.  Longer ones are many rows of few tokens over long contexts,
    // whose tiles run up to a fifth faster than that (their loads overlap across rows) and whose blocks read every key up to eight times: of 700
    // such launches 51 were slower as blocks than as tiles (five rows of 20 to 130 tokens over 600 to 8 000, 8-bit 65.9 -> 84.3), with this 15.
    constexpr int64_t LONG_NS = 38000;
    if (best_tiles > LONG_NS) best_tiles = LONG_NS + (best_tiles - LONG_NS) * 6 / 10;
    return 100 * best <= 97 * best_tiles;
}

// Append items: consecutive runs of packed rows, whatever request they belong to (a decode batch of 96 rows is two items,
// not 96); each names the request and token its first row belongs to.
void add_append_items(const Plan& plan, int rows, std::vector<Item>& items) {
    int r = 0;
    for (int64_t row = 0; row < plan.sum_L; row += rows) {
        while (row >= (int64_t)plan.reqs[r].row_off + plan.reqs[r].L) ++r;
        items.push_back(Item{r, pack_heads(0, 0, 0, KIND_APPEND), (int32_t)(row - plan.reqs[r].row_off),
                             (int32_t)std::min<int64_t>(rows, plan.sum_L - row), 0, 0, -1, plan.reqs[r].C,
                             plan.reqs[r].row_off, plan.reqs[r].L, {0, 0}});
    }
}

Item null_item() { return Item{-1, pack_heads(0, 0, 0, KIND_NULL), 0, 0, 0, 0, -1, 0, 0, 0, {0, 0}}; }

// What a tile table says of the launch as a whole, and its rows; false when it has no room for them.  row_of (one entry per request):
// the table's row.
bool begin_tiles(const Shape& s, int32_t chunk, int32_t few_chunk, bool blocks, const Plan& out, TileTable& t, std::vector<int32_t>& row_of) {
    const int G = s.Hq / s.Hkv;
    if (G > 32 || s.Hkv > 64 || out.combs.size() > (size_t)TILE_TABLE_COMBS) return false;
    t.n_rows = 0;
    t.n_combs = (int32_t)out.combs.size();
    t.chunk = chunk;
    t.few_chunk = few_chunk;
    t.tq = (blocks ? 1 : ATTN_WAVES) * (32 / G);
    t.kind = blocks ? KIND_NARROW : KIND_WIDE;
    t.G = G;
    t.D = s.D;
    t.sum_L = (int32_t)out.sum_L;
    // These launches end with their append items, so an item is small: two 16-byte chunks of K and of V per thread, one trip to
    // memory (one prefill of 509 tokens over 8 heads of 128, 64 rows an item -> 16 -> 8: 59.6 -> 53.8 -> 53.2 us on the GPU).
    t.append_rows = std::max(4, std::min(APPEND_ITEM_ROWS, 8192 / (s.Hkv * s.D)));
    row_of.assign(out.reqs.size(), -1);
    for (const ReqInfo& r : out.reqs) {
        if (r.L <= 0) continue;
        if (t.n_rows == TILE_TABLE_ROWS) return false;
        row_of[r.req] = t.n_rows;
        t.rows[t.n_rows++] = r;
    }
    return true;
}

// A launch of blocks (out.reqs holds the rows): items, combine tiles, launch order.  In a launch that fits one round the blocks that
// would make one tile read the same keys at the same rate, so they go next to each other on one die, as tiles of one stream do, larger
// groups first, each to the shortest queue; null items pad the shorter dies' queues.  Where that is more than a round, or more on
// a die than it has slots: longest first.  All KV heads of a row are alike and its groups are known when the blocks are made, so no
// more than one head's items is ever sorted, and a list that travels in the arguments is written as its codes straight away: planning
// 256 tokens over 2 048 (8 KV heads) takes 1.7 us; the launch as tiles took 13, blocks by sorted items and a vector per group 34.
void build_blocks(const Shape& s, int32_t chunk, int32_t few_chunk, const PlanOptions& opt, Plan& out) {
    const int G = s.Hq / s.Hkv, tq = 32 / G, tile = ATTN_WAVES * tq, slots = opt.wg_slots;
    struct Block { int32_t req, q0, nq, pieces; };             // of one KV head
    struct Row { int32_t block0, block1, group0, group1, chunk; };
    std::vector<Block> blocks;
    std::vector<Row> rows;
    blocks.reserve(slots);
    rows.reserve(out.reqs.size());
    int64_t items = 0;
    for (const ReqInfo& r : out.reqs) {
        if (r.L <= 0) continue;
        Row row{(int32_t)blocks.size(), 0, 0, 0, r.L <= tq ? few_chunk : chunk};
        const int32_t rest = r.L % tq;
        for (int q0 = 0, nq = rest ? rest : tq; q0 < r.L; q0 += nq, nq = tq) {
            blocks.push_back(Block{r.req, q0, nq, (int32_t)ceil_div(r.C + q0 + nq, row.chunk)});
            items += (int64_t)blocks.back().pieces * s.Hkv;
        }
        row.block1 = (int32_t)blocks.size();
        rows.push_back(row);
    }

    struct Place { int32_t block, kvh, piece; };
    std::vector<Place> launch;
    auto by_die = [&]() {
        struct Group { int32_t block, n, piece; };             // piece `piece` of blocks [block, block + n)
        std::vector<Group> groups;
        groups.reserve(slots);
        uint32_t sizes = 0;                                    // of groups, one bit each (at most 9: the first block may be a remainder)
        for (Row& row : rows) {
            row.group0 = (int32_t)groups.size();
            for (int piece = 0; piece < blocks[row.block1 - 1].pieces; ++piece)
                for (int i = row.block0, j = i; i < row.block1; i = j) {
                    const int tile_end = (blocks[i].q0 / tile + 1) * tile;
                    while (j < row.block1 && blocks[j].q0 < tile_end) ++j;
                    while (i < j && blocks[i].pieces <= piece) ++i;     // (later blocks see more keys)
                    if (i == j) continue;
                    groups.push_back(Group{i, j - i, piece});
                    sizes |= 1u << (j - i);
                }
            row.group1 = (int32_t)groups.size();
        }
        launch.assign(slots, Place{-1, 0, 0});
        int queue[NUM_XCD] = {0}, n = 0;
        for (int size = 31; size > 0; --size) {
            if (!(sizes >> size & 1)) continue;
            for (const Row& row : rows)
                for (int kvh = 0; kvh < s.Hkv; ++kvh)
                    for (int g = row.group0; g < row.group1; ++g) {
                        if (groups[g].n != size) continue;
                        int x = 0;
                        for (int y = 1; y < NUM_XCD; ++y)
                            if (queue[y] < queue[x]) x = y;
                        if (queue[x] + size > slots / NUM_XCD) return false;
                        for (int k = 0; k < size; ++k) launch[queue[x]++ * NUM_XCD + x] = Place{groups[g].block + k, kvh, groups[g].piece};
                        n = std::max(n, (queue[x] - 1) * NUM_XCD + x + 1);
                    }
        }
        launch.resize(n);
        return true;
    };
    if (items > slots || !by_die()) {
        std::vector<Cost> order;                               // KV head 0
        order.reserve(items / s.Hkv);
        for (const Row& row : rows)
            for (int i = row.block0; i < row.block1; ++i) {
                int32_t keys = out.reqs[blocks[i].req].C + blocks[i].q0 + blocks[i].nq;
                for (int piece = 0; piece < blocks[i].pieces; ++piece, keys -= row.chunk) order.push_back(Cost{std::min(keys, row.chunk), i, piece});
            }
        longest_first(order);
        launch.resize(items);
        Place* to = launch.data();
        for (size_t i = 0, j = 0; i < order.size(); i = j) {   // equal ones of a row, head by head
            const int32_t req = blocks[order[i].idx].req;
            while (j < order.size() && order[j].cost == order[i].cost && blocks[order[j].idx].req == req) ++j;
            for (int kvh = 0; kvh < s.Hkv; ++kvh)
                for (size_t k = i; k < j; ++k) *to++ = Place{order[k].idx, kvh, order[k].piece};
        }
    }
    const int n = (int)launch.size();

    std::vector<int32_t> comb_of(blocks.size() * s.Hkv, -1);   // [KV head][block]
    int32_t max_pieces = 0, max_blocks = 0;
    for (const Row& row : rows) {
        max_blocks = std::max(max_blocks, row.block1 - row.block0);
        for (int kvh = 0; kvh < s.Hkv; ++kvh)
            for (int i = row.block0; i < row.block1; ++i) {
                const Block& b = blocks[i];
                if (b.pieces == 1) continue;
                max_pieces = std::max(max_pieces, b.pieces);
                const int32_t slot = b.nq * G * (s.D + 2);
                comb_of[kvh * blocks.size() + i] = (int32_t)out.combs.size();
                out.combs.push_back(CombItem{b.req, pack_heads(kvh, 0, G, KIND_NARROW), b.q0, b.nq, (int32_t)out.partial_floats, b.pieces, slot, 0});
                out.partial_floats += (int64_t)slot * b.pieces;
            }
    }
    out.num_narrow = items;

    std::vector<int32_t> row_of;
    TileTable& t = out.tiles;
    if (opt.kv_bytes == 2 && n <= TILE_TABLE_ITEMS && max_pieces <= 128 && max_blocks <= 256 && begin_tiles(s, chunk, few_chunk, true, out, t, row_of)) {
        auto code_of = [&](int32_t i, int32_t kvh, int32_t piece, int32_t comb) {
            const int32_t row = row_of[blocks[i].req];
            return (uint32_t)row | (uint32_t)kvh << 4 | (uint32_t)(i - rows[row].block0) << 10 | (uint32_t)piece << 18 | (uint32_t)comb << 25;
        };
        t.n_items = n;
        for (int i = 0; i < n; ++i) {
            const Place& e = launch[i];
            t.items[i] = e.block < 0 ? TILE_NULL : code_of(e.block, e.kvh, e.piece, std::max(0, comb_of[e.kvh * blocks.size() + e.block]));
        }
        for (const Row& row : rows)
            for (int kvh = 0; kvh < s.Hkv && t.n_combs > 0; ++kvh)
                for (int i = row.block0; i < row.block1; ++i) {
                    const int32_t comb = comb_of[kvh * blocks.size() + i];
                    if (comb >= 0) t.combs[comb] = TileComb{code_of(i, kvh, 0, 0), out.combs[comb].part_off};
                }
        out.by_tiles = true;
        return;
    }
    out.items.reserve(n + (opt.append_items ? ceil_div(out.sum_L, APPEND_ITEM_ROWS) : 0));
    for (const Place& e : launch) {
        if (e.block < 0) {
            out.items.push_back(null_item());
            continue;
        }
        const Block& b = blocks[e.block];
        const ReqInfo& r = out.reqs[b.req];
        const int32_t comb = comb_of[e.kvh * blocks.size() + e.block], ch = r.L <= tq ? few_chunk : chunk, keys = r.C + b.q0 + b.nq;
        Item it{b.req, pack_heads(e.kvh, 0, G, KIND_NARROW), b.q0, b.nq, e.piece * ch, keys, -1, r.C, r.row_off, r.L, {0, 0}};
        if (comb >= 0) {
            it.kv_end = std::min(keys - it.kv_begin, ch) + it.kv_begin;
            it.part_off = out.combs[comb].part_off + e.piece * out.combs[comb].part_stride;
        }
        out.items.push_back(it);
    }
}

// The row table of a batch of decode rows alone (out.reqs holds the rows).
void build_table(const Shape& s, int32_t chunk, const PlanOptions& opt, Plan& out) {
    RowTable& t = out.table;
    t.chunk = chunk;
    t.Hkv = s.Hkv;
    t.G = s.Hq / s.Hkv;
    t.D = s.D;
    t.sum_L = (int32_t)out.sum_L;
    int n = 0;
    std::pair<int32_t, int32_t> by_rest[ROW_TABLE_MAX];        // (keys of the remainder, request)
    for (size_t r = 0; r < out.reqs.size(); ++r)
        if (out.reqs[r].L > 0) by_rest[n++] = {(out.reqs[r].C + out.reqs[r].L) % chunk, (int32_t)r};
    std::stable_sort(by_rest, by_rest + n, [](const auto& a, const auto& b) { return a.first > b.first; });
    t.n = n;
    int32_t whole = 0, rests = 0;
    int64_t keys_sum = 0;
    t.max_rows = 0;
    for (int i = 0; i < n; ++i) {
        const ReqInfo& r = out.reqs[by_rest[i].second];
        const int32_t keys = r.C + r.L, pieces = (int32_t)ceil_div(keys, chunk), slot = r.L * t.G * (s.D + 2);
        t.e[i] = RowEntry{r.C, r.row_off, by_rest[i].second | r.L << 24, whole, -1};
        keys_sum += (int64_t)keys * s.Hkv;
        t.max_rows = std::max(t.max_rows, r.L * t.G);
        whole += keys / chunk * s.Hkv;
        rests += by_rest[i].first > 0 ? s.Hkv : 0;
        if (pieces > 1) {
            t.e[i].part_off = (int32_t)out.partial_floats;
            out.partial_floats += (int64_t)slot * pieces * s.Hkv;
            out.num_combs += s.Hkv;
        }
    }
    t.n_whole = whole;
    t.n_items = whole + rests;
    // Small workgroups pay where rows are cut into two or more items per CU and a CU's share of the keys is small enough for
    // the items' fixed costs to show, since neighbours on the CU hide them.  us per call, 8 waves -> 4, rows of 0.4-4, 1.6-16
    // and 3.2-32 k tokens over 8 KV heads, 25 rows (1.7, 6.9, 14 k keys per CU): bf16 48.7 -> 44.8, 147.7 -> 143.3, 313 -> 316;
    // 8-bit 33.8 -> 28.1, 86.6 -> 83.1, 175.7 -> 183.9; 40 rows of 1.6-16 k (11 k keys per CU): 230 -> 235, 129.9 -> 133.8.  Rows
    // that are not cut: 40 rows of 0.2-2 k 8-bit 28.1 -> 33.4, 96 bf16 rows of 2-16 k 552 -> 578; one item per CU: 8 rows of
    // 2-16 k 8-bit 33.8 -> 39.4.  All of these are d = 128 (the only head dimension with such a kernel); over 1 to 16 KV heads,
    // groups of 1 to 16 and pages of 16 to 64, 200 drawn decode batches run at 0.86 of their time before this table, the worst at 1.04.
    const int64_t slots = opt.wg_slots;
    t.small = t.n_items >= 2 * slots && 2 * n * s.Hkv < 3 * slots && keys_sum <= 8192 * slots;
    out.by_table = true;
    out.num_narrow = t.n_items;
    out.num_append = opt.append_items ? ceil_div(out.sum_L, APPEND_ITEM_ROWS) : 0;
    out.num_items = out.num_narrow + out.num_append;
    out.grid = (int32_t)out.num_items;
    out.total_bytes = std::max<int64_t>(256, round_up(out.partial_floats * 4, 256));
}

// The tile table of a launch of uncut or evenly cut tiles (out.items without append items, out.combs in the order of their
// partial results); false when it does not fit.
bool build_tiles(const Shape& s, int32_t chunk, Plan& out) {
    TileTable& t = out.tiles;
    std::vector<int32_t> row_of;
    if (out.num_narrow > 0 || out.items.size() > (size_t)TILE_TABLE_ITEMS || !begin_tiles(s, chunk, 1 << 30, false, out, t, row_of))
        return false;
    bool fits = true;                      // (a row of more than 256 tiles, a tile of more than 128 pieces: no)
    auto code_of = [&](int32_t req, int32_t heads, int32_t q0, int32_t nq, int32_t kv_begin) {
        const uint32_t tile = q0 == 0 ? 0 : (uint32_t)((q0 + nq + t.tq - 1) / t.tq - 1);   // (the first tile holds the remainder)
        if (tile > 255) fits = false;
        return (uint32_t)row_of[req] | (uint32_t)(heads & 0xff) << 4 | tile << 10 | (uint32_t)(kv_begin / chunk) << 18;
    };
    for (int i = 0; i < t.n_combs; ++i) {
        const CombItem& c = out.combs[i];
        if (c.nsplit > 128) return false;
        t.combs[i] = TileComb{code_of(c.req, c.heads, c.q0, c.nq, 0), c.part_off};
    }
    t.n_items = (int32_t)out.items.size();
    for (int i = 0; i < t.n_items; ++i) {
        const Item& it = out.items[i];
        t.items[i] = TILE_NULL;
        if (it.req < 0) continue;
        uint32_t code = code_of(it.req, it.heads, it.q0, it.nq, it.kv_begin);
        if (it.part_off >= 0) {                                    // its cut tile: the last one whose partial results start at or before
            const auto c = std::upper_bound(out.combs.begin(), out.combs.end(), it.part_off,
                                            [](int32_t off, const CombItem& x) { return off < x.part_off; });
            code |= (uint32_t)(c - out.combs.begin() - 1) << 25;
        }
        t.items[i] = code;
    }
    return fits;
}

// Append items, launch size and byte layout of a plan whose attention items (or tile table) and combine tiles are there.
void finish_plan(const PlanOptions& opt, Plan& out) {
    out.num_combs = (int64_t)out.combs.size();
    if (opt.append_items) out.num_append = ceil_div(out.sum_L, out.by_tiles ? out.tiles.append_rows : APPEND_ITEM_ROWS);
    if (out.by_tiles) {
        out.items.clear();
        out.num_items = out.tiles.n_items + out.num_append;
        out.grid = (int32_t)out.num_items;
        out.total_bytes = std::max<int64_t>(256, round_up(out.partial_floats * 4, 256));
        return;
    }
    if (opt.append_items) add_append_items(out, APPEND_ITEM_ROWS, out.items);
    out.num_items = (int64_t)out.items.size();
    out.off_reqs = 0;
    out.off_items = round_up((int64_t)out.reqs.size() * sizeof(ReqInfo), 256);
    out.off_combs = out.off_items + round_up((int64_t)out.items.size() * sizeof(Item), 256);
    out.off_queues = out.off_combs + round_up((int64_t)out.combs.size() * sizeof(CombItem), 256);
    out.plan_bytes = out.off_queues + 256;
    // persistent workgroups pay off where tiles are in the launch (the dies finish together: -1.2 % on configuration 2, -3.5 % on
    // the fused mixed launch of configuration 3); a launch of decode rows alone gains nothing from them (+-1 %)
    out.grid = (int32_t)(out.num_wide > 0 ? std::min<int64_t>((int64_t)out.items.size(), opt.wg_slots) : (int64_t)out.items.size());
    for (int q = 0; q < NUM_QUEUES; ++q) out.queue_heads[q] = out.grid > q ? (out.grid - q + NUM_QUEUES - 1) / NUM_QUEUES : 0;
    out.off_partial = out.plan_bytes;
    out.total_bytes = out.off_partial + round_up(out.partial_floats * 4, 256);
    if (out.total_bytes == 0) out.total_bytes = 256;
}

}  // namespace

void plan_items(const Plan& plan, std::vector<Item>& out) {
    if (!plan.by_table && !plan.by_tiles) {
        out = plan.items;
        return;
    }
    out.clear();
    if (plan.by_tiles) {
        for (int i = 0; i < plan.tiles.n_items; ++i) out.push_back(plan.tiles.items[i] == TILE_NULL ? null_item() : tile_item(plan.tiles, plan.tiles.items[i]));
        if (plan.num_append > 0) add_append_items(plan, plan.tiles.append_rows, out);
        return;
    }
    const RowTable& t = plan.table;
    int row = 0;
    for (int i = 0; i < t.n_items; ++i) {
        if (i < t.n_whole)
            while (row + 1 < t.n && t.e[row + 1].first <= i) ++row;
        else
            row = (i - t.n_whole) / t.Hkv;
        out.push_back(table_item(t, t.e[row], i));
    }
    if (plan.num_append > 0) add_append_items(plan, APPEND_ITEM_ROWS, out);
}

void build_plan(const Shape& s, int num_reqs, const int32_t* ctx_len, const int32_t* incr_len,
                const PlanOptions& opt, Plan& out) {
    out = Plan();
    const int G = s.Hq / s.Hkv;
    const int nhb = (G + 31) / 32;                 // head blocks of at most 32 heads per KV head
    out.reqs.resize(num_reqs);
    int64_t off = 0;
    for (int r = 0; r < num_reqs; ++r) {
        out.reqs[r] = ReqInfo{ctx_len[r], incr_len[r], (int32_t)off, r};
        off += incr_len[r];
    }
    out.sum_L = off;

    // A batch of decode rows alone whose list travels in the kernel's arguments (see RowTable)
    bool by_table = opt.force_kv_splits <= 0 && nhb == 1 && num_reqs < (1 << 24);
    int active = 0;
    for (int r = 0; r < num_reqs && by_table; ++r) {
        by_table = (int64_t)incr_len[r] * G <= 32;
        active += incr_len[r] > 0;
    }
    by_table = by_table && active > 0 && active <= ROW_TABLE_MAX;

    // 1. query blocks
    int64_t block_chunk = 1 << 30;
    const bool blocks = !by_table && opt.force_kv_splits <= 0 && nhb == 1 && take_blocks(s, out.reqs, opt, &block_chunk);
    int64_t narrow_keys = 0;
    int64_t n_wide = 0;
    // (keys, number of blocks with that many): what the split policy needs to know of the blocks; noted for KV head 0
    // and multiplied by the number of KV heads afterwards
    std::vector<std::pair<int32_t, int32_t>> narrow_runs, wide_runs;
    auto note = [](std::vector<std::pair<int32_t, int32_t>>& runs, int32_t keys) {
        if (!runs.empty() && runs.back().first == keys)
            ++runs.back().second;
        else
            runs.emplace_back(keys, 1);
    };
    // f(first token, tokens) of every tile of tq tokens of a row of L.  A tile that is not full costs its workgroup nearly
    // as much per key as a full one, so the remainder of the row goes into the FIRST tile, which sees the fewest keys.
    auto each_tile = [](int32_t L, int tq, auto&& f) {
        const int first = L % tq ? L % tq : tq;
        for (int q0 = 0; q0 < L; q0 += q0 ? tq : first) f(q0, q0 ? tq : first);
    };
    narrow_runs.reserve(num_reqs);
    for (int r = 0; r < num_reqs; ++r) {
        const int C = ctx_len[r], L = incr_len[r];
        for (int g0 = 0; g0 < G && L > 0; g0 += 32) {
            const int gn = std::min(32, G - g0);
            if ((int64_t)L * gn <= 32) {
                narrow_keys += (int64_t)s.Hkv * (C + L);
                note(narrow_runs, C + L);
            } else if (!blocks) {
                each_tile(L, ATTN_WAVES * (32 / gn), [&](int q0, int nq) {
                    n_wide += s.Hkv;
                    note(wide_runs, C + q0 + nq);
                });
            }
        }
    }

    for (auto& r : narrow_runs) r.second *= s.Hkv;
    for (auto& r : wide_runs) r.second *= s.Hkv;

    // 2. split policy (chunk sizes in keys, multiples of KV_TILE)
    // An item costs a few microseconds around its key range (item, Q, page ids and first block before the first key;
    // merge of the waves or the store of a partial result after the last), and a CU runs one item at a time, so
    // nothing hides that: few, long items win as long as the slots (resident workgroups) stay evenly loaded.
    // Candidates are the smallest chunks whose items fit ONE round on all, half or a quarter of the slots, the chunks
    // that give ~2, 3, 4 items per slot, and (tiles) no cut at all.  One round lasts as long as its longest piece; several rounds about a slot's
    // share of the keys plus half a longest piece; every item adds its fixed cost (item_keys, in keys streamed), and
    // every piece of a cut block the cost of its partial result (split_keys: written, and read again by the combine pass).
    int64_t narrow_chunk = 1 << 30, wide_chunk = 1 << 30;
    bool wide_first = false;                               // all tiles before all decode rows
    auto choose_chunk = [&](const std::vector<std::pair<int32_t, int32_t>>& runs, int64_t slots, int64_t granule,
                            int64_t min_chunk, int64_t item_keys, int64_t split_keys) {
        auto count_items = [&](int64_t chunk, int64_t* pieces_of_cut_blocks = nullptr) {
            int64_t n = 0, cut = 0;
            for (const auto& r : runs) {
                const int64_t pieces = ceil_div(r.first, chunk);
                n += pieces * r.second;
                if (pieces > 1) cut += pieces * r.second;
            }
            if (pieces_of_cut_blocks) *pieces_of_cut_blocks = cut;
            return n;
        };
        int64_t n_blocks = 0, max_len = 0, keys = 0;
        for (const auto& r : runs) {
            n_blocks += r.second;
            max_len = std::max<int64_t>(max_len, r.first);
            keys += (int64_t)r.first * r.second;
        }
        const int64_t base = ceil_div(keys, slots);
        int64_t best_cost = -1, best = 1 << 30;
        auto consider = [&](int64_t chunk) {
            int64_t cut = 0;
            const int64_t n = count_items(chunk, &cut);
            const int64_t piece = std::min(chunk, max_len);
            const int64_t cost = (n <= slots ? piece + item_keys : base + piece / 2 + ceil_div(item_keys * n, slots)) +
                                 ceil_div(split_keys * cut, slots);
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                best = chunk;
            }
        };
        // one round on all, half or a quarter of the slots: the smallest chunk whose items fit
        for (int64_t target = slots; target >= slots / 4 && target >= n_blocks; target /= 2) {
            int64_t lo = min_chunk / granule - 1, hi = std::max<int64_t>(min_chunk / granule, ceil_div(max_len, granule));
            while (lo + 1 < hi) {                          // count(hi) = n_blocks <= target
                const int64_t mid = (lo + hi) / 2;
                (count_items(mid * granule) > target ? lo : hi) = mid;
            }
            consider(hi * granule);
        }
        // ~2, 3, 4 items per slot
        for (int per_slot = n_blocks <= slots ? 2 : 1; per_slot <= 4; ++per_slot) {
            const int64_t chunk = std::max<int64_t>(min_chunk, round_up(ceil_div(base, per_slot), granule));
            consider(chunk);
            if (chunk == min_chunk) break;                 // (smaller chunks are not allowed)
        }
        if (split_keys > 0) consider(round_up(max_len, granule));    // whole blocks
        return best;
    };
    if (opt.force_kv_splits <= 0) {
        const int64_t slots = opt.wg_slots;
        if (narrow_keys > 0) {
            // Three or more (row, KV head) blocks for every two slots: whole rows balance well by themselves (longest first),
            // since half of the slots streaming is enough to keep HBM busy to the end; only where a row is a quarter longer
            // than a slot's share of the keys are rows cut, to that share (a cut costs the launch a combine pass, 5 us).
            // Measured for decode rows over 8 KV heads, cut as for fewer blocks -> whole: 48 rows of 1-6 k tokens 113 -> 104 us
            // (8-bit cache 68 -> 59), 50 equal rows 107 -> 103 (64 -> 61), 62 equal rows 125 -> 121 (71 -> 69); 40 rows of
            // 0.5-6 k are better cut (91 against 101 us; 53 against 89).
            int64_t n_blocks = 0, longest = 0;
            for (const auto& r : narrow_runs) {
                n_blocks += r.second;
                longest = std::max<int64_t>(longest, r.first);
            }
            if (2 * n_blocks >= (s.D == 64 ? 4 : 3) * slots) {
                const int64_t share = std::max<int64_t>(MIN_NARROW_CHUNK, round_up(ceil_div(narrow_keys, slots), KV_TILE));
                if (4 * longest > 5 * share) narrow_chunk = share;
            } else {
                narrow_chunk = choose_chunk(narrow_runs, slots, KV_TILE, MIN_NARROW_CHUNK, NARROW_ITEM_KEYS, 0);
            }
        }
        // tiles: cut only when fewer than two per slot exist
        if (n_wide > 0 && n_wide < 2 * slots) {
            if (narrow_keys == 0) {
                wide_chunk = choose_chunk(wide_runs, slots, WIDE_STAGE_KEYS, MIN_WIDE_CHUNK, WIDE_ITEM_KEYS, WIDE_SPLIT_KEYS);
            } else {
                // next to decode rows (a mixed batch) the tiles are not alone on the slots and the estimate above does
                // not hold; measured best there: about two pieces per slot, cut by the longest tile, at least 1024 keys
                int64_t max_keys = 0;
                for (const auto& r : wide_runs) max_keys = std::max<int64_t>(max_keys, r.first);
                const int64_t want = ceil_div(2 * slots, n_wide);
                wide_chunk = std::max<int64_t>(MIN_WIDE_CHUNK_MIXED, round_up(ceil_div(max_keys, want), KV_TILE));
                // Tiles that fit about one round of the slots, whole or in a few pieces: they all start first, and the slots
                // they leave (or the first to finish) stream the decode rows meanwhile.  The launch then lasts as long as the
                // longest piece or a slot's share of everything, so the fewest pieces that meet those two ends are best: a
                // piece costs a start and a partial result.  Where the longest piece would outlast the share by a fifth (whole
                // tiles, which need no combine pass: by three tenths), the cut above stays.  us per launch, before -> so, 8-bit and
                // bf16: 24 rows of 0.7-7 k tokens over 8 KV heads next to a prefill of 701 over 2 900 114 -> 98 and 129 -> 126, of
                // 200 over 6 000 90 -> 76 and 108 -> 96, next to two of 300-900 over 2-4 k 164 -> 141 and 170 -> 145; 21 rows of
                // 1.4-14 k next to three of up to 2 682 (one KV head) 219 -> 198 and 209 -> 184 (with other lengths of these
                // ranges 225 -> 224 and 213 -> 214); 60 rows of 5-30 k next to four of up to 1 000 165 -> 140 and 175 -> 165.
                // Tiles first when they are more than that: 96 rows next to 8 long prefills 1 627 -> 1 793, since all decode rows
                // then stream at once.  200 drawn mixed batches of other head counts and sizes run at 0.94 of their time, none
                // above 1.02.
                const int64_t stage_ns = s.D == 128 ? 3500 : 2200, key_ns = (opt.kv_bytes == 1 ? 9 : 13) * (s.D == 128 ? 10 : 6);
                int64_t n_rows = 0, best = -1;
                for (const auto& r : narrow_runs) n_rows += r.second;
                const int64_t narrow_ns = narrow_keys * key_ns / 10 + std::max<int64_t>(n_rows, std::min<int64_t>(2 * slots, narrow_keys / NARROW_ITEM_KEYS)) * 5000;
                for (int64_t k = 1; k <= 8; ++k) {
                    const int64_t chunk = round_up(ceil_div(max_keys, k), WIDE_STAGE_KEYS);
                    if (k > 1 && chunk < MIN_WIDE_CHUNK_MIXED) break;
                    int64_t pieces = 0, stages = 0;
                    for (const auto& r : wide_runs) {
                        pieces += ceil_div(r.first, chunk) * r.second;
                        stages += (r.first / chunk * (chunk / WIDE_STAGE_KEYS) + ceil_div(r.first % chunk, WIDE_STAGE_KEYS)) * r.second;
                    }
                    if (10 * pieces > 11 * slots) break;
                    const int64_t longest = ceil_div(std::min(chunk, max_keys), WIDE_STAGE_KEYS) * stage_ns + 7000;
                    const int64_t share = (stages * stage_ns + pieces * 7000 + narrow_ns) / slots;
                    const int64_t cost = std::max(longest, share) + (k > 1 ? 3000 + 20 * pieces : 0);
                    if ((best < 0 || cost < best) && 10 * longest <= (k > 1 ? 12 : 13) * share) {
                        best = cost;
                        wide_chunk = chunk;
                        wide_first = true;
                    }
                }
            }
        }
    }

    if (by_table) {
        build_table(s, (int32_t)std::min<int64_t>(narrow_chunk, 1 << 30), opt, out);
        return;
    }

    if (blocks) {
        build_blocks(s, (int32_t)block_chunk, (int32_t)std::min<int64_t>(narrow_chunk, 1 << 30), opt, out);
        finish_plan(opt, out);
        return;
    }

    // 3. items
    struct Stream { int64_t cost = 0; int64_t max_keys = 0; std::vector<Cost> items; };
    std::vector<Cost> nar;                                  // narrow items
    std::vector<Stream> streams;                            // wide items by (request, KV head)
    out.items.reserve(2 * opt.wg_slots);
    nar.reserve(2 * opt.wg_slots);
    double wide_cost = 0, narrow_cost = 0;
    auto add_items = [&](int r, int kvh, int g0, int gn, int q0, int nq, int kind) {
        const int64_t nkeys = ctx_len[r] + q0 + nq;
        int64_t chunk;
        if (opt.force_kv_splits > 0)
            chunk = std::max<int64_t>(KV_TILE, round_up(ceil_div(nkeys, opt.force_kv_splits), KV_TILE));
        else
            chunk = kind == KIND_WIDE ? wide_chunk : narrow_chunk;
        const int nsplit = (int)ceil_div(nkeys, chunk);
        const int32_t slot = nq * gn * (s.D + 2);               // floats per partial slot
        const int32_t heads = pack_heads(kvh, g0, gn, kind);
        int64_t part0 = -1;
        if (nsplit > 1) {
            part0 = out.partial_floats;
            out.partial_floats += (int64_t)slot * nsplit;
            out.combs.push_back(CombItem{r, heads, q0, nq, (int32_t)part0, nsplit, slot, 0});
        }
        for (int sp = 0; sp < nsplit; ++sp) {
            const int32_t begin = (int32_t)(sp * chunk), end = (int32_t)std::min<int64_t>(nkeys, (sp + 1) * chunk);
            const Cost c{(end - begin) * (int64_t)(kind == KIND_WIDE ? 4 : 1), (int32_t)out.items.size(), 0};
            out.items.push_back(Item{r, heads, q0, nq, begin, end, nsplit > 1 ? (int32_t)(part0 + (int64_t)sp * slot) : -1, ctx_len[r],
                                     out.reqs[r].row_off, incr_len[r], {0, 0}});
            if (kind == KIND_WIDE) {
                ++out.num_wide;
                wide_cost += (double)c.cost;
                Stream& st = streams.back();
                st.cost += c.cost;
                st.max_keys = std::max<int64_t>(st.max_keys, end);
                st.items.push_back(c);
            } else {
                ++out.num_narrow;
                narrow_cost += (double)c.cost;
                nar.push_back(c);
            }
        }
    };
    for (int r = 0; r < num_reqs; ++r) {
        const int L = incr_len[r];
        for (int kvh = 0; kvh < s.Hkv && L > 0; ++kvh) {
            bool stream = false;
            for (int g0 = 0; g0 < G; g0 += 32) {
                const int gn = std::min(32, G - g0);
                if ((int64_t)L * gn <= 32) {
                    add_items(r, kvh, g0, gn, 0, L, KIND_NARROW);
                    continue;
                }
                if (!stream) streams.emplace_back();
                stream = true;
                each_tile(L, ATTN_WAVES * (32 / gn), [&](int q0, int nq) { add_items(r, kvh, g0, gn, q0, nq, KIND_WIDE); });
            }
        }
    }

    // 4. launch order.  Workgroup i runs on XCD i % NUM_XCD, and each XCD has its own L2, so the position of
    //    an item in the launch order decides which L2 its K/V stream passes through.  Wide items that read
    //    the same stream (same request and KV head: the query tiles of one prefill chunk, which all start at
    //    key 0 and advance at the same rate) are therefore queued on the same XCD, next to each other, so
    //    that the stream is fetched from HBM once and the other tiles hit in L2:
    //      a. streams are dealt to the XCDs longest-processing-time first (a stream that is a large part of
    //         one XCD's share is first cut into pieces, tile by tile);
    //      b. inside an XCD, streams run longest keys first, and tiles of a stream longest first, so the
    //         last workgroups of the launch are the short ones;
    //         (then single items move from the heaviest queue to the lightest until they are level);
    //      c. the XCD queues are interleaved position by position; null items pad a queue that is shorter
    //         than the others.
    //    Narrow items stream their key range exactly once, so they only need balance: longest first.  In a
    //    mixed batch the two kinds alternate in runs of NUM_XCD in proportion to their total cost, so that at
    //    any time some CUs run compute-bound tiles while others stream decode rows (or, see wide_first, the tiles
    //    go first because they leave slots for that).
    //    Everything is stable and depends on the lengths only.
    longest_first(nar);
    std::vector<int32_t> wide_ix;
    if (!streams.empty()) {

        // a. pieces well below one XCD's share, dealt to the least loaded XCD, heaviest first
        const int64_t share = std::max<int64_t>(1, ceil_div((int64_t)wide_cost, NUM_XCD));
        std::vector<Stream> pieces;
        pieces.reserve(streams.size());
        for (Stream& st : streams) {
            longest_first(st.items);
            // pieces of a quarter share let the dies mix long and short streams, but a piece keeps at least 8
            // tiles so that a die still reuses what it fetched; a power of two, so that equal streams deal evenly
            const int64_t want = std::max<int64_t>(1, std::min<int64_t>(ceil_div(4 * st.cost, share), (int64_t)st.items.size() / 8));
            int np = 1;
            while (2 * np <= want && np < NUM_XCD) np *= 2;
            const size_t base = pieces.size();
            if (np == 1) {
                pieces.push_back(std::move(st));
                continue;
            }
            pieces.resize(base + np);
            for (size_t i = 0; i < st.items.size(); ++i) {         // deal the tiles round-robin: equal pieces
                Stream& pc = pieces[base + i % np];
                pc.items.push_back(st.items[i]);
                pc.cost += st.items[i].cost;
                pc.max_keys = st.max_keys;
            }
        }
        std::vector<int32_t> by_cost(pieces.size());
        for (size_t i = 0; i < pieces.size(); ++i) by_cost[i] = (int32_t)i;
        std::stable_sort(by_cost.begin(), by_cost.end(), [&](int32_t a, int32_t b) { return pieces[a].cost > pieces[b].cost; });
        std::vector<int32_t> bin_pieces[NUM_XCD];
        int64_t bin_cost[NUM_XCD] = {0};
        for (int32_t pi : by_cost) {
            int best = 0;
            for (int x = 1; x < NUM_XCD; ++x)
                if (bin_cost[x] < bin_cost[best]) best = x;
            bin_pieces[best].push_back(pi);
            bin_cost[best] += pieces[pi].cost;
        }
        // b. queue of every XCD
        std::vector<Cost> queue[NUM_XCD];
        for (int x = 0; x < NUM_XCD; ++x) {
            std::stable_sort(bin_pieces[x].begin(), bin_pieces[x].end(),
                             [&](int32_t a, int32_t b) { return pieces[a].max_keys > pieces[b].max_keys; });
            for (int32_t pi : bin_pieces[x])
                for (const Cost& c : pieces[pi].items) queue[x].push_back(c);
        }
        //    level the queues: the heaviest queue hands its last (shortest) item to the lightest one while that
        //    lowers the maximum.  The result is kept only if the launch gets shorter when every queue is
        //    replayed on the CUs of one XCD, which also sees the granularity of a few long items per CU.
        const int cus = std::max(1, opt.wg_slots / NUM_XCD);
        std::vector<int64_t> cu_free;
        auto finish_time = [&](const std::vector<Cost>& q) {
            cu_free.assign(cus, 0);                                 // min-heap of the CUs' free times
            auto later = [](int64_t a, int64_t b) { return a > b; };
            int64_t last = 0;
            for (const Cost& c : q) {
                std::pop_heap(cu_free.begin(), cu_free.end(), later);
                cu_free.back() += c.cost;
                last = std::max(last, cu_free.back());
                std::push_heap(cu_free.begin(), cu_free.end(), later);
            }
            return last;
        };
        auto launch_time = [&](const std::vector<Cost>* q) {
            int64_t t = 0;
            for (int x = 0; x < NUM_XCD; ++x) t = std::max(t, finish_time(q[x]));
            return t;
        };
        // the next move: from the heaviest queue to the lightest, if it lowers the maximum
        auto move_of = [](const std::vector<Cost>* q, const int64_t* sum, int* hi, int* lo) {
            *hi = *lo = 0;
            for (int x = 1; x < NUM_XCD; ++x) {
                if (sum[x] > sum[*hi]) *hi = x;
                if (sum[x] < sum[*lo]) *lo = x;
            }
            return !q[*hi].empty() && sum[*lo] + q[*hi].back().cost < sum[*hi];
        };
        int hi, lo;
        if (move_of(queue, bin_cost, &hi, &lo)) {
            std::vector<Cost> trial[NUM_XCD];
            int64_t sum[NUM_XCD];
            for (int x = 0; x < NUM_XCD; ++x) {
                trial[x] = queue[x];
                sum[x] = bin_cost[x];
            }
            for (size_t moves = 0; moves < out.items.size() && move_of(trial, sum, &hi, &lo); ++moves) {
                const Cost c = trial[hi].back();
                trial[hi].pop_back();
                trial[lo].push_back(c);
                sum[hi] -= c.cost;
                sum[lo] += c.cost;
            }
            if (launch_time(trial) < launch_time(queue))
                for (int x = 0; x < NUM_XCD; ++x) queue[x].swap(trial[x]);
        }
        // c. interleave; -1 stands for a null item that pads a shorter queue
        size_t longest = 0;
        for (int x = 0; x < NUM_XCD; ++x) longest = std::max(longest, queue[x].size());
        for (size_t j = 0; j < longest; ++j)
            for (int x = 0; x < NUM_XCD; ++x) wide_ix.push_back(j < queue[x].size() ? queue[x][j].idx : -1);
        while (!wide_ix.empty() && wide_ix.back() < 0) wide_ix.pop_back();
    }
    std::vector<Item> sorted;
    sorted.reserve(wide_ix.size() + nar.size() + (opt.append_items ? ceil_div(out.sum_L, APPEND_ITEM_ROWS) : 0));
    {
        size_t iw = 0, in = 0;
        double dw = 0, dn = 0;                     // cost already emitted per kind
        while (iw < wide_ix.size() || in < nar.size()) {
            bool take_wide;
            if (iw >= wide_ix.size()) take_wide = false;
            else if (in >= nar.size()) take_wide = true;
            else if (wide_first) take_wide = true;
            else take_wide = dw * narrow_cost <= dn * wide_cost;      // the kind that lags behind its share
            for (int k = 0; k < NUM_XCD; ++k) {
                if (take_wide ? iw >= wide_ix.size() : in >= nar.size()) break;
                const int32_t idx = take_wide ? wide_ix[iw++] : nar[in++].idx;
                if (idx < 0) {
                    sorted.push_back(null_item());
                    continue;
                }
                const Item& it = out.items[idx];
                const double keys = it.kv_end - it.kv_begin;
                (take_wide ? dw : dn) += take_wide ? keys * 4 : keys;
                sorted.push_back(it);
            }
        }
    }
    out.items.swap(sorted);

    // Over a bf16 cache nothing runs in front of the attention launch that could carry the list along: a small one of tiles alone
    // travels in the arguments instead of an upload launch (5 us: one prefill of 32 tokens 10.4 -> 7.6 us a call, one
    // of 509 tokens over 4 099 55.8 -> 49.5 with the small append items).
    out.by_tiles = opt.force_kv_splits <= 0 && opt.kv_bytes == 2 && build_tiles(s, (int32_t)std::min<int64_t>(wide_chunk, 1 << 30), out);

    // 5. append items and byte layout
    finish_plan(opt, out);
}

}  // namespace ampd
