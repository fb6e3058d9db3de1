// Host-side work planner: cuts a batch of (C_r, L_r) rows into GPU work items.
//
// A prefill task is described to the scheduler by its history length and incremental
// length only (paper Section 3, T_pre(l_hist, l_incr)); a decode step by one token per
// request (T_dec).  From these lengths alone the planner derives, per request and KV head:
//   * wide items   -- tiles of up to 256 query rows (tokens x grouped heads) whose 8 waves
//                     share K/V tiles staged in LDS (compute-bound prefill work), and
//   * narrow items -- blocks of at most 32 query rows (decode rows, very short chunks, and all rows of a small launch)
//                     whose 8 waves split the key range (bandwidth-bound work),
//   * append items -- (bf16 cache, append-then-attend calls) runs of packed new rows to be copied into
//                     their pages by the same launch; they close the work list, where they fill the CUs
//                     that run out of attention work first,
// optionally cutting an item's key range into pieces (split-KV) that a combine pass merges.
// Workgroup i of a launch runs on accelerator die (XCD) i % 8, each with its own L2, so the
// launch order also decides which L2 a K/V stream passes through; null items (no work) pad the
// per-die queues to equal length.
// Everything is computed from logical positions, never from physical page ids, so results
// are bitwise independent of where pages live in the pool.
#pragma once
#include <cstdint>
#include <vector>

namespace ampd {

enum : int32_t { KIND_WIDE = 0, KIND_NARROW = 1, KIND_NULL = 2, KIND_APPEND = 3 };

constexpr int ATTN_WAVES = 8;      // waves of an attention workgroup (one workgroup per CU)
constexpr int NUM_QUEUES = 8;      // accelerator dies (XCDs): workgroup i of a launch is dispatched to die i % 8
constexpr int APPEND_MAX_REQS = 128;   // requests per append launch (their lengths travel as kernel arguments)

struct ReqInfo {          // 16 B, one per request, device-visible
    int32_t C, L, row_off, req;
};

struct Item {             // 48 B, one per attention workgroup, device-visible
    int32_t req;          // -1 for a null item
    int32_t heads;        // kvh | g0 << 8 | gn << 16 | kind << 24
    int32_t q0, nq;       // first new-token index and token count of this item
    int32_t kv_begin, kv_end;   // key range [begin, end) in logical positions
    int32_t part_off;     // float offset of this item's partial slot, or -1: write final output
    int32_t C;            // context length of the request and the first row of its packed q / out rows:
    int32_t row_off;      // copies of its ReqInfo, so that a workgroup starts with one dependent load less
    int32_t row_L;        // and the request's new tokens
    int32_t pad[2];
};
static_assert(sizeof(Item) == 48, "device layout");

struct CombItem {         // 32 B, one per query tile whose key range was split
    int32_t req;
    int32_t heads;
    int32_t q0, nq;
    int32_t part_off;     // float offset of split 0
    int32_t nsplit;
    int32_t part_stride;  // floats between consecutive splits
    int32_t pad;
};

#if defined(__HIP__)
#define AMPD_HD __attribute__((host)) __attribute__((device)) inline __attribute__((always_inline))
#else
#define AMPD_HD inline
#endif

AMPD_HD int32_t pack_heads(int kvh, int g0, int gn, int kind) {
    return kvh | (g0 << 8) | (gn << 16) | (kind << 24);
}

struct Shape {
    int Hq, Hkv, D, P;
};

// The work list of a launch of decode rows alone, small enough to travel in the kernel's arguments: no list in the
// workspace, no staging buffer and no upload in front of the launch.  One entry per row with new tokens; a row's key range
// is cut into pieces of `chunk` keys and a remainder.  Items in launch order: the whole pieces of all rows, then the
// remainders, longest first (rows are sorted by their remainder), each row's items by piece and KV head.
constexpr int ROW_TABLE_MAX = 128;
struct RowEntry {         // 20 B
    int32_t C, row_off;
    int32_t req_L;        // req | L << 24 (L <= 32)
    int32_t first;        // item index of the row's first whole piece (= whole pieces of the rows before it)
    int32_t part_off;     // float offset of the row's first partial slot, or -1: the key range is not cut
};
struct RowTable {
    int32_t n, chunk;     // entries; keys per piece
    int32_t n_whole, n_items;   // items that are whole pieces; all attention items (append items follow them)
    int32_t sum_L, Hkv, G, D;
    int32_t max_rows;     // query rows of the tallest item
    int32_t small;        // workgroups of 4 waves, several to a CU, where the kernel has them (see build_table)
    RowEntry e[ROW_TABLE_MAX];
};

// Item idx (< n_items) of the table; row: its entry (see row_of_item).
AMPD_HD Item table_item(const RowTable& t, const RowEntry& e, int idx) {
    const int L = e.req_L >> 24, keys = e.C + L, whole = keys / t.chunk;
    const int pieces = whole + (whole * t.chunk < keys ? 1 : 0);
    int piece, kvh;
    if (idx < t.n_whole) {
        piece = (idx - e.first) / t.Hkv;
        kvh = idx - e.first - piece * t.Hkv;
    } else {
        piece = whole;
        kvh = (idx - t.n_whole) % t.Hkv;
    }
    Item it;
    it.req = e.req_L & 0xffffff;
    it.heads = pack_heads(kvh, 0, t.G, KIND_NARROW);
    it.q0 = 0;
    it.nq = L;
    it.kv_begin = piece * t.chunk;
    it.kv_end = it.kv_begin + t.chunk < keys ? it.kv_begin + t.chunk : keys;
    it.part_off = e.part_off < 0 ? -1 : e.part_off + (kvh * pieces + piece) * (L * t.G * (t.D + 2));
    it.C = e.C;
    it.row_off = e.row_off;
    it.row_L = L;
    it.pad[0] = it.pad[1] = 0;
    return it;
}
// The combine work of row e, KV head kvh (nsplit = 1: none).
AMPD_HD CombItem table_comb(const RowTable& t, const RowEntry& e, int kvh) {
    const int L = e.req_L >> 24, keys = e.C + L, pieces = (keys + t.chunk - 1) / t.chunk;
    const int slot = L * t.G * (t.D + 2);
    return CombItem{e.req_L & 0xffffff, pack_heads(kvh, 0, t.G, KIND_NARROW), 0, L, e.part_off + kvh * pieces * slot, pieces, slot, 0};
}

// The work list of a small launch of tiles alone, or of blocks of at most 32 query rows alone, in the kernel's arguments for the
// same reason: one word per item and 8 bytes per cut tile (or block: "tile" below is either).
constexpr int TILE_TABLE_ROWS = 16, TILE_TABLE_ITEMS = 256, TILE_TABLE_COMBS = 128;
constexpr uint32_t TILE_NULL = 0xffffffffu;
struct TileComb {
    uint32_t code;            // as an item's, piece 0
    int32_t part_off;         // float offset of split 0
};
struct TileTable {
    int32_t n_rows, n_items, n_combs;
    int32_t chunk, tq;        // keys per piece; tokens of a full tile (a row's first tile takes the remainder)
    int32_t G, D, sum_L;
    int32_t append_rows;      // packed rows per append item
    int32_t kind;             // KIND_WIDE, or KIND_NARROW: blocks of at most 32 query rows
    int32_t few_chunk;        // ... then: keys per piece of a row that is one block (a decode row)
    ReqInfo rows[TILE_TABLE_ROWS];          // rows with new tokens
    uint32_t items[TILE_TABLE_ITEMS];       // row | kvh << 4 | tile << 10 | piece << 18 | cut tile << 25, or TILE_NULL
    TileComb combs[TILE_TABLE_COMBS];
};

AMPD_HD int32_t tile_chunk(const TileTable& t, int32_t L) { return t.kind == KIND_NARROW && L <= t.tq ? t.few_chunk : t.chunk; }

// Tile and piece of a code.
AMPD_HD Item tile_item(const TileTable& t, uint32_t code) {
    const ReqInfo& r = t.rows[code & 15];
    const int kvh = (code >> 4) & 63, tile = (code >> 10) & 255, piece = (code >> 18) & 127;
    const int rest = r.L % t.tq, first = rest ? rest : t.tq;
    Item it;
    it.req = r.req;
    it.heads = pack_heads(kvh, 0, t.G, t.kind);
    it.q0 = tile ? first + (tile - 1) * t.tq : 0;
    it.nq = tile ? t.tq : first;
    const int keys = r.C + it.q0 + it.nq, chunk = tile_chunk(t, r.L);
    it.kv_begin = piece * chunk;
    it.kv_end = keys - it.kv_begin > chunk ? it.kv_begin + chunk : keys;
    it.part_off = keys > chunk ? t.combs[code >> 25].part_off + piece * (it.nq * t.G * (t.D + 2)) : -1;
    it.C = r.C;
    it.row_off = r.row_off;
    it.row_L = r.L;
    it.pad[0] = it.pad[1] = 0;
    return it;
}
AMPD_HD CombItem tile_comb(const TileTable& t, int i) {
    const Item it = tile_item(t, t.combs[i].code);
    const int keys = it.C + it.q0 + it.nq, chunk = tile_chunk(t, t.rows[t.combs[i].code & 15].L);
    return CombItem{it.req, it.heads, it.q0, it.nq, t.combs[i].part_off, (keys + chunk - 1) / chunk, it.nq * t.G * (t.D + 2), 0};
}

// Whether the page slots up to position C (a row's one new token) all lie in the 32-key block of a narrow item that holds the
// token.  Blocks start at multiples of 32 and pages at multiples of P, so only the upper half of a 64-slot page shares its page
// with the block before it.
AMPD_HD bool page_in_last_block(int C, int P) { return ((C & (P - 1)) & 32) == 0; }

constexpr int APPEND_ITEM_ROWS = 64;   // packed rows (new tokens, all heads, K and V) that one append item moves

struct PlanOptions {
    int force_kv_splits = 0;
    int wg_slots = 256;   // workgroups resident at once: one per CU
    int kv_bytes = 2;     // bytes of a cached element
    bool append_items = false;   // the page writes of the call ride in the attention launch (bf16 cache): append items
                                 // of APPEND_ITEM_ROWS packed rows each (TileTable::append_rows in a launch by that table)
                                 // close the work list
};

struct Plan {
    std::vector<ReqInfo> reqs;
    std::vector<Item> items;
    std::vector<CombItem> combs;
    // A launch of decode rows alone (at most ROW_TABLE_MAX of them): the table stands for items and combs, which stay empty
    // (plan_items() writes the items out for a caller that wants to see them).
    bool by_table = false;
    RowTable table;
    // A small launch of tiles or blocks alone over a bf16 cache: `tiles` stands for items, which stay empty, and says the same as combs.
    bool by_tiles = false;
    TileTable tiles;
    int64_t num_items = 0, num_combs = 0;
    int64_t num_wide = 0, num_narrow = 0, num_append = 0;
    int64_t partial_floats = 0;
    int64_t sum_L = 0;
    // A launch with tiles in it and more items than workgroup slots runs `grid` persistent workgroups (otherwise grid = the
    // number of items, one workgroup each): workgroup i starts with item i
    // and then takes items from the queue of its die (queue q = items q, q + NUM_QUEUES, ...; queue_heads[q] = the
    // queue's position of the first item nobody has started), helping out on other queues when its own is empty.
    int32_t grid = 0;
    int32_t queue_heads[NUM_QUEUES] = {0, 0, 0, 0, 0, 0, 0, 0};
    // byte layout of the device copy: [reqs][items][combs][queue heads], each 256 B aligned
    int64_t off_reqs = 0, off_items = 0, off_combs = 0, off_queues = 0, plan_bytes = 0;
    int64_t off_partial = 0, total_bytes = 0;
};

// The items of a plan in launch order (a table's written out).
void plan_items(const Plan& plan, std::vector<Item>& out);

// ctx_len / incr_len must already be validated (non-negative, no overflow).
void build_plan(const Shape& s, int num_reqs, const int32_t* ctx_len, const int32_t* incr_len,
                const PlanOptions& opt, Plan& out);

}  // namespace ampd
