// Kernel parameter blocks and launcher declarations shared by kernels.hip and api.cpp.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plan.h"

namespace ampd {

enum : int { KV_BF16 = 0, KV_FP8 = 1 };

struct AttnParams {
    const void* q;             // bf16 [sum L][Hq][D]
    void* out;                 // bf16 [sum L][Hq][D]
    const void* k_new;         // bf16 [sum L][Hkv][D]: the new tokens of this call when their page writes ride in the
    const void* v_new;         //   attention launch (bf16 cache: keys >= C are then read from here), else null
    const void* k_pool;        // [pages][Hkv][P][D]
    const void* v_pool;
    const float* k_scale;      // [pages][Hkv] (8-bit cache) or null
    const float* v_scale;
    const int32_t* block_table;
    const ReqInfo* reqs;
    const Item* items;
    const CombItem* combs;
    float* partial;
    int32_t Hq, Hkv, P, logP, max_pages;
    float c_log2;              // softmax_scale * log2(e)
    // The host's pinned staging slot this call's work list came from may be reused once this launch runs (every copy
    // out of the slot precedes it in stream order): the first workgroup stores slot_seq to *slot_flag (pinned host memory).
    uint32_t* slot_flag;
    uint32_t slot_seq;
    // Persistent launch (more items than workgroups): per-die queue heads in the workspace, see Plan::queue_heads.
    int32_t* queue_heads;
    int32_t nitems;
};

struct alignas(16) AppendRow {
    int32_t C, L;
    int32_t row_off;           // first packed row
    int32_t pg_off;            // pages of the rows before it that new tokens fall into
};
struct AppendParams {
    const void* k_new;         // bf16 [sum L][Hkv][D]
    const void* v_new;
    void* k_pool;
    void* v_pool;
    float* k_scale;
    float* v_scale;
    const int32_t* block_table;
    int32_t Hkv, D, P, logP, max_pages, req0;
    int32_t h0, hn;            // KV heads [h0, h0 + hn) of the pool; the packed rows hold hn heads
    // Optional rider: the work list of the attention launch that follows, copied from pinned host memory into the workspace by
    // the first up_blocks workgroups of this launch (up_n16 16-byte vectors; 0: none).
    const void* up_src;
    void* up_dst;
    int32_t up_n16, up_blocks;
    // One workgroup column per page that new tokens fall into: pages [pg0, pg0 + gridDim.x - up_blocks) of the n rows' pages
    // laid end to end.
    int32_t n, pg0;
    AppendRow rows[APPEND_MAX_REQS];
};

// h_src: pinned, device-visible host memory; bytes is rounded up to 16
hipError_t launch_upload(const void* h_src, void* d_dst, size_t bytes, hipStream_t st);
// tiles: the list holds some (otherwise grid is the number of items)
hipError_t launch_attn(const AttnParams& p, int D, int kvt, bool tiles, int grid, hipStream_t st);
// a batch of decode rows alone, whose list travels in the arguments; p.k_new: the call appends (both kinds of cache)
hipError_t launch_rows(const AttnParams& p, const RowTable& t, int kvt, int grid, hipStream_t st);
// a small launch of tiles alone over a bf16 cache, likewise
hipError_t launch_tiles(const AttnParams& p, const TileTable& t, int grid, hipStream_t st);
// max_rows: the largest nq * heads among the split tiles (sizes the second grid dimension)
// t, tt: the launch went by this table (at most one of them), or null
hipError_t launch_combine(const AttnParams& p, const RowTable* t, const TileTable* tt, int D, int ncombs, int max_rows, int max_splits,
                          hipStream_t st);
// pages: pages of the p.n rows that new tokens fall into; the launchers fill pg0 and up_blocks in p.  0: nothing is launched
hipError_t launch_append(AppendParams& p, int kvt, int64_t pages, hipStream_t st);
// bf16 only: pack = pages -> packed rows (k_new / v_new are written), otherwise packed rows -> pages
hipError_t launch_kv_move(AppendParams& p, bool pack, int64_t pages, hipStream_t st);

}  // namespace ampd
