// What the two prefill kernels (prefill.hip, prefill_short.hip) share: their arguments.
#pragma once
#include "esp_common.h"

namespace esp {

struct PrefillArgs {
    const uint16_t* q; const uint16_t* k; const uint16_t* v;
    const int32_t* q_pos; const int32_t* kv_pos; const int32_t* cu_q; const int32_t* cu_kv;
    const int32_t* retain_slot;       // [Tkv] pool slot of every shard row (negative: not kept), or null: nothing is kept
    const int32_t* kv_slot;           // [Tkv] pool slot of every shard row when k and v ARE the token pools; null: dense shard
    uint16_t* k_pool; uint16_t* v_pool;
    void* O; float* LSE;              // O: bf16 [Tq, Hq, 128], or fp32 of the same shape when o_f32 is set
    int32_t batch, Tq, Tkv, Hq, Hkv, causal, o_f32;
    // Packed rows: the rows of a KV head are the (token, query head of the group) pairs in memory order, row rho of a
    // request being token rho / G, query head kvh * G + rho % G, and a query tile is 256 of them.  A group's heads
    // see the same keys, so nothing else changes; but a tile spans 256 / G tokens instead of 256: less of it is masked at
    // the diagonal, a short chunk fills a tile G times better, and its Q and O rows are contiguous runs of G.
    // Measured (one tile per query head -> packed, 32 / 8 heads): six prompts of 37 .. 2047 tokens 79.7 -> 69.1 us, a
    // batch of 1000 .. 8192 tokens against two shards, rows kept, 1.470 -> 1.415 ms, 300 tokens against 20300
    // 379.6 -> 368.3 us.
    int32_t G;                        // query heads per KV head
    float inv_G;
    // Split KV: every request's KV tiles in `splits` parts, an item each ("KV head" h * splits + part in the deal of the
    // items); part p's O and LSE lie p * o_part and p * lse_part bytes behind the first part's
    int32_t splits;
    int64_t o_part, lse_part;
    int32_t q_tiles, heads_per_xcd;   // upper bound of the number of query tiles of a KV head; (KV head, part) pairs per XCD (0: no split)
    unsigned long long* pool;         // counter of the item pool: launch tag (high word), draws so far (low word)
    uint32_t tag;                     // this launch's tag
    int32_t by_head;                  // items of an XCD in order of KV head (and part), not of query tile
    int32_t group_sync;               // the workgroups of an XCD start their dealt rounds together
    int32_t sync_ticks;               // longest such wait, in ticks of the 100 MHz wall clock
    float scale_log2;
    int32_t q_odd;                    // q does not lie on 16 bytes
};

// The kernel for calls with few query rows (prefill_short.hip): a.splits parts; the other fields as for the main kernel.
constexpr int kShortRows = 32;        // packed rows of a workgroup
constexpr int kShortWaves = 8;        // wavefronts, each on tiles of 32 keys of its own
esp_status launch_prefill_short(const PrefillArgs& a, hipStream_t stream);

}  // namespace esp
