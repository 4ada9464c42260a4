// esp_partial_attn_prefill: a causal query chunk against ONE local key-value shard, masked by
// global token position (sequence-parallel prefill, Sec. 2.3 / Fig. 1: instance i attends its
// local q_i to the segment kv_j of the current round; striped layout and tile-skipping remarks
// in Sec. 6).  Emits the un-merged output, normalised within the shard, and its log-sum-exp.
//
// Mapping to gfx950 (64-wide wavefronts, MFMA 32x32x16 bf16, 160 KiB LDS):
//   * one persistent workgroup of 8 wavefronts per CU works through items; an item is 256 query
//     rows of one KV head: each wavefront owns 32 rows and keeps their Q fragment (B operand), the
//     softmax state and the fp32 output accumulator in registers for the whole KV sweep.  The rows
//     of a KV head are its (token, query head) pairs in memory order, so with G query heads per
//     KV head a tile covers 256 / G tokens (see "packed rows" at PrefillArgs).  Most
//     items are dealt to the workgroups beforehand, the light ones at the end are drawn from a
//     device-wide counter as workgroups become free (see the item loop at the end of the kernel);
//   * K/V tiles of 64 rows are fetched straight from global memory into a 4-stage LDS ring
//     (global_load ... lds, no register staging), K four tiles and V two tiles ahead of their use;
//   * the K tile is the A operand of S^T = K Q^T, so a lane ends up with scores of ONE query
//     row (its column); P^T stays in registers and is the B operand of O^T = V^T P^T, whose A
//     operand comes from transposing LDS reads of the row-major V tile;
//   * the 16-byte chunks of K and V rows are XOR-swizzled in LDS, so that the operand reads spread over all banks;
//   * one uniform instruction stream per wavefront, software pipelined at the level of single
//     MFMAs: every step issues one MFMA of S^T for tile j+1, the exp2 of two scores of tile j,
//     one MFMA of O^T += V^T P^T that trails the probabilities by one chunk of 16 keys, and the
//     sum / bf16 pack of the two probabilities.  A wavefront issues an instruction only every
//     6-8 cycles and a 32x32x16 MFMA lasts 32, so with the two wavefronts of a SIMD running the
//     same mix the matrix pipe always has an MFMA of one of them to run;
//   * the softmax offset is optimistic: probabilities are taken against the offset in use
//     without looking at the scores first; one compare per tile on the probability sum tells
//     whether the offset has to move (exact rescale by a power of two), and a workgroup whose
//     scores leave the range this can handle redoes its rows with a plain, exact sweep;
//   * the minimum / maximum position of every KV tile (found by the workgroup itself while its
//     first tiles are in flight) decide: tiles past the last one any row can see are never
//     processed; tiles below every row of a wavefront run the branch-free "plain" iteration;
//     the others apply the element-wise test kv_pos <= q_pos; past the last tile any of its own
//     rows can see a wavefront stops its arithmetic and only keeps up transfers and barriers.
#include <limits.h>
#include <math.h>
#include <stdlib.h>

#include <atomic>
#include <chrono>
#include <random>

#include "mfma_tile.h"
#include "prefill.h"

namespace esp {

constexpr int kBM = 256;   // query rows per workgroup
constexpr int kBN = 64;    // KV rows per tile
constexpr int kPfWaves = 8;
constexpr long long kSyncTicks = 15000;   // longest wait at a round start, in ticks of the 100 MHz wall clock (150 us)
constexpr int kTileBytes = kBN * kHeadDim * 2;   // 16 KiB: a V tile in LDS, rows of 256 bytes
constexpr int kORow = 272;                       // LDS row pitch of the results on their way out: 256 bytes + 16 of padding
constexpr int kKTileBytes = kBN * kORow;         // a stage of K: its tile, and room for the results (see the epilogue)

// Where K lies in a stage.  LDS has 64 banks, 256 bytes in a row, and reads 16 lanes of 16 bytes at a time, here one chunk of 16 rows: the chunks
// of a row are swizzled by the row modulo 8, which spreads eight rows over half of the banks, and every second eight rows lie half a row
// on.  (A swizzle by the row modulo 16 would do the same, with eight address registers for four.)  With all rows 256 bytes apart 34.5 of
// the 105 million cycles that the LDS of all CUs was busy in a call of 8192 on 8192 rows, 32 / 32 heads, were conflicts, now 0.1 of 71.  The loop does
// not wait for them: six prompts of 37 .. 2047 tokens, 32 / 8 heads, 59.6 -> 59.3 us, other calls within 0.2 %.
constexpr int kKGroup = 8 * 256 + 128;
__host__ __device__ constexpr int k_row(int r) { return r * 256 + (r >> 3) * 128; }
__host__ __device__ constexpr int k_chunk(int r, int c) { return k_row(r) + ((c ^ (r & 7)) << 4); }
constexpr bool k_reads_spread() {
    for (int c = 0; c < 16; ++c)
        for (int first = 0; first < kBN; first += 16) {
            unsigned seen = 0;
            for (int r = first; r < first + 16; ++r) seen |= 1u << (k_chunk(r, c) / 16 % 16);
            if (seen != 0xffff) return false;
        }
    return k_row(8) == kKGroup && k_row(kBN) <= kKTileBytes;
}
static_assert(k_reads_spread(), "an operand read of K must touch every bank once");


// upper bound of the query tiles of one KV head: Tq * G packed rows, and one ragged tile per request
static int32_t prefill_q_tiles_bound(int32_t Tq, int32_t G, int32_t batch) {
    const int64_t rows = (int64_t)Tq * G;
    return (int32_t)(batch == 1 ? (rows + kBM - 1) / kBM : rows / kBM + batch);
}

// Global scratch memory of the prefill path: one 64-bit item counter (the first word of the block, the second is
// spare) and the arrival counts of the start-of-round waits (one per XCD).
// Every launch
// gets a tag of its own, so that a counter left by an earlier launch, or never written, is told from the current
// one without clearing it first (a clearing kernel ahead of each launch costs about 6 us).  Tags start at a random
// 32-bit value per process: stale memory passes for the current launch's counter with probability 2^-32.
static uint32_t next_launch_tag() {
    static std::atomic<uint32_t> tag{[] {
        uint32_t seed = (uint32_t)std::chrono::steady_clock::now().time_since_epoch().count();
        try { seed ^= std::random_device{}(); } catch (...) {}
        return seed;
    }()};
    const uint32_t t = tag.fetch_add(1, std::memory_order_relaxed) + 1;
    return t ? t : tag.fetch_add(1, std::memory_order_relaxed) + 1;   // never 0: cleared counters carry tag 0
}
// Longest start-of-round wait.  The default comes from ESP_PREFILL_SYNC_TICKS in the environment, read once when the
// library is loaded; esp_debug_set_prefill_sync_ticks replaces it (0: every wait gives up at once, the path a
// missing workgroup would cause).
static std::atomic<int32_t> g_sync_ticks{[] {
    if (const char* e = getenv("ESP_PREFILL_SYNC_TICKS")) {
        const long v = strtol(e, nullptr, 10);
        if (v >= 0 && v <= 1000000) return (int32_t)v;
    }
    return (int32_t)kSyncTicks;
}()};
int32_t set_prefill_sync_ticks(int32_t ticks) {
    return g_sync_ticks.exchange(ticks < 0 ? (int32_t)kSyncTicks : ticks > 1000000 ? 1000000 : ticks, std::memory_order_relaxed);
}

// Which kernel a call runs on, and in how many parts its key-value rows are cut.  A query tile of the main kernel is one item, and
// few of them (a follow-up turn of a few hundred tokens, a shard with few heads) leave most of the 256 CUs idle, or busy for one
// round and a fraction.  Then every request's KV tiles are cut into S equal parts, each an item of its own with its partial result
// in fp32 in the workspace, and the merge kernel combines them.  Few rows, or few keys, are better off on the kernel of
// prefill_short.hip, cut or not.  The choice is the least of these estimates of the call's time, in us, fitted to 57 shapes of
// 1 .. 3000 tokens on 27 .. 262000 rows, 4 / 4 .. 64 / 8 heads, each with up to sixteen choices; the one taken was within 6 % of
// the best of them in all but a few (10 %, 32 / 8 heads, 130 tokens on 3130 rows).
// Main kernel: an item costs a set-up and an epilogue (8.5) beside its tiles (1.45 each; 0.8 where only one wavefront has rows,
// as the others then only move tiles), the merge a launch (4) and its traffic.  Items of a chunk at the end of a long context are
// alike, so rounds count whole; where the chunk is most of the shard the sweeps are a triangle, which the item pool evens out.
// In a triangle a tile costs less, but for an owner of kept rows (1.05: a wavefront past its last one leaves the matrix pipe to the
// other), and where the items are one round and uncut, halves of query tiles are paired (PAIRED at the kernel): 12 beside
// 0.5 .. 0.9 a tile of the longest sweep, the more the more CUs are at it.
// Short kernel: 4.5 beside its steps of 8 x 32 keys (1.85 each, 1.3 in a triangle, while K and V come from the caches, 2.5 once they are
// more than the 256 MB that the last of those holds; on average 0.75 of the last row block's in a triangle), but no faster than its
// row blocks can be fed from the L2 (12.5 TB/s).  Several row blocks of a head share its K and V only on one XCD, i.e. where heads times
// parts is a multiple of 8 (51 tokens on 29013 rows, 12 / 12 heads: 54 us in 8 parts, 47 in 10, 63 in 9).
// Measured (main kernel, best cut -> this, best cut): 27 tokens on 27, 32 / 8 heads, 9.3 -> 5.8 us, 256 on 512, 4 / 4, 17.2 -> 8.1,
// 1024 on 1024, 8 / 8, 23.2 -> 11.9, 16 on 2016, 32 / 8, 19.5 -> 12.1, 100 on 3100, 8 / 8, 21.4 -> 13.5, 31 on 70195, 4 / 4, 67.3
// -> 58.1; where it ends: 512 on 512, 32 / 8, 16.9 -> 14.4, 200 on 5200, 16 / 16, 29.8 -> 25.0, and 600 on 1200, 32 / 8, stays at
// 29.4 (the short kernel 31.9), eight prompts of 64, 32 / 8, at 11.1 (12.5).
// Triangle or not: a chunk that is a good part of its shard (two fifths) may be the shard's own tokens, or a stripe of them, and see a
// triangle of it; or lie behind it (every shard but the last of a contiguous sequence), or have no mask, and see all, where
// nothing is paired away and items are as long as each other.  Without a mask the estimate is the latter's.  With one the sizes do not
// say; the plan is the one that is least far from the best in the worse of the two, which costs the triangle up to a tenth (7370 on 7370,
// 4 / 4 heads: 83 us in two parts, 75 in three; behind the shard 109 and 139).  Where rows are kept it is the triangle's: over 32 such
// shapes that is 0.2 % from the best in a triangle and 2.6 % behind the shard, the other 2.3 % and 1.1 %.
// Over 136 shapes of 126 .. 10000 tokens on 205 .. 10000 rows, 4 / 4 .. 64 / 8 heads, with up to thirteen plans each, the choice is 0.5 % from the
// best on average in a triangle, 0.2 % behind the shard and 0.3 % without a mask (11 % at most; by the triangle's terms alone, whatever
// the call, 0.6, 2.1 and 2.1 %, up to 39 %): 2427 on 3640, 4 / 4, behind it 37.0 in five parts (the short kernel 51.1), 510 on 1275, 32 / 8,
// 25.6 (uncut on the main kernel 31.9), 2427 on 2427, 8 / 8, 40.6 in three parts (uncut 49.6); 512 on 512, 32 / 8, 14.1 (main kernel 17.7).
// Kept: 700 on 700, 32 / 8, 25.0 (main kernel 28.6), two of 2000, 16 / 16, 113 in two parts (uncut 117).
// Cut on the main kernel: 300 tokens on 20300 rows, 32 / 8 heads, 326 -> 99 us (of the pool 368 -> 104); 1488 on 101488, 32 / 32, 2.13 -> 1.97 ms.
// Requests of unequal length: the average says nothing of the longest one's walk, which may start as late as the round before the
// last ends.  With that in the estimate such a batch is cut differently where it promises a fifth less time; the estimate is rough, as
// which rows the longest request has is not known.  Over 265 batches that it would cut differently, most of them random (time against
// the even cut's): any gain promised 0.77 on average, 15 of them 3 .. 21 % slower; a fifth 0.78 and 8; three tenths 0.83 and 1.
// Measured (by the average -> by the longest, 32 / 8 heads): 16 tokens on 8192 rows beside seven of 16 on 512 53.0 -> 28.8 us, 8 on 200000
// beside 63 of 8 on 512 2205 -> 479, 300 on 20300 beside three of 300 on 600 328 -> 156; 32 on 60000 beside 31 of 32 on 64, 4 / 4,
// 405 -> 87; left alone: 20 tokens each on 700 .. 10000, 32 / 4, 46.1 (30.9).
// Where the chunk is a good part of the shard the rows are as good as known, in proportion to the keys, and the plan follows the longest
// request without that margin (46 batches of 2 .. 16 prompts: 0.7 % from the best on average, before 2.9 %): 2000 tokens beside
// fifteen of 32, 8 / 8, 34.4 -> 29.8 us; 4000 beside seven of 32, 4 / 4, 55.0 -> 44.2; 6000 beside fifteen of 32, 4 / 4, 75.1 -> 70.6.
struct PrefillPlan { int32_t splits, use_short; };
// What the estimate is told of a call beside its sizes.  `kept`: rows are kept on the way; such items stay side by side (each owns the
// tiles on its diagonal).
struct PrefillKind { bool causal, kept; };
static thread_local int32_t t_forced_plan = 0;                      // this thread's choice instead (set_prefill_plan); 0: none
constexpr double kCus = 256;                                        // of the card that these times are of (a launch fills whatever there is)
// rounds of the main kernel's items, uncut (the lengths of a batch's requests are not known: half a ragged tile each)
static double prefill_rounds(int32_t Tq, int32_t batch, int32_t Hq, int32_t Hkv) {
    const double rows = (double)Tq * (Hq / Hkv);
    return Hkv * (batch == 1 ? ceil(rows / kBM) : rows / kBM + 0.5 * batch) / kCus;
}
// calls whose query tiles are halves in pairs
static bool prefill_paired(PrefillKind kind, double rounds, int32_t S) { return kind.causal && !kind.kept && S == 1 && rounds <= 1; }
// the chunk is so much of the shard that a causal mask may hide a triangle of it
static bool prefill_near(int32_t Tq, int32_t Tkv) { return Tq >= 0.4 * Tkv; }
static PrefillPlan prefill_plan(int32_t Tq, int32_t Tkv, int32_t batch, int32_t max_kv, int32_t Hq, int32_t Hkv, PrefillKind kind,
                                int32_t most_splits) {
    constexpr double kTileLeast = 0.7, kTileRows = 0.75, kTileTriangle = 1.05, kItem = 8.5, kMerge = 4, kBytesPerUs = 4e6;
    constexpr double kPairTile = 0.5, kPairTileFull = 0.4, kPairItem = 12;
    constexpr double kShortItem = 4.5, kShortStep = 1.85, kShortFar = 2.5, kShortTriangle = 1.3, kShortLater = 0.9, kShortBytesPerUs = 12.5e6;
    constexpr double kUnevenGain = 0.8;
    if (Tq <= 0 || Tkv <= 0) return {1, 0};
    if (t_forced_plan != 0) {
        const int32_t parts = t_forced_plan < 0 ? -t_forced_plan : t_forced_plan, S = parts <= most_splits ? parts : 1;
        return {S, t_forced_plan < 0 ? 1 : 0};
    }
    const bool near = prefill_near(Tq, Tkv);
    const double rows = (double)Tq * (Hq / Hkv), tiles = ceil((double)Tkv / batch / kBN);
    const double at_end = Tq < Tkv ? 1.0 - 0.5 * Tq / Tkv : 0.5;      // of the tiles, seen on average by a chunk at the shard's end
    const double rounds = prefill_rounds(Tq, batch, Hq, Hkv);
    const double blocks = Hkv * (batch == 1 ? ceil(rows / kShortRows) : rows / kShortRows + 0.5 * batch);
    const double kv_bytes = (double)Tkv * Hkv * (4 * kHeadDim);
    // `longest`: tiles of the longest request, or of all alike (`tiles`); `triangle`: the chunk is at the end of a shard that it is a good
    // part of.  There the requests of a batch are taken to have rows as they have keys, and a batch takes no less than its longest alone.
    auto rows_of = [&](double longest) { return rows * fmin(longest * kBN / Tkv, 1); };
    auto merge_us = [&](int32_t S) { return S > 1 ? kMerge + S * rows * Hkv * (2 * 4 * kHeadDim) / kBytesPerUs : 0.0; };
    auto main_us = [&](int32_t S, double longest, bool triangle) {
        if (triangle && prefill_paired(kind, rounds, S)) {
            const double alike = Tq < Tkv ? 1 - (double)Tq / Tkv : 0;   // of the tiles, seen by all rows
            return longest * (alike * kTileTriangle + (1 - alike) * (kPairTile + kPairTileFull * rounds)) + kPairItem;
        }
        const double seen = near && !triangle ? 1 : at_end;
        const double tile = fmin(kTileLeast + kTileRows * fmin(rows / batch / kBM, 1), triangle && !kind.kept ? kTileTriangle : HUGE_VAL);
        auto item_of = [&](double t) { return seen * t / S * tile + kItem; };
        auto rounds_us = [&](double n, double t) { return triangle ? fmax(t / S * tile + kItem, (n + 0.3) * item_of(t)) : ceil(n) * item_of(t); };
        double us = rounds_us(rounds * S, tiles);
        if (longest > tiles) {
            us = fmax(us, fmax(rounds * S - 1, 0) * item_of(tiles) + longest / S * tile + kItem);
            if (near) us = fmax(us, rounds_us(Hkv * ceil(rows_of(longest) / kBM) / kCus * S, longest));
        }
        return us + merge_us(S);
    };
    auto short_us = [&](int32_t S, double longest, bool triangle) {
        const double seen = near && !triangle ? 1 : at_end;
        const double step = kv_bytes > 2e8 ? kShortFar : triangle ? kShortTriangle + (kShortStep - kShortTriangle) * (seen - 0.5) / 0.3 : kShortStep;
        auto item_of = [&](double t) { return kShortItem + step * ceil(2 * t / S / kShortWaves); };
        auto rounds_us = [&](double n, double t) {
            const double item = item_of(t);
            if (!triangle) return (1 + (near ? kShortLater : 1) * (ceil(n) - 1)) * item;
            return n <= 1 ? item : fmax(item, (n + 0.3) * (kShortItem + (0.5 + 0.5 * seen) * (item - kShortItem)));
        };
        double us = rounds_us(blocks * S / kCus, tiles), swept = blocks / Hkv / batch * seen * kv_bytes;
        if (longest > tiles) {
            us = fmax(us, fmax(blocks * S / kCus - 1, 0) * item_of(tiles) + item_of(longest));
            const double their_rows = near ? rows_of(longest) / kShortRows * seen * Hkv : blocks / batch;
            swept = fmax(swept, their_rows * longest * kBN * (4 * kHeadDim));
            if (near) us = fmax(us, rounds_us(Hkv * ceil(rows_of(longest) / kShortRows) / kCus * S, longest));
        }
        return fmax(us, swept / kShortBytesPerUs) + merge_us(S);
    };
    auto us_of = [&](const PrefillPlan& p, double longest, bool triangle) {
        return p.use_short ? short_us(p.splits, longest, triangle) : main_us(p.splits, longest, triangle);
    };
    // Of a causal call with a near shard the sizes do not say whether its rows see a triangle of it or, lying behind it, all: its plan
    // is the one whose time, as a multiple of the best plan's, is least in the worse of the two (where rows are kept: in the triangle).
    const bool may_be[2] = {!(near && kind.causal && kind.kept), near && kind.causal};   // all rows see alike; a triangle
    auto least = [&](double longest) {
        PrefillPlan plans[2 * ESP_MAX_PARTIALS];
        double us[2][2 * ESP_MAX_PARTIALS], least_us[2] = {HUGE_VAL, HUGE_VAL};
        int32_t n = 0;
        auto add = [&](int32_t S, int32_t use_short) {
            plans[n] = {S, use_short};
            for (int triangle = 0; triangle < 2; ++triangle) {
                if (!may_be[triangle]) continue;
                us[triangle][n] = us_of(plans[n], longest, triangle != 0);
                least_us[triangle] = fmin(least_us[triangle], us[triangle][n]);
            }
            ++n;
        };
        for (int32_t S = 1; S <= most_splits && (S == 1 || longest >= 4 * S); ++S) add(S, 0);
        for (int32_t S = 1; S <= most_splits && (S == 1 || 2 * longest >= kShortWaves * S); ++S) {
            if (S > 1 && blocks > Hkv * batch && Hkv * S % 8 != 0) continue;
            if ((rows / kShortRows + batch) * Hkv * S > 4e6) break;  // one workgroup each: what a launch holds
            add(S, 1);
        }
        int32_t best = 0;
        double best_cost = HUGE_VAL;
        for (int32_t i = 0; i < n; ++i) {
            double cost = 0;
            for (int triangle = 0; triangle < 2; ++triangle)
                if (may_be[triangle]) cost = fmax(cost, us[triangle][i] / least_us[triangle]);
            if (cost < (plans[i].use_short == plans[best].use_short ? 0.97 : 1.0) * best_cost) { best = i; best_cost = cost; }
        }
        return plans[best];
    };
    const double longest = ceil((double)max_kv / kBN);
    if (longest <= tiles) return least(tiles);
    const PrefillPlan uneven = least(longest);
    if (near) return uneven;
    const PrefillPlan even = least(tiles);
    return us_of(uneven, longest, false) < kUnevenGain * us_of(even, longest, false) ? uneven : even;
}
// bytes of the parts' results: O [S][Tq, Hq, 128] fp32, then LSE [S][Tq, Hq], each part on a 256-byte boundary
static size_t split_o_bytes(int32_t Tq, int32_t Hq) { return (size_t)Tq * Hq * kHeadDim * 4; }
static size_t split_lse_bytes(int32_t Tq, int32_t Hq) { return ((size_t)Tq * Hq * 4 + 255) / 256 * 256; }
static size_t split_bytes(int32_t S, int32_t Tq, int32_t Hq) { return S > 1 ? S * (split_o_bytes(Tq, Hq) + split_lse_bytes(Tq, Hq)) : 0; }

// Parts that a call may run in.  For a batch the workspace is asked for before the longest request is known: it has room for what
// equal requests are cut in, and for what the batch would be cut in if one request held all keys, the latter as far as kUnevenBytes go
// (which few rows fit, and cutting helps only those: the merge of 64 MB of parts takes 30 us).
constexpr size_t kUnevenBytes = 64 << 20;
static int32_t prefill_most_splits(int32_t Tq, int32_t Tkv, int32_t batch, int32_t Hq, int32_t Hkv) {
    auto splits = [&](int32_t max_kv) {                              // (what kind of call: not known either; without a mask, kept rows change nothing)
        int32_t S = 1;
        for (const PrefillKind kind : {PrefillKind{true, false}, PrefillKind{true, true}, PrefillKind{false, false}}) {
            const int32_t its = prefill_plan(Tq, Tkv, batch, max_kv, Hq, Hkv, kind, ESP_MAX_PARTIALS).splits;
            if (its > S) S = its;
            if (!prefill_near(Tq, Tkv)) break;                      // all kinds alike
        }
        return S;
    };
    int32_t most = splits(0);
    if (batch > 1) {
        int32_t uneven = splits(Tkv);
        while (uneven > most && split_bytes(uneven, Tq, Hq) > kUnevenBytes) --uneven;
        if (uneven > most) most = uneven;
    }
    return most;
}
size_t prefill_workspace_bytes(int32_t Tq, int32_t Tkv, int32_t batch, int32_t Hq, int32_t Hkv) {
    return kPrefillCounterBytes + split_bytes(prefill_most_splits(Tq, Tkv, batch, Hq, Hkv), Tq, Hq);
}

int32_t set_prefill_plan(int32_t plan) {
    const int32_t before = t_forced_plan;
    t_forced_plan = plan;
    return before;
}
// what a call with a workspace of so many bytes runs on
static PrefillPlan prefill_plan_in(size_t workspace_bytes, int32_t Tq, int32_t Tkv, int32_t batch, int32_t max_kv, int32_t Hq, int32_t Hkv, PrefillKind kind) {
    PrefillPlan plan = prefill_plan(Tq, Tkv, batch, max_kv, Hq, Hkv, kind, ESP_MAX_PARTIALS);
    if (batch > 1 && plan.splits > 1) {                            // (a larger workspace than was asked for changes nothing)
        const int32_t most = prefill_most_splits(Tq, Tkv, batch, Hq, Hkv);
        if (plan.splits > most) plan = prefill_plan(Tq, Tkv, batch, max_kv, Hq, Hkv, kind, most);
    }
    int32_t fit = plan.splits;
    while (fit > 1 && workspace_bytes < kPrefillCounterBytes + split_bytes(fit, Tq, Hq)) --fit;
    return fit == plan.splits ? plan : prefill_plan(Tq, Tkv, batch, max_kv, Hq, Hkv, kind, fit);   // a block without room for all parts
}
int32_t query_prefill_plan(size_t workspace_bytes, int32_t Tq, int32_t Tkv, int32_t batch, int32_t max_kv, int32_t Hq, int32_t Hkv, bool causal, bool kept) {
    const PrefillPlan plan = prefill_plan_in(workspace_bytes, Tq, Tkv, batch, max_kv, Hq, Hkv, PrefillKind{causal, kept});
    return plan.use_short ? -plan.splits : plan.splits;
}

constexpr int kStages = 4;            // LDS stages per operand; tile j lives in stage j % 4
constexpr float kSumLimit = 1048576.f;  // 2^20: a tile's probability sum above this refreshes the offset

template <int V> struct IC { static constexpr int value = V; };

// MODE 0: the plain kernel.
// RETAIN (MODE 1): the variant that also keeps rows of the shard in the token pool while they pass through LDS (proactive
// scale-down, Sec. 4.1 / Fig. 7).  Every KV tile of a request and KV head is OWNED by one item, which stores its K
// and V rows to the pool slots that are not negative:
//   * a request whose shard rows are about as many as its query rows (a striped shard, causal self-attention): the
//     item of query tile i owns the KV tiles of its tokens, from 4i / G up to (4i + 4) / G (the last query tile: all
//     that remain).  Under a causal mask these are the tiles on its diagonal, the last ones of its sweep, which
//     run the masked iteration anyway: the work is spread evenly over the items and costs each of them little;
//   * any other request (a chunk against a long prefix): one item owns every tile, the last query tile's, or the
//     first one's where the workgroups of an XCD walk a KV head's rows together (its turn comes last of that head's).
// An owner sweeps at least up to its last owned tile (tiles it cannot see pass through LDS without arithmetic), runs
// the masked iteration from its first owned tile on, finds the slots in a ring of 8 LDS stages (the first four owned
// tiles' slots are fetched at the start, the others with their K tiles), and stores the sweep's last four tiles, which
// stay in LDS, after the sweep; an earlier tile j at the top of iteration j: complete in LDS by then, and issued
// ahead of the iteration's transfers, so that the hand-counted waits still see those as the newest operations in
// flight (they have to sit out the stores, though, which is why the tiles at the end are left for later).
//
// MODE 3: MODE 1 for a Q that does not lie on 16 bytes.  (The other modes ask a.q_odd.  This one has no scalar register left for the
// question: 1000 .. 8192 tokens, kept, 32 / 8 heads, 654 us without it, 661 with; Q through registers in every call 0.4 .. 1 % more.)
//
// POOL (MODE 2): the shard's rows live in the token pool (a.k / a.v are the pools, a.kv_slot the slot of every shard
// row, Sec. 4.1 / 4.2: KV that an instance kept stays where it was placed).  The tile transfers take each row from its
// slot: the slots of tile t travel to a ring of 4 LDS stages (stage t % 4) one iteration before the tile's first
// transfer is issued, every lane reads the slot of the row its 16 bytes belong to and forms the address itself.
//
// ONE (with MODE 0): one request, one query head per KV head, keys uncut: the chunk or the stripe of a multi-head model.  What
// bounds a short call of that kind is the chain of instructions in front of its first transfer and at its end, and here the
// rows of a tile are Hq rows apart, known when it is compiled: no float arithmetic for every row that is loaded and stored, no
// search for request, part and query head.  Measured, 32 / 32 heads (any call -> ONE): 700 on 700 23.4 -> 22.3 us, against two of 700
// 49.8 -> 46.9 us; 1500 on 1500 39.4 -> 38.1; 4000 on 20000 962 -> 960; 8192 against four of 8192 1824 -> 1808 us.  The
// same for MODE 1 and 2 gained nothing: 1500 against two of 1500, kept, 8 / 8 heads, 81.9 -> 82.4 us, 2048 against 8192 rows
// of the pool, 32 / 32 heads, 237.5 -> 237.7 us.
//
// PAIRED (with MODE 0 and 2, uncut): where a causal call's items are one round of workgroups, its time is the longest sweep's, the last query
// tile's, while a workgroup of the first ones has nothing left to do.  So a tile is 128 rows from the end of the request and the 128 as
// far from its start: every workgroup has a long and a short half, and where only the long one is left, one wavefront per SIMD,
// a tile takes 0.75 us in place of 1.05.  The wavefronts' rows are counted from each one's own first row then.  Over more than one round the deal
// evens the items out, and one wavefront per SIMD leaves the matrix pipe idle: 1200 and 1100 tokens, 32 / 8 heads (296 items), 36.7 us
// side by side, 46.4 paired, 3000, 32 / 8, 78.4 and 88.5, 8192, 32 / 32, 446 and 486.  Measured (side by side -> paired, or the best cut ->
// paired): 2048 on 2048, 32 / 8, 49.4 -> 43.6 us; 1000, 32 / 32, 28.1 -> 24.7; 4000, 16 / 16, 81.7 -> 70.8; 3000, 12 / 12, 50.2 -> 45.4;
// 6000, 8 / 8, 88.6 -> 83.2; 4000, 300, 1500, 600 and 900, 8 / 8, 76.2 -> 60.8; 2000 on 2000 rows of the pool, 32 / 8, 57.0 -> 50.1.
template <int MODE, bool ONE, bool PAIRED>
__global__ __launch_bounds__(kPfWaves * 64) void prefill_kernel(PrefillArgs a) {
    constexpr bool RETAIN = MODE == 1 || MODE == 3, POOL = MODE == 2;
    constexpr int kTileRow = PAIRED ? 0 : 32, kHalf = kBM / 2;      // rows of the tile ahead of each wavefront's own (PAIRED: counted from its own)
    // One LDS block, V stages first: an LDS instruction adds a 16-bit immediate to its address register, so with
    // each array's base folded into the per-lane register every operand read of the loop needs no address math.
    constexpr int kLdsV = 0, kLdsK = kLdsV + kStages * kTileBytes, kLdsPos = kLdsK + kStages * kKTileBytes,
                  kLdsQmm = kLdsPos + kStages * kBN * 4, kLdsSched = kLdsQmm + 2 * kPfWaves * 4,
                  kLdsFlag = kLdsSched + kPfWaves * 64 * 8, kLdsSlot = kLdsFlag + 16,
                  kLdsK0 = kLdsSlot + (RETAIN ? 8 * kBN * 4 : POOL ? (kStages + 1) * kBN * 4 : 0), kLdsTotal = kLdsK0 + kKTileBytes;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kLdsTotal];
    int32_t (*lds_pos)[kBN] = (int32_t (*)[kBN])(smem + kLdsPos);
    int32_t (*lds_qmm)[kPfWaves] = (int32_t (*)[kPfWaves])(smem + kLdsQmm);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = ONE ? 1 : a.G;

    // ---- one query tile of one KV head (rank: position in the heaviest-first order of query tiles).  Returns false
    //      if there is no such tile.  With `claim_from` set, thread 0 also draws the workgroup's next item from that
    //      counter (a device-wide atomic, issued when the sweep is done; its latency hides behind the epilogue) and
    //      leaves the counter's old value in LDS (lds_next), to be read after the next workgroup barrier.
    int32_t* lds_next = (int32_t*)(smem + kLdsFlag + 4);
    // The pool counter needs no clearing between launches: its high word names the launch that counted in it.  A
    // draw is one fetch-and-add; if the old value carries this launch's tag, its low word is the ticket.  If not
    // (a draw before this launch's count was started finds the previous launch's count, or whatever a fresh workspace
    // holds), the drawer starts it with a compare-and-swap, or draws again if another one has done so.
    auto draw_finish = [&](unsigned long long* ctr, unsigned long long old) {
        if ((uint32_t)(old >> 32) == a.tag) return (int)(uint32_t)old;
        for (unsigned long long cur = old + 1;;) {
            if (__hip_atomic_compare_exchange_strong(ctr, &cur, ((unsigned long long)a.tag << 32) | 1ULL, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                return 0;
            if ((uint32_t)(cur >> 32) == a.tag)
                return (int)(uint32_t)__hip_atomic_fetch_add(ctr, 1ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    auto process = [&](const int rank, const int vhead, unsigned long long* claim_from) {
    const bool cut = !ONE && !PAIRED && a.splits > 1;
    const int kvh = cut ? vhead / a.splits : vhead, part = cut ? vhead - kvh * a.splits : 0;
    int row0, n_rows, g0, kv_lo, kv_hi;   // first row of this tile (PAIRED: of this wavefront) in the [token, head] order, how many it has, query head of
                                          // the group it starts at; rows of its request in the shard
    int tok0;                       // token of the first row
    int own_lo = 0, own_hi = 0;     // KV tiles of the request whose rows this item keeps in the pool (none: equal)
    {
        // query tiles of request r; a request without query rows whose shard rows may have to be kept gets one
        // (empty) tile, so that it has a keeper
        auto tiles_of = [&](int r) {
            const int len = a.cu_q ? a.cu_q[r + 1] - a.cu_q[r] : a.Tq;
            int nt = (len * G + kBM - 1) / kBM;
            if (RETAIN && nt == 0 && a.retain_slot && a.cu_kv && a.cu_kv[r + 1] > a.cu_kv[r]) nt = 1;
            return nt;
        };
        // later tiles of a causal request see more keys: they come first, the last request's before the others'.
        // The requests are looked at 64 at a time, one per lane, from the last one down: a scan of their tile counts
        // finds the one that holds tile `rank`.
        int tl = 0, r = 0, nt = 0;
        if (ONE || a.batch == 1) {
            nt = __builtin_amdgcn_readfirstlane(tiles_of(0));
            if (rank >= nt) return false;
            tl = nt - 1 - rank;
        } else {
            int skip = rank;
            bool found = false;
            int ln = lane;                                          // (opaque: keeps the scan's lane arithmetic out of the item
            asm volatile("" : "+v"(ln));                            // loop's invariants, i.e. out of registers that live through the sweep)
            for (int top = a.batch - 1; top >= 0; top -= 64) {
                const int n = ln <= top ? tiles_of(top - ln) : 0;
                int upto = n;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int below = __shfl_up(upto, d);
                    if (ln >= d) upto += below;
                }
                const uint64_t hit = __builtin_amdgcn_ballot_w64(upto > skip);
                if (hit) {
                    const int l = __builtin_ctzll(hit);
                    r = top - l;
                    nt = __builtin_amdgcn_readlane(n, l);
                    tl = __builtin_amdgcn_readlane(upto, l) - 1 - skip;
                    found = true;
                    break;
                }
                skip -= __builtin_amdgcn_readlane(upto, 63);
            }
            if (!found) return false;
        }
        const int qs = a.cu_q ? a.cu_q[r] : 0, qe = a.cu_q ? a.cu_q[r + 1] : a.Tq;
        int rho = tl * kBM;
        n_rows = min(kBM, (qe - qs) * G - rho);
        if constexpr (PAIRED) {                                     // (of this wavefront; without rows, any of the tile's will do for what is loaded)
            const int total = (qe - qs) * G, lower = nt - 1 - tl, upper = (total + kHalf - 1) / kHalf - 1 - lower;
            rho = (wave < kPfWaves / 2 ? lower : upper) * kHalf + (wave & (kPfWaves / 2 - 1)) * 32;
            n_rows = wave >= kPfWaves / 2 && upper == lower ? 0 : max(min(32, total - rho), 0);
            if (n_rows == 0) rho = lower * kHalf;
        }
        tok0 = qs + rho / G;
        g0 = rho % G;
        row0 = tok0 * a.Hq + kvh * G + g0;
        kv_lo = a.cu_kv ? a.cu_kv[r] : 0;
        kv_hi = a.cu_kv ? a.cu_kv[r + 1] : a.Tkv;
        if (RETAIN && a.retain_slot != nullptr) {                // which KV tiles this item owns (see the kernel's head)
            const int tiles = (kv_hi - kv_lo + kBN - 1) / kBN, per = kBM / kBN;
            if (!a.group_sync && a.causal && (int64_t)tiles * G <= (int64_t)per * nt + per * G) {
                own_lo = min(per * tl / G, tiles);
                own_hi = tl == nt - 1 ? tiles : min(per * (tl + 1) / G, tiles);
            } else if (tl == (a.group_sync ? 0 : nt - 1)) {
                own_hi = tiles;
            }
        }
        if (cut) {                                                  // this part's share of the request's tiles, as if it were the shard
            const int tiles = (kv_hi - kv_lo + kBN - 1) / kBN;
            const int t_lo = (int)((int64_t)tiles * part / a.splits), t_hi = (int)((int64_t)tiles * (part + 1) / a.splits);
            kv_hi = min(kv_hi, kv_lo + t_hi * kBN);
            kv_lo = min(kv_lo + t_lo * kBN, kv_hi);
            if (RETAIN) {
                own_lo = min(max(own_lo - t_lo, 0), t_hi - t_lo);
                own_hi = min(max(own_hi - t_lo, 0), t_hi - t_lo);
            }
        }
    }
    // the same for every lane by construction; said explicitly, since base addresses of the tile transfers derive
    // from them and must sit in scalar registers
    row0 = __builtin_amdgcn_readfirstlane(row0); n_rows = __builtin_amdgcn_readfirstlane(n_rows);
    tok0 = __builtin_amdgcn_readfirstlane(tok0); g0 = __builtin_amdgcn_readfirstlane(g0);
    kv_lo = __builtin_amdgcn_readfirstlane(kv_lo); kv_hi = __builtin_amdgcn_readfirstlane(kv_hi);
    own_lo = __builtin_amdgcn_readfirstlane(own_lo); own_hi = __builtin_amdgcn_readfirstlane(own_hi);
    // token of row i of this tile, counted from tok0 (with G > 1 exact: i + g0 is far below 2^21), and the row's distance from row0
    auto token_of = [&](int i) { return ONE ? i : (int)(((float)(i + g0) + 0.5f) * a.inv_G); };
    auto row_of = [&](int i) { return ONE ? i * a.Hq : i + token_of(i) * (a.Hq - G); };
    // The rest of the item exists twice in the keeping kernel: as everywhere else, and with an owner's extras.
    // (One body with the extras behind a run-time flag costs the items that own nothing dearly: measured +25 % on
    // a GQA batch, where three items in four own nothing, against +1.6 % with two bodies.)
    auto body = [&](auto keep_c) {
    constexpr bool KEEP = RETAIN && decltype(keep_c)::value != 0;
    const int kv_len = kv_hi - kv_lo;
    const int nkt = (kv_len + kBN - 1) / kBN;
    const int tail_rows = kv_len - (nkt - 1) * kBN;    // rows of the last tile (64 when not ragged)
    const int ragged_tile = tail_rows < kBN ? nkt - 1 : -8;          // index of the ragged last tile, if any

    // ---- global -> LDS in transfers of 64 lanes x 16 bytes = 1 KiB of consecutive LDS bytes.
    //      K and V tiles have rows of 256 B, their chunks XOR-swizzled: wavefront w moves rows 8w .. 8w+7 of either, 2 KiB in a row, in two
    //      transfers; lane L writes LDS chunk L % 16 of row r = base + L / 16, so it fetches the global chunk
    //      (L % 16) ^ f(r).  Wavefront 0 also moves the positions.
    //      (K rows padded to 272 bytes instead: operand reads with one address register for four, but 17 transfers, of which each lane's
    //      bytes fell into rows of their own, and wavefront 7 had one more.  Padded -> swizzled, 32 / 8 heads: 1000 .. 8192 against two
    //      shards, kept, 1374 -> 1343 us; 32 / 32: 8192 against four of 8192 1866 -> 1841, merge included, 32768 on 262144 103.8 -> 103.3 ms, 1000 on 1000
    //      24.8 -> 24.5; pool rows below.)
    const uint32_t kv_row_bytes = (uint32_t)a.Hkv * kHeadDim * 2;
    const int64_t tile_bytes = (int64_t)kBN * kv_row_bytes;
    const int st_sub = lane >> 4, st_p = lane & 15;
    const int st_r0 = wave * 8 + st_sub, st_r1 = st_r0 + 4;
    auto v_goff = [&](int r_lds, int r_glb) { return r_glb * kv_row_bytes + ((st_p ^ ((r_lds & 3) << 2)) << 4); };
    auto k_goff = [&](int r_lds, int r_glb) { return r_glb * kv_row_bytes + ((st_p ^ (r_lds & 7)) << 4); };
    const uint32_t gv0 = v_goff(st_r0, st_r0), gv1 = v_goff(st_r1, st_r1);
    const uint32_t gk0 = k_goff(st_r0, st_r0), gk1 = k_goff(st_r1, st_r1);
    const uint32_t lds_base0 = (uint32_t)(uintptr_t)(ESP_LDS unsigned char*)smem;
    // row kv_lo, head kvh (POOL: slot 0, head kvh)
    const char* kreq = (const char*)a.k + ((int64_t)(POOL ? 0 : kv_lo) * a.Hkv + kvh) * (kHeadDim * 2);
    const char* vreq = (const char*)a.v + ((int64_t)(POOL ? 0 : kv_lo) * a.Hkv + kvh) * (kHeadDim * 2);
    // POOL: one read of the ring (stage kStages: tile 0) has the slots of both rows that a lane moves of K or V.  From a slot to a row's
    // address: one 32 x 32 -> 64-bit multiply-add on where this lane's 16 bytes lie in slot 0.
    // The loop is bound by issue and by power (the LDS is busy in 35 % of its cycles); with padded rows of K it took five slot reads a wavefront and
    // tile, each an instruction and a round trip in front of a transfer, now two for two rows each.  Padded -> swizzled: a tile 2666 -> 2577 cycles; 300 tokens on 20300 rows of
    // the pool, 32 / 8 heads, 108.8 -> 105.9 us, 2000 on 2000 51.7 -> 48.7, 8000 on 30000 2733 -> 2680, 2048 on 10240, 32 / 32, 285 -> 279.
    const ESP_LDS int32_t* const slot_rd = (const ESP_LDS int32_t*)(uintptr_t)(lds_base0 + kLdsSlot + st_r0 * 4);
    auto pool_slot = [&](int st, int part) { return slot_rd[st * kBN + 4 * part]; };
    const char* const pk0 = kreq + ((st_p ^ (st_r0 & 7)) << 4);
    const char* const pk1 = kreq + ((st_p ^ (st_r1 & 7)) << 4);
    const char* const pv = vreq + ((st_p ^ ((st_r0 & 3) << 2)) << 4);
    auto pool_at = [&](const char* at, int32_t slot) { return at + (uint64_t)(uint32_t)slot * kv_row_bytes; };
    // slots of tile t into ring stage st (wavefront 6); rows past the end of a ragged last tile repeat the last row's
    // slot, so their transfers re-read that row (their scores get masked)
    const int32_t* slot_req = POOL ? a.kv_slot + kv_lo : nullptr;
    auto fetch_pool_slots = [&](int t, int st) {
        if (!POOL || wave != 6 || t >= nkt) return;
        const int rows = min(kBN, kv_len - t * kBN);
        load_to_lds_b32(lds_base0, kLdsSlot + st * (kBN * 4), slot_req + t * kBN, min(lane, rows - 1) * 4);
    };
    // the same inside the sweep's plain iterations, where the tile is a full one that exists: nothing to work out
    const uint32_t lane4 = lane * 4;
    auto fetch_pool_slots_full = [&](int t, int st) {
        load_to_lds_b32(lds_base0, kLdsSlot + st * (kBN * 4), slot_req + t * kBN, lane4);
    };
    const int32_t* preq = a.kv_pos + kv_lo;
    const uint32_t lds_base = lds_base0;
    const uint32_t lds_k0 = lds_base + kLdsK, lds_v0 = lds_base + kLdsV;
    const uint32_t lds_w = lds_base + wave * 2048, lds_wk = lds_base + wave * kKGroup;   // this wavefront's first pieces of V and K tiles

    // K tile at kt into K stage st: 2 transfers per wavefront; `part` picks one of them, so that
    // the sweep can spread them over an iteration (a burst of transfers from all wavefronts at once backs up the
    // memory pipeline and stalls the issuing wavefronts).  `tail`: it is the ragged last tile, whose rows past the
    // end re-read the last row (their scores get masked).
    auto fetch_k_part = [&](const char* kt, int st, bool tail, int part) {
        const int off = (st == kStages ? kLdsK0 : kLdsK + st * kKTileBytes) + 1024 * part;
        if constexpr (POOL) { load_to_lds_b128_at(lds_wk, off, pool_at(part == 0 ? pk0 : pk1, pool_slot(st, part))); return; }
        if (__builtin_expect(tail, 0)) {
            const int r = part == 0 ? st_r0 : st_r1;
            load_to_lds_b128(lds_wk, off, kt, k_goff(r, min(r, tail_rows - 1)));
        } else {
            load_to_lds_b128(lds_wk, off, kt, part == 0 ? gk0 : gk1);
        }
    };
    // V tile at vt and its positions at pt into V stage st: 2 transfers per wavefront, 3 for wavefront 0
    auto fetch_v_part = [&](const char* vt, const int32_t* pt, int st, bool tail, int part, int slot_st = -1) {
        const int off = kLdsV + st * kTileBytes + 1024 * part;
        const int last = tail_rows - 1;
        if (part == 2) {
            if (wave != 0) return;
            load_to_lds_b32(lds_base, kLdsPos + st * (kBN * 4), pt, (tail ? min(lane, last) : lane) * 4);
        } else if constexpr (POOL) {
            load_to_lds_b128_at(lds_w, off, pool_at(pv, pool_slot(slot_st < 0 ? st : slot_st, part)));
        } else if (__builtin_expect(tail, 0)) {
            const int r = part == 0 ? st_r0 : st_r1;
            load_to_lds_b128(lds_w, off, vt, v_goff(r, min(r, last)));
        } else {
            load_to_lds_b128(lds_w, off, vt, part == 0 ? gv0 : gv1);
        }
    };
    auto fetch_k = [&](const char* kt, int st, bool tail) {
        fetch_k_part(kt, st, tail, 0); fetch_k_part(kt, st, tail, 1);
    };
    auto fetch_v = [&](const char* vt, const int32_t* pt, int st, bool tail) {
        fetch_v_part(vt, pt, st, tail, 0); fetch_v_part(vt, pt, st, tail, 1); fetch_v_part(vt, pt, st, tail, 2);
    };
    // positions past the end of a ragged last tile become INT_MAX, hidden from every query
    auto seal_tail = [&](int st) {
        if (wave == 0 && lane >= tail_rows) lds_pos[st][lane] = INT_MAX;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // written before the barrier that follows
    };

    // an owner's extras: slots of an owned tile t into stage t % 8 of the slot ring (wavefront 6), and the stores of
    // owned tiles' K and V rows from LDS to the pool (wavefront w: rows 8w .. 8w+7)
    const int32_t* sreq = KEEP ? a.retain_slot + kv_lo : nullptr;
    auto fetch_slots = [&](int t) {
        if (!KEEP || wave != 6 || t < own_lo || t >= own_hi) return;
        const int rows = min(kBN, kv_len - t * kBN);
        load_to_lds_b32(lds_base, kLdsSlot + (t & 7) * (kBN * 4), sreq + t * kBN, min(lane, rows - 1) * 4);
    };
    // Slots past the end of a ragged last tile become -1 (wavefront 6, once the tile's slots have landed and a
    // barrier before anyone reads them), so that the stores test the slot alone.
    auto seal_slots = [&]() {
        if (!KEEP || wave != 6 || ragged_tile < own_lo || ragged_tile >= own_hi) return;
        if (lane >= tail_rows) ((int32_t*)(smem + kLdsSlot))[(ragged_tile & 7) * kBN + lane] = -1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    // K and V rows of tile t (both in stage st, K(0) in its own place) to the pool, at the top of iteration t.  Every wavefront stores
    // exactly the LDS bytes its own transfers fill, rows 8w .. 8w+7 of either.  The K stage is refilled during this very iteration, but each
    // wavefront's own refills follow its own reads in program order, and it reads nobody else's bytes.
    // All LDS reads first (slots and rows, one round trip), then the stores.
    auto keep_tile = [&](int t, int st) {
        if (!KEEP) return;
        if (t < own_lo || t >= own_hi) return;
        const int32_t* ring = (const int32_t*)(smem + kLdsSlot) + (t & 7) * kBN;
        const unsigned char* kt = smem + (t == 0 ? kLdsK0 : kLdsK + st * kKTileBytes);
        const unsigned char* vt = smem + kLdsV + st * kTileBytes;
        const int r0 = wave * 8 + st_sub, r1 = r0 + 4;
        const int32_t s0 = ring[r0], s1 = ring[r1];
        const uint4 wk0 = *(const uint4*)(kt + k_chunk(r0, st_p));
        const uint4 wk1 = *(const uint4*)(kt + k_chunk(r1, st_p));
        const uint4 wv0 = *(const uint4*)(vt + r0 * 256 + ((st_p ^ ((r0 & 3) << 2)) << 4));
        const uint4 wv1 = *(const uint4*)(vt + r1 * 256 + ((st_p ^ ((r1 & 3) << 2)) << 4));
        // address of a pool row's piece: one 32 x 32 -> 64-bit multiply-add each
        const uint32_t row_pitch = (uint32_t)a.Hkv * (kHeadDim * 2);
        ESP_GLOBAL char* kb = (ESP_GLOBAL char*)a.k_pool + (uint32_t)kvh * (kHeadDim * 2) + 16 * st_p;
        ESP_GLOBAL char* vb = (ESP_GLOBAL char*)a.v_pool + (uint32_t)kvh * (kHeadDim * 2) + 16 * st_p;
        if (s0 >= 0) *(ESP_GLOBAL u32x4*)(kb + (uint64_t)(uint32_t)s0 * row_pitch) = u32x4{wk0.x, wk0.y, wk0.z, wk0.w};
        if (s1 >= 0) *(ESP_GLOBAL u32x4*)(kb + (uint64_t)(uint32_t)s1 * row_pitch) = u32x4{wk1.x, wk1.y, wk1.z, wk1.w};
        if (s0 >= 0) *(ESP_GLOBAL u32x4*)(vb + (uint64_t)(uint32_t)s0 * row_pitch) = u32x4{wv0.x, wv0.y, wv0.z, wv0.w};
        if (s1 >= 0) *(ESP_GLOBAL u32x4*)(vb + (uint64_t)(uint32_t)s1 * row_pitch) = u32x4{wv1.x, wv1.y, wv1.z, wv1.w};
    };

    // ---- this lane's query row (column of S^T); its position is needed first (schedule scan), so it is loaded first
    const int qi = lane & 31, hi = lane >> 5;
    int bl = lane, bw = wave;                                       // opaque, as at the scan of the requests: what is worked out from
    asm volatile("" : "+v"(bl), "+s"(bw));                          // these once per item does not live through the sweep
    const int ld_i = PAIRED ? max(min(bl & 31, n_rows - 1), 0) : min(bw * 32 + (bl & 31), n_rows - 1);
    const bool any_row = PAIRED || n_rows > 0;                        // (an empty tile of the keeping variant: any row will do)
    // effective query position: non-causal rows see every real key
    const int my_qpos = a.causal ? a.q_pos[any_row ? tok0 + token_of(ld_i) : 0] : INT_MAX - 1;   // INT_MAX marks rows past a ragged tail

    // ---- smallest / largest key position of the KV tiles of this request, to LDS, 512 tiles at a time: 16 lanes a tile, four
    //      positions a lane, so that a load is 1 KiB in a row, at any 4-byte alignment; past the request's end the last four
    //      again.  (So a last tile of one to three rows takes rows of the tile before in: it may be seen or masked where it need
    //      not be, never the other way round.)  A thread per tile touched 64 cache lines with each of sixteen loads, and took the
    //      positions one by one where a request's rows do not start on 16 bytes: 6 us of the 11 before an item's first tile.
    int2* lds_mm = (int2*)(smem + kLdsSched);
    constexpr int kBoundTiles = kPfWaves * 64;
    struct __attribute__((packed, aligned(4))) Pos4 { int32_t x, y, z, w; };
    auto load_bounds = [&](auto& v, int base, int g0) {              // groups of four tiles: g0 + wave, + 8, ...
#pragma unroll
        for (int u = 0; u < (int)(sizeof v / sizeof v[0]); ++u) {
            const int row = (base + 4 * (g0 + 8 * u + bw)) * kBN + 4 * bl;
            v[u] = *(const Pos4*)(preq + min(row, kv_len - 4));
        }
    };
    auto least = [](int x, int y) { return min(x, y); };
    auto most = [](int x, int y) { return max(x, y); };
    auto row16 = [](int x, auto op) {                               // over the 16 lanes of a tile, by rotations
        x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false));
        x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, false));
        x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x122, 0xf, 0xf, false));
        return op(x, __builtin_amdgcn_update_dpp(0, x, 0x121, 0xf, 0xf, false));
    };
    auto store_bounds = [&](const auto& v, int g0) {                 // (of tiles past the last: not read)
#pragma unroll
        for (int u = 0; u < (int)(sizeof v / sizeof v[0]); ++u) {
            const int mn = row16(min(min(v[u].x, v[u].y), min(v[u].z, v[u].w)), least);
            const int mx = row16(max(max(v[u].x, v[u].y), max(v[u].z, v[u].w)), most);
            const int at = 4 * (g0 + 8 * u + bw) + (bl >> 4);
            if ((bl & 15) == 0 && at < kBoundTiles) lds_mm[at] = make_int2(mn, mx);
        }
    };
    const bool few_keys = kv_len < 4;                               // no four rows to load: see below
    Pos4 pos_first[4] = {};
    if (a.causal && !few_keys) load_bounds(pos_first, 0, 0);

    // ---- the item's first requests, in two groups, so that what the schedule and the scores of tile 0 wait for does not queue
    //      behind the rest.  First: query positions, bounds, K(0) with its positions, and Q.  K(0) has a place of its own, outside
    //      the ring: iteration 0 fetches K(4) into stage 0, while a wavefront that is behind may still be at the scores of tile 0.
    //      Q goes through LDS, laid out in whole rows (chunk c of row r at c ^ (r % 16)): fetched as fragments, 16-byte pieces of 32
    //      rows with every load, it took as long as all the tiles' transfers.  It lies where V(1), V(2), K(4) and K(3) go later.
    //      POOL: the slots of the first five tiles go first (tile 0's to a fifth ring stage, so that tile 4's need not wait for its
    //      readers), and K(0) is in the second group.
    //      An item's set-up, measured (all transfers, then positions, then bounds, then Q, each waiting for the one before -> this):
    //      11.0 -> 7.4 us with six prompts of 37 .. 2047 tokens, 32 / 8 heads, 9.8 -> 8.1 us with 8192 rows on 8192, 32 / 32 heads.
    //      Calls: the six prompts 65.0 -> 59.3 us, 300 tokens on 20300 rows of the pool, 32 / 8 heads, 110.6 -> 108.0, 1000 .. 8192
    //      against two shards, kept, 1504 -> 1464, 8192 against four shards and their merge 2038 -> 2024 (that one is bound by power).
    const uint32_t q_off = bw < 4 ? kLdsV + kTileBytes + bw * 8192 : kLdsK + (bw < 6 ? 0 : 3 * kKTileBytes) + (bw & 1) * 8192;
    if constexpr (POOL) {
        fetch_pool_slots(0, kStages); fetch_pool_slots(1, 1); fetch_pool_slots(2, 2); fetch_pool_slots(3, 3); fetch_pool_slots(4, 0);
    } else if (nkt > 0) {
        fetch_k(kreq, kStages, 0 == ragged_tile);
    }
    if (nkt > 0) fetch_v_part(vreq, preq, 0, 0 == ragged_tile, 2);
    {
        const char* qp = (const char*)a.q + (any_row ? (int64_t)row0 * (kHeadDim * 2) : 0);
        auto q_src = [&](int n) {
            const int r = 4 * n + (bl >> 4), i = max(min(kTileRow * bw + r, n_rows - 1), 0);
            return qp + (int64_t)row_of(i) * (kHeadDim * 2) + (((bl ^ r) & 15) << 4);
        };
        struct __attribute__((packed, aligned(2))) Any16 { uint32_t x, y, z, w; };
        if (MODE == 3 || (!RETAIN && __builtin_expect(a.q_odd, 0))) {   // not on 16 bytes: through registers, whose loads take any alignment
#pragma unroll 1
            for (int n = 0; n < 8; ++n)
                *(ESP_LDS u32x4*)(uintptr_t)(lds_base + q_off + 1024 * n + 16 * bl) = __builtin_bit_cast(u32x4, *(const Any16*)q_src(n));
        } else {
#pragma unroll
            for (int n = 0; n < 8; ++n) load_to_lds_b128_at(lds_base + q_off, 1024 * n, q_src(n));
        }
    }
    // V stage 3 stands in for the tile before the first one (the loop multiplies the last chunk of tile j-1 at the
    // start of iteration j): zero it, since stale LDS contents could be NaN patterns; V(3) arrives there later
    {
        const uint4 z = make_uint4(0u, 0u, 0u, 0u);
        uint4* dst = (uint4*)(smem + kLdsV + 3 * kTileBytes) + tid * 2;
        dst[0] = z;
        dst[1] = z;
        if (tid == 0) *(int32_t*)(smem + kLdsFlag) = 0;      // "redo with the plain sweep" flag, see below
    }

    wait_vm<0>();
    if (ragged_tile == 0) seal_tail(0);
    // the wavefront's smallest and largest query position (lanes l and l | 32 hold the same row)
    auto of_two = [](int x, auto op) { return op(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)); };
    const int wave_qmin = of_two(row16(my_qpos, least), least), wave_qmax = of_two(row16(my_qpos, most), most);
    if (lane == 0) { lds_qmm[0][wave] = wave_qmin; lds_qmm[1][wave] = wave_qmax; }

    // ---- tile schedule of this workgroup: n_vis = 1 + last tile some row can see (tiles before it that are
    //      hidden, possible only with unordered positions, are swept fully masked); first_mask = first tile
    //      this wavefront has to mask (every later tile is masked too, which is exact for ascending positions
    //      and merely redundant otherwise); n_need = 1 + last tile a row of this wavefront can see: beyond it
    //      the wavefront only keeps up its share of the transfers and the barriers.
    //      The bounds of 512 tiles at a time go through LDS; every wavefront then reads them all,
    //      64 per step, and wavefront-wide ballots turn its three tests into bit masks whose highest / lowest set
    //      bit is the answer: no exchange of candidates, and one barrier for requests of up to 512 tiles.
    int n_vis = nkt, first_mask = nkt, n_need = nkt;
    auto rest_of_bounds = [&](int base) {
        for (int g = base == 0 ? 4 * kPfWaves : 0; 4 * g < min(kBoundTiles, nkt - base); g += 8 * kPfWaves) {
            Pos4 v[8];
            load_bounds(v, base, g);
            store_bounds(v, g);
        }
    };
    if (a.causal && !few_keys) {
        store_bounds(pos_first, 0);
        rest_of_bounds(0);
    } else if (a.causal && tid == 0 && kv_len > 0) {
        int mn = INT_MAX, mx = INT_MIN;
        for (int e = 0; e < kv_len; ++e) { mn = min(mn, preq[e]); mx = max(mx, preq[e]); }
        lds_mm[0] = make_int2(mn, mx);
    }
    wg_barrier();
    // second group: what iteration 0 needs, in flight under the schedule scan and the scores of tile 0 (tiles the scan finds hidden are
    // fetched for nothing, which is harmless: they exist)
    fetch_slots(own_lo); fetch_slots(own_lo + 1); fetch_slots(own_lo + 2); fetch_slots(own_lo + 3);
    if (nkt > 4) {                                                   // the usual case, without a conditional in it
        if constexpr (POOL) fetch_k(kreq, kStages, false);
        fetch_k(kreq + tile_bytes, 1, false);
        fetch_v_part(vreq, preq, 0, false, 0, kStages); fetch_v_part(vreq, preq, 0, false, 1, kStages);
        fetch_k(kreq + 2 * tile_bytes, 2, false);
        fetch_v_part(vreq, preq + kBN, 1, false, 2);
    } else if (nkt > 0) {
        const bool tail = 0 == ragged_tile;
        if constexpr (POOL) fetch_k(kreq, kStages, tail);
        if (nkt > 1) fetch_k(kreq + tile_bytes, 1, 1 == ragged_tile);
        fetch_v_part(vreq, preq, 0, tail, 0, kStages); fetch_v_part(vreq, preq, 0, tail, 1, kStages);
        if (nkt > 2) fetch_k(kreq + 2 * tile_bytes, 2, 2 == ragged_tile);
        if (nkt > 1) fetch_v_part(vreq, preq + kBN, 1, 1 == ragged_tile, 2);
    }
    bf16x8 qf[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
        qf[t] = *(const ESP_LDS bf16x8*)(uintptr_t)((lds_base + q_off + (bl & 31) * 256 + (((bl >> 5) ^ (bl & 15)) << 4)) ^ (t << 5));
    if (a.causal) {
        int wg_qmax = lds_qmm[1][0];
#pragma unroll
        for (int w = 1; w < kPfWaves; ++w) wg_qmax = max(wg_qmax, lds_qmm[1][w]);
        int last_vis = -1, fm = nkt, lw = -1;
        for (int base = 0; base < nkt; base += kBoundTiles) {
            if (base > 0) {
                wg_barrier();                                       // everyone has read the previous 512
                rest_of_bounds(base);
                wg_barrier();
            }
            const int cnt = min(kBoundTiles, nkt - base);
            for (int t0 = 0; t0 < cnt; t0 += 64) {
                const int2 mm = t0 + lane < cnt ? lds_mm[t0 + lane] : make_int2(INT_MAX, INT_MIN);   // past the last tile: hidden, needs no mask
                const uint64_t vis = __builtin_amdgcn_ballot_w64(mm.x <= wg_qmax);
                if (vis) last_vis = base + t0 + 63 - __builtin_clzll(vis);
                const uint64_t mk = __builtin_amdgcn_ballot_w64(mm.y > wave_qmin);
                if (mk && fm == nkt) fm = base + t0 + __builtin_ctzll(mk);
                const uint64_t vw = __builtin_amdgcn_ballot_w64(mm.x <= wave_qmax);
                if (vw) lw = base + t0 + 63 - __builtin_clzll(vw);
            }
        }
        n_vis = last_vis + 1;
        first_mask = fm;
        n_need = lw + 1;
        if (KEEP) n_vis = max(n_vis, own_hi);                       // every owned tile passes through LDS, seen or not
    }
    if (kTileRow * wave >= n_rows) n_need = 0;                           // a wavefront without rows: transfers and barriers only

    // ---- operand read offsets
    // K (A operand of S^T): row 32*kvb + qi, chunk 2t + hi -> four bases per lane, by the bits of t that the swizzle changes; the
    // rest are immediates
    uint32_t k_rd[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) k_rd[x] = lds_k0 + k_chunk(qi, 2 * x + hi);
    // V (A operand of O^T) by transposing reads: 16 lanes fetch a 4 (kv) x 16 (d) patch
    const int j16 = lane & 15, jq = j16 >> 2, dblk = (lane >> 4) & 1;
    uint32_t v_rd[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
        v_rd[db] = lds_v0 + (4 * hi + jq) * 256 + ((((db ^ jq) << 2) + 2 * dblk + ((j16 & 3) >> 1)) << 4) + (j16 & 1) * 8;

    floatx16 oacc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
    // softmax state.  The offset m_use subtracted from the scaled scores moves in whole steps (so every change
    // of it rescales by an exact power of two) and only when it has to: lim is the largest tile sum
    // accepted without a move, -1 while the row has not seen a key yet (m_use is then a stand-in 0).
    float m_use = 0.f, lim = -1.f;
    float lsum = 0.f;          // running sum of exp2 over this lane's half of the keys (for the log-sum-exp)
    float lcorr = 0.f;         // what rounding the probabilities to bf16 added to that sum, over the tiles that track it
    float psum = 0.f, psum_r = 0.f, p0 = 0.f, p1 = 0.f;

    floatx16 sbuf[2][2];       // S^T of two tiles in flight: [tile parity][kvb]
    union PFrag { uint32_t u[4]; bf16x8 v; };
    PFrag pf[2][2];            // P^T packed to bf16, one fragment per chunk of 16 keys: [kvb][t2]
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) pf[c >> 1][c & 1].u[e] = 0u;
    union VFrag { short4_t s[2]; bf16x8 v; };
    VFrag frk[2], frv[2];      // operand fragments, fetched two steps ahead of their use

    // K fragment i = (t, kvb) = (i / 2, i % 2) of the tile in K stage st; V^T fragment p = (kvb, t2, db) =
    // (p / 8, (p / 4) % 2, p % 4) of the tile at byte offset stage_off of the V stages
    auto read_k = [&](int slot, int st, int i) {
        const int t = i >> 1;
        frk[slot].v = *(const ESP_LDS bf16x8*)(uintptr_t)(k_rd[t & 3] + st * kKTileBytes + (i & 1) * k_row(32) + (t >> 2) * 128);
    };
    auto read_v = [&](int slot, uint32_t stage_off, int p) {
        const uint32_t vp = v_rd[p & 3] + stage_off + (32 * (p >> 3) + 16 * ((p >> 2) & 1)) * 256;
        frv[slot].s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ESP_LDS short4_t*)(uintptr_t)(vp));
        frv[slot].s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ESP_LDS short4_t*)(uintptr_t)(vp + 8 * 256));
    };

    // mask of a tile: key positions in lds_pos[st] against this lane's query position
    auto apply_mask = [&](floatx16 (&sc)[2], int st) {
#pragma unroll
        for (int kvb = 0; kvb < 2; ++kvb)
#pragma unroll
            for (int bb = 0; bb < 4; ++bb) {
                const int4 kp = *(const int4*)(&lds_pos[st][32 * kvb + 8 * bb + 4 * hi]);
                if (kp.x > my_qpos) sc[kvb][4 * bb + 0] = -INFINITY;
                if (kp.y > my_qpos) sc[kvb][4 * bb + 1] = -INFINITY;
                if (kp.z > my_qpos) sc[kvb][4 * bb + 2] = -INFINITY;
                if (kp.w > my_qpos) sc[kvb][4 * bb + 3] = -INFINITY;
            }
    };
    // largest score of this lane's query row in a tile, in exp2 units (-inf if every key is masked)
    auto row_max = [&](const floatx16 (&sc)[2]) {
        float tmax = sc[0][0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, sc[0][r]);
#pragma unroll
        for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sc[1][r]);
        return half_swap_max(tmax) * a.scale_log2;
    };

    // probabilities of score pair c (0..15) of the current tile, in two parts placed behind the two MFMAs of a
    // step: exp2 first, then the fp32 partial sum (of the unrounded values: the log-sum-exp has to be good to
    // 1e-4) and the bf16 pack.  O^T accumulates the ROUNDED probabilities, so O is best normalised by their sum:
    // then it is a convex combination of value rows whatever the rounding did, an error common to the weights
    // cancels, and a row that sees a single key returns that key's value row exactly.  Summing the packed values
    // too (one dot product with (1, 1) per pair) costs 4 % of the loop's issue slots, though, and matters only
    // where few keys carry a row: so `track` is set in the masked iterations around the diagonal (a row with
    // fewer than 64 keys has no other) and in the exact sweep, and a tile at which the offset moves (a late,
    // dominant key) is accounted for in close_tile.  The plain iterations sum the unrounded values only.
    auto pair_exp = [&](const floatx16 (&sc)[2], int c) {
        const int kvb = c >> 3, r = 2 * (c & 7);
        p0 = __builtin_amdgcn_exp2f(fmaf(sc[kvb][r], a.scale_log2, -m_use));
        p1 = __builtin_amdgcn_exp2f(fmaf(sc[kvb][r + 1], a.scale_log2, -m_use));
    };
    auto packed_sum = [](uint32_t pk, float acc) {            // acc + both bf16 halves of pk
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), __builtin_bit_cast(bf16x2, 0x3f803f80u), acc, false);
    };
    auto pair_sum_pack = [&](int c, bool track) {
        if (c == 0) psum = p0 + p1;
        else { psum += p0; psum += p1; }
        const uint32_t pk = pack_bf16(p0, p1);
        if (track) {
            psum_r = packed_sum(pk, c == 0 ? 0.f : psum_r);
            asm volatile("" :: "v"(psum_r));
        }
        asm volatile("" :: "v"(pk), "v"(psum));   // sum and pack here, not in a bunch further down
        pf[c >> 3][(c >> 2) & 1].u[c & 3] = pk;
    };

    // End of a tile in the pipelined sweep.  The probabilities were taken against the offset in use, without
    // looking at the scores first; that is exact as long as nothing left the range of fp32 / bf16, whatever their
    // size.  The tile sum tells: up to lim nothing needs doing (the common case: one compare); above it the
    // offset moves up to the tile's row maximum, and everything accumulated so far (the sum, O^T, and the last
    // chunk's P^T, which is multiplied only in the next iteration) is rescaled by the exact power of two.  A sum
    // that is not finite or beyond 2^100, or a first visible tile whose maximum is further than 2^64 from the
    // stand-in offset, means the optimistic pass cannot be trusted: the workgroup then redoes its rows with the
    // plain sweep below (`unsafe` is only ever set, never cleared).
    int32_t* lds_unsafe = (int32_t*)(smem + kLdsFlag);
    auto close_tile = [&](const floatx16 (&sc)[2], bool tracked) {
        lsum += psum;
        if (tracked) lcorr += psum_r - psum;
        if (__builtin_amdgcn_ballot_w64(!(psum <= lim)) != 0) {
            const float tm = row_max(sc);
            // A query row is held by two lanes (l and l | 32), each with the sum over its half of the tile's keys:
            // the decision must be the row's, or one half would go on with the old offset while the other one
            // moves.  Coded as a number so that a NaN sum counts too: 1 = above the limit, 3 = also out of range.
            const float mine = !(psum <= 0x1p100f) ? 3.f : !(psum <= lim) ? 1.f : 0.f;
            const float rows = half_swap_max(mine);
            const bool move = rows >= 1.f && tm != -INFINITY;        // a fresh row whose tile is all masked stays fresh
            const bool bad = move && (rows >= 3.f || (lim < 0.f && !(fabsf(tm) <= 64.f)));
            if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) *lds_unsafe = 1;
            if (!tracked) {
                // a tile whose rounded sum was not kept: its packed probabilities are all still in pf (the next
                // tile has not begun to overwrite them), so the sum is taken here; rows that stay where they are
                // have nothing dominant in this tile and go without
                float d = 0.f;
#pragma unroll
                for (int c = 0; c < 16; ++c) d = packed_sum(pf[c >> 3][(c >> 2) & 1].u[c & 3], d);
                if (move) lcorr += d - psum;
            }
            const float m_new = move ? m_use + ceilf(tm - m_use) : m_use;     // whole steps: alpha is a power of two
            const float alpha = __builtin_amdgcn_exp2f(m_use - m_new);        // 1 where nothing moves
            m_use = m_new;
            if (move) lim = kSumLimit;
            lsum *= alpha;
            lcorr *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t w = pf[1][1].u[e];
                pf[1][1].u[e] = pack_bf16(bf16_lo(w) * alpha, bf16_hi(w) * alpha);
            }
        }
    };

    const int mask_from = min(first_mask, tail_rows < kBN ? nkt - 1 : nkt);   // first tile this wavefront masks
    const char* k_next = kreq + 4 * tile_bytes;                       // K tile that iteration 0 fetches
    const char* v_next = vreq + 2 * tile_bytes;                       // V tile that iteration 0 fetches
    const int32_t* p_next = preq + 2 * kBN;

    // One tile per iteration, one workgroup barrier at its end; every wavefront runs the same uniform stream of
    // 16 steps, each with two MFMAs and one score pair:
    //   step m:  S^T MFMA m of tile j+1 (into sbuf[PAR^1]);  exp2 of pair m of tile j;
    //            O^T MFMA p = (m + 12) % 16;                 sum and pack of pair m
    // The O^T MFMAs trail the pairs by four steps, i.e. by one chunk of 16 keys: chunk c of tile j is multiplied
    // in steps 4c+4 .. 4c+7, and the last chunk in steps 0 .. 3 of iteration j+1 (after the loop for the last
    // tile).  With two wavefronts per SIMD, each issuing an instruction about every 6-8 cycles, this keeps an
    // MFMA (32 cycles) in front of every 5-6 other instructions of both wavefronts.
    // On entry: scores of tile j in sbuf[PAR]; frk = K fragments 0, 1 of tile j+1; frv = V^T fragments 12, 13
    // of tile j-1; pf[1][1] = last chunk of tile j-1 (zeros, and a zeroed V stage, when j = 0).
    // LDS stages: K(t), V(t) and the positions of tile t live in stage t % 4 (K(0): in a place of its own).  Iteration j reads K(j+1), the
    // first two fragments of K(j+2), V(j-1) (steps 0, 1) and V(j); it fetches K(j+4) over K(j), last read in
    // iteration j-1, and V(j+2) over V(j-2), last read in the first steps of iteration j-1: both before the
    // barrier that ended iteration j-1.  What a wavefront fetched in iteration j-1 has landed before the barrier
    // that ends its iteration j, and is first read in iteration j+1.
    // POOL, plain iterations: wavefront 6 fetches the slots of tile j+5 while j is below this (the sweep reaches that
    // tile, and it is a full one: see n_plain); no other wavefront does
    const int plain_slots = POOL && wave == 6 ? n_vis - 5 : INT_MIN;
    auto iteration = [&](auto st_c, auto par_c, auto plain_c, int j) {
        constexpr int ST = decltype(st_c)::value, PAR = decltype(par_c)::value;
        constexpr bool PLAIN = decltype(plain_c)::value != 0;
        constexpr int ST1 = (ST + 1) % kStages, ST2 = (ST + 2) % kStages, ST3 = (ST + 3) % kStages;
        floatx16 (&sc)[2] = sbuf[PAR];
        floatx16 (&sn)[2] = sbuf[PAR ^ 1];
        if (KEEP && !PLAIN && j < n_vis - 4) keep_tile(j, ST);
        if (!PLAIN && j >= mask_from) apply_mask(sc, ST);
        const bool do_k = PLAIN || j < n_vis - 4, do_v = PLAIN || j < n_vis - 2;
        const bool tail_k = !PLAIN && j + 4 == ragged_tile, tail_v = !PLAIN && j + 2 == ragged_tile;
        int32_t pslot0 = 0, pslot1 = 0;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int t = m >> 1, kvb = m & 1;
            // POOL: the slots of this step's transfer and of the operand's other one are read first, ahead of the step's fragment reads:
            // LDS answers in order, so a read placed next to the transfer would wait for those as well
            if constexpr (POOL) {
                if (m == 3 && do_k) { pslot0 = pool_slot(ST, 0); pslot1 = pool_slot(ST, 1); }
                if (m == 9 && do_v) { pslot0 = pool_slot(ST2, 0); pslot1 = pool_slot(ST2, 1); }
            }
            if (t == 0) {                                 // S^T of tile j+1 (after the last tile: stale data, unused)
                floatx16 zero;
#pragma unroll
                for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                sn[kvb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frk[m & 1].v, qf[t], zero, 0, 0, 0);
            } else {
                sn[kvb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frk[m & 1].v, qf[t], sn[kvb], 0, 0, 0);
            }
            pair_exp(sc, m);
            __builtin_amdgcn_sched_barrier(0);
            const int p = (m + 12) & 15;                  // O^T += V^T P^T, one chunk behind the pairs
            oacc[p & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frv[m & 1].v, pf[p >> 3][(p >> 2) & 1].v, oacc[p & 3], 0, 0, 0);
            // both fragments of step m+2; the K fragment last, so that the wait in front of its MFMA covers the
            // V^T fragment too (LDS reads return in order) and one wait per step is enough
            read_v(m & 1, (m < 2 ? ST3 : ST) * kTileBytes, (m + 14) & 15);
            read_k(m & 1, m + 2 < 16 ? ST1 : ST2, (m + 2) & 15);
            pair_sum_pack(m, !PLAIN);
            // the transfers of this iteration, spread out (a burst from all wavefronts at once backs up the memory
            // pipeline); the odd ones, wavefront 0's positions and wavefront 6's slots, go first, so that "all but the last four have landed"
            // is the same wait for every wavefront.  (Issued last instead, with a wait count per wavefront, they
            // would have a whole iteration more to land; measured, that is slower: 1.6 % on the 8K x 8K causal
            // shard, 6 % on a chunk against a 256K prefix.)
            if (m == 1) {
                if constexpr (POOL) {                   // over tile j+1's slots, last read in iteration j-1
                    if (PLAIN) { if (j < plain_slots) fetch_pool_slots_full(j + 5, ST1); }
                    else if (j + 5 < n_vis) fetch_pool_slots(j + 5, ST1);
                }
                if (KEEP && !PLAIN && do_k && j >= own_lo) fetch_slots(j + 4);
                if (do_v) fetch_v_part(v_next, p_next, ST2, tail_v, 2);
            }
            if constexpr (POOL) {
                if (do_k && (m == 3 || m == 6))
                    load_to_lds_b128_at(lds_wk, kLdsK + ST * kKTileBytes + 1024 * (m / 6), pool_at(m == 3 ? pk0 : pk1, m == 3 ? pslot0 : pslot1));
                if (do_v && (m == 9 || m == 12))
                    load_to_lds_b128_at(lds_w, kLdsV + ST2 * kTileBytes + 1024 * (m / 12), pool_at(pv, m == 9 ? pslot0 : pslot1));
            } else {
                if (do_k && (m == 3 || m == 6)) fetch_k_part(k_next, ST, tail_k, m / 6);
                if (do_v && (m == 9 || m == 12)) fetch_v_part(v_next, p_next, ST2, tail_v, m / 12);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        close_tile(sc, !PLAIN);
        k_next += tile_bytes; v_next += tile_bytes; p_next += kBN;
        // what iteration j-1 fetched must have landed; this iteration's own transfers may stay in flight
        if (do_k) wait_vm<4>();
        else if (do_v) wait_vm<2>();
        else wait_vm<0>();
        if (__builtin_expect(j + 1 == ragged_tile, 0)) { seal_tail(ST1); seal_slots(); }   // its positions landed with V(j+1), its slots before
        asm volatile("s_barrier" :: "v"(sn[0]), "v"(sn[1]), "v"(oacc[0]), "v"(oacc[1]), "v"(oacc[2]), "v"(oacc[3]),
                                    "v"(pf[1][1].v) : "memory");
    };

    // ---- prologue: S^T of tile 0 (POOL: once K(0) has landed with the rest of the second group); then, behind the barrier at which
    //      all wavefronts have read their Q rows, V(1) and K(3); first fragments
    auto first_scores = [&]() {
        if (n_need <= 0) return;
        auto read_k0 = [&](int slot, int i) {
            const int t = i >> 1;
            frk[slot].v = *(const ESP_LDS bf16x8*)(uintptr_t)(k_rd[t & 3] + (uint32_t)(kLdsK0 - kLdsK) + (i & 1) * k_row(32) + (t >> 2) * 128);
        };
        read_k0(0, 0);
        read_k0(1, 1);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int t = m >> 1, kvb = m & 1;
            if (t == 0) {
#pragma unroll
                for (int r = 0; r < 16; ++r) sbuf[0][kvb][r] = 0.f;
            }
            sbuf[0][kvb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frk[m & 1].v, qf[t], sbuf[0][kvb], 0, 0, 0);
            if (m + 2 < 16) read_k0(m & 1, m + 2);
        }
        // the offset starts at the exact row maximum of tile 0 wherever the row sees a key there (with ascending
        // positions: whenever it sees any key at all), so that the largest probability of a short row is exactly 1
        // and takes no bf16 rounding; rows still without a key keep the stand-in 0
        if (0 >= mask_from) apply_mask(sbuf[0], 0);
        const float tm0 = row_max(sbuf[0]);
        if (tm0 != -INFINITY) { m_use = tm0; lim = kSumLimit; }
    };
    if constexpr (!POOL) first_scores();
    // (POOL: the slots of tile 1 are read ahead of the barrier, since iteration 0 fetches those of tile 5 over them)
    int32_t v1_slot0 = 0, v1_slot1 = 0;
    if constexpr (POOL) { v1_slot0 = pool_slot(1, 0); v1_slot1 = pool_slot(1, 1); }
    wait_vm<0>();
    if (ragged_tile == 1) seal_tail(1);
    if (ragged_tile >= 0 && ragged_tile < 2) seal_slots();          // (in every other case before the iteration ahead of its own)
    wg_barrier();
    // what iterations 1 and 2 need (a sweep that is shorter does not wait for it)
    if (n_vis > 1) {
        if constexpr (POOL) {
            load_to_lds_b128_at(lds_w, kLdsV + kTileBytes, pool_at(pv, v1_slot0));
            load_to_lds_b128_at(lds_w, kLdsV + kTileBytes + 1024, pool_at(pv, v1_slot1));
        } else {
            fetch_v_part(vreq + tile_bytes, preq, 1, 1 == ragged_tile, 0);
            fetch_v_part(vreq + tile_bytes, preq, 1, 1 == ragged_tile, 1);
        }
    }
    if (n_vis > 3) fetch_k(kreq + 3 * tile_bytes, 3, 3 == ragged_tile);
    if constexpr (POOL) first_scores();
    if (n_need > 0) {
        read_k(0, 1, 0);                                            // (stale if there is no tile 1)
        read_k(1, 1, 1);
        read_v(0, 3 * kTileBytes, 12);                              // the zeroed stage: there is no tile -1
        read_v(1, 3 * kTileBytes, 13);
    }
    // the sweep: a loop with a single exit over groups of four tiles (the stage of a tile is a compile-time
    // constant), then the zero to three tiles left over
    //   1. "plain" iterations: every transfer is a full tile that exists and this wavefront masks nothing, so the
    //      stream has no conditional code at all (a wavefront may leave this part earlier than its neighbours:
    //      the barriers and transfers per iteration are the same in both kinds);
    //   2. general iterations for the rest, again in groups of four, then one by one.
    //      (an owner: also short of its first owned tile, unless that is one of the sweep's last four, which are
    //      stored after the sweep)
    //      (one tile earlier than its K tile asks for before a ragged last tile: POOL's plain iterations do not fetch that
    //      tile's slot list, and the calls on dense and on pool rows agree bit for bit)
    const int n_plain = max(0, min(min(min(min(n_vis - 4, n_need), mask_from), ragged_tile >= 0 ? nkt - 6 : INT_MAX),
                                   KEEP && own_lo < n_vis - 4 ? own_lo : INT_MAX)) & ~3;
    int j = 0;
    for (; j < n_plain; j += 4) {
        iteration(IC<0>{}, IC<0>{}, IC<1>{}, j);
        iteration(IC<1>{}, IC<1>{}, IC<1>{}, j + 1);
        iteration(IC<2>{}, IC<0>{}, IC<1>{}, j + 2);
        iteration(IC<3>{}, IC<1>{}, IC<1>{}, j + 3);
    }
    for (; j + 4 <= n_need; j += 4) {
        iteration(IC<0>{}, IC<0>{}, IC<0>{}, j);
        iteration(IC<1>{}, IC<1>{}, IC<0>{}, j + 1);
        iteration(IC<2>{}, IC<0>{}, IC<0>{}, j + 2);
        iteration(IC<3>{}, IC<1>{}, IC<0>{}, j + 3);
    }
    if (j < n_need) {
        iteration(IC<0>{}, IC<0>{}, IC<0>{}, j);
        if (j + 1 < n_need) {
            iteration(IC<1>{}, IC<1>{}, IC<0>{}, j + 1);
            if (j + 2 < n_need) iteration(IC<2>{}, IC<0>{}, IC<0>{}, j + 2);
        }
    }
    if (n_need > 0) {                                               // last chunk of this wavefront's last tile
        const uint32_t last_off = (uint32_t)((n_need - 1) & 3) * kTileBytes;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            oacc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frv[m & 1].v, pf[1][1].v, oacc[m], 0, 0, 0);
            if (m < 2) read_v(m & 1, last_off, 14 + m);
        }
    }
    //   3. tiles that only other wavefronts can see: no arithmetic, but the same transfers, waits and barrier as
    //      in every other iteration (stages computed at run time here)
    for (int jj = n_need; jj < n_vis; ++jj) {
        const bool do_k = jj < n_vis - 4, do_v = jj < n_vis - 2;
        const bool tail_k = jj + 4 == ragged_tile, tail_v = jj + 2 == ragged_tile;
        if (KEEP && jj < n_vis - 4) keep_tile(jj, jj & 3);
        if (do_k && jj >= own_lo) fetch_slots(jj + 4);
        if (POOL && jj + 5 < n_vis) fetch_pool_slots(jj + 5, (jj + 1) & 3);
        if (do_v) fetch_v_part(v_next, p_next, (jj + 2) & 3, tail_v, 2);
        if (do_k) { fetch_k_part(k_next, jj & 3, tail_k, 0); fetch_k_part(k_next, jj & 3, tail_k, 1); }
        if (do_v) { fetch_v_part(v_next, p_next, (jj + 2) & 3, tail_v, 0); fetch_v_part(v_next, p_next, (jj + 2) & 3, tail_v, 1); }
        k_next += tile_bytes; v_next += tile_bytes; p_next += kBN;
        if (do_k) wait_vm<4>();
        else if (do_v) wait_vm<2>();
        else wait_vm<0>();
        if (__builtin_expect(jj + 1 == ragged_tile, 0)) { seal_tail((jj + 1) & 3); seal_slots(); }
        asm volatile("s_barrier" ::: "memory");
    }

    // The last four tiles of the sweep are still in their stages, with nothing in flight any more: an owner stores
    // those it owns now (under a causal mask the tiles on its diagonal, i.e. all it owns), where no hand-counted
    // wait has to sit out the stores.
    if (KEEP) {
        for (int t = max(max(own_lo, n_vis - 4), 0); t < own_hi; ++t) keep_tile(t, t & 3);
    }

    // ---- the plain sweep, for a workgroup whose optimistic pass met scores outside its range: one tile at a
    //      time through stage 0, row maximum before the exponentials, nothing overlapped.  Slow and exact.
    float m_fin = m_use;
    wg_barrier();                                                   // everyone's flag write and last LDS reads are done
    // the draw of the next item: as late as possible, so that items go out in the order in which workgroups
    // really become free, and early enough for the answer to arrive while the results are written
    unsigned long long next_item = 0;
    if (claim_from && tid == 0) {
        // an index the compiler cannot see through: with a provably uniform address it rewrites the atomic into
        // its one-per-wavefront form, which needs the answer at once instead of after the epilogue
        int idx = 0;
        asm volatile("" : "+v"(idx));
        next_item = __hip_atomic_fetch_add(claim_from + idx, 1ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__builtin_amdgcn_readfirstlane(*lds_unsafe) != 0) {
        float m_ref = -INFINITY;
        lsum = 0.f;
        lcorr = 0.f;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
        for (int t = 0; t < n_vis; ++t) {
            wg_barrier();
            if constexpr (POOL) {
                fetch_pool_slots(t, 0);
                wait_vm<0>();
                wg_barrier();
            }
            fetch_k(kreq + (int64_t)t * tile_bytes, 0, t == ragged_tile);
            fetch_v(vreq + (int64_t)t * tile_bytes, preq + t * kBN, 0, t == ragged_tile);
            wait_vm<0>();
            if (t == ragged_tile) seal_tail(0);
            wg_barrier();
            floatx16 (&sc)[2] = sbuf[0];
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                const int tt = m >> 1, kvb = m & 1;
                if (tt == 0) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) sc[kvb][r] = 0.f;
                }
                read_k(0, 0, m);
                sc[kvb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frk[0].v, qf[tt], sc[kvb], 0, 0, 0);
            }
            apply_mask(sc, 0);
            const float m_new = fmaxf(m_ref, row_max(sc));
            const float alpha = (m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_ref - m_new);
            m_ref = m_new;
            lsum *= alpha;
            lcorr *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
            m_use = (m_ref == -INFINITY) ? 0.f : m_ref;             // nothing visible yet: exp2(-inf - 0) = 0
#pragma unroll
            for (int c = 0; c < 16; ++c) { pair_exp(sc, c); pair_sum_pack(c, true); }
            lsum += psum;
            lcorr += psum_r - psum;
#pragma unroll
            for (int p = 0; p < 16; ++p) {
                read_v(0, 0, p);
                oacc[p & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frv[0].v, pf[p >> 3][(p >> 2) & 1].v, oacc[p & 3], 0, 0, 0);
            }
        }
        m_fin = m_use;
        wg_barrier();                                               // the epilogue reuses the K stages
    }

    // ---- epilogue: normalise, write O (bf16) and LSE (natural log)
    const float ltot = half_swap_sum(lsum);
    const float ltot_r = half_swap_sum(lsum + lcorr);
    const float inv = ltot_r > 0.f ? 1.0f / ltot_r : 0.f;
    // -inf says that the row saw no key (a sum of 0, exactly), and a merge leaves the row out; a sum that is NaN has to show
    // (first, while no store is in flight that a wait for anything else would have to sit out)
    int el = lane, ew = wave;                                       // opaque: the addresses are worked out here, not before the sweep
    asm volatile("" : "+v"(el), "+s"(ew));
    const int my_i = kTileRow * ew + el, e_qi = el & 31, e_hi = el >> 5;
    if (el < 32 && my_i < n_rows)
        *(float*)((char*)(a.LSE + row0 + row_of(my_i)) + part * a.lse_part) = ltot != 0.f ? (m_fin + __builtin_amdgcn_logf(ltot)) * kLn2 : -INFINITY;
    // O goes through LDS so that it leaves in whole rows: a lane holds 8-byte pieces of one row, 16 of them spread
    // over the 256 bytes; written to a wavefront-private 32 x 272-byte block (the K stages are free by now: the
    // barrier above ended all tile reads) they come back as 16 lanes x 16 bytes per row, four rows per store.
    // rows of this wavefront that exist (may be <= 0); a part of a split call in which none of them sees a key leaves O
    // unwritten: its LSE, -inf, keeps it out of the merge
    const int rows_here = cut && n_need == 0 ? 0 : min(32, n_rows - kTileRow * ew);
    char* const O_part = (char*)a.O + part * a.o_part;
    if (!a.o_f32) {
        unsigned char* blk = smem + kLdsK + ew * (32 * kORow);
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int bb = 0; bb < 4; ++bb) {
                uint2 w;
                w.x = pack_bf16(oacc[db][4 * bb + 0] * inv, oacc[db][4 * bb + 1] * inv);
                w.y = pack_bf16(oacc[db][4 * bb + 2] * inv, oacc[db][4 * bb + 3] * inv);
                *(uint2*)(blk + e_qi * kORow + (32 * db + 8 * bb + 4 * e_hi) * 2) = w;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // same wavefront wrote what it reads next
        const int rsub = el >> 4, c16 = el & 15;
        uint16_t* orow = (uint16_t*)O_part + (int64_t)(ONE ? row0 + row_of(kTileRow * ew + rsub) : row0) * kHeadDim + 8 * c16;
        auto out = [&](int i) { return (uint4*)(orow + (int64_t)(ONE ? row_of(4 * i) : row_of(kTileRow * ew + 4 * i + rsub)) * kHeadDim); };
        if (rows_here >= 32) {                                      // all rows exist: eight stores in a row, no branches
            uint4 w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = *(const uint4*)(blk + (4 * i + rsub) * kORow + 16 * c16);
#pragma unroll
            for (int i = 0; i < 8; ++i) *out(i) = w[i];
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r = 4 * i + rsub;
                const uint4 w = *(const uint4*)(blk + r * kORow + 16 * c16);
                if (r < rows_here) *out(i) = w;
            }
        }
    } else {
        // fp32 output (a partial that stays on this GPU until the merge): rows of 512 bytes, padded to 528 in LDS;
        // the eight blocks of 32 rows fill the V and K stages exactly.  Two rows per store, 16 stores.
        constexpr int kFRow = 4 * kHeadDim + 16;
        static_assert(kPfWaves * 32 * kFRow <= kStages * (kTileBytes + kKTileBytes), "fp32 output staging must fit the tile stages");
        unsigned char* blk = smem + kLdsV + ew * (32 * kFRow);
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int bb = 0; bb < 4; ++bb)
                *(float4*)(blk + e_qi * kFRow + (32 * db + 8 * bb + 4 * e_hi) * 4) =
                    make_float4(oacc[db][4 * bb + 0] * inv, oacc[db][4 * bb + 1] * inv, oacc[db][4 * bb + 2] * inv, oacc[db][4 * bb + 3] * inv);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int rsub = el >> 5, c32 = el & 31;
        float* orow = (float*)O_part + (int64_t)(ONE ? row0 + row_of(kTileRow * ew + rsub) : row0) * kHeadDim + 4 * c32;
        auto out = [&](int i) { return (uint4*)(orow + (int64_t)(ONE ? row_of(2 * i) : row_of(kTileRow * ew + 2 * i + rsub)) * kHeadDim); };
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint4 w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = *(const uint4*)(blk + (2 * (8 * half + i) + rsub) * kFRow + 16 * c32);
            if (rows_here >= 32) {
#pragma unroll
                for (int i = 0; i < 8; ++i) *out(8 * half + i) = w[i];
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (2 * (8 * half + i) + rsub < rows_here) *out(8 * half + i) = w[i];
            }
        }
    }
    if (claim_from && tid == 0) *lds_next = draw_finish(claim_from, next_item);
    return true;
    };
    if constexpr (RETAIN) {
        if (own_hi > own_lo) return body(IC<1>{});
    }
    return body(IC<0>{});
    };

    // ---- persistent workgroups, one per CU.  Consecutive workgroup ids land on consecutive XCDs, each with a
    //      private L2, so XCD x keeps the KV heads (times parts) [x * per, (x + 1) * per):
    //      a queue of M items, heaviest first (later query tiles of a causal request see more keys), or where their
    //      sizes differ less (by_head) one head after the other, so that the workgroups share a head's K/V in the L2.  All but the
    //      last one or two rounds of a queue are dealt to the XCD's L workgroups back and forth (0 .. L-1,
    //      L-1 .. 0, ...), which for the linear size profile of a causal sweep gives every workgroup the same
    //      total.  XCDs do not run at quite the same speed, though, so the light items at the end of all queues
    //      form one pool that every workgroup draws from, through a device-wide counter, as it becomes free:
    //      a faster XCD takes more of them, and a workgroup whose dealt items were lighter a heavier one.  Pool
    //      items mostly miss their XCD's L2, but they are few and small.  Without the XCD split (head count not
    //      a multiple of 8) the same scheme runs with one queue over all workgroups.
    {
        const int P = gridDim.x, p = blockIdx.x;
        const bool split = a.heads_per_xcd > 0;
        const int L = split ? P >> 3 : P, l = split ? p >> 3 : p, x = split ? p & 7 : 0;
        const int width = split ? a.heads_per_xcd : a.Hkv * a.splits;
        const int M = a.q_tiles * width;
        // Rounds dealt statically (M <= L: one item each).  With start-of-round waits the items are long and alike: a pool of them does not
        // even out the workgroups of an XCD, and its items walk K/V alone (of two to four rounds the last drawn from the pool: 0.3 .. 1 %
        // slower).  But XCDs differ by 7 % and more, and from eight rounds on that is an item's time or near it: then the pool has the last
        // full round all the same, and what there is of a next one (L .. 2 L - 1 items).  All dealt -> these drawn, two cards: 32768 tokens on
        // 262144, 32 / 32 heads, 106.5 -> 104.7 and 112.1 -> 105.5 ms, 16384 on 180000 37.0 -> 35.5, 10000 on 90000, 64 / 8 (57 items of 32
        // workgroups), 21.3 -> 21.1; one more round drawn 105.8 and 21.1.
        const int S = M <= L ? 1 : a.group_sync && M < 8 * L ? (M + L - 1) / L : max(1, (M - L) / L);
        const int synced = min(S, M / L);                             // dealt rounds that are full: all but the first start together
        const int pool_items = M > S * L ? (M - S * L) * (split ? 8 : 1) : 0;
        // One workgroup starts this launch's count of the pool while the others are at their first items (a single round trip: the
        // last draw of the launch before left a 0).  Without that the first draws start it themselves, and where many items end
        // at about the same time their failing compare-and-swaps held everyone up: 333, 444, 1111 and 95 tokens against two
        // shards, 32 / 8 heads (264 items, 256 workgroups), 207 -> 88 us, the rows kept 263 -> 105; four of 512 122 -> 67; six
        // prompts of 37 .. 2047 against one 69.8 -> 66.4 us.
        if (pool_items > 0 && p == P - 1 && tid == 0) {
            for (unsigned long long cur = 0; (uint32_t)(cur >> 32) != a.tag;)
                if (__hip_atomic_compare_exchange_strong(a.pool, &cur, (unsigned long long)a.tag << 32, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
        }
        int i_pool = 0;
        bool drew = false;
        long long item_started = 0;
        for (int s = 0;; ++s) {
            // Long requests: the workgroups of an XCD walk K/V of one head together (by_head), and the L2 serves all but
            // the first of them, as long as they stay within the 128 or so tiles it can hold.  Their items differ in
            // length, so they would start the next round up to that far apart, and since all run at the same speed
            // the gap never closes: K/V then comes from memory several times over.  So they wait for each other at
            // the start of a dealt round: an arrival count per XCD, tagged like the pool counter, and a wait that ends by
            // itself: after 1/64 of the time this workgroup's previous item took (waiting pays only where the items are
            // long and alike; where they differ a lot, as in a triangular sweep, it must cost next to nothing), at
            // most after kSyncTicks.  Every workgroup arrives at every waiting round whether its wait is cut short or
            // not, so the total a count reaches is known beforehand, and the arrival that completes it clears the count (a
            // launch replayed from a captured graph carries the tag it was recorded with and must not find its own
            // earlier counts).
            if (a.group_sync && s >= 1 && s < synced && tid == 0) {
                unsigned long long* ctr = a.pool + 2 + x;
                const uint32_t target = (uint32_t)(L * s), total = (uint32_t)(L * (synced - 1));   // rounds up to this one; all that wait
                const int before_me = draw_finish(ctr, __hip_atomic_fetch_add(ctr, 1ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                if ((uint32_t)before_me + 1 == total) {
                    __hip_atomic_store(ctr, 0ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else if ((uint32_t)before_me + 1 < target) {
                    const long long t0 = wall_clock64();
                    const long long patience = min((long long)a.sync_ticks, (t0 - item_started) >> 6);
                    for (;;) {
                        const unsigned long long cur = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        // a count that is no longer this launch's was cleared by its last arrival (see above)
                        if ((uint32_t)(cur >> 32) != a.tag || (uint32_t)cur >= target) break;
                        if (wall_clock64() - t0 > patience) break;
                        __builtin_amdgcn_s_sleep(16);
                    }
                }
            }
            if (s > 0) wg_barrier();                                  // every wavefront is done with the LDS of the previous item
            if (drew) i_pool = __builtin_amdgcn_readfirstlane(*lds_next);
            // every workgroup draws once per item from its last dealt one on, until a draw comes back empty: P draws
            // plus one per pool item.  The very last one clears the counter (replayed launches, see above).
            if (drew && i_pool == pool_items + P - 1 && tid == 0)
                __hip_atomic_store(a.pool, 0ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int qu, m;
            if (s < S) {
                qu = x;
                m = s * L + ((s & 1) ? L - 1 - l : l);
            } else {
                if (i_pool >= pool_items) break;
                qu = split ? i_pool & 7 : 0;                          // the queues take turns: still heaviest first
                m = S * L + (split ? i_pool >> 3 : i_pool);
            }
            if (m >= M) break;                                        // a last dealt round that is not full
            unsigned long long* claim = (s >= S - 1 && pool_items > 0) ? a.pool : nullptr;
            if (a.group_sync) item_started = wall_clock64();
            const int run = a.by_head ? a.q_tiles : width, major = m / run, minor = m - major * run;
            const bool ran = process(a.by_head ? minor : major, qu * width + (a.by_head ? major : minor), claim);
            drew = claim != nullptr;
            if (drew && !ran) {                                       // no such query tile: it drew nothing
                wg_barrier();                                         // everyone has read the previous answer
                if (tid == 0)
                    *lds_next = draw_finish(claim, __hip_atomic_fetch_add(claim, 1ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
        }
    }
}

static esp_status merge_parts(const PrefillArgs& a, void* O, float* LSE, int32_t o_f32, hipStream_t stream) {
    MergeArgs parts = {};
    for (int32_t p = 0; p < a.splits; ++p) {
        parts.O_parts[p] = (const char*)a.O + p * a.o_part;
        parts.LSE_parts[p] = (const float*)((const char*)a.LSE + p * a.lse_part);
    }
    return launch_merge(parts, a.splits, (int64_t)a.Tq * a.Hq, 1, O, LSE, stream, o_f32);
}

esp_status launch_prefill(const void* q, const void* k, const void* v, const int32_t* q_pos, const int32_t* kv_pos,
                          const int32_t* cu_q, const int32_t* cu_kv, int32_t batch, int32_t Tq, int32_t Tkv,
                          int32_t max_kv, int32_t Hq, int32_t Hkv, float softmax_scale,
                          int32_t causal, int32_t o_f32, void* O, float* LSE, void* workspace, size_t workspace_bytes,
                          const int32_t* retain_slot, void* k_pool, void* v_pool, const int32_t* kv_slot,
                          hipStream_t stream) {
    PrefillArgs a;
    a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v;
    a.q_pos = q_pos; a.kv_pos = kv_pos; a.cu_q = cu_q; a.cu_kv = cu_kv;
    const size_t counters = kPrefillCounterBytes;
    const PrefillKind kind = {causal != 0, retain_slot != nullptr};
    const PrefillPlan plan = prefill_plan_in(workspace_bytes, Tq, Tkv, batch, max_kv, Hq, Hkv, kind);
    const int32_t S = plan.splits;
    a.splits = S;
    if (S > 1) {
        a.O = (char*)workspace + counters;
        a.LSE = (float*)((char*)workspace + counters + S * split_o_bytes(Tq, Hq));
        a.o_f32 = 1;
        a.o_part = (int64_t)split_o_bytes(Tq, Hq);
        a.lse_part = (int64_t)split_lse_bytes(Tq, Hq);
    } else {
        a.O = O; a.LSE = LSE; a.o_f32 = o_f32 ? 1 : 0;
        a.o_part = a.lse_part = 0;
    }
    a.kv_slot = kv_slot;
    a.retain_slot = retain_slot; a.k_pool = (uint16_t*)k_pool; a.v_pool = (uint16_t*)v_pool;
    a.batch = batch; a.Tq = Tq; a.Tkv = Tkv; a.Hq = Hq; a.Hkv = Hkv; a.causal = causal ? 1 : 0;
    a.scale_log2 = softmax_scale * kLog2e;
    a.G = Hq / Hkv;
    a.inv_G = 1.0f / (float)a.G;
    a.q_odd = ((uintptr_t)q & 15) != 0;
    if (kv_slot && retain_slot) return fail(ESP_ERR_INVALID_ARG, "prefill: rows that are read from the pool are in it already");
    if (plan.use_short) {
        const esp_status st = launch_prefill_short(a, stream);
        return st != ESP_OK || S == 1 ? st : merge_parts(a, O, LSE, o_f32, stream);
    }
    a.q_tiles = prefill_q_tiles_bound(Tq, a.G, batch);
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return fail(ESP_ERR_HIP, "prefill: cannot query the device");
    const int32_t vheads = Hkv * S;
    const int64_t items = (int64_t)a.q_tiles * vheads;
    // one workgroup per CU (a workgroup fills a CU's registers and LDS); fewer if there are fewer items
    a.heads_per_xcd = (vheads % 8 == 0 && cus % 8 == 0 && items >= cus) ? vheads / 8 : 0;
    const unsigned grid = (unsigned)(items < cus ? items : cus);
    a.pool = (unsigned long long*)workspace;
    a.tag = next_launch_tag();
    // Order of the items: head by head where the query tiles of a head do not differ much (the shard reaches at least a
    // quarter of the chunk's length before the chunk), so that all workgroups of an XCD walk one head's K/V at a time and a
    // head comes through the L2 once per (workgroups / query tiles); by query tile, heaviest first, where the sweeps
    // are a triangle: there the light items have to come last.  Measured in turn, by query tile -> by head, 32 / 32 heads: 1488
    // rows on 210407 4.84 -> 4.24 ms, 32768 on 262144 105.4 -> 103.9 ms, 8 / 8 heads, 5999 on 8578 159 -> 151 us, 32 / 8, 4096 on
    // 65536 the same; against it 8192 on 8192: 1.934 -> 1.965 ms for four shards.  Without the XCD split consecutive items sit on different XCDs and
    // "by head" would spread a head over all of them (300 on 20300 rows, 32 / 8 heads: 114 -> 117 us).
    a.by_head = a.heads_per_xcd > 0 && batch == 1 && 4 * (int64_t)Tkv >= 5 * (int64_t)Tq;
    // start-of-round waits: one request with at least 512 KV tiles and a query chunk of at most an eighth of them
    // (a chunk against a long prefix: every query tile then sees nearly all of the shard, the items are alike)
    a.group_sync = a.by_head && S == 1 && Tkv >= 512 * kBN && (int64_t)Tkv >= 8 * (int64_t)Tq;
    const bool paired = prefill_paired(kind, prefill_rounds(Tq, batch, Hq, Hkv), S);
    a.sync_ticks = g_sync_ticks.load(std::memory_order_relaxed);
#define ESP_PREFILL_LAUNCH(...) hipLaunchKernelGGL((prefill_kernel<__VA_ARGS__>), dim3(grid), dim3(kPfWaves * 64), 0, stream, a)
    const bool one = a.G == 1 && batch == 1 && S == 1;
    if (kv_slot && paired) ESP_PREFILL_LAUNCH(2, false, true);
    else if (kv_slot) ESP_PREFILL_LAUNCH(2, false, false);
    else if (retain_slot && a.q_odd) ESP_PREFILL_LAUNCH(3, false, false);
    else if (retain_slot) ESP_PREFILL_LAUNCH(1, false, false);
    else if (one && paired) ESP_PREFILL_LAUNCH(0, true, true);
    else if (one) ESP_PREFILL_LAUNCH(0, true, false);
    else if (paired) ESP_PREFILL_LAUNCH(0, false, true);
    else ESP_PREFILL_LAUNCH(0, false, false);
#undef ESP_PREFILL_LAUNCH
    const esp_status st = check_launch("prefill_kernel");
    if (st != ESP_OK || S == 1) return st;
    return merge_parts(a, O, LSE, o_f32, stream);
}

}  // namespace esp
