// Prefill partial attention for calls with few query rows: a small chunk, a follow-up turn, short prompts, few heads.  The main
// kernel (prefill.hip) gives a workgroup 256 packed rows of a KV head and lets all its wavefronts walk the keys together: such a
// call has a handful of items, each a serial walk (set-up 7 us, 1.5 us per 64 keys whatever it holds), and leaves the chip idle.
// What bounds it is that chain, so here the chain is cut: a workgroup has 32 packed rows (the columns of one MFMA tile), its
// eight wavefronts take the tiles of 32 keys in turn, each alone, with an LDS block of its own and no barrier until the end,
// and combine their results through LDS (column_tile.h).  A row block re-reads all of its K and V from the L2, eight times as often
// as there, and a row costs several times as much: the launcher picks by an estimate of both times (prefill.hip).
// A wavefront's own chain is two round trips before its first product (the request's bounds; everything else; with pool rows a third, as
// their slots have to be there first) and one for each tile that follows, which starts as soon as the block that it lands in has
// been read.  Measured (positions, then queries and rows, each tile's rows asked for when the one before is done -> this; kernel alone):
// 256 on 512, 4 / 4 heads, 9.9 -> 8.3 us, 16 on 2016 rows of the pool, 32 / 8, 9.5 -> 8.3, 64 on 576 11.7 -> 9.9, 64 kept 8.4 -> 7.7, a
// single tile (27 on 27) 5.7 -> 5.8; calls: 130 on 3130, 32 / 8, 26.8 -> 23.5, 200 on 5200, 16 / 16, 28.4 -> 25.7, 17 on 517, 40 / 8, 9.7
// -> 8.4, 31 on 70195, 4 / 4, 63.2 -> 59.8.  The next tile's rows in registers while this one is in LDS (64 of them, 228 in all) was slower
// everywhere, 27 on 27 5.6 -> 6.8, 300 on 20300 280 -> 298 us.
#include <limits.h>
#include <math.h>

#include "column_tile.h"
#include "prefill.h"

namespace esp {

// MODE as for the main kernel: 0 dense rows, 1 (KEEP) dense rows that are also kept in the token pool, 2 (POOL) rows of the pool.  To be kept,
// tile t of a request and KV head is stored by row block t % (row blocks of the request), from LDS, after its products, also where no
// row sees it; a request without query rows has one block without rows for that.
template <int MODE>
__global__ __launch_bounds__(kShortWaves * 64, 2) void prefill_short_kernel(PrefillArgs a) {
    constexpr bool KEEP = MODE == 1, POOL = MODE == 2;
    constexpr int kListStages = 4;
    constexpr int kQAt = kShortWaves * kColWaveBytes, kListAt = kQAt + kShortRows * kHeadDim * 2, kQPosAt = kListAt + kShortWaves * kListStages * 256;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kQPosAt + kShortWaves * 256];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qi = lane & 31, hi = lane >> 5;
    // the row blocks of a (KV head, part) lie heads x parts workgroups apart: on one XCD where that is a multiple of 8
    const uint32_t vheads = a.Hkv * a.splits, block = blockIdx.x / vheads, vhead = blockIdx.x - block * vheads;
    const int kvh = a.splits == 1 ? vhead : vhead / (uint32_t)a.splits, part = vhead - kvh * a.splits;
    const int G = a.G;

    // ---- the request and the row block in it: requests are looked at 64 at a time, one per lane
    auto blocks_of = [&](int r) {
        const int n = ((a.cu_q ? a.cu_q[r + 1] - a.cu_q[r] : a.Tq) * G + kShortRows - 1) / kShortRows;
        return KEEP && n == 0 && a.cu_kv && a.cu_kv[r + 1] > a.cu_kv[r] ? 1 : n;
    };
    int r = 0, blk = block;
    if (a.batch > 1) {
        bool found = false;
        for (int base = 0; base < a.batch; base += 64) {
            const int n = base + lane < a.batch ? blocks_of(base + lane) : 0;
            int upto = n;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int below = __shfl_up(upto, d);
                if (lane >= d) upto += below;
            }
            const uint64_t hit = __builtin_amdgcn_ballot_w64(upto > blk);
            if (hit) {
                const int l = __builtin_ctzll(hit);
                r = base + l;
                blk -= __builtin_amdgcn_readlane(upto, l) - __builtin_amdgcn_readlane(n, l);
                found = true;
                break;
            }
            blk -= __builtin_amdgcn_readlane(upto, 63);
        }
        if (!found) return;                                         // the grid is an upper bound
    }
    const int qs = a.cu_q ? a.cu_q[r] : 0, qe = a.cu_q ? a.cu_q[r + 1] : a.Tq;
    const int rho = blk * kShortRows;
    const int n_rows = min(kShortRows, (qe - qs) * G - rho);
    const bool any_row = n_rows > 0;
    if (!KEEP && !any_row) return;
    int kv_lo = a.cu_kv ? a.cu_kv[r] : 0;
    const int kv_end = a.cu_kv ? a.cu_kv[r + 1] : a.Tkv;
    const int all_tiles = (kv_end - kv_lo + 31) / 32;
    int t_lo = 0, t_hi = all_tiles;
    if (a.splits > 1) {                                             // (32 bits: at most 2^26 tiles and 16 parts)
        t_lo = (uint32_t)(all_tiles * part) / (uint32_t)a.splits;
        t_hi = (uint32_t)(all_tiles * (part + 1)) / (uint32_t)a.splits;
    }
    const int kv_len = min(kv_end - kv_lo, t_hi * 32) - t_lo * 32;  // this part's rows (may be none)
    kv_lo += t_lo * 32;
    const int tiles = (kv_len + 31) / 32;

    // ---- row i of the block: token and query head of the group (rows past the end repeat the last)
    const int tok0 = qs + (int)((uint32_t)rho / (uint32_t)G), g0 = (uint32_t)rho % (uint32_t)G, row0 = tok0 * a.Hq + kvh * G + g0;
    auto row_of = [&](int i, int& tok) {
        const int j = min(i, n_rows - 1), t = (int)(((float)(j + g0) + 0.5f) * a.inv_G);   // (exact: j + g0 is far below 2^21)
        tok = tok0 + t;
        return row0 + j + t * (a.Hq - G);
    };
    const uint32_t row_bytes = (uint32_t)a.Hkv * (kHeadDim * 2);
    const char* kbase = (const char*)a.k + (uint32_t)kvh * (kHeadDim * 2);
    const char* vbase = (const char*)a.v + (uint32_t)kvh * (kHeadDim * 2);
    const uint32_t lds = (uint32_t)(uintptr_t)(ESP_LDS unsigned char*)smem;
    const uint32_t lds_k = lds + wave * kColWaveBytes, lds_v = lds_k + kColKBytes;

    // ---- everything that the first tile needs is asked for at once, by transfers whose waits are counted by hand: queries, positions,
    //      lists and, of dense rows, the rows, seen or not (they exist).  Taken one after the other, positions, then queries and rows,
    //      these were two round trips; and queries fetched by every wavefront as fragments, 16-byte pieces of 32 rows, took as
    //      long as a tile.
    // Lists of a tile: lane L holds the position of tile row L % 32, or in the upper half (KEEP, POOL) its pool slot; rows past the end
    // repeat the last.  They lie in a ring of four stages.
    const int32_t* my_list = a.causal ? a.kv_pos + kv_lo : POOL ? a.kv_slot + kv_lo : (const int32_t*)a.k;
    if (KEEP && hi) my_list = a.retain_slot + kv_lo;
    if (POOL && hi) my_list = a.kv_slot + kv_lo;
    const uint32_t lds_list = lds + kListAt + wave * (kListStages * 256);
    auto fetch_list = [&](int i, int st) { load_to_lds_b32_at(lds_list + st * 256, my_list + min(32 * i + qi, kv_len - 1)); };
    auto list = [&](int st) { return (int32_t*)(smem + kListAt + (wave * kListStages + st) * 256); };
    const uint32_t row_at = (lane >> 4) * row_bytes;
    auto fetch = [&](uint32_t to, const char* base, int i, int st, bool is_k) {
        const uint32_t last = min(32, kv_len - 32 * i) - 1;
        const char* tile = base + (int64_t)(kv_lo + 32 * i) * row_bytes;
        if constexpr (POOL) {
            int32_t slot[8];
#pragma unroll
            for (int n = 0; n < 8; ++n) slot[n] = list(st)[32 + col_row(n, lane)];
#pragma unroll
            for (int n = 0; n < 8; ++n)
                load_to_lds_b128_at(to + 1024 * n, base + ((uint64_t)(uint32_t)slot[n] * row_bytes + (is_k ? col_k_within(n, lane) : col_v_within(lane))));
        } else {
#pragma unroll
            for (int n = 0; n < 8; ++n)
                load_to_lds_b128(to + 1024 * n, tile, min(row_at + 4 * n * row_bytes, last * row_bytes) + (is_k ? col_k_within(n, lane) : col_v_within(lane)));
        }
    };
    if (wave < tiles) {
        fetch_list(wave, 0);
        fetch_list(wave + kShortWaves, 1);
        if constexpr (!POOL) fetch(lds_k, kbase, wave, 0, true);
    }
    int tok = 0, row = 0;                                           // this lane's (column of S^T)
    if (any_row) row = row_of(qi, tok);
    if (a.causal) load_to_lds_b32_at(lds + kQPosAt + wave * 256, a.q_pos + tok);
    {
        int t;
        const int r4 = 4 * wave + (lane >> 4), at = any_row ? row_of(r4, t) : 0;
        const char* src = (const char*)a.q + (int64_t)at * (kHeadDim * 2) + (((lane ^ r4) & 15) << 4);
        struct __attribute__((packed, aligned(2))) Any16 { uint32_t x, y, z, w; };
        if (__builtin_expect(a.q_odd, 0)) *(ESP_LDS u32x4*)(uintptr_t)(lds + kQAt + 1024 * wave + 16 * lane) = __builtin_bit_cast(u32x4, *(const Any16*)src);
        else load_to_lds_b128_at(lds + kQAt + 1024 * wave, src);
    }
    if (!POOL && wave < tiles) {
        fetch(lds_v, vbase, wave, 0, false);
        wait_vm<8>();
    } else {
        wait_vm<0>();
    }
    const int my_qpos = a.causal ? ((const int32_t*)(smem + kQPosAt))[wave * 64 + lane] : INT_MAX - 1;   // non-causal rows see every key that exists

    Columns cols;
    cols.place(lds_k, lane);
    cols.clear();

    auto least = [](int x, int y) { return min(x, y); };
    auto most = [](int x, int y) { return max(x, y); };
    auto of_rows = [](int x, auto op) {                             // over the 32 rows: rotations within 16 lanes, then two of those
        x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false));
        x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, false));
        x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x122, 0xf, 0xf, false));
        x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x121, 0xf, 0xf, false));
        return op(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16));
    };
    const int q_min = of_rows(my_qpos, least), q_max = of_rows(my_qpos, most);
    const int n_blk = KEEP ? blocks_of(r) : 1;
    // position of tile row lane % 32; of rows past the end one that nobody sees
    auto tile_pos = [&](int i, int st) { return 32 * i + qi >= kv_len ? INT_MAX : a.causal ? list(st)[qi] : 0; };
    // (a key may sit at the lowest position there is: a block without rows sees nothing all the same)
    auto is_seen = [&](int pos) { return any_row && of_rows(pos, least) <= q_max; };
    auto is_owned = [&](int i) { return KEEP && (t_lo + i) % n_blk == blk; };

    int pos = INT_MAX;
    bool seen = false, owned = false;
    if (wave < tiles) { pos = tile_pos(wave, 0); seen = is_seen(pos); owned = is_owned(wave); }
    if constexpr (POOL) {
        if (seen) { fetch(lds_k, kbase, wave, 0, true); fetch(lds_v, vbase, wave, 0, false); }
    }
    wg_barrier();                                                   // all queries are there
    bf16x8 qf[8];
    const uint32_t q_rd = lds + kQAt + qi * 256 + ((hi ^ (qi & 15)) << 4);
#pragma unroll
    for (int t = 0; t < 8; ++t) qf[t] = *(const ESP_LDS bf16x8*)(uintptr_t)(q_rd ^ (t << 5));

    int st = 0;
    for (int i = wave; i < tiles; i += kShortWaves, st = (st + 1) % kListStages) {
        // Here the rows of tile i are on their way where it is seen or owned, V last; the lists of the next tile before them.
        const int next = i + kShortWaves, st1 = (st + 1) % kListStages, st2 = (st + 2) % kListStages;
        const bool has_next = next < tiles;
        if (seen || owned) wait_vm<8>(); else wait_vm<0>();
        const int pos_next = has_next ? tile_pos(next, st1) : INT_MAX;
        const bool seen_next = has_next && is_seen(pos_next), owned_next = has_next && is_owned(next), wanted_next = seen_next || owned_next;
        // The next tile's K follows as soon as the scores are taken, its V as soon as this tile's has been read; not past an owned tile,
        // whose rows leave after its products, and whose stores the waits would count.
        const bool ahead = !KEEP || !owned;
        floatx16 sc;
        if (seen) sc = cols.scores(qf);
        if (ahead && has_next) {
            if (seen) asm volatile("" :: "v"(sc));                  // K has been read
            fetch_list(next + kShortWaves, st2);
            if (wanted_next) fetch(lds_k, kbase, next, st1, true);
        }
        if (seen) {
            if (of_rows(pos, most) > q_min) {
                int32_t* const lds_pos = list(st);
                if (32 * i + 32 > kv_len && lane < 32) lds_pos[lane] = pos;   // the ragged last tile: positions past the end
#pragma unroll
                for (int bb = 0; bb < 4; ++bb) {
                    const int4 kp = *(const int4*)(lds_pos + 8 * bb + 4 * hi);
                    if (kp.x > my_qpos) sc[4 * bb + 0] = -INFINITY;
                    if (kp.y > my_qpos) sc[4 * bb + 1] = -INFINITY;
                    if (kp.z > my_qpos) sc[4 * bb + 2] = -INFINITY;
                    if (kp.w > my_qpos) sc[4 * bb + 3] = -INFINITY;
                }
            }
            Columns::PFrag pf[2];
            cols.weigh(sc, a.scale_log2, pf);
            if (ahead && wanted_next) wait_vm<9>(); else wait_vm<0>();
            cols.accumulate(pf);
        }
        if (owned) {
            if (!seen) wait_vm<0>();
            // what this wavefront fetched, to the rows' slots (lane L of transfer n: the 16 bytes it brought)
            auto keep = [&](char* pool, int lds_at, int n, int within) {
                const int32_t slot = 32 * i + col_row(n, lane) < kv_len ? list(st)[32 + col_row(n, lane)] : -1;
                const uint4 w = *(const uint4*)(smem + wave * kColWaveBytes + lds_at + 16 * lane);
                if (slot >= 0) *(uint4*)(pool + (uint32_t)kvh * (kHeadDim * 2) + ((uint64_t)(uint32_t)slot * row_bytes + within)) = w;
            };
#pragma unroll
            for (int n = 0; n < 8; ++n) keep((char*)a.k_pool, 1024 * n, n, col_k_within(n, lane));
#pragma unroll
            for (int n = 0; n < 8; ++n) keep((char*)a.v_pool, kColKBytes + 1024 * n, n, col_v_within(lane));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // read before the next tile's transfers overwrite it
        }
        if (!ahead && has_next) {
            wait_vm<0>();
            fetch_list(next + kShortWaves, st2);
            if (wanted_next) fetch(lds_k, kbase, next, st1, true);
        }
        if (wanted_next) fetch(lds_v, vbase, next, st1, false);
        pos = pos_next; seen = seen_next; owned = owned_next;
    }
    wait_vm<0>();

    constexpr int N = 64 / kShortWaves;
    float out[N], mx, lsum;
    cols.combine<kShortWaves>(smem, wave, lane, out, mx, lsum);
    if (qi >= n_rows) return;
    // a row that saw no key: O = 0, LSE = -inf; a NaN sum shows in both
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    const int64_t at = (int64_t)row * kHeadDim + Columns::first_element<kShortWaves>(wave, lane);
    if (a.o_f32) {
        float* dst = (float*)((char*)a.O + part * a.o_part) + at;
#pragma unroll
        for (int e = 0; e < N; e += 4) *(float4*)(dst + 2 * e) = make_float4(out[e] * inv, out[e + 1] * inv, out[e + 2] * inv, out[e + 3] * inv);
    } else {
        uint16_t* dst = (uint16_t*)a.O + at;
#pragma unroll
        for (int e = 0; e < N; e += 4) *(uint2*)(dst + 2 * e) = make_uint2(pack_bf16(out[e] * inv, out[e + 1] * inv), pack_bf16(out[e + 2] * inv, out[e + 3] * inv));
    }
    if (wave == 0 && hi == 0) *(float*)((char*)(a.LSE + row) + part * a.lse_part) = lsum != 0.f ? (mx + __builtin_amdgcn_logf(lsum)) * kLn2 : -INFINITY;
}

esp_status launch_prefill_short(const PrefillArgs& a, hipStream_t stream) {
    const int64_t rows = (int64_t)a.Tq * a.G;
    const int64_t blocks = a.batch == 1 ? (rows + kShortRows - 1) / kShortRows : rows / kShortRows + a.batch;
    if (blocks * a.Hkv * a.splits > UINT32_MAX / (kShortWaves * 64)) return fail(ESP_ERR_UNSUPPORTED, "prefill: too many rows for one launch of the kernel for few");
    const dim3 grid((unsigned)(blocks * a.Hkv * a.splits));
    if (a.kv_slot) hipLaunchKernelGGL((prefill_short_kernel<2>), grid, dim3(kShortWaves * 64), 0, stream, a);
    else if (a.retain_slot) hipLaunchKernelGGL((prefill_short_kernel<1>), grid, dim3(kShortWaves * 64), 0, stream, a);
    else hipLaunchKernelGGL((prefill_short_kernel<0>), grid, dim3(kShortWaves * 64), 0, stream, a);
    return check_launch("prefill_short_kernel");
}

}  // namespace esp
