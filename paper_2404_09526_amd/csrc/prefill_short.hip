// Prefill partial attention for calls with few query rows: a small chunk, a follow-up turn, short prompts, few heads.  The main
// kernel (prefill.hip) gives a workgroup 256 packed rows of a KV head and lets all its wavefronts walk the keys together: such a
// call has a handful of items, each a serial walk (set-up 7 us, 1.5 us per 64 keys whatever it holds), and leaves the chip idle.
// What bounds it is that chain, so here the chain is cut: a workgroup has 32 packed rows (the columns of one MFMA tile), its
// eight wavefronts take the tiles of 32 keys in turn, each alone, with an LDS block of its own and no barrier until the end,
// and combine their results through LDS (column_tile.h).  A row block re-reads all of its K and V from the L2, eight times as often
// as there, and a row costs several times as much: the launcher picks by an estimate of both times (prefill.hip).
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
    constexpr int kPosAt = kShortWaves * kColWaveBytes;             // key positions of a tile that has to be masked, per wavefront
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kPosAt + kShortWaves * 32 * 4];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qi = lane & 31, hi = lane >> 5;
    // the row blocks of a (KV head, part) lie heads x parts workgroups apart: on one XCD where that is a multiple of 8
    const int vheads = a.Hkv * a.splits, vhead = blockIdx.x % vheads;
    const int kvh = vhead / a.splits, part = vhead - kvh * a.splits;
    const int G = a.G;

    // ---- the request and the row block in it: requests are looked at 64 at a time, one per lane
    auto blocks_of = [&](int r) {
        const int n = ((a.cu_q ? a.cu_q[r + 1] - a.cu_q[r] : a.Tq) * G + kShortRows - 1) / kShortRows;
        return KEEP && n == 0 && a.cu_kv && a.cu_kv[r + 1] > a.cu_kv[r] ? 1 : n;
    };
    int r = 0, blk = blockIdx.x / vheads;
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
    const int t_lo = (int)((int64_t)all_tiles * part / a.splits), t_hi = (int)((int64_t)all_tiles * (part + 1) / a.splits);
    const int kv_len = min(kv_end - kv_lo, t_hi * 32) - t_lo * 32;  // this part's rows (may be none)
    kv_lo += t_lo * 32;
    const int tiles = (kv_len + 31) / 32;

    // ---- this lane's row (column of S^T; rows past the end repeat the last): token and query head of the group
    const int my = any_row ? rho + min(qi, n_rows - 1) : 0, tok = any_row ? qs + my / G : 0, row = tok * a.Hq + kvh * G + my % G;
    const int my_qpos = a.causal ? a.q_pos[tok] : INT_MAX - 1;      // non-causal rows see every key that exists

    const uint32_t row_bytes = (uint32_t)a.Hkv * (kHeadDim * 2);
    const char* kbase = (const char*)a.k + (uint32_t)kvh * (kHeadDim * 2);
    const char* vbase = (const char*)a.v + (uint32_t)kvh * (kHeadDim * 2);
    // position and pool slot of tile row lane % 32; rows past the end: a position nobody sees, the last row's slot (KEEP: none)
    auto tile_pos = [&](int i) {
        const int at = 32 * i + qi;
        const int p = a.causal ? a.kv_pos[kv_lo + min(at, kv_len - 1)] : 0;
        return at < kv_len ? p : INT_MAX;
    };
    auto tile_slots = [&](int i) {
        const int at = 32 * i + qi;
        if (KEEP) return at < kv_len ? a.retain_slot[kv_lo + at] : -1;
        return POOL ? a.kv_slot[kv_lo + min(at, kv_len - 1)] : 0;
    };
    int pos = 0, slots = 0;
    if (wave < tiles) { pos = tile_pos(wave); slots = tile_slots(wave); }
    bf16x8 qf[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) qf[t] = __builtin_bit_cast(bf16x8, *(const uint4*)(a.q + (int64_t)row * kHeadDim + 8 * hi + 16 * t));

    const uint32_t lds_k = (uint32_t)(uintptr_t)(ESP_LDS unsigned char*)smem + wave * kColWaveBytes;
    const uint32_t lds_v = lds_k + kColKBytes;
    int32_t* const lds_pos = (int32_t*)(smem + kPosAt) + wave * 32;
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

    for (int i = wave; i < tiles; i += kShortWaves) {
        // (a key may sit at the lowest position there is: a block without rows sees nothing all the same)
        const bool seen = any_row && of_rows(pos, least) <= q_max, mask = of_rows(pos, most) > q_min;
        const bool owned = KEEP && (t_lo + i) % n_blk == blk;
        const int last = min(32, kv_len - 32 * i) - 1, next = i + kShortWaves;
        int pos_next = 0, slots_next = 0;
        if (!seen && !owned) {                                      // a tile that no row can see
            if (next < tiles) { pos_next = tile_pos(next); slots_next = tile_slots(next); }
            pos = pos_next; slots = slots_next;
            continue;
        }
        const int64_t tile_at = (int64_t)(kv_lo + 32 * i) * row_bytes;
        auto fetch = [&](uint32_t lds, const char* base, ColPiece at) {
            if constexpr (POOL) load_to_lds_b128_at(lds, base + ((uint64_t)(uint32_t)__shfl(slots, at.row) * row_bytes + at.within));
            else load_to_lds_b128(lds, base + tile_at, (uint32_t)min(at.row, last) * row_bytes + at.within);
        };
#pragma unroll
        for (int n = 0; n < 9; ++n) fetch(lds_k + 1024 * n, kbase, col_k_piece(n, lane));
        if (next < tiles) { pos_next = tile_pos(next); slots_next = tile_slots(next); }
#pragma unroll
        for (int n = 0; n < 8; ++n) fetch(lds_v + 1024 * n, vbase, col_v_piece(n, lane));
        wait_vm<8>();                                               // K (and what the next tile needs first) has landed

        if (seen) {
            floatx16 sc = cols.scores(qf);
            if (mask) {
                if (lane < 32) lds_pos[lane] = pos;
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
            wait_vm<0>();
            asm volatile("" :: "v"(pos_next), "v"(slots_next));
            cols.accumulate(pf);
        }
        if (owned) {
            if (!seen) wait_vm<0>();
            // what this wavefront fetched, to the rows' slots (lane L of transfer n: the 16 bytes it brought)
            auto keep = [&](char* pool, int lds_at, ColPiece at, bool is_row) {
                const int32_t slot = __shfl(slots, at.row);
                const uint4 w = *(const uint4*)(smem + wave * kColWaveBytes + lds_at + 16 * lane);
                if (is_row && slot >= 0) *(uint4*)(pool + (uint32_t)kvh * (kHeadDim * 2) + ((uint64_t)(uint32_t)slot * row_bytes + at.within)) = w;
            };
#pragma unroll
            for (int n = 0; n < 9; ++n)
                keep((char*)a.k_pool, 1024 * n, col_k_piece(n, lane), (1024 * n + 16 * lane) % kColKRow < 256 && 1024 * n + 16 * lane < 32 * kColKRow);
#pragma unroll
            for (int n = 0; n < 8; ++n) keep((char*)a.v_pool, kColKBytes + 1024 * n, col_v_piece(n, lane), true);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // read before the next tile's transfers overwrite it
        }
        pos = pos_next; slots = slots_next;
    }

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
    if (blocks * a.Hkv * a.splits > 0x7fffffff) return fail(ESP_ERR_UNSUPPORTED, "prefill: too many rows for one launch of the kernel for few");
    const dim3 grid((unsigned)(blocks * a.Hkv * a.splits));
    if (a.kv_slot) hipLaunchKernelGGL((prefill_short_kernel<2>), grid, dim3(kShortWaves * 64), 0, stream, a);
    else if (a.retain_slot) hipLaunchKernelGGL((prefill_short_kernel<1>), grid, dim3(kShortWaves * 64), 0, stream, a);
    else hipLaunchKernelGGL((prefill_short_kernel<0>), grid, dim3(kShortWaves * 64), 0, stream, a);
    return check_launch("prefill_short_kernel");
}

}  // namespace esp
