// Decode of short requests in one launch: a workgroup has a whole request and one KV head (a chunk of its query heads), and leaves the
// result, with the peers' partials folded in; no partials, no kernel to combine them.  Such a call is a chain of round trips: offsets, slots,
// rows, and a second launch with three of its own (3.6 us), longer than one CU takes for the rows of a few hundred tokens (46 .. 56 GB/s a
// workgroup on the matrix cores, 43 on the vector ALU, when few are at it).  Which calls: decode_whole (decode.hip), with both sides'
// figures.  A step of four requests of 224 .. 485 tokens, 4 / 4 heads, three peers, its append included: 12.0 -> 9.0 us.
#include "column_tile.h"
#include "decode_merge.h"

namespace esp {

constexpr int kWholeWaves = 16;      // of the vector kernel; on the matrix cores eight (an LDS block of 16.5 KiB each)
constexpr int kWholeGqWaves = 8;
constexpr int kPeersAhead = 4;       // peers whose rows are asked for at the start

// N elements of head `pair` from element `at` on, in pieces of four that lie `step` apart, of peers p0 .. p0 + 3
template <int N>
struct PeerRows {
    float lse[kPeersAhead];
    U32x2 o[kPeersAhead][N / 4];
    __device__ __forceinline__ void load(const MergeArgs& peers, int p0, int n_peers, int64_t pair, int at, int step) {
#pragma unroll
        for (int u = 0; u < kPeersAhead; ++u) {
            const int p = min(p0 + u, n_peers - 1);
            lse[u] = peers.LSE_parts[p][pair];
#pragma unroll
            for (int e = 0; e < N / 4; ++e) o[u][e] = ((const U32x2*)peers.O_parts[p])[pair * (kHeadDim / 4) + (at + step * e) / 4];
        }
    }
    __device__ __forceinline__ void add_to(Weighted<N>& sum, int p0, int n_peers) const {
        float m[kPeersAhead], l[kPeersAhead], v[kPeersAhead][N];
#pragma unroll
        for (int u = 0; u < kPeersAhead; ++u) {
            m[u] = lse[u] * kLog2e;
            l[u] = p0 + u < n_peers && lse[u] != -INFINITY ? 1.f : 0.f;   // a peer's rows are normalised
#pragma unroll
            for (int e = 0; e < N / 4; ++e) {
                v[u][4 * e] = bf16_lo(o[u][e].x); v[u][4 * e + 1] = bf16_hi(o[u][e].x);
                v[u][4 * e + 2] = bf16_lo(o[u][e].y); v[u][4 * e + 3] = bf16_hi(o[u][e].y);
            }
        }
        sum.template add<true>(m, l, v);
    }
};
// the rest of the peers, and the result
template <bool PEERS, int N>
__device__ __forceinline__ void finish(Weighted<N>& sum, PeerRows<N>& rows, const MergeArgs& peers, int n_peers, int64_t pair, int at, int step,
                                       U32x2* O, float* LSE, bool writes_lse) {
    if constexpr (PEERS) {
        rows.add_to(sum, 0, n_peers);
        for (int p0 = kPeersAhead; p0 < n_peers; p0 += kPeersAhead) {
            rows.load(peers, p0, n_peers, pair, at, step);
            rows.add_to(sum, p0, n_peers);
        }
    }
    const float inv = sum.L == 0.f ? 0.f : 1.0f / sum.L;            // no token anywhere: exactly 0
#pragma unroll
    for (int e = 0; e < N / 4; ++e)
        O[pair * (kHeadDim / 4) + (at + step * e) / 4] = U32x2{pack_bf16(sum.acc[4 * e] * inv, sum.acc[4 * e + 1] * inv),
                                                               pack_bf16(sum.acc[4 * e + 2] * inv, sum.acc[4 * e + 3] * inv)};
    if (writes_lse) LSE[pair] = sum.L == 0.f ? -INFINITY : (sum.M + __builtin_amdgcn_logf(sum.L)) * kLn2;
}

// the same between neighbouring rows of 16 lanes as half_swap_* between the halves
__device__ __forceinline__ void row_pair(float x, float& lo, float& hi) {
    int a = __builtin_bit_cast(int, x), b = a;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    lo = __builtin_bit_cast(float, a);
    hi = __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float row_swap_max(float x) {
    float lo, hi;
    row_pair(x, lo, hi);
    return fmaxf(lo, hi);
}
__device__ __forceinline__ float row_swap_sum(float x) {
    float lo, hi;
    row_pair(x, lo, hi);
    return lo + hi;
}

// One or two query heads per KV head, on the vector ALU (as the row-burst kernel of decode.hip): 16 lanes have a token's 256 bytes of K
// and of V, a wavefront four tokens a load; four loads of each (two with two query heads) are a step, 256 tokens (128) a workgroup, and the first two steps are asked
// for together.
template <int G, bool PEERS>
__global__ __launch_bounds__(kWholeWaves * 64, 4) void decode_whole_kernel(
    const uint16_t* __restrict__ q, const char* __restrict__ k_pool, const char* __restrict__ v_pool, const int32_t* __restrict__ slot_idx,
    const int32_t* __restrict__ seq_offsets, int32_t total_tokens, int32_t Hkv, float scale_log2, int32_t n_peers, U32x2* O, float* LSE, MergeArgs peers) {
    constexpr int U = 4 / G;
    __shared__ float lds_acc[kWholeWaves][G][kHeadDim];
    __shared__ float2 lds_ml[kWholeWaves][G];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.x, kvh = blockIdx.y;
    const int32_t s0 = seq_offsets[b], s1 = min(seq_offsets[b + 1], total_tokens);   // (never past the slot list)
    // tokens are counted from the request's first on, without a sign: steps that are looked ahead to may start past 2^31
    const uint32_t n = max(s1 - s0, 0);
    const int32_t* const list = slot_idx + s0;
    const int dseg = (lane & 15) * 8;
    const uint32_t row_bytes = (uint32_t)Hkv * (kHeadDim * 2), within = (uint32_t)kvh * (kHeadDim * 2) + dseg * 2;
    const int64_t pair0 = ((int64_t)b * Hkv + kvh) * G;

    float qf[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint4 w = *(const uint4*)(q + (pair0 + g) * kHeadDim + dseg);
        unpack8(w, qf[g]);
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[g][e] *= scale_log2;
    }

    float m[G], l[G], acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = -INFINITY; l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
    }
    const uint32_t first = wave * 4 + (lane >> 4);                      // of a step's tokens: this one, and every 64th after it
    struct Rows { uint4 k[U], v[U]; };
    auto slots_of = [&](uint32_t t, uint32_t (&s)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) s[u] = (uint32_t)list[min(t + first + 64 * u, n - 1)];
    };
    auto load = [&](Rows& r, const uint32_t (&s)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t at = (uint64_t)s[u] * row_bytes + within;
            r.k[u] = load_once((const uint4*)(k_pool + at));
            r.v[u] = load_once((const uint4*)(v_pool + at));
        }
    };
    auto attend = [&](const Rows& r, uint32_t t) {
        float s[U][G];
        bool here[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            here[u] = t + first + 64 * u < n;
            float kf[8];
            unpack8(r.k[u], kf);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float d = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) d = fmaf(qf[g][e], kf[e], d);
                d = row16_sum(d);
                s[u][g] = here[u] ? d : -INFINITY;
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float mx = m[g];
#pragma unroll
            for (int u = 0; u < U; ++u) mx = fmaxf(mx, s[u][g]);
            const float ref = finite_offset(mx), alpha = __builtin_amdgcn_exp2f(m[g] - ref);
            m[g] = mx;
            l[g] *= alpha;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[g][e] *= alpha;
#pragma unroll
            for (int u = 0; u < U; ++u) s[u][g] = __builtin_amdgcn_exp2f(s[u][g] - ref);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint4 w = r.v[u];
            if (!here[u]) w = make_uint4(0u, 0u, 0u, 0u);           // (a row taken twice adds nothing, whatever it holds)
            float vf[8];
            unpack8(w, vf);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                l[g] += s[u][g];
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[g][e] = fmaf(s[u][g], vf[e], acc[g][e]);
            }
        }
    };
    constexpr uint32_t kStep = kWholeWaves * 4 * U;
    if (n > 0) {
        Rows a, c;
        uint32_t sa[U], sc[U];
        slots_of(0, sa);
        slots_of(kStep, sc);
        load(a, sa);
        uint32_t t = 0;
        for (; t + kStep < n; t += 2 * kStep) {
            load(c, sc);
            const bool more = t + 2 * kStep < n;
            if (more) { slots_of(t + 2 * kStep, sa); slots_of(t + 3 * kStep, sc); }
            attend(a, t);
            if (more) load(a, sa);
            attend(c, t + kStep);
        }
        if (t < n) attend(a, t);
    }

    // the lanes that are left at the end (32 a head, four elements each) ask for the peers' rows
    PeerRows<4> rows;
    const int out_lane = lane & 31, out_g = wave * 2 + (lane >> 5);
    if (PEERS && out_g < G) rows.load(peers, 0, n_peers, pair0 + out_g, 4 * out_lane, 0);
    // ---- four tokens a load: the four groups of 16 lanes combine by exchanges, then the wavefronts through LDS
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float mx = half_swap_max(row_swap_max(m[g])), c = __builtin_amdgcn_exp2f(m[g] - finite_offset(mx));
        const float lt = half_swap_sum(row_swap_sum(l[g] * c));
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = half_swap_sum(row_swap_sum(acc[g][e] * c));
        if (lane < 16) {
            float4* dst = (float4*)&lds_acc[wave][g][dseg];
            dst[0] = make_float4(acc[g][0], acc[g][1], acc[g][2], acc[g][3]);
            dst[1] = make_float4(acc[g][4], acc[g][5], acc[g][6], acc[g][7]);
            if (lane == 0) lds_ml[wave][g] = make_float2(mx, lt);
        }
    }
    __syncthreads();
    if (out_g >= G) return;
    Weighted<4> sum;
#pragma unroll
    for (int w = 0; w < kWholeWaves; w += 4) {
        float wm[4], wl[4], wv[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float2 ml = lds_ml[w + u][out_g];
            const float4 x = *(const float4*)&lds_acc[w + u][out_g][4 * out_lane];
            wm[u] = ml.x; wl[u] = ml.y;
            wv[u][0] = x.x; wv[u][1] = x.y; wv[u][2] = x.z; wv[u][3] = x.w;
        }
        sum.template add<false>(wm, wl, wv);
    }
    sum.own = sum.L != 0.f;
    finish<PEERS>(sum, rows, peers, n_peers, pair0 + out_g, 4 * out_lane, 0, O, LSE, out_lane == 0);
}

// Every other layout, on the matrix cores (as decode_gq.hip): eight wavefronts, a tile of 32 tokens each in turn.
template <bool PEERS>
__global__ __launch_bounds__(kWholeGqWaves * 64, 2) void decode_whole_gq_kernel(
    const uint16_t* __restrict__ q, const char* __restrict__ k_pool, const char* __restrict__ v_pool, const int32_t* __restrict__ slot_idx,
    const int32_t* __restrict__ seq_offsets, int32_t total_tokens, int32_t Hq, int32_t Hkv, float scale_log2, int32_t n_peers, U32x2* O, float* LSE,
    MergeArgs peers) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kWholeGqWaves * kColWaveBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qi = lane & 31, hi = lane >> 5;
    const int b = blockIdx.x, kvh = blockIdx.y;
    const int32_t s0 = seq_offsets[b], s1 = min(seq_offsets[b + 1], total_tokens);   // (never past the slot list)
    const uint32_t n = max(s1 - s0, 0);                             // (without a sign, as above)
    const int32_t* const list = slot_idx + s0;
    // slots of a tile: lane holds that of tile row lane % 32 (rows past the end: the last)
    auto tile_slots = [&](uint32_t i) { return list[min(32 * i + qi, n - 1)]; };
    int32_t slots = 0, slots_next = 0;
    if (32 * wave < n) { slots = tile_slots(wave); slots_next = tile_slots(wave + kWholeGqWaves); }
    const int G = Hq / Hkv, g0 = blockIdx.z * 32;
    const int ng = min(32, G - g0);                                 // query heads of this chunk: columns 0 .. ng-1
    const uint32_t row_bytes = (uint32_t)Hkv * (kHeadDim * 2);
    const char* kbase = k_pool + (uint32_t)kvh * (kHeadDim * 2);
    const char* vbase = v_pool + (uint32_t)kvh * (kHeadDim * 2);
    const uint32_t lds_k = (uint32_t)(uintptr_t)(ESP_LDS unsigned char*)smem + wave * kColWaveBytes, lds_v = lds_k + kColKBytes;
    const int64_t pair = (int64_t)b * Hq + kvh * G + g0 + min(qi, ng - 1);   // of this column (columns past the chunk: zeros, nothing written)

    bf16x8 qf[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        uint4 raw = *(const uint4*)(q + pair * kHeadDim + 16 * t + 8 * hi);
        if (qi >= ng) raw = make_uint4(0u, 0u, 0u, 0u);
        qf[t] = __builtin_bit_cast(bf16x8, raw);
    }
    constexpr int N = 64 / kWholeGqWaves;
    const int at = Columns::first_element<kWholeGqWaves>(wave, lane);
    PeerRows<N> rows;
    if (PEERS) rows.load(peers, 0, n_peers, pair, at, 8);
    Columns cols;
    cols.place(lds_k, lane);
    cols.clear();
    auto fetch = [&](uint32_t to, const char* base, int32_t of, bool is_k) {
#pragma unroll
        for (int x = 0; x < 8; ++x)
            load_to_lds_b128_at_nt(to + 1024 * x, base + ((uint64_t)(uint32_t)__shfl(of, col_row(x, lane)) * row_bytes + (is_k ? col_k_within(x, lane) : col_v_within(lane))));
    };
    if (32 * wave < n) { fetch(lds_k, kbase, slots, true); fetch(lds_v, vbase, slots, false); }
    for (uint32_t i = wave; 32 * i < n; i += kWholeGqWaves) {
        const int here = min(32u, n - 32 * i);
        const bool next = 32 * (i + kWholeGqWaves) < n;
        wait_vm<8>();                                               // K has landed; V may be on its way
        floatx16 sc = cols.scores(qf);
        // the next tile's K follows as soon as the scores are taken, its V as soon as this one's has been read
        if (next) {
            asm volatile("" :: "v"(sc));
            fetch(lds_k, kbase, slots_next, true);
        }
        if (here < 32) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + 4 * hi + (r & 3) >= here) sc[r] = -INFINITY;
        }
        Columns::PFrag pf[2];
        cols.weigh(sc, scale_log2, pf);
        if (next) wait_vm<8>(); else wait_vm<0>();
        cols.accumulate(pf);
        if (next) {
            fetch(lds_v, vbase, slots_next, false);
            slots_next = tile_slots(i + 2 * kWholeGqWaves);
        }
    }
    Weighted<N> sum;
    cols.combine<kWholeGqWaves>(smem, wave, lane, sum.acc, sum.M, sum.L);
    if (qi >= ng) return;
    sum.own = sum.L != 0.f;
    if (!sum.own) {                                                 // no token of this request here: nothing that it left counts
        sum.M = -INFINITY;
#pragma unroll
        for (int e = 0; e < N; ++e) sum.acc[e] = 0.f;
    }
    finish<PEERS>(sum, rows, peers, n_peers, pair, at, 8, O, LSE, wave == 0 && hi == 0);
}

esp_status launch_decode_whole(const void* q, const void* k_pool, const void* v_pool, const int32_t* slot_idx, const int32_t* seq_offsets,
                               int32_t B, int32_t total_tokens, int32_t Hq, int32_t Hkv, bool burst, float scale_log2, void* O, float* LSE,
                               const MergeArgs* peers, int32_t n_peers, hipStream_t stream) {
    const int G = Hq / Hkv;
    const bool with_peers = peers != nullptr && n_peers > 0;
    const MergeArgs none = {};
    if (B > (int32_t)(UINT32_MAX / (kWholeWaves * 64)) || Hkv > 65535 || (G + 31) / 32 > 65535)   // (only where a test asks for this form)
        return fail(ESP_ERR_UNSUPPORTED, "decode: too many requests or heads for one launch of a workgroup each");
#define ESP_WHOLE_LAUNCH(KERNEL, WAVES, Z, ...)                                                                                          \
    hipLaunchKernelGGL(KERNEL, dim3(B, Hkv, Z), dim3(WAVES * 64), 0, stream, (const uint16_t*)q, (const char*)k_pool, (const char*)v_pool, \
                       slot_idx, seq_offsets, total_tokens, __VA_ARGS__, scale_log2, n_peers, (U32x2*)O, LSE, with_peers ? *peers : none)
    if (burst && G == 1 && with_peers) ESP_WHOLE_LAUNCH((decode_whole_kernel<1, true>), kWholeWaves, 1, Hkv);
    else if (burst && G == 1) ESP_WHOLE_LAUNCH((decode_whole_kernel<1, false>), kWholeWaves, 1, Hkv);
    else if (burst && with_peers) ESP_WHOLE_LAUNCH((decode_whole_kernel<2, true>), kWholeWaves, 1, Hkv);
    else if (burst) ESP_WHOLE_LAUNCH((decode_whole_kernel<2, false>), kWholeWaves, 1, Hkv);
    else if (with_peers) ESP_WHOLE_LAUNCH(decode_whole_gq_kernel<true>, kWholeGqWaves, (G + 31) / 32, Hq, Hkv);
    else ESP_WHOLE_LAUNCH(decode_whole_gq_kernel<false>, kWholeGqWaves, (G + 31) / 32, Hq, Hkv);
#undef ESP_WHOLE_LAUNCH
    return check_launch("decode_whole_kernel");
}

}  // namespace esp
