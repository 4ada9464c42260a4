// Internal declarations shared by the translation units of libesp (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "esp.h"

namespace esp {

constexpr int kHeadDim = 128;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Records a message for esp_last_error() and returns `code`.
esp_status fail(esp_status code, const char* fmt, ...);
// Returns ESP_OK or converts the pending launch error into ESP_ERR_HIP.
esp_status check_launch(const char* what);

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float floatx2;

// bf16 bit pattern (low or high half of a 32-bit word) to float: exact.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

// Two floats to packed bf16 (round to nearest even), a in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    floatx2 f = {a, b};
    bf16x2 h = __builtin_convertvector(f, bf16x2);
    return __builtin_bit_cast(uint32_t, h);
}

// Loads and stores of data that passes once (pool rows under a decode pass, partials on their way to a merge):
// marked non-temporal, so that they do not displace what the caches hold.  Measured on the decode kernel: 74 % -> 82 %
// of the HBM rate.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_once(const uint4* p) {
    const u32x4 t = __builtin_nontemporal_load((const u32x4*)p);
    return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ float4 load_once(const float4* p) {
    const floatx4 t = __builtin_nontemporal_load((const floatx4*)p);
    return make_float4(t[0], t[1], t[2], t[3]);
}
__device__ __forceinline__ void store_once(uint4* p, const uint4& v) {
    __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, (u32x4*)p);
}

// Grids of one thread block after another along rows.  A launch counts its work-items in 32 bits a dimension, and one that asks for more
// starts, without an error, with what the count keeps of them; so block i is (i % kGridX, i / kGridX), and blocks past the last
// find no row.
constexpr int kGridX = 1 << 23;
constexpr int64_t kGridMost = (int64_t)65535 * kGridX;
inline dim3 row_grid(int64_t blocks) { return dim3((unsigned)(blocks < kGridX ? blocks : kGridX), (unsigned)((blocks + kGridX - 1) / kGridX)); }
__device__ __forceinline__ int64_t row_block() { return (int64_t)blockIdx.y * kGridX + blockIdx.x; }

// ---- launchers (one per kernel file) -------------------------------------------------
struct MergeArgs {
    const void* O_parts[ESP_MAX_PARTIALS];
    const float* LSE_parts[ESP_MAX_PARTIALS];
};
esp_status launch_kv_append(const void* k, const void* v, const int32_t* slot_idx, int32_t T, void* k_pool,
                            void* v_pool, int32_t row_bytes, hipStream_t stream);
esp_status launch_kv_gather(const void* k_pool, const void* v_pool, const int32_t* slot_idx, int32_t T, int64_t num_slots,
                            void* k, void* v, int32_t row_bytes, hipStream_t stream);
esp_status launch_probe_mfma(const void* operands, int64_t operand_bytes, int32_t iters, void* sink, int64_t* flops,
                             hipStream_t stream);
esp_status launch_probe_read(const void* src, int64_t bytes, void* sink, hipStream_t stream);
esp_status launch_merge(const MergeArgs& parts, int32_t P, int64_t pairs, int32_t parts_f32, void* O, float* LSE_out,
                        hipStream_t stream, int32_t o_f32 = 0);

size_t decode_workspace_bytes(int32_t B, int32_t total_tokens, int32_t Hq, int32_t Hkv);
size_t decode_least_workspace_bytes(int32_t B, int32_t total_tokens, int32_t Hq, int32_t Hkv);
esp_status launch_decode(const void* q, const void* k_pool, const void* v_pool, const int32_t* slot_idx,
                         const int32_t* seq_offsets, int32_t B, int32_t total_tokens, int32_t max_len, int32_t Hq,
                         int32_t Hkv, float softmax_scale, void* O, float* LSE, void* workspace, size_t workspace_bytes,
                         hipStream_t stream, const MergeArgs* peers = nullptr, int32_t n_peers = 0);

// The request that holds token t, the last b with seq_offsets[b] <= t, and where it ends; found by a wavefront 64 candidates at a
// time (a binary search is six dependent loads, about 3 us, at 64 requests; this is one).
struct RequestAt { int32_t b, end; };
__device__ __forceinline__ RequestAt request_of(int32_t t, const int32_t* seq_offsets, int32_t B, int lane) {
    int lo = 0, hi = B, end = 0;   // invariant: seq_offsets[lo] <= t < seq_offsets[hi]
    do {
        const int stride = (hi - lo + 63) >> 6, i = min(lo + lane * stride, hi), next = min(i + 1, B);
        const int32_t at = seq_offsets[i], after = seq_offsets[next];
        const uint64_t below = __builtin_amdgcn_ballot_w64(i < hi && at <= t);
        const int l = max(__builtin_popcountll(below) - 1, 0);
        lo += l * stride;
        hi = min(hi, lo + stride);
        end = __builtin_amdgcn_readlane(after, l);
    } while (hi - lo > 1);
    return {lo, end};
}

// Ranges counted from each request's first token on: workgroup i of a launch works on tokens t0 .. t1 - 1 of request b, its partial is that of
// range w along the list.
struct RequestRange { int32_t b, t0, t1, w; };
// `parts` of them for each request (the last one takes what is left of a request longer than the caller said).
// The parts of a request and the requests of a part lie on all XCDs in turn: consecutive workgroups do, so that takes an odd
// number of them from one part to the next (all parts of a request on one XCD: 31 us for 16 requests of 900, 32 / 8 heads, against 21).
__device__ __forceinline__ RequestRange request_part(int32_t i, int32_t parts, int32_t range, int32_t B, const int32_t* seq_offsets) {
    const int32_t part = i / B, at = i - part * B, b = (B & 1) != 0 ? at : (at + B - part % B) % B;
    const int32_t s0 = seq_offsets[b], s1 = seq_offsets[b + 1], t0 = s0 + min(part * range, s1 - s0);   // (s0 + part * range may be past 2^31)
    return {b, t0, part == parts - 1 ? s1 : t0 + min(range, s1 - t0), s0 / range + part};
}
// As many as each request has: the whole ranges of all requests first, then what is left of each, so that workgroups which find no
// room at first have little to do.  Requests are looked at 64 at a time, one per lane; a scan finds the one that holds range i.
__device__ __forceinline__ RequestRange request_range(int32_t i, int32_t range, int32_t B, const int32_t* seq_offsets, int lane) {
#pragma unroll 1
    for (int rest = 0; rest < 2; ++rest) {
#pragma unroll 1
        for (int base = 0; base < B; base += 64) {
            const int b = min(base + lane, B - 1);
            const int32_t s0 = seq_offsets[b], s1 = seq_offsets[b + 1], whole = (s1 - s0) / range;
            const int32_t n = base + lane >= B ? 0 : rest ? (s1 - s0 > whole * range ? 1 : 0) : whole;
            int32_t upto = n;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int32_t below = __shfl_up(upto, d);
                if (lane >= d) upto += below;
            }
            const uint64_t hit = __builtin_amdgcn_ballot_w64(upto > i);
            if (hit) {
                const int l = __builtin_ctzll(hit);
                const int32_t start = __builtin_amdgcn_readlane(s0, l), end = __builtin_amdgcn_readlane(s1, l);
                const int32_t part = rest ? __builtin_amdgcn_readlane(whole, l) : i - (__builtin_amdgcn_readlane(upto, l) - __builtin_amdgcn_readlane(n, l));
                const int32_t t0 = start + part * range;
                return {base + l, t0, t0 + min(range, end - t0), start / range + part};
            }
            i -= __builtin_amdgcn_readlane(upto, 63);
        }
    }
    return {0, 0, 0, 0};                                            // the launch is an upper bound
}

constexpr int kGqWaves = 4;       // wavefronts per workgroup of decode_gq.hip

// the partial kernel on the matrix cores (decode_gq.hip): one partial per (range + request, head)
esp_status launch_decode_gq(const void* q, const void* k_pool, const void* v_pool, const int32_t* slot_idx,
                            const int32_t* seq_offsets, int32_t B, int32_t total_tokens, int32_t range, int32_t parts, int32_t nwg,
                            int32_t Hq, int32_t Hkv, float scale_log2, float* part_acc, float* part_ml, hipStream_t stream);

// short requests in one launch (decode_whole.hip); `burst`: the layouts that decode.hip has on the vector ALU
esp_status launch_decode_whole(const void* q, const void* k_pool, const void* v_pool, const int32_t* slot_idx, const int32_t* seq_offsets,
                               int32_t B, int32_t total_tokens, int32_t Hq, int32_t Hkv, bool burst, float scale_log2, void* O, float* LSE,
                               const MergeArgs* peers, int32_t n_peers, hipStream_t stream);

// whether decode calls of this thread work in ranges (1), in one launch (2), or by estimate (0); returns the previous value; and what a
// call of these sizes would do
int32_t set_decode_plan(int32_t plan);
int32_t query_decode_plan(int32_t B, int32_t total_tokens, int32_t max_len, int32_t Hq, int32_t Hkv);

int32_t set_prefill_sync_ticks(int32_t ticks);   // returns the previous value; negative restores the built-in default
// which kernel prefill calls of this thread run on, in how many parts: n: the main one in n, -n: the one for few rows in n, 0: by
// estimate.  Returns the previous value.
int32_t set_prefill_plan(int32_t plan);
// what a call of these sizes would run on (the same form; never 0)
int32_t query_prefill_plan(size_t workspace_bytes, int32_t Tq, int32_t Tkv, int32_t batch, int32_t max_kv, int32_t Hq, int32_t Hkv, bool causal, bool kept);
esp_status launch_decode_static(const void* q, const void* k_pool, const void* v_pool, const int32_t* slot_idx,
                                const int32_t* seq_offsets, int32_t B, int32_t total_tokens, int32_t max_len, int32_t Hq,
                                int32_t Hkv, float softmax_scale, void* O, float* LSE, hipStream_t stream);

constexpr size_t kPrefillCounterBytes = 256;      // what every prefill call needs: its item counter and arrival counts
// the same, and room for the partial results of the calls that split the key-value rows
size_t prefill_workspace_bytes(int32_t Tq, int32_t Tkv, int32_t batch, int32_t Hq, int32_t Hkv);
esp_status launch_prefill(const void* q, const void* k, const void* v, const int32_t* q_pos, const int32_t* kv_pos,
                          const int32_t* cu_q, const int32_t* cu_kv, int32_t batch, int32_t Tq, int32_t Tkv,
                          int32_t max_kv, int32_t Hq, int32_t Hkv, float softmax_scale,
                          int32_t causal, int32_t o_f32, void* O, float* LSE, void* workspace, size_t workspace_bytes,
                          const int32_t* retain_slot, void* k_pool, void* v_pool, const int32_t* kv_slot,
                          hipStream_t stream);

}  // namespace esp
