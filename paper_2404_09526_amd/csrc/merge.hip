// esp_merge_partials: log-sum-exp weighted combination of P partial attention results of the
// same (token, head) pairs into the result over the union of their key sets (the final
// output after all sequence-parallel rounds, Sec. 2.3; the results returned to the master in
// distributed decoding, Sec. 4.2).  HBM-streaming: 16 lanes share one (token, head) pair,
// each owning 8 of the 128 output elements, or with fp32 partials 32 lanes, each owning 4: one 16-byte load of each
// partial, a pair's bytes in a row.
// (Partials that never leave this GPU, the rounds of a sequence-parallel prefill, may stay in fp32,
// so that the merged result is rounded to bf16 once and not twice.)  The parts of a prefill call that split its
// key-value rows come here too, and leave as fp32 where the call's own result is a partial (OUT32).
#include "esp_common.h"

namespace esp {

// Bound by the memory.  What the lanes of a wavefront load together lies in a row: with 16 lanes on a pair of fp32 partials, two loads of
// 16 bytes each, every load touched all of its lines for half of them.  Before -> now, one merge after another: four of 8192 x 32 pairs 112 ->
// 99.8 us (6.1 TB/s), two of 15336 x 32 107.6 -> 99.9, four of 1488 x 32 21.6 -> 17.6, six of 300 x 32 7.6 -> 6.8; behind the prefill calls that
// wrote them the first 103.5 -> 95.1, the second 104.2 -> 104.7.  (Loads through the caches while these hold all partials: 5.3 us for the
// six of 300 x 32, but the rows that they displace are the next call's: 300 tokens against four shards, 32 / 8 heads, 62.1 -> 62.6 us.)
// The partials are loaded N at a time, in up to GROUPS groups: all of them up to four; beyond, four at a time where the call is bound
// by the chain of loads (up to 4096 pairs), one at a time where it is bound by the memory and registers for more only cost
// wavefronts (one at a time, each behind a test for P -> this, with 16 lanes on a pair: sixteen of 31 x 4 9.7 -> 7.2, eight of 32 x 32 5.6 -> 4.7,
// twelve of 64 x 32 8.8 -> 7.0; six fp32 ones of 300 x 32 7.6, with four at a time 8.2).
template <bool F32, bool OUT32, int N, int GROUPS>
__global__ __launch_bounds__(256) void merge_kernel(int32_t P, int64_t pairs, void* O, float* LSE_out, MergeArgs parts) {
    constexpr int LANES = F32 ? 32 : 16, E = kHeadDim / LANES;       // of a pair; output elements of a lane
    const int64_t i = row_block() * 256 + threadIdx.x, pair = i / LANES;
    if (pair >= pairs) return;
    const int seg = (int)(i % LANES);

    float m = -INFINITY;
    float lse[GROUPS][N];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
#pragma unroll
        for (int u = 0; u < N; ++u) lse[g][u] = g == 0 || N * g + u < P ? parts.LSE_parts[N * g + u][pair] : -INFINITY;
#pragma unroll
        for (int u = 0; u < N; ++u) m = fmaxf(m, lse[g][u]);
    }
    // The maximum passes a NaN log-sum-exp over; its weight is NaN and makes the pair NaN, also where there is nothing but -inf
    // beside it: the weights are then taken against 0.  (A test of all sixteen for NaN took 0.25 us of the 28.7 of a split call
    // of 64 tokens on 4096 rows, 32 / 8 heads.)
    const float ref = m == -INFINITY ? 0.f : m;
    float acc[E] = {};
    float wsum = 0.f;
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        if (g > 0 && N * g >= P) continue;
        uint4 piece[N] = {};
#pragma unroll
        for (int u = 0; u < N; ++u) {
            if (g > 0 && N * g + u >= P) continue;
            piece[u] = load_once((const uint4*)parts.O_parts[N * g + u] + pair * LANES + seg);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const uint4 o = piece[u];
            float f[E];
            if constexpr (F32) {
                const float4 x = __builtin_bit_cast(float4, o);
                f[0] = x.x; f[1] = x.y; f[2] = x.z; f[3] = x.w;
            } else {
                f[0] = bf16_lo(o.x); f[1] = bf16_hi(o.x); f[2] = bf16_lo(o.y); f[3] = bf16_hi(o.y);
                f[4] = bf16_lo(o.z); f[5] = bf16_hi(o.z); f[6] = bf16_lo(o.w); f[7] = bf16_hi(o.w);
            }
            // an empty partial (LSE = -inf) gets weight exp(-inf) = 0
            const float w = __expf(lse[g][u] - ref);
            wsum += w;
            if (w != 0.f) {  // keeps non-finite garbage of an empty partial out of the sum
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] += w * f[e];
            }
        }
    }
    const float inv = wsum == 0.f ? 0.f : 1.0f / wsum;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] *= inv;
    if (LSE_out != nullptr && seg == 0) LSE_out[pair] = wsum == 0.f ? -INFINITY : m + __logf(wsum);
    if constexpr (OUT32) {
        ((float4*)O)[pair * LANES + seg] = make_float4(acc[0], acc[1], acc[2], acc[3]);
    } else if constexpr (F32) {
        ((uint2*)O)[pair * LANES + seg] = make_uint2(pack_bf16(acc[0], acc[1]), pack_bf16(acc[2], acc[3]));
    } else {
        ((uint4*)O)[pair * LANES + seg] = make_uint4(pack_bf16(acc[0], acc[1]), pack_bf16(acc[2], acc[3]), pack_bf16(acc[4], acc[5]), pack_bf16(acc[6], acc[7]));
    }
}

esp_status launch_merge(const MergeArgs& parts, int32_t P, int64_t pairs, int32_t parts_f32, void* O, float* LSE_out,
                        hipStream_t stream, int32_t o_f32) {
    const int64_t per_block = parts_f32 ? 8 : 16;
    const int64_t blocks = (pairs + per_block - 1) / per_block;
    if (blocks > kGridMost) return fail(ESP_ERR_INVALID_ARG, "merge: too many rows for one launch");
#define ESP_MERGE_KERNEL(F32, OUT32, N, GROUPS) \
    hipLaunchKernelGGL((merge_kernel<F32, OUT32, N, GROUPS>), row_grid(blocks), dim3(256), 0, stream, P, pairs, O, LSE_out, parts)
#define ESP_MERGE_LAUNCH(F32, OUT32)                                  \
    if (P == 1) ESP_MERGE_KERNEL(F32, OUT32, 1, 1);                   \
    else if (P == 2) ESP_MERGE_KERNEL(F32, OUT32, 2, 1);              \
    else if (P == 3) ESP_MERGE_KERNEL(F32, OUT32, 3, 1);              \
    else if (P == 4) ESP_MERGE_KERNEL(F32, OUT32, 4, 1);              \
    else if (pairs <= 4096) ESP_MERGE_KERNEL(F32, OUT32, 4, ESP_MAX_PARTIALS / 4); \
    else ESP_MERGE_KERNEL(F32, OUT32, 1, ESP_MAX_PARTIALS);
    if (parts_f32 && o_f32) { ESP_MERGE_LAUNCH(true, true) }
    else if (parts_f32) { ESP_MERGE_LAUNCH(true, false) }
    else { ESP_MERGE_LAUNCH(false, false) }
#undef ESP_MERGE_LAUNCH
#undef ESP_MERGE_KERNEL
    return check_launch("merge_kernel");
}

}  // namespace esp
