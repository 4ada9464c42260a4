// esp_merge_partials: log-sum-exp weighted combination of P partial attention results of the
// same (token, head) pairs into the result over the union of their key sets (the final
// output after all sequence-parallel rounds, Sec. 2.3; the results returned to the master in
// distributed decoding, Sec. 4.2).  HBM-streaming: 16 lanes share one (token, head) pair,
// each owning 8 of the 128 output elements (one 16-byte load per bf16 partial, two per fp32 partial:
// partials that never leave this GPU, the rounds of a sequence-parallel prefill, may stay in fp32,
// so that the merged result is rounded to bf16 once and not twice).  The parts of a prefill call that split its
// key-value rows come here too, and leave as fp32 where the call's own result is a partial (OUT32).
#include "esp_common.h"

namespace esp {

// The partials are loaded N at a time, in up to GROUPS groups: all of them up to four; beyond, four at a time where the call is bound
// by the chain of loads (up to 4096 pairs), one at a time where it is bound by the memory and registers for more only cost
// wavefronts.  Measured, us (one at a time, each behind a test for P -> this): two fp32 partials of 256 x 4 pairs 3.5 -> 3.0, sixteen of
// 31 x 4 9.7 -> 7.2, eight of 32 x 32 5.6 -> 4.7, twelve of 64 x 32 8.8 -> 7.0, four of 1488 x 32 23.7 -> 21.7, four bf16 ones of 8192 x 32 59.5
// -> 56.1; six fp32 ones of 300 x 32 7.6, with four at a time 8.2; four of 8192 x 32 113 -> 112 (5.4 TB/s).
template <bool F32, bool OUT32, int N, int GROUPS>
__global__ __launch_bounds__(256) void merge_kernel(MergeArgs parts, int32_t P, int64_t pairs,
                                                    uint4* O, float* LSE_out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t pair = i >> 4;
    if (pair >= pairs) return;
    int seg = (int)(i & 15);

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
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float wsum = 0.f;
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        if (g > 0 && N * g >= P) continue;
        constexpr int kPieces = F32 ? 2 : 1;
        uint4 piece[N][kPieces] = {};
#pragma unroll
        for (int u = 0; u < N; ++u) {
            if (g > 0 && N * g + u >= P) continue;
            const uint4* src = (const uint4*)parts.O_parts[N * g + u] + (pair * 16 + seg) * kPieces;
#pragma unroll
            for (int e = 0; e < kPieces; ++e) piece[u][e] = load_once(&src[e]);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            float f[8];
            if (F32) {
                const float4 x = __builtin_bit_cast(float4, piece[u][0]), y = __builtin_bit_cast(float4, piece[u][kPieces - 1]);
                f[0] = x.x; f[1] = x.y; f[2] = x.z; f[3] = x.w; f[4] = y.x; f[5] = y.y; f[6] = y.z; f[7] = y.w;
            } else {
                const uint4 o = piece[u][0];
                f[0] = bf16_lo(o.x); f[1] = bf16_hi(o.x); f[2] = bf16_lo(o.y); f[3] = bf16_hi(o.y);
                f[4] = bf16_lo(o.z); f[5] = bf16_hi(o.z); f[6] = bf16_lo(o.w); f[7] = bf16_hi(o.w);
            }
            // an empty partial (LSE = -inf) gets weight exp(-inf) = 0
            const float w = __expf(lse[g][u] - ref);
            wsum += w;
            if (w != 0.f) {  // keeps non-finite garbage of an empty partial out of the sum
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] += w * f[e];
            }
        }
    }
    const float inv = wsum == 0.f ? 0.f : 1.0f / wsum;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= inv;
    if (LSE_out != nullptr && seg == 0) LSE_out[pair] = wsum == 0.f ? -INFINITY : m + __logf(wsum);
    if (OUT32) {
        float4* dst = (float4*)O + (pair * 16 + seg) * 2;
        dst[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        dst[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
        return;
    }
    uint4 out;
    out.x = pack_bf16(acc[0], acc[1]);
    out.y = pack_bf16(acc[2], acc[3]);
    out.z = pack_bf16(acc[4], acc[5]);
    out.w = pack_bf16(acc[6], acc[7]);
    O[pair * 16 + seg] = out;
}

esp_status launch_merge(const MergeArgs& parts, int32_t P, int64_t pairs, int32_t parts_f32, void* O, float* LSE_out,
                        hipStream_t stream, int32_t o_f32) {
    int64_t threads = pairs * 16;
    int64_t blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffff) return fail(ESP_ERR_INVALID_ARG, "merge: too many rows for one launch");
#define ESP_MERGE_KERNEL(F32, OUT32, N, GROUPS) \
    hipLaunchKernelGGL((merge_kernel<F32, OUT32, N, GROUPS>), dim3((unsigned)blocks), dim3(256), 0, stream, parts, P, pairs, (uint4*)O, LSE_out)
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
