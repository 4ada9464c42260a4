// Decode partial attention on the matrix cores: every head layout but MHA-like ones that the row-burst kernel
// covers (MQA, GQA with any number of KV heads and query heads per KV head; Sec. 2.3 / Sec. 6: the method serves MHA,
// GQA and MQA alike).  With G query heads per KV head, a resident key row meets G queries: per token
// 2 * 2 * 128 * G flops on 512 bytes, which the vector ALU cannot keep up with from G = 4 or so on (a per-head kernel
// on it reached 11 % of the HBM rate for 32 / 1 heads, the row-burst kernel 46 % for 64 / 8), but which is a dense
// contraction.  The query heads of a request's KV head are the 32 columns of an MFMA tile (unused columns are zero):
//   S^T [32 keys x 32 heads] = K_tile [32 x 128] Q^T [128 x 32],   O^T [128 x 32 heads] += V_tile^T [128 x 32] P^T [32 x 32]
// The products are far from binding (16 MFMAs per 16 KiB gathered), so the kernel's time does not depend on G.
// Work is split as in the row-burst kernel: the concatenated token list in equal ranges, one workgroup per
// (range, KV head, chunk of up to 32 query heads); inside it every wavefront works alone, on every 4th tile of 32
// tokens of a request's part of the range, with an LDS block of its own (no workgroup barrier inside the sweep): it
// gathers the tile's K and V rows from their pool slots straight into LDS (16-byte pieces, a full address per
// lane), multiplies (the scores as soon as K is there) and keeps an exact running maximum; when the request's part of the
// range is done, the wavefronts combine their results through LDS and leave one partial (accumulator, maximum, sum) per
// (range + request, head) for the combine kernel.  (A partial per wavefront made the combine kernel read 145 MB for
// 32 / 1 heads and 64 requests: a quarter of the call's time.)
// A workgroup is four wavefronts, so that two fit a CU (LDS and registers) and one gathers while the other starts or
// combines: a start (search of the request, queries, first slots) and an end take about as long as two steps of
// gathers.  With the ranges of decode_range (decode.hip) and the 64-way search of the first request, measured against one
// workgroup of eight wavefronts per CU: 64 requests of 4K, 32 / 1 heads, 55.7 -> 42.5 us; 128 of 16K, 32 / 8 heads,
// 2337 -> 2291 us (6.45 TB/s; processes differ by as much); 16 of 600, 32 / 8 heads, partial kernel 20.1 -> 16.5 us.
#include "column_tile.h"

namespace esp {

template <bool BY_REQUEST>
__global__ __launch_bounds__(kGqWaves * 64, 2) void decode_partial_gq_kernel(
    const uint16_t* __restrict__ q, const char* __restrict__ k_pool, const char* __restrict__ v_pool,
    const int32_t* __restrict__ slot_idx, const int32_t* __restrict__ seq_offsets, int32_t B, int32_t total_tokens,
    int32_t range, int32_t parts, int32_t Hq, int32_t Hkv, float scale_log2, float* __restrict__ part_acc, float* __restrict__ part_ml) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kGqWaves * kColWaveBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qi = lane & 31, hi = lane >> 5;
    const int kvh = blockIdx.y;
    const int G = Hq / Hkv;
    const int g0 = blockIdx.z * 32;
    const int ng = min(32, G - g0);                             // query heads of this chunk: columns 0 .. ng-1
    const int h0 = kvh * G + g0;
    int w = blockIdx.x;
    const uint32_t row_bytes = (uint32_t)Hkv * (kHeadDim * 2);
    const char* kbase = k_pool + (uint32_t)kvh * (kHeadDim * 2);
    const char* vbase = v_pool + (uint32_t)kvh * (kHeadDim * 2);
    const uint32_t lds_k = (uint32_t)(uintptr_t)(ESP_LDS unsigned char*)smem + wave * kColWaveBytes;
    const uint32_t lds_v = lds_k + kColKBytes;

    Columns cols;
    cols.place(lds_k, lane);

    int b;
    int32_t t0, t1, req_end, slots;
    if (BY_REQUEST) {
        const RequestRange at = parts > 0 ? request_part(w, parts, range, B, seq_offsets) : request_range(w, range, B, seq_offsets, lane);
        b = at.b; t0 = at.t0; t1 = req_end = min(at.t1, total_tokens); w = at.w;   // (never past the slot list)
        if (t0 >= t1) return;
        slots = slot_idx[t0 + min(32 * wave + qi, t1 - 1 - t0)];
    } else {
        t0 = w * range;
        t1 = t0 + min(range, total_tokens - t0);                    // (t0 + range may be past 2^31)
        if (t0 >= t1) return;
        // slots of this wavefront's first tile, as far as they do not depend on where its request ends: asked for before the search
        slots = slot_idx[min(t0 + 32 * wave + qi, total_tokens - 1)];
        const RequestAt at = request_of(t0, seq_offsets, B, lane);
        b = at.b; req_end = at.end;
    }
    bool first = true;

    while (t0 < t1 && b < B) {                                  // (tokens past the offsets' end belong to no request)
        if (!first) req_end = seq_offsets[b + 1];
        if (req_end <= t0) { ++b; continue; }                   // empty request, or the last one where the range starts past its end
        const int32_t pe = min(t1, req_end);
        const int32_t seg = pe - t0;                            // tokens of request b inside this range

        // Q^T fragments of the request's heads: column qi = head h0 + qi (columns past the chunk: zeros)
        bf16x8 qf[8];
        {
            const uint16_t* qp = q + ((int64_t)b * Hq + h0 + (qi < ng ? qi : 0)) * kHeadDim + 8 * hi;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                uint4 raw = *(const uint4*)(qp + 16 * t);
                if (qi >= ng) raw = make_uint4(0u, 0u, 0u, 0u);
                qf[t] = __builtin_bit_cast(bf16x8, raw);
            }
        }
        cols.clear();

        // slots of a tile: lane holds the slot of tile row lane % 32 (rows past the end: the last)
        auto tile_slots = [&](int i) {
            const int rows = min(32, seg - 32 * i);
            return slot_idx[t0 + 32 * i + min(qi, rows - 1)];
        };
        if (!first) slots = 32 * wave < seg ? tile_slots(wave) : 0;
        else if (32 * wave < seg) slots = __shfl(slots, min(qi, min(32, seg - 32 * wave) - 1));
        first = false;
        for (int i = wave; 32 * i < seg; i += kGqWaves) {
            const int rows = min(32, seg - 32 * i);
            // ---- gather
            uint64_t row_at[8];
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                row_at[n] = (uint64_t)(uint32_t)__shfl(slots, col_row(n, lane)) * row_bytes;
                load_to_lds_b128_at_nt(lds_k + 1024 * n, kbase + (row_at[n] + col_k_within(n, lane)));
            }
#pragma unroll
            for (int n = 0; n < 8; ++n) load_to_lds_b128_at_nt(lds_v + 1024 * n, vbase + (row_at[n] + col_v_within(lane)));
            int32_t slots_next = 0;
            if (32 * (i + kGqWaves) < seg) slots_next = tile_slots(i + kGqWaves);
            wait_vm<8>();                                           // K has landed; V and the next slots may be on their way

            floatx16 sc = cols.scores(qf);
            // keys past the end are hidden
            if (rows < 32) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + 4 * hi + (r & 3) >= rows) sc[r] = -INFINITY;
            }
            Columns::PFrag pf[2];
            cols.weigh(sc, scale_log2, pf);
            wait_vm<0>();
            asm volatile("" :: "v"(slots_next));
            cols.accumulate(pf);
            slots = slots_next;
        }

        // ---- the partial of (range + request): one per head leaves the workgroup.  (The combine kernel divides by the sum that
        //      travels with the partial, and takes the log-sum-exp from it.)
        float out[64 / kGqWaves], mx, lsum;
        cols.combine<kGqWaves>(smem, wave, lane, out, mx, lsum);
        if (qi < ng) {
            const int64_t ph = (int64_t)(w + b) * Hq + h0 + qi;
            float* dst = part_acc + ph * kHeadDim + Columns::first_element<kGqWaves>(wave, lane);
#pragma unroll
            for (int e = 0; e < 64 / kGqWaves; e += 4) *(float4*)(dst + 2 * e) = make_float4(out[e], out[e + 1], out[e + 2], out[e + 3]);
            if (wave == 0 && hi == 0) *(float2*)(part_ml + ph * 2) = make_float2(mx, lsum);
        }
        __syncthreads();                                        // the blocks are read: the next request may gather into them
        t0 = pe;
        ++b;
    }
}

esp_status launch_decode_gq(const void* q, const void* k_pool, const void* v_pool, const int32_t* slot_idx,
                            const int32_t* seq_offsets, int32_t B, int32_t total_tokens, int32_t range, int32_t parts, int32_t nwg,
                            int32_t Hq, int32_t Hkv, float scale_log2, float* part_acc, float* part_ml, hipStream_t stream) {
    const int G = Hq / Hkv;
    const int chunks = (G + 31) / 32;
    if (Hkv > 65535 || chunks > 65535) return fail(ESP_ERR_UNSUPPORTED, "decode: too many heads for one launch");
#define ESP_GQ_LAUNCH(BY_REQUEST, RANGES)                                                                                                 \
    hipLaunchKernelGGL(decode_partial_gq_kernel<BY_REQUEST>, dim3(RANGES, Hkv, chunks), dim3(kGqWaves * 64), 0, stream, (const uint16_t*)q, \
                       (const char*)k_pool, (const char*)v_pool, slot_idx, seq_offsets, B, total_tokens, range, parts, Hq, Hkv,            \
                       scale_log2, part_acc, part_ml)
    if (parts > 0) ESP_GQ_LAUNCH(true, B * parts);
    else if (parts < 0) ESP_GQ_LAUNCH(true, nwg + B);
    else ESP_GQ_LAUNCH(false, nwg);
#undef ESP_GQ_LAUNCH
    return check_launch("decode_partial_gq_kernel");
}

}  // namespace esp
