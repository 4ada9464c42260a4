// What a wavefront that works alone on tiles of 32 keys does with each of them (decode_gq.hip, prefill_short.hip; gfx950 only): 32
// columns (the query heads of a KV head, or packed (token, query head) rows) against the tile's K and V rows in an LDS block of
// the wavefront's own, with an exact running maximum:
//   S^T [32 keys x 32 columns] = K_tile [32 x 128] Q^T [128 x 32],   O^T [128 x 32 columns] += V_tile^T [128 x 32] P^T [32 x 32]
// and how the wavefronts of a workgroup combine their results when their tiles are done.
#pragma once
#include "mfma_tile.h"

namespace esp {

constexpr int kColKBytes = 32 * 256;          // K and V rows of 256 bytes, their 16-byte chunks XOR-swizzled by the row
constexpr int kColVBytes = 32 * 256;
constexpr int kColWaveBytes = 66 * 256;       // the tile, and two rows more for the combination

// Both tiles are moved by eight transfers of 1 KiB: lane L of transfer n fills chunk L % 16 of row col_row, with these bytes of the row
// in memory: chunk c of row r holds chunk c ^ (r % 16) of K, c ^ 4 (r % 4) of V.  (K padded to rows of 272 bytes took nine, and a lookup of the
// slots of its own; decode, before -> now: 64 requests of 8K, 32 / 8 heads, 551.3 -> 548.4 us, 100 of 2K, 40 / 8, 236.1 -> 234.1, 24 of
// 950, 32 / 4, 24.0 -> 23.9.)
__device__ __forceinline__ int col_row(int n, int lane) { return 4 * n + (lane >> 4); }
__device__ __forceinline__ int col_k_within(int n, int lane) { return ((lane & 15) ^ (lane >> 4) ^ (4 * (n & 3))) << 4; }
__device__ __forceinline__ int col_v_within(int lane) { return ((lane & 15) ^ (lane >> 4 << 2)) << 4; }

struct Columns {
    floatx16 oacc[4];
    float m;                 // running maximum of this column's scaled scores (both halves of the wavefront hold the same)
    float l, l_r;            // this half's sums of the probabilities: as computed, and as rounded to bf16
    uint32_t k_rd, v_rd[4];  // operand read addresses

    __device__ __forceinline__ void place(uint32_t lds_k, int lane) {
        const int qi = lane & 31, hi = lane >> 5, j16 = lane & 15, jq = j16 >> 2, dblk = (lane >> 4) & 1;
        k_rd = lds_k + qi * 256 + ((hi ^ (qi & 15)) << 4);
#pragma unroll
        for (int db = 0; db < 4; ++db)
            v_rd[db] = lds_k + kColKBytes + (4 * hi + jq) * 256 + ((((db ^ jq) << 2) + 2 * dblk + ((j16 & 3) >> 1)) << 4) + (j16 & 1) * 8;
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
        m = -INFINITY;
        l = l_r = 0.f;
    }
    // K has landed.  Register r of a lane is the score of key 8 (r / 4) + 4 (lane / 32) + r % 4 of the tile.
    __device__ __forceinline__ floatx16 scores(const bf16x8 (&qf)[8]) const {
        floatx16 sc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const bf16x8 kf = *(const ESP_LDS bf16x8*)(uintptr_t)(k_rd ^ (t << 5));
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[t], sc, 0, 0, 0);
        }
        return sc;
    }
    union PFrag { uint32_t u[4]; bf16x8 v; };
    union VFrag { short4_t s[2]; bf16x8 v; };
    // scores to probabilities: pf holds them in bf16 (hidden keys: scores of -inf)
    __device__ __forceinline__ void weigh(const floatx16& sc, float scale_log2, PFrag (&pf)[2]) {
        float tmax = sc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, sc[r]);
        tmax = half_swap_max(tmax) * scale_log2;
        const float m_new = fmaxf(m, tmax);
        // nothing visible so far and nothing in this tile (or only scores of -inf and NaN): exp2(-inf - -inf) must not leak
        // a NaN into sums that are still zero
        const float alpha = (m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
            l *= alpha; l_r *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
        }
        const float m_sub = (m == -INFINITY) ? 0.f : m;
        float psum = 0.f, psum_r = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[2 * c], scale_log2, -m_sub));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[2 * c + 1], scale_log2, -m_sub));
            psum += p0 + p1;
            const uint32_t pk = pack_bf16(p0, p1);
            psum_r = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), __builtin_bit_cast(bf16x2, 0x3f803f80u), psum_r, false);
            pf[c >> 2].u[c & 3] = pk;
        }
        l += psum; l_r += psum_r;
    }
    // V has landed: O^T += V^T P^T, 16 keys per step.  The tile's LDS reads are complete when this returns.
    __device__ __forceinline__ void accumulate(const PFrag (&pf)[2]) {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const int t2 = p >> 2, db = p & 3;
            const uint32_t vp = v_rd[db] + (16 * t2) * 256;
            VFrag fv;
            fv.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ESP_LDS short4_t*)(uintptr_t)(vp));
            fv.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ESP_LDS short4_t*)(uintptr_t)(vp + 8 * 256));
            oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv.v, pf[t2].v, oacc[db], 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }

    // Combination of the WAVES wavefronts of a workgroup, whose LDS blocks lie kColWaveBytes apart from smem on.  O^T accumulated the
    // ROUNDED probabilities, so each wavefront first brings it to the scale of its unrounded sum; then register rho of every lane
    // goes to row rho of the wavefront's block (64 lanes x 4 bytes a row), maximum and sum to two more.  Wavefront j combines
    // the registers from 64 / WAVES * j on of all of them into out, with the column's maximum mx and sum lsum.  out[e] is
    // element first_element() + 2 e + e' of the column for e = 0, 4, ... and e' = 0 .. 3.
    template <int WAVES>
    __device__ __forceinline__ void combine(unsigned char* smem, int wave, int lane, float (&out)[64 / WAVES], float& mx, float& lsum) const {
        constexpr int N = 64 / WAVES;
        const float l_tot = half_swap_sum(l), lr_tot = half_swap_sum(l_r);
        const float fix = lr_tot > 0.f ? l_tot / lr_tot : 0.f;
        float* mine = (float*)(smem + wave * kColWaveBytes);
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) mine[(16 * db + r) * 64 + lane] = oacc[db][r] * fix;
        mine[64 * 64 + lane] = m;
        mine[65 * 64 + lane] = l_tot;
        __syncthreads();
        float mw[WAVES];
        mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < WAVES; ++u) {
            mw[u] = ((const float*)(smem + u * kColWaveBytes))[64 * 64 + lane];
            mx = fmaxf(mx, mw[u]);
        }
        lsum = 0.f;
#pragma unroll
        for (int e = 0; e < N; ++e) out[e] = 0.f;
#pragma unroll
        for (int u = 0; u < WAVES; ++u) {
            const float* blk = (const float*)(smem + u * kColWaveBytes);
            const float lu = blk[65 * 64 + lane];
            // a wavefront that saw no key (sum 0) has nothing to add; a NaN sum shows in lu * c
            const float c = lu > 0.f ? __builtin_amdgcn_exp2f(mw[u] - mx) : 0.f;
            lsum += lu * c;
#pragma unroll
            for (int e = 0; e < N; ++e) out[e] += blk[(N * wave + e) * 64 + lane] * c;
        }
    }
    template <int WAVES>
    static __device__ __forceinline__ int first_element(int wave, int lane) { return 2 * (64 / WAVES) * wave + 4 * (lane >> 5); }
};

}  // namespace esp
