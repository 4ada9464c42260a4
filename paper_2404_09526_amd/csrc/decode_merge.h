// The log-sum-exp combination of partial results as the decode kernels do it (decode.hip, decode_whole.hip): U partials at a time, N
// output elements a lane.
#pragma once
#include "esp_common.h"

namespace esp {

struct U32x2 { uint32_t x, y; };      // O and the peers' O: the calls ask for 4-byte alignment, not for 8
__device__ __forceinline__ float finite_offset(float m) { return m == -INFINITY ? 0.f : m; }

__device__ __forceinline__ float row16_sum(float x) {
    // all-reduce over the 16 lanes of a DPP row by rotations (8, 4, 2, 1)
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xf, 0xf, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x124, 0xf, 0xf, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x122, 0xf, 0xf, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x121, 0xf, 0xf, false));
    return x;
}

__device__ __forceinline__ void unpack8(const uint4& w, float (&f)[8]) {
    f[0] = bf16_lo(w.x); f[1] = bf16_hi(w.x); f[2] = bf16_lo(w.y); f[3] = bf16_hi(w.y);
    f[4] = bf16_lo(w.z); f[5] = bf16_hi(w.z); f[6] = bf16_lo(w.w); f[7] = bf16_hi(w.w);
}

// A partial whose every score is NaN has the maximum -inf (maxima pass NaN over) and the sum NaN.  It must not be taken for
// an empty one: only a sum of exactly 0 is, and where no maximum is finite the exponentials are taken against 0.
//
// A peer may mark "no token" with a large negative number instead of -inf and leave its O unwritten, so an output whose weight
// is 0 is left out rather than multiplied.  In a group that holds peers only (not `own`) that goes for the group's whole sum: it may be
// such a peer's, taken at weight 1 before anything larger was seen.  (Not for this instance's own partials: those are written
// whenever their sum is not 0, and a NaN in them has to show.)
template <int N>
struct Weighted {
    float M = -INFINITY, L = 0.f;                                   // base-2 maximum and sum of the weights so far
    float acc[N] = {};
    bool own = false;                                               // holds partials of this instance
    // adds U partials (m: base-2 maximum, l: sum, 0 = nothing; v: l-weighted output)
    template <bool PEER, int U>
    __device__ __forceinline__ void add(const float (&m)[U], const float (&l)[U], const float (&v)[U][N]) {
        float mx = M;
#pragma unroll
        for (int u = 0; u < U; ++u) mx = fmaxf(mx, l[u] != 0.f ? m[u] : -INFINITY);
        const float ref = finite_offset(mx);
        const float c_old = __builtin_amdgcn_exp2f(M - ref);
        M = mx;
        L *= c_old;
        const bool drop = PEER && !own && c_old == 0.f;
#pragma unroll
        for (int e = 0; e < N; ++e) acc[e] = drop ? 0.f : acc[e] * c_old;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (l[u] != 0.f) {                                      // keeps the garbage of an empty partial out of the sum
                const float c = __builtin_amdgcn_exp2f(m[u] - ref);
                L += l[u] * c;
                if (PEER && c == 0.f) continue;
#pragma unroll
                for (int e = 0; e < N; ++e) acc[e] += v[u][e] * c;
            }
        }
    }
};

}  // namespace esp
