// esp_partial_attn_decode: one query token per request against the key/value rows this
// instance holds in its token-granular pool (distributed decoding, Sec. 4.2 / Fig. 8; pool at
// single-token granularity, Sec. 6).  The path is HBM-bound (about one flop per byte), so the
// design is about the gather:
//   * a pool row [Hkv, 128] bf16 is contiguous; a wavefront reads 1 KiB of it per load
//     instruction (4 KV heads x 128 elements, 16 bytes per lane), and the 8 wavefronts of a
//     workgroup cover neighbouring 1 KiB pieces of the same rows at the same time, so each
//     random slot is one multi-KiB burst;
//   * split-K with an even share: the concatenated token list of all requests is cut
//     into equal ranges, one per workgroup; a range that crosses request boundaries yields
//     one partial per (workgroup, request), stored at slot workgroup + request, which is
//     unique because both indices only grow along the token list;
//   * dot products on the vector ALU with a 16-lane butterfly per head, online softmax in
//     the exp2 domain per batch of tokens, fp32 accumulation;
//   * a second kernel combines the partials of each (request, head) and writes O, LSE;
//   * short requests go without ranges and combination (decode_whole below, decode_whole.hip).
#include <math.h>

#include <mutex>

#include "decode_merge.h"

namespace esp {

// Split-K partials of the entry point that allocates nothing: a fixed block of device memory that every GPU the
// library runs on holds until the process ends.  In host code the array's name is only a stand-in; its device
// address is asked for once per device (static_scratch below) and that pointer is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[ESP_DECODE_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device (looked up on the first call on that device).
static esp_status static_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return fail(ESP_ERR_HIP, "decode (static scratch): cannot identify the current device");
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr)
            return fail(ESP_ERR_HIP, "decode (static scratch): hipGetSymbolAddress failed on device %d: %s", dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return ESP_OK;
}

constexpr int kDecWaves = 8;         // wavefronts per workgroup
constexpr int kDecTB = 4;            // tokens per wavefront per loop step
constexpr int kDecMaxWG = 1024;      // ranges (workgroups) along the token list

struct DecodeGeom {
    int32_t nwg;        // ranges
    int32_t range;      // tokens per range
    int32_t nhb_wg;     // 1 KiB head blocks handled by one workgroup (1, 2, 4 or 8)
    int32_t nt;         // wavefronts sharing one head block (token interleave) = 8 / nhb_wg
    int32_t ygroups;    // workgroups along y when a row has more than 8 head blocks
    int32_t kept;       // ranges (with nt partials each) that a workspace always has to hold, see decode_range
};

// Head counts of the row-burst kernel: whole 1 KiB head blocks (4 KV heads) that split the 8 wavefronts evenly, and
// one or two query heads per KV head.  Everything else (other KV head counts, larger query groups) goes to the
// matrix-core kernel of decode_gq.hip, which gathers one KV head's 256 bytes of a row at a time but does not pay for
// the size of the group: measured against it, this kernel's dot products on the vector ALU fall behind from four
// query heads per KV head on (16/4: 59 % of the HBM rate here, 71 % there; 64/8: 46 % and 68 %), and lead with one
// or two (32/32: 74 % and 69 %; 32/16: 68 % and 65 %).
static bool decode_burst_layout(int32_t Hq, int32_t Hkv) {
    const int G = Hq / Hkv;
    return (Hkv == 4 || Hkv == 8 || Hkv == 16 || Hkv % 32 == 0) && (G == 1 || G == 2);
}

// Tokens per range.  Two workgroups of either kernel fit a CU, and a call that is only a few times what the chip holds at once
// must not end with a round of a few workgroups: of the ranges that fill 1 .. 16 rounds of workgroups (`rows` of them per
// range; none finer than `least` steps of `step` tokens, at most kDecMaxWG ranges) the one is taken for which the rounds, each
// with a start (search, queries, first slots, combination) and its steps (64 KiB of rows), take the least time.  Measured
// with 1 / 2 / 4 / 8 rounds, us: 32 requests of 2K, 32 / 32 heads 328 / 345 / 344 / 345; 64 of 8K 2158 / 2190 / 2189 / 2186;
// 250 of 20K, 32 / 1 525 / 543 / 541 / 541; 128 of 16K, 32 / 8 2399 / 2244 / 2198 / 2212; 64 of 8K, 64 / 8 430 / 412 / 412 / 428;
// 32 / 4 210 / 213 / 221 / 233.  Where eight or more workgroups gather from the same rows, a head each, a long single round falls
// behind (2 rounds against 1: 128 of 4K, 32 / 8 433 / 456, 30 of 20K, 40 / 8 357 / 373, 100 of 6K, 12 / 12 697 / 706; short ones
// not: 32 of 2K, 32 / 8 50.0 / 50.3), with two to four it does not (24 / 3, 6 / 3, 16 / 2, 32 / 4: one is best by 0 .. 6 %).
// The 8 % stand for the former and do not decide the latter.  Over 18 shapes with 1, 2, 3, 4, 6, 8 and 16 rounds the rule's choice was
// within 3 % of the best in fifteen and 5 % in all.  64 requests of 4K, 32 / 1 heads: 598 workgroups of 512 tokens were three
// rounds of 256, 479 of 640 are one of 512.
// `room`: ranges that the workspace holds (as far as the built-in block would, so that both calls agree); `kept`: ranges that
// every workspace holds which is not refused (those of a simpler rule, by which workspaces are also measured).
static int32_t decode_range(int32_t total_tokens, int64_t step, int64_t least, int64_t rows, int64_t kept, int64_t room) {
    constexpr int64_t kResident = 512;
    constexpr double kStart = 6, kStep = 4.8;                     // microseconds
    const double lag = rows > 1 ? 0.08 : 0;
    int64_t most = kept > room ? kept : room;
    if (most < 1) most = 1;
    if (most > kDecMaxWG) most = kDecMaxWG;
    const int64_t steps = ((int64_t)total_tokens + step - 1) / step;
    int64_t finest = (steps + most - 1) / most;
    if (finest < least) finest = least;
    int64_t best = finest;
    double best_us = 0;
    for (int64_t rounds = 1; rounds <= 16; ++rounds) {
        const int64_t fit = rounds * kResident / rows;             // ranges in so many rounds
        const int64_t s = fit > 0 ? (steps + fit - 1) / fit : steps;
        const int64_t take = s > finest ? s : finest;
        const int64_t wgs = (steps + take - 1) / take * rows;
        const double us = ((double)((wgs + kResident - 1) / kResident) + lag) * (kStart + kStep * (double)take);
        if (rounds == 1 || us < best_us) { best = take; best_us = us; }
        if (take == finest) break;
    }
    return (int32_t)(best * step);
}

// Ranges by request.  Where calls are short, a range that crosses into the next request costs more than its share of the work: its
// requests are worked on one after the other, each with a start and an end (3 us), and such a workgroup ends last.  Then the
// ranges are counted from each request's first token on.  Partials lie at (first token's range + part + request): as far apart as along
// the list, in the same number of slots.  Returns 0: ranges along the whole list; n > 0: n of them for each request, enough for the longest
// by the caller's bound (request_part: no search, but the workgroups of parts that a request does not have start for nothing); -1: as many
// as each request has (request_range).
// Measured in turn, along the list -> by request (* with n for each): 16 of 900, 32 / 8 heads, 23.6 -> 21.7 us; 25 of 196, 32 / 8, 23.8 -> 16.1;
// 99 of 182, 4 / 4, 28.0 -> 20.3; 24 of 950, 32 / 4, 24.9 -> 22.1; 64 of 4800, 32 / 1, 42.8 -> 40.8; 7 of 430, 8 / 8, 17.4 -> 15.1; 6 of 250,
// 8 / 8, 14.3 -> 11.3*; 10 of 183, 32 / 8, 14.4 -> 11.5*.  Found by search where n for each would do: 0.1 .. 0.5 us more (11.5 -> 12.0 us, 10 of
// 183), 25 of 121, 40 / 8, 12.1 -> 14.2.
// The lines, over 240 shapes of 2 .. 226 requests: by request only where its ranges are on the chip at once, expected half a range more
// than along the list for each request.  Beyond, the shorter ranges at the end wait for a whole one: 78 of 3400, 8 / 8 heads, 547
// workgroups for 508, 182 -> 212 us, 43 of 5300, 12 / 12, 238 -> 274 (a few calls of one to five steps would gain: 45 of 176, 40 / 8, 672 for
// 496, 24.9 -> 21.4).  Up to there every call gained or was within 3 %; beyond twelve steps a range nothing is left to gain (10 of 4300, 32 / 32,
// 22 steps, 128.9 / 130.0; 14 of 29600, 4 / 4, 26 steps, 143.5 / 147.4).  n for each: up to 256 workgroups, and up to 512 where
// requests are at least 3 to 20 ranges or ranges are single steps.
static int32_t decode_parts(const DecodeGeom& g, int32_t B, int32_t max_len, int32_t Hq, int32_t Hkv) {
    if (B <= 1) return 0;
    const bool gq = g.nhb_wg == 0;
    const int64_t rows = gq ? (int64_t)Hkv * ((Hq / Hkv + 31) / 32) : g.ygroups;
    const int64_t parts = ((int64_t)max_len + g.range - 1) / g.range;
    const int32_t steps = g.range / (gq ? kGqWaves * 32 : g.nt * kDecTB);
    const bool crossed = (int64_t)B * 20 >= (int64_t)g.nwg * 3, single = gq && steps == 1;
    if (B * parts * rows <= (crossed || single ? 512 : 256)) return (int32_t)parts;
    return (g.nwg + (int64_t)B / 2) * rows <= 512 && steps <= 12 ? -1 : 0;
}

// Short requests, each by one workgroup and KV head (decode_whole.hip), where all of them are on the chip at once, one to a CU, and the
// estimates of both forms' times, in us, say so.  In one launch: a start and an end, then the longest request's walk, which the others'
// traffic slows down, or the traffic where that takes longer (16 wavefronts a CU, or eight with a tile each in flight, do not
// reach the memory's rate: 5.9 TB/s, 6.3 on the matrix cores, 6.8 with one KV head; ranges 6.5 .. 6.8).  In ranges: the lesser of two lines
// in the traffic.  With few KV heads rows are read in shorter pieces by fewer workgroups at a time, and ranges of many short requests cross;
// but more than 32 query heads read a row again, from the caches in ranges.  The lines were fitted to 3770 calls of 1 .. 256 requests of up to
// 64000 tokens, all alike, down to 0.6 and down to 0.1 of the longest, 18 head layouts, rows not cached and repeated.  Of those calls 0.04 of the time
// promised keeps all but nine from losing more than 1.5 % to ranges (at most 8.6 %); to the better form the choice loses
// 0.1 .. 0.4 % on average.  Beyond the stated lengths the estimates are no closer than what there is to gain.
// Measured, all requests alike, rows not cached (in ranges -> in one launch; * stays in ranges): 64 of 1000 and 4000, 4 / 4 heads, 31.1 -> 26.4,
// 89.4 -> 93.3*; 8 of 1000 and 4000, 32 / 32, 31.1 -> 26.2, 90.8 -> 88.6*; 64 of 1000, 8000 and 64000, 8 / 4, 39.0 -> 27.9, 186 -> 182, 1259 -> 1404*; 8 of
// 1000, 16 / 8, 15.1 -> 19.4*; 32 of 1000, 4000 and 64000, 32 / 8, 30.5 -> 26.9, 94.2 -> 89.0, 1258 -> 1340*; 256 of 1000 and 16000, 32 / 1,
// 32.7 -> 25.3, 329 -> 313.  Unequal ones: 64 of 700 .. 7000, 32 / 4, 94.8 -> 113.8*, 16 of 106 .. 3077, 32 / 8 (the longest would walk for 23).
// With more than 256 workgroups the second round's longest request decides: 10 of 186, 32 / 32, 15.1 -> 16.2*, 16 of 57, 64 / 32, 17.4 -> 24.1*,
// though equal lengths gain (16 of 400, 32 / 32, 27.7 -> 23.0*).
constexpr int32_t kWholeMost = 256;                                 // CUs of the card that these times are of
static thread_local int32_t t_forced_decode = 0;                    // this thread's choice instead (set_decode_plan); 0: none
static bool decode_whole(int32_t B, int32_t total_tokens, int32_t max_len, int32_t Hq, int32_t Hkv) {
    const int G = Hq / Hkv;
    const int64_t chunks = (G + 31) / 32;
    if (B > 0 && t_forced_decode != 0) return t_forced_decode == 2;
    const bool burst = decode_burst_layout(Hq, Hkv), few = !burst && Hkv <= 3 && chunks == 1;
    if (total_tokens <= 0 || B * (int64_t)Hkv * chunks > kWholeMost || max_len > (few ? 16384 : 8192)) return false;
    struct Lines { double step, start, token, beside, alone, short_start, short_traffic, long_start, long_traffic; };
    constexpr Lines kBurst1 = {256, 3.2, 0.0104, 0.49, 1.15, 9.2, 1.05, 11, 1.04}, kBurst2 = {128, 4.9, 0.0108, 0.55, 1.15, 11.1, 1.3, 17.4, 1.15};
    constexpr Lines kFew = {1, 5.5, 0.0084, 0.41, 1.035, 9.2, 1.17, 12.8, 1.06}, kMany = {1, 5.0, 0.0095, 0.48, 1.11, 8.6, 1.13, 15, 1.05};
    const Lines& at = burst ? (G == 1 ? kBurst1 : kBurst2) : few ? kFew : kMany;
    const double traffic = (double)total_tokens * Hkv * chunks * (4 * kHeadDim) / 7e6;   // us at 7 TB/s
    const double whole = at.start + fmax(ceil(max_len / at.step) * at.step * at.token + at.beside * traffic, at.alone * traffic);
    const double ranges = fmin(at.short_start + at.short_traffic * traffic, at.long_start + at.long_traffic * traffic);
    return whole < 0.96 * ranges;
}
int32_t set_decode_plan(int32_t plan) {
    const int32_t before = t_forced_decode;
    t_forced_decode = plan;
    return before;
}
int32_t query_decode_plan(int32_t B, int32_t total_tokens, int32_t max_len, int32_t Hq, int32_t Hkv) {
    return decode_whole(B, total_tokens, max_len, Hq, Hkv) ? 2 : 1;
}

static int64_t partial_bytes(int32_t Hq) { return (int64_t)Hq * (kHeadDim + 2) * (int64_t)sizeof(float); }

static DecodeGeom decode_geom(int32_t B, int32_t total_tokens, int32_t Hq, int32_t Hkv, size_t bytes) {
    DecodeGeom g;
    if (bytes > (size_t)ESP_DECODE_STATIC_SCRATCH_BYTES) bytes = ESP_DECODE_STATIC_SCRATCH_BYTES;
    const int64_t room = ((int64_t)bytes - 256) / partial_bytes(Hq) - B;
    // ranges of total_tokens in `unit`s, at least `least` tokens each and at most kDecMaxWG of them
    auto ranges = [&](int64_t least, int64_t unit) {
        int64_t want = ((int64_t)total_tokens + kDecMaxWG - 1) / kDecMaxWG;
        if (want < least) want = least;
        want = (want + unit - 1) / unit * unit;
        return (int32_t)(((int64_t)total_tokens + want - 1) / want);
    };
    if (!decode_burst_layout(Hq, Hkv)) {
        // matrix-core kernel: every wavefront of a workgroup works on the same KV head, a tile of 32 tokens each per step
        g.nhb_wg = 0;
        g.nt = 1;
        g.ygroups = Hkv;
        g.kept = ranges(512, 256);
        g.range = decode_range(total_tokens, kGqWaves * 32, 1, (int64_t)Hkv * ((Hq / Hkv + 31) / 32), g.kept, room);
    } else {
        const int nhb = Hkv / 4;
        g.nhb_wg = nhb < 8 ? nhb : 8;
        g.nt = kDecWaves / g.nhb_wg;
        g.ygroups = (nhb + 7) / 8;
        const int64_t step = (int64_t)g.nt * kDecTB;                 // tokens one workgroup consumes per loop step
        g.kept = ranges(8 * step, step);
        g.range = decode_range(total_tokens, step, 2, g.ygroups, g.kept, room);
    }
    g.nwg = (int32_t)(((int64_t)total_tokens + g.range - 1) / g.range);
    if (g.nwg < 1) g.nwg = 1;
    if (g.kept < 1) g.kept = 1;
    return g;
}

// workspace: fp32 accumulators [slots][Hq][128], then (m, l) pairs [slots][Hq][2]
static size_t decode_slots(const DecodeGeom& g, int32_t B) { return (size_t)g.nwg + (size_t)B; }

// the least a call takes, and what it asks for: room for the ranges it would like to have
size_t decode_least_workspace_bytes(int32_t B, int32_t total_tokens, int32_t Hq, int32_t Hkv) {
    const DecodeGeom g = decode_geom(B, total_tokens, Hq, Hkv, 0);
    return ((size_t)g.kept + (size_t)B) * (size_t)g.nt * (size_t)partial_bytes(Hq) + 256;
}
size_t decode_workspace_bytes(int32_t B, int32_t total_tokens, int32_t Hq, int32_t Hkv) {
    const DecodeGeom g = decode_geom(B, total_tokens, Hq, Hkv, ESP_DECODE_STATIC_SCRATCH_BYTES);
    const size_t want = decode_slots(g, B) * (size_t)partial_bytes(Hq) + 256, least = decode_least_workspace_bytes(B, total_tokens, Hq, Hkv);
    return want > least ? want : least;
}

// Bound by HBM.  A step is a chain: slots, rows (8 KiB a wavefront), products.  The chains of two steps overlap: rows are
// loaded a step ahead and slots two (scalar loads: they do not queue behind the rows), in registers that still leave room
// for two workgroups per CU.  The wavefronts that share a head block (rows of less than 8 KiB) leave one partial together;
// one each made the combination read up to eight times as much.  With decode_range's rounds, before -> now: 32 requests of 2K,
// 32 / 32 heads 346 -> 331 us (the combination 9.5 -> 6.9), 64 of 8K 2208 -> 2155 us (6.75 TB/s), 100 of 10K, 8 / 8 heads,
// the rounds alone 751 -> 741 us.
template <int G>
__global__ __launch_bounds__(kDecWaves * 64, 4) void decode_partial_kernel(
    const uint16_t* __restrict__ q, const uint4* __restrict__ k_pool, const uint4* __restrict__ v_pool,
    const int32_t* __restrict__ slot_idx, const int32_t* __restrict__ seq_offsets, int32_t B, int32_t total_tokens,
    int32_t range, int32_t parts, int32_t nhb_wg, int32_t Hq, int32_t Hkv, float scale_log2, float* __restrict__ part_acc,
    float* __restrict__ part_ml) {
    // accumulators (8 per lane and query head), maximum and sum of every wavefront, for the combination within the workgroup
    __shared__ float lds[kDecWaves][G][10][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nt = kDecWaves / nhb_wg;
    const int nt_log = __builtin_ctz(nt);
    const int hb_wg = wave & (nhb_wg - 1);
    const int hb = blockIdx.y * 8 + hb_wg;           // 1 KiB head block of the row
    const int tsub = wave / nhb_wg;                  // token interleave index among nt wavefronts
    int w = blockIdx.x;
    const uint32_t row_bytes = (uint32_t)Hkv * (kHeadDim * 2);
    const uint32_t lane_off = (uint32_t)(hb * 64 + lane) * 16;  // this lane's piece within a row
    const int kvh = hb * 4 + (lane >> 4);                      // KV head of this lane
    const int dseg = (lane & 15) * 8;                          // first of its 8 elements

    int b;
    int32_t r0, t1, req_end;
    if (parts != 0) {
        const RequestRange at = parts > 0 ? request_part(w, parts, range, B, seq_offsets) : request_range(w, range, B, seq_offsets, lane);
        b = at.b; r0 = at.t0; t1 = req_end = min(at.t1, total_tokens); w = at.w;   // (never past the slot list)
        if (r0 >= t1) return;
    } else {
        r0 = w * range;
        t1 = r0 + min(range, total_tokens - r0);                    // (r0 + range may be past 2^31)
        if (r0 >= t1) return;
        const RequestAt at = request_of(r0, seq_offsets, B, lane);
        b = at.b; req_end = at.end;
    }
    int32_t t0 = r0;
    while (t0 < t1 && b < B) {                                  // (tokens past the offsets' end belong to no request)
        if (t0 > r0) req_end = seq_offsets[b + 1];
        if (req_end <= t0) { ++b; continue; }                   // empty request, or the last one where the range starts past its end
        const int32_t pe = min(t1, req_end);
        // this wavefront's tokens of the request: i0 .. i1 - 1
        const int i0 = max(t0 - r0 - tsub + nt - 1, 0) >> nt_log, i1 = max(pe - r0 - tsub + nt - 1, 0) >> nt_log;

        // slots of tokens i .. i + 3 of those (past the last: the last one's again, hidden below), the same for all lanes; then
        // their K and V pieces
        struct Slots { uint32_t s[kDecTB]; };
        auto slots_of = [&](int i) {
            Slots r;
#pragma unroll
            for (int u = 0; u < kDecTB; ++u) r.s[u] = (uint32_t)slot_idx[r0 + tsub + (min(i + u, i1 - 1) << nt_log)];
            return r;
        };
        auto load = [&](uint4 (&kw)[kDecTB], uint4 (&vw)[kDecTB], const Slots& sl) {
#pragma unroll
            for (int u = 0; u < kDecTB; ++u) {
                const uint64_t row = (uint64_t)sl.s[u] * row_bytes;
                kw[u] = load_once((const uint4*)((const char*)k_pool + row + lane_off));
                vw[u] = load_once((const uint4*)((const char*)v_pool + row + lane_off));
            }
        };
        uint4 ka[kDecTB], va[kDecTB], kb[kDecTB], vb[kDecTB];
        Slots ahead = {};
        if (i0 < i1) {
            load(ka, va, slots_of(i0));
            ahead = slots_of(i0 + kDecTB);
        }

        float qf[G][8];
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            uint4 qw = *(const uint4*)(q + ((int64_t)b * Hq + kvh * G + gi) * kHeadDim + dseg);
            unpack8(qw, qf[gi]);
#pragma unroll
            for (int e = 0; e < 8; ++e) qf[gi][e] *= scale_log2;
        }
        float m[G], l[G], acc[G][8];
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            m[gi] = -INFINITY; l[gi] = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[gi][e] = 0.f;
        }

        auto attend = [&](const uint4 (&kw)[kDecTB], const uint4 (&vw)[kDecTB], int i) {
            float s[kDecTB][G];
#pragma unroll
            for (int u = 0; u < kDecTB; ++u) {
                float kf[8];
                unpack8(kw[u], kf);
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
                    float d = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) d = fmaf(qf[gi][e], kf[e], d);
                    d = row16_sum(d);
                    s[u][gi] = i + u < i1 ? d : -INFINITY;
                }
            }
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
                float mx = m[gi];
#pragma unroll
                for (int u = 0; u < kDecTB; ++u) mx = fmaxf(mx, s[u][gi]);
                // the first token of a step is always valid, so mx is finite here
                float alpha = __builtin_amdgcn_exp2f(m[gi] - mx);
                m[gi] = mx;
                l[gi] *= alpha;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[gi][e] *= alpha;
#pragma unroll
                for (int u = 0; u < kDecTB; ++u) s[u][gi] = __builtin_amdgcn_exp2f(s[u][gi] - mx);
            }
#pragma unroll
            for (int u = 0; u < kDecTB; ++u) {
                float vf[8];
                unpack8(vw[u], vf);
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
                    l[gi] += s[u][gi];
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[gi][e] = fmaf(s[u][gi], vf[e], acc[gi][e]);
                }
            }
        };
        // two steps per trip: while one is worked on, the next one's rows and the slots of the one after it are on their way
        // (no condition within a trip: a path that may have skipped a load makes the compiler wait for all of them)
        int i = i0;
        for (; i + 2 * kDecTB < i1; i += 2 * kDecTB) {
            load(kb, vb, ahead);
            ahead = slots_of(i + 2 * kDecTB);
            attend(ka, va, i);
            load(ka, va, ahead);
            ahead = slots_of(i + 3 * kDecTB);
            attend(kb, vb, i + kDecTB);
        }
        if (i + kDecTB < i1) {
            load(kb, vb, ahead);
            attend(ka, va, i);
            attend(kb, vb, i + kDecTB);
        } else if (i < i1) {
            attend(ka, va, i);
        }

        // partial of (range w, request b): slot w + b.  The wavefronts that share a head block combine theirs through LDS,
        // each for 8 / nt of a lane's 8 elements.
        const int64_t pslot = (int64_t)(w + b) * Hq;
        if (nt == 1) {
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
                const int64_t ph = pslot + kvh * G + gi;
                float4* dst = (float4*)(part_acc + ph * kHeadDim + dseg);
                dst[0] = make_float4(acc[gi][0], acc[gi][1], acc[gi][2], acc[gi][3]);
                dst[1] = make_float4(acc[gi][4], acc[gi][5], acc[gi][6], acc[gi][7]);
                if ((lane & 15) == 0) *(float2*)(part_ml + ph * 2) = make_float2(m[gi], l[gi]);
            }
        } else {
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
#pragma unroll
                for (int e = 0; e < 8; ++e) lds[wave][gi][e][lane] = acc[gi][e];
                lds[wave][gi][8][lane] = m[gi];
                lds[wave][gi][9][lane] = l[gi];
            }
            __syncthreads();
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
                const int64_t ph = pslot + kvh * G + gi;
                float mx = -INFINITY, lsum = 0.f;
                for (int u = 0; u < nt; ++u) mx = fmaxf(mx, lds[hb_wg + u * nhb_wg][gi][8][lane]);
                float out[4] = {0.f, 0.f, 0.f, 0.f};
                const int per = 8 >> nt_log;                        // 4, 2 or 1
                for (int u = 0; u < nt; ++u) {
                    const float (&src)[10][64] = lds[hb_wg + u * nhb_wg][gi];
                    const float lu = src[9][lane];
                    const float c = lu > 0.f ? __builtin_amdgcn_exp2f(src[8][lane] - mx) : 0.f;   // no token of this request: nothing to add (a NaN sum shows in lu * c)
                    lsum += lu * c;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (e < per) out[e] += src[tsub * per + e][lane] * c;
                }
                float* dst = part_acc + ph * kHeadDim + dseg + tsub * per;
                if (per == 4) *(float4*)dst = make_float4(out[0], out[1], out[2], out[3]);
                else if (per == 2) *(float2*)dst = make_float2(out[0], out[1]);
                else dst[0] = out[0];
                if (tsub == 0 && (lane & 15) == 0) *(float2*)(part_ml + ph * 2) = make_float2(mx, lsum);
            }
            __syncthreads();                                        // read: the next request may overwrite it
        }
        t0 = pe;
        ++b;
    }
}

// Combination of the partials of a (request, head) pair: groups of 32 lanes, four output elements a lane, take the
// partials in turn, four at a time, and then combine among themselves.  The time is latency (offsets -> partials -> result)
// and, for long requests, the number of trips through the partials; so the loads of a trip are issued together, and a pair
// gets a workgroup (GROUPS = 8) where its request may have more than 32 partials, a wavefront (GROUPS = 2, four
// pairs per workgroup, no LDS) otherwise.  Measured (64 lanes a partial, one at a time, always a workgroup -> this):
// 32 requests of 2K, 32 / 32 heads, 1006 ranges, 3 peers 20.7 -> 9.6 us; 64 of 4K, 32 / 1 heads 12.0 -> 5.7 us; 128 of 16K,
// 32 / 8 heads 15.9 -> 12.4 us; 89 of 172, 32 / 1 heads, 3 peers 5.3 -> 4.6 us.
//
// PEERS: the master of a multi-master decode (Sec. 4.2) also holds the partial results its peers returned for the
// same queries (bf16 O, natural-log LSE).  They enter the same log-sum-exp combination here, shared out among the groups
// like the partials, so the local result is never rounded to bf16 on its own and no separate merge launch follows.
constexpr int kCombineShort = 32;
template <int GROUPS, bool PEERS>
__global__ __launch_bounds__(256) void decode_combine_kernel(const int32_t* __restrict__ seq_offsets,
                                                             int32_t range, int32_t parts, int32_t Hq, int32_t pairs,
                                                             const float* __restrict__ part_acc,
                                                             const float* __restrict__ part_ml,
                                                             MergeArgs peers, int32_t n_peers,
                                                             U32x2* __restrict__ O, float* __restrict__ LSE) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 31, grp = threadIdx.x >> 5;
    const int64_t at = row_block() * (8 / GROUPS) + grp / GROUPS;
    if (at >= pairs) return;                                        // (a whole workgroup, or a pair is a wavefront and no barrier follows)
    const int pair = (int)at, g = grp % GROUPS;
    const int b = pair / Hq, h = pair - b * Hq;
    const int32_t s0 = seq_offsets[b], s1 = seq_offsets[b + 1];
    Weighted<4> sum;
    if (s1 > s0) {
        const int w_lo = s0 / range;
        const int64_t first = w_lo + b;                             // the slots of consecutive ranges
        const int whole = (s1 - s0 - 1) / range + 1, n = parts == 0 ? (s1 - 1) / range - w_lo + 1 : parts > 0 ? min(parts, whole) : whole;
        for (int i = g; i < n; i += GROUPS * U) {
            float m[U], l[U];
            float v[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = i + u * GROUPS;
                const int64_t ph = (first + min(k, n - 1)) * Hq + h;
                const float2 ml = *(const float2*)(part_ml + ph * 2);
                const float4 x = load_once((const float4*)(part_acc + ph * kHeadDim + lane * 4));
                v[u][0] = x.x; v[u][1] = x.y; v[u][2] = x.z; v[u][3] = x.w;
                m[u] = ml.x;
                l[u] = k < n ? ml.y : 0.f;
            }
            sum.template add<false>(m, l, v);
        }
    }
    if (PEERS) {
        sum.own = sum.L != 0.f;
        for (int p0 = g; p0 < n_peers; p0 += GROUPS * U) {
            float m[U], l[U];
            float v[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = p0 + u * GROUPS, q = min(p, n_peers - 1);
                const float lse = peers.LSE_parts[q][pair];
                const U32x2 o = ((const U32x2*)peers.O_parts[q])[(int64_t)pair * (kHeadDim / 4) + lane];
                m[u] = lse * kLog2e;
                l[u] = p < n_peers && lse != -INFINITY ? 1.f : 0.f;  // a peer's rows are normalised
                v[u][0] = bf16_lo(o.x); v[u][1] = bf16_hi(o.x); v[u][2] = bf16_lo(o.y); v[u][3] = bf16_hi(o.y);
            }
            sum.template add<true>(m, l, v);
        }
    }
    const float M = sum.M, L = sum.L;
    const float (&acc)[4] = sum.acc;
    const bool own = sum.own;
    // ---- the groups' results: exchanged by shuffles within a wavefront, through LDS otherwise
    float mx, Lt = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
    if (GROUPS == 2) {
        const float M2 = __shfl_xor(M, 32);
        mx = fmaxf(M, M2);
        const float c = __builtin_amdgcn_exp2f(M - finite_offset(mx));
        Lt = L * c;
        Lt += __shfl_xor(Lt, 32);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = PEERS && !own && c == 0.f ? 0.f : acc[e] * c;
            o[e] += __shfl_xor(o[e], 32);
        }
    } else {
        __shared__ float sm[8], sl[8];
        __shared__ bool so[8];
        __shared__ float4 sa[8][32];
        if (lane == 0) { sm[grp] = M; sl[grp] = L; so[grp] = own; }
        sa[grp][lane] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        __syncthreads();
        if (g != 0) return;
        mx = sm[0];
#pragma unroll
        for (int u = 1; u < 8; ++u) mx = fmaxf(mx, sm[u]);
        const float ref = finite_offset(mx);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float c = __builtin_amdgcn_exp2f(sm[u] - ref);      // exp2(-inf) = 0 for an idle group
            const float4 t = sa[u][lane];
            Lt += sl[u] * c;
            if (PEERS && !so[u] && c == 0.f) continue;
            o[0] += t.x * c; o[1] += t.y * c; o[2] += t.z * c; o[3] += t.w * c;
        }
    }
    if (g != 0) return;
    const float inv = Lt == 0.f ? 0.f : 1.0f / Lt;                  // no token anywhere: exactly 0
    O[(int64_t)pair * (kHeadDim / 4) + lane] = U32x2{pack_bf16(o[0] * inv, o[1] * inv), pack_bf16(o[2] * inv, o[3] * inv)};
    if (lane == 0) LSE[pair] = Lt == 0.f ? -INFINITY : (mx + __builtin_amdgcn_logf(Lt)) * kLn2;
}

esp_status launch_decode_static(const void* q, const void* k_pool, const void* v_pool, const int32_t* slot_idx,
                                const int32_t* seq_offsets, int32_t B, int32_t total_tokens, int32_t max_len, int32_t Hq,
                                int32_t Hkv, float softmax_scale, void* O, float* LSE, hipStream_t stream) {
    const size_t need = decode_least_workspace_bytes(B, total_tokens, Hq, Hkv);
    if (need > (size_t)ESP_DECODE_STATIC_SCRATCH_BYTES)
        return fail(ESP_ERR_WORKSPACE, "decode (static scratch): this call needs %zu bytes of scratch memory, the built-in block holds %zu; "
                    "use esp_partial_attn_decode with a workspace", need, (size_t)ESP_DECODE_STATIC_SCRATCH_BYTES);
    void* ws = nullptr;
    const esp_status st = static_scratch(&ws);
    if (st != ESP_OK) return st;
    return launch_decode(q, k_pool, v_pool, slot_idx, seq_offsets, B, total_tokens, max_len, Hq, Hkv, softmax_scale, O, LSE, ws,
                         (size_t)ESP_DECODE_STATIC_SCRATCH_BYTES, stream);
}

esp_status launch_decode(const void* q, const void* k_pool, const void* v_pool, const int32_t* slot_idx,
                         const int32_t* seq_offsets, int32_t B, int32_t total_tokens, int32_t max_len, int32_t Hq,
                         int32_t Hkv, float softmax_scale, void* O, float* LSE, void* workspace, size_t workspace_bytes,
                         hipStream_t stream, const MergeArgs* peers, int32_t n_peers) {
    if (decode_whole(B, total_tokens, max_len, Hq, Hkv))
        return launch_decode_whole(q, k_pool, v_pool, slot_idx, seq_offsets, B, total_tokens, Hq, Hkv, decode_burst_layout(Hq, Hkv),
                                   softmax_scale * kLog2e, O, LSE, peers, n_peers, stream);
    if ((int64_t)B * Hq > INT32_MAX) return fail(ESP_ERR_INVALID_ARG, "decode: too many rows for one launch");
    const int32_t pairs = B * Hq;
    DecodeGeom g = decode_geom(B, total_tokens, Hq, Hkv, workspace_bytes);
    const int32_t parts = decode_parts(g, B, max_len, Hq, Hkv);
    size_t n = decode_slots(g, B) * (size_t)Hq;
    float* part_acc = (float*)workspace;
    float* part_ml = part_acc + n * kHeadDim;
    const int G = Hq / Hkv;
    if (total_tokens > 0 && g.nhb_wg == 0) {
        esp_status st = launch_decode_gq(q, k_pool, v_pool, slot_idx, seq_offsets, B, total_tokens, g.range, parts, g.nwg, Hq, Hkv,
                                         softmax_scale * kLog2e, part_acc, part_ml, stream);
        if (st != ESP_OK) return st;
    } else if (total_tokens > 0) {
        dim3 grid(parts > 0 ? B * parts : parts < 0 ? g.nwg + B : g.nwg, g.ygroups), block(kDecWaves * 64);
        float sl2 = softmax_scale * kLog2e;
#define ESP_DECODE_LAUNCH(GG)                                                                                   \
    hipLaunchKernelGGL(decode_partial_kernel<GG>, grid, block, 0, stream, (const uint16_t*)q,                   \
                       (const uint4*)k_pool, (const uint4*)v_pool, slot_idx, seq_offsets, B, total_tokens,      \
                       g.range, parts, g.nhb_wg, Hq, Hkv, sl2, part_acc, part_ml)
        switch (G) {
            case 1: ESP_DECODE_LAUNCH(1); break;
            case 2: ESP_DECODE_LAUNCH(2); break;
            default: return fail(ESP_ERR_UNSUPPORTED, "decode: Hq/Hkv=%d unsupported", G);
        }
#undef ESP_DECODE_LAUNCH
        esp_status st = check_launch("decode_partial_kernel");
        if (st != ESP_OK) return st;
    }
    const bool with_peers = peers != nullptr && n_peers > 0;
    const bool wave = (int64_t)max_len / g.range + 2 <= kCombineShort;
#define ESP_COMBINE_LAUNCH(GROUPS, PEERS)                                                                                 \
    hipLaunchKernelGGL((decode_combine_kernel<GROUPS, PEERS>), row_grid(((int64_t)pairs + 8 / GROUPS - 1) / (8 / GROUPS)), dim3(256), 0, \
                       stream, seq_offsets, g.range, parts, Hq, pairs, (const float*)part_acc, (const float*)part_ml,        \
                       with_peers ? *peers : MergeArgs{}, n_peers, (U32x2*)O, LSE)
    if (wave && with_peers) ESP_COMBINE_LAUNCH(2, true);
    else if (wave) ESP_COMBINE_LAUNCH(2, false);
    else if (with_peers) ESP_COMBINE_LAUNCH(8, true);
    else ESP_COMBINE_LAUNCH(8, false);
#undef ESP_COMBINE_LAUNCH
    return check_launch("decode_combine_kernel");
}

}  // namespace esp
