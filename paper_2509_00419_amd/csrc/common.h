// Shared declarations of the library's translation units: the context, the
// per-op launch entry points (host side) and a few device helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <stdio.h>

#include "../../include/lvlm.h"

struct lvlm_ctx {
    int device;
    void *ws;
    size_t ws_bytes;
    char err[256];
    // optional per-kernel timing (eager launches only): one event pair per bracket of launches
    bool prof_on;
    bool prof_open, prof_first;  // a bracket is open / it has launched nothing yet
    int prof_n, prof_cap;
    hipEvent_t *prof_ev;        // 2 * prof_cap events
    const char **prof_name;     // prof_cap static strings
};

namespace lvlm {

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---- workspace layouts (host arithmetic shared by the size query and the launch) ----
// The keys of all (batch, KV head) pairs, one pair behind the other in steps, in consecutive shares: the first `longer` of
// them of size + 1 steps, the others of `size`.  A share is part of one pair or reaches into the next ones.
struct KeyRuns {
    int steps;              // of a pair
    int shares, size, longer;
#if defined(__HIPCC__)
    __device__ __forceinline__ int begin(int j) const { return j * size + (j < longer ? j : longer); }
    __device__ __forceinline__ int share_of(int step) const {
        const int cut = longer * (size + 1);
        return step < cut ? step / (size + 1) : longer + (step - cut) / size;
    }
    __device__ __forceinline__ int first(int pair) const { return share_of(pair * steps); }       // share with the pair's first step
    __device__ __forceinline__ int count(int pair) const { return share_of(pair * steps + steps - 1) - first(pair) + 1; }
#endif
};
struct ScoreShares {
    int waves;     // per workgroup, two query chunks each; 0: not that form
    KeyRuns runs1, runs2;   // the normaliser sweep over all keys, the column sums over the image keys
};
// Position of query row 0 as the kernels take it.  A row at or behind the last key sees every key, so all positions beyond the
// keys are one, and a row's number (below 2^16) added to this one cannot overflow.
inline int first_row_position(const lvlm_score_desc &d) { return d.q_pos0 < d.N ? d.q_pos0 : d.N; }
// Whole steps of the keys [jb, je), from jb on, that a row at position `pos` sees: inside the range whatever the position is.
__host__ __device__ inline int steps_seen(int jb, int je, int pos, int step) {
    const int last = pos < je - 1 ? pos : je - 1;
    return last >= jb + step - 1 ? (last - jb + 1) / step : 0;
}
struct ScoreWs {
    size_t part_m, part_l, lse2, colpart, total;
    int nkb;       // key blocks of the normaliser pass
    int block_keys;
    int rs, cps;   // row splits per key block, query chunks per split
    bool single;   // short sequence: both passes in one launch, one part of column sums per query chunk
    bool shared_tiles;   // ... with four query chunks per workgroup sharing the key tiles through LDS
    int key_segs;        // ... and the keys cut into this many runs, a launch per sweep (1 = one launch)
    ScoreShares shares, shares_given;   // much work: the keys in equal shares, a launch per sweep; the same with the normalisers given
    int rows, rows_given;   // few query rows: chunks of 16 of them, one workgroup each, in one launch (0: not that form); the
                            // same with the normalisers given
};
ScoreWs score_ws(const lvlm_score_desc &d);

struct ProbsWs {
    size_t colpart, total;
    int rs;        // row groups of 32 rows (heads of a group x query rows) that are summed separately
};
ProbsWs probs_ws(const lvlm_probs_desc &d);

struct PrefillWs {
    size_t lse_t, score, total;   // normalisers of the last T rows, the score pass's workspace
};
PrefillWs prefill_ws(const lvlm_prefill_desc &d);
lvlm_score_desc prefill_score_desc(const lvlm_prefill_desc &d);   // the score call the last T rows amount to

struct MergeWs {
    size_t rank_part, kept, partial, sorted, total;
    int n_split;   // always 1: the rank kernel leaves complete ranks
    int n_chunk;   // source-row chunks of the gather kernel (partial sums per chunk)
    int rows_per_chunk;
    int max_row_elems;
};
MergeWs merge_ws(const lvlm_merge_desc &d, const lvlm_plane *planes);

struct SimWs {
    size_t rank, dom_of, keep_idx, rest_idx, inv_norm, best, assign, rank2, order, owner, sorted, total;
};
SimWs sim_ws(const lvlm_merge_desc &d);

struct KvWs {
    size_t src, total;
};
KvWs kv_ws(const lvlm_kv_desc &d);
// Keys per thread (0: any number, from memory), threads and waves per SIMD of kv_select_kernel, by length and number of heads
// (times of the kernel alone, us, other form -> this one).
//   One head to a compute unit: 1024 threads beyond 1024 entries (512 threads: 64 heads of 2048 13.4 -> 12.9, 256 heads of 1500
//   13.4 -> 13.0, 64 heads of 4096 18.3 -> 15.8), but 512 threads to 1024 (256 heads of 500 13.0 -> 12.5) and, with five keys
//   instead of four, to 2560 (256 heads of 2300 14.6 -> 14.5).
//   More: as many heads on a unit as may be.  256 threads to 1280 entries (512 threads: 1000 heads of 1280 25.3 -> 18.1); to 2048
//   entries 512 threads while three heads to a unit are all of them (256 threads: 640 heads of 2048 19.9 -> 18.4), then 256
//   (1000 heads of 2048 27.6 -> 22.1); 512 threads to 8192 (1024 threads: 300 heads of 2560 26.2 -> 17.2, 768 heads of 4096
//   42.2 -> 27.3; whole calls: 320 heads of 8192 59.9 -> 51.1, 2048 heads 265 -> 214).
//   Eight keys per thread do not fit the registers of six waves per SIMD (four go to scratch memory): that form only where it
//   saves a turn of the chip (1536 heads of 2048 by 256 threads 33.7 -> 28.2, 640 heads of 4096 by 512 33.4 -> 26.6), the other
//   where it does not (1000 heads 23.4 -> 22.1, 2048 heads of 1600 36.9 -> 35.8; 512 heads of 4096 22.8 -> 21.6).
struct SelectForm { int keys, threads, waves; };
inline SelectForm kv_select_form(int bound, long long heads) {
    const bool one = heads <= 256;      // a compute unit's
    auto turns = [&](int per_unit) { return (heads + 256 * per_unit - 1) / (256 * per_unit); };
    if (bound <= 1024) return one ? SelectForm{4, 512, 6} : SelectForm{5, 256, 6};
    if (bound <= 1280 && !one) return {5, 256, 6};
    if (bound <= 2048) return one ? SelectForm{2, 1024, 4} : heads <= 768 ? SelectForm{4, 512, 6} : SelectForm{8, 256, turns(6) < turns(5) ? 6 : 5};
    if (bound <= 2560) return {5, 512, 6};
    if (bound <= 4096) return one ? SelectForm{4, 1024, 4} : SelectForm{8, 512, turns(3) < turns(2) ? 6 : 4};
    if (bound <= 8192) return one ? SelectForm{8, 1024, 4} : SelectForm{16, 512, 4};
    return bound <= 17408 ? SelectForm{17, 1024, 4} : SelectForm{0, 1024, 4};
}
constexpr int kFillRows = 32;      // moves per batch of kv_fill_kernel
// Workgroups of kv_fill_kernel per head: one for every batch of moves the longest head can have, while that is at most 16384 in all
// -- or 32768 where a head has no more than 33 -- and an odd number of them.
// Heads can be shorter than their bound, and workgroups that find nothing cost as much to start as the others: 112 heads of 2115
// entries, 16512 reserved, 259 per head 12.9 us, 147 10.5.  Fewer than the batches there are cost the heads that evict their first
// entries and move half of what they keep: 8 heads of 4000, a half kept, 33 instead of 63 per head 10.6 against 7.3 us, 800 heads of
// 2000, 17 instead of 33, 156 against 144; 1536 heads of 1888, 11 instead of 23, 136 against 130 at a third kept by mass.
// Odd: a head's first workgroups find its moves and the others nothing, and
// workgroups go to the 8 XCDs and the 4 shader engines of each in turn: by an even number per head, the ones with work are the
// same few engines' in every head (32 per head -> 33, caches just read: 800 heads of 2000 entries of 256 bytes at a third kept by mass
// 98 -> 64 us, with a budget of 200 83 -> 35, 500 heads 64 -> 40).
inline int kv_fill_workgroups(long long heads, int max_moves) {
    const long long batches = (max_moves + kFillRows - 1) / kFillRows;
    const long long sixteen = (16384 + heads - 1) / heads, more = (32768 + heads - 1) / heads;
    const long long most = sixteen > 33 ? sixteen : (more < 33 ? more : 33);
    return (int)(batches < most ? batches : most) | 1;
}
// Whether kv_fill_kernel loads the rows of a head of `entries` entries past the caches: where all heads, taken as long as this one,
// hold more rows than the 256 MB cache in front of the memory, so that those written or read last push the others out.  The
// lengths count, not what the caller reserves.  Moves loaded through the caches -> past them, us: 1536 heads of 1888 entries of
// 256 bytes 182 -> 133 where the caches have just been written, 131 -> 121 just read, 183 -> 132 long before; 500 heads of 2000
// (488 MB) 52 -> 50, 42 -> 41, 76 -> 52; 112 heads of 2115 (115 MB), 16512 reserved, 11 -> 14, 10 -> 11, 21 -> 16.
// (The same call again at once, its moved rows all cached, has the faster loads through the caches up to 512 MB -- 200 heads of
// 3000 19 against 29 -- but slots are not compressed again before they are written.)
__host__ __device__ inline bool fill_past_caches(long long heads, long long entries, int row_bytes) {
    return 2 * heads * entries * row_bytes > (256ll << 20);
}

struct AttnWs {
    size_t part_ml, part_o, logits, cur_len, total;
    int n_split, split_len, lcap, tail_entry;
};
AttnWs attn_ws(const lvlm_attn_desc &d);

// Names the kernel launches between begin() and end() for the optional timing.  The events are bound to the
// kernels themselves (the start event to the first launch of the bracket, the stop event to its last), so what
// is read back is the time from that kernel's first wave to its last -- the duration a kernel trace reports --
// without the dispatch gaps that events recorded around a launch would add.
struct Prof {
    lvlm_ctx *ctx;
    hipStream_t stream;
    void begin(const char *name) const {
        if (!ctx->prof_on || ctx->prof_n >= ctx->prof_cap) return;
        ctx->prof_name[ctx->prof_n] = name;
        ctx->prof_open = ctx->prof_first = true;
    }
    void end() const {
        if (!ctx->prof_open) return;
        ctx->prof_open = false;
        if (!ctx->prof_first) ++ctx->prof_n;     // a bracket without a launch leaves no entry
    }
    // the events the next launch carries (null: none), or false when no bracket is open
    bool events(hipEvent_t *start, hipEvent_t *stop) const {
        if (!ctx->prof_open) return false;
        *start = ctx->prof_first ? ctx->prof_ev[2 * ctx->prof_n] : nullptr;
        *stop = ctx->prof_ev[2 * ctx->prof_n + 1];
        ctx->prof_first = false;
        return true;
    }
};

// hipLaunchKernelGGL with a Prof in front: the same launch, carrying the open bracket's events if there is one.
#define LVLM_LAUNCH(prof, kernel, grid, block, lds_bytes, stream_, ...)                                      \
    do {                                                                                                     \
        hipEvent_t lvlm_ev0_, lvlm_ev1_;                                                                     \
        if ((prof).events(&lvlm_ev0_, &lvlm_ev1_))                                                           \
            hipExtLaunchKernelGGL(kernel, grid, block, lds_bytes, stream_, lvlm_ev0_, lvlm_ev1_, 0, __VA_ARGS__); \
        else                                                                                                 \
            hipLaunchKernelGGL(kernel, grid, block, lds_bytes, stream_, __VA_ARGS__);                        \
    } while (0)

// ---- launches (defined in the .hip files; all asynchronous on `stream`) ----
// How the sorted blocks of long sequences are searched: `groups` times 64 tokens to a workgroup, `parts` workgroups to a token.
// One group while every workgroup has a compute unit of its own, then two, then four: each halves what is staged in all (ranking
// alone, one group -> the form taken, us: 5 x 4800 tokens 11.9 -> 9.4, 8 x 8192 21.6 -> 15.7, 32 x 4096 34.9 -> 20.7; the other way
// round four groups -> one at 1 x 12000 13.6 -> 9.8, -> two at 2 x 16384 16.0 -> 12.1).  Beyond 32 blocks the few workgroups, each with
// five rounds or more, leave the last turn of the chip uneven: every round goes to a workgroup of its own, which adds its counts to the
// rank, and a further launch finishes it (rounds in turn -> shared: 1 x 33000 24.4 -> 22.5, 1 x 100000 87 -> 71, 1 x 400000 1000 -> 849;
// below, 2 x 24000 20.1 -> 22.7).
struct SearchForm {
    int groups, parts;
};
inline SearchForm rank_search_form(int n, int B) {
    const long long alone = (long long)B * ((n + 63) / 64), pairs = (long long)B * ((n + 127) / 128);
    const int blocks = (n + 1023) / 1024;
    SearchForm f;
    f.groups = alone <= 256 ? 1 : pairs <= 256 ? 2 : 4;
    f.parts = blocks > 32 ? (blocks + 7) / 8 : 1;
    return f;
}
// scratch: rank_scratch_bytes(n, B) bytes for the sorted blocks of long sequences, or null (counting at any length)
size_t rank_scratch_bytes(int n, int B);
// kept: [B, ceil(n / 64)], how many of every 64 tokens have a rank below n_kept (null: not counted)
// norm: 1 / |row| of these rows on the side, in the same launch (null: none)
struct NormJob {
    const char *src;        // row 0 of sequence 0; rows of row_bytes (a multiple of 16)
    long long stride_b;     // bytes from sequence to sequence
    float *inv_norm;        // [B, n]
    int row_bytes, dtype, n;
};
void launch_rank(const Prof &prof, const float *score, int32_t *rank, int n, int B, void *scratch, const NormJob *norm = nullptr,
                 int32_t *kept = nullptr, int n_kept = 0);
// Which dominant token every other token joined, and what the similarity merge makes of it: the tokens ordered by
// (owner, index), the dominant ones behind.
struct OwnerJob {
    const int32_t *dom_of;              // [B, n]  p >= 0: dominant position; -(q+1): q-th other token
    const unsigned long long *best;     // [B, r]  (order-preserving key of the cosine, ~dominant position); 0: none comparable
    int32_t *order, *owner, *assign;    // [B, n]  token and owner of every place, owner of every token
    int r;
#if defined(__HIPCC__)
    __device__ __forceinline__ int joined(int b, int d) const {
        const unsigned long long w = best[(long long)b * r - d - 1];
        return w == 0ull ? 0 : (int)(0xffffffffu - (uint32_t)w);
    }
#endif
};
void launch_owner_order(const Prof &prof, const OwnerJob &owners, int32_t *rank, int n, int B, void *scratch);
hipError_t launch_score(const Prof &prof, const lvlm_score_desc &d, const ScoreWs &w, char *ws,
                        const void *q, const void *k, const float *row_lse, float *score_head,
                        float *score_mean);
hipError_t launch_score_probs(const Prof &prof, const lvlm_probs_desc &d, const ProbsWs &w, char *ws, const void *probs,
                              float *score_head, float *score_mean);
hipError_t launch_prefill_attn(const Prof &prof, const lvlm_prefill_desc &d, const PrefillWs &w, char *ws, const void *q,
                               const void *k, const void *v, void *out, float *row_lse, float *score_head,
                               float *score_mean);
hipError_t launch_merge(const Prof &prof, const lvlm_merge_desc &d, const MergeWs &w, char *ws,
                        const float *score_mean, const float *wtab, const lvlm_plane *planes,
                        int32_t *keep_idx, int32_t *merged_idx);
hipError_t launch_merge_similar(const Prof &prof, const lvlm_merge_desc &d, const SimWs &w, char *ws,
                                const float *score_mean, const lvlm_plane *planes, const float *size_in,
                                float *size_out, int32_t *keep_idx, int32_t *assign);
hipError_t launch_kv_compress(const Prof &prof, const lvlm_kv_desc &d, const KvWs &w, char *ws,
                              void *k_cache, void *v_cache, float *score, uint8_t *kind,
                              int32_t *orig_pos, int32_t *len, int32_t *n_evicted);
hipError_t launch_decode_attn(const Prof &prof, const lvlm_attn_desc &d, const AttnWs &w, char *ws,
                              const void *q, const void *k_new, const void *v_new, void *k_cache,
                              void *v_cache, float *score, uint8_t *kind, int32_t *orig_pos,
                              int32_t *len, void *out);

hipError_t launch_stream_probe(const Prof &prof, const void *src, size_t bytes, int n_workgroups, unsigned int *sink);

// Device address and size of the fixed scratch array that lvlm_decode_attn_static uses on the current device
// (looked up once per device; no allocation).
hipError_t attn_static_scratch(int device, char **ptr, size_t *bytes);

#if defined(__HIPCC__)
// ---- device helpers ----
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Loads and stores of what passes through once and should not take up a cache.
template <class T>
__device__ __forceinline__ T load_once(const T *p) {
    if constexpr (sizeof(T) == 16) {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        return __builtin_bit_cast(T, __builtin_nontemporal_load(reinterpret_cast<const u4 *>(p)));
    } else {
        return __builtin_nontemporal_load(p);
    }
}
template <class T>
__device__ __forceinline__ void store_once(T *p, T v) {
    if constexpr (sizeof(T) == 16) {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(__builtin_bit_cast(u4, v), reinterpret_cast<u4 *>(p));
    } else {
        __builtin_nontemporal_store(v, p);
    }
}

// round-to-nearest-even; NaN stays NaN
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Order-preserving map float -> u32: a < b  <=>  key(a) < key(b); -0 == +0;
// NaN maps to 0, below -inf.  Descending importance = descending key.
__device__ __forceinline__ uint32_t score_key(float x) {
    if (x != x) return 0u;
    x += 0.0f;
    uint32_t b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Exact fixed-point image of a score used for cumulative thresholds:
// floor(clamp(score, 0, 2^16) * 2^32); NaN and negatives give 0.
// Computed as two 32-bit halves (integer part, then the fraction scaled by 2^32: both conversions
// truncate and both products are exact), which is much cheaper than a float -> u64 conversion.
__device__ __forceinline__ unsigned long long score_fixed(float s) {
    if (!(s > 0.0f)) return 0ull;
    s = fminf(s, 65536.0f);
    const unsigned int hi = (unsigned int)s;
    const unsigned int lo = (unsigned int)((s - (float)hi) * 4294967296.0f);
    return ((unsigned long long)hi << 32) | lo;
}

// Wave reductions that leave the result in every lane, without the LDS permute unit: inside a row of 16 lanes by
// data-parallel-primitive moves (swap neighbours, swap pairs, mirror the halves of 8, mirror the row), across the
// rows and the two half-waves by the lane-swap instructions.
__device__ __forceinline__ float dpp_quad1(float v) { return __int_as_float(__hip_move_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true)); }   // lanes 1,0,3,2
__device__ __forceinline__ float dpp_quad2(float v) { return __int_as_float(__hip_move_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true)); }   // lanes 2,3,0,1
__device__ __forceinline__ float dpp_half_mirror(float v) { return __int_as_float(__hip_move_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true)); }
__device__ __forceinline__ float dpp_row_mirror(float v) { return __int_as_float(__hip_move_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true)); }
__device__ __forceinline__ float swap_rows(float x) {          // the value of the lane 16 places away
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float((threadIdx.x & 16) ? r.x : r.y);
}
__device__ __forceinline__ float swap_halves(float x) {        // the value of the lane 32 places away
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float((threadIdx.x & 32) ? r.x : r.y);
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_quad1(v));
    v = fmaxf(v, dpp_quad2(v));
    v = fmaxf(v, dpp_half_mirror(v));
    v = fmaxf(v, dpp_row_mirror(v));
    v = fmaxf(v, swap_rows(v));
    return fmaxf(v, swap_halves(v));
}
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_quad1(v);
    v += dpp_quad2(v);
    v += dpp_half_mirror(v);
    v += dpp_row_mirror(v);
    v += swap_rows(v);
    return v + swap_halves(v);
}
// Minimum of a 64-bit key over the wave, in every lane (the moves are bitwise: the halves travel as floats).
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
#define LVLM_MIN_STEP(MOVE)                                                                          \
    {                                                                                                \
        const unsigned ph = __float_as_uint(MOVE(__uint_as_float((unsigned)(v >> 32))));             \
        const unsigned pl = __float_as_uint(MOVE(__uint_as_float((unsigned)v)));                     \
        const unsigned long long o = ((unsigned long long)ph << 32) | pl;                            \
        v = o < v ? o : v;                                                                           \
    }
    LVLM_MIN_STEP(dpp_quad1)
    LVLM_MIN_STEP(dpp_quad2)
    LVLM_MIN_STEP(dpp_half_mirror)
    LVLM_MIN_STEP(dpp_row_mirror)
    LVLM_MIN_STEP(swap_rows)
    LVLM_MIN_STEP(swap_halves)
#undef LVLM_MIN_STEP
    return v;
}
// Orders the wave's LDS accesses before and after it, for values that lanes of one wave hand each other there: no workgroup barrier,
// and no instruction (a wave's LDS operations run in order), but the compiler moves none of them across.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Any associative, commutative OP over the wave's 32-bit or 64-bit values, in every lane, by the same moves.
template <class OP>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t v, OP op) {
#define LVLM_RED_STEP(MOVE) v = op(v, __float_as_uint(MOVE(__uint_as_float(v))));
    LVLM_RED_STEP(dpp_quad1)
    LVLM_RED_STEP(dpp_quad2)
    LVLM_RED_STEP(dpp_half_mirror)
    LVLM_RED_STEP(dpp_row_mirror)
    LVLM_RED_STEP(swap_rows)
    LVLM_RED_STEP(swap_halves)
#undef LVLM_RED_STEP
    return v;
}
template <class OP>
__device__ __forceinline__ unsigned long long wave_reduce_u64(unsigned long long v, OP op) {
#define LVLM_RED_STEP(MOVE)                                                                          \
    {                                                                                                \
        const unsigned ph = __float_as_uint(MOVE(__uint_as_float((unsigned)(v >> 32))));             \
        const unsigned pl = __float_as_uint(MOVE(__uint_as_float((unsigned)v)));                     \
        v = op(v, ((unsigned long long)ph << 32) | pl);                                              \
    }
    LVLM_RED_STEP(dpp_quad1)
    LVLM_RED_STEP(dpp_quad2)
    LVLM_RED_STEP(dpp_half_mirror)
    LVLM_RED_STEP(dpp_row_mirror)
    LVLM_RED_STEP(swap_rows)
    LVLM_RED_STEP(swap_halves)
#undef LVLM_RED_STEP
    return v;
}
#endif

}  // namespace lvlm
