// Steps 2-4 -- partition by importance, merge P_merged into one token, compact
// every plane that shares the token axis (Sec. 3.2.1, par. 4).
//
//   rank_kernel      rank[j] = number of image tokens that precede j in
//                    descending score order (ties: lower index first).  It is
//                    the counting definition itself, spread over the chip:
//                    64 tokens per workgroup, the keys staged in LDS and split
//                    over the 16 waves.  Nothing iterative or data dependent.
//                    Long sequences: rank_block_kernel + rank_search_kernel
//                    (blocks of 1024 tokens sorted by counting, then one
//                    binary search per token and block).  Counts the kept
//                    tokens of every 64 on the way.
//   gather_kernel    works out where its rows' tokens go (and emits keep_idx,
//                    ascending, and merged_idx, in rank order); then
//                    one streaming pass over every source row of every plane:
//                    a kept row is copied to its new place with 128-bit loads
//                    and stores, a merged row is multiplied by its rank weight
//                    and accumulated in fp32 registers; each row chunk leaves
//                    one partial sum.
//   finalize_kernel  adds the partial sums in chunk order, rounds once and
//                    writes P_new behind P_unmerged.
#include <limits.h>

#include "common.h"
#include "planes.h"

namespace lvlm {
namespace {

constexpr int kGatherRows = 8;     // rows per batch (all of a batch's loads are in flight together)
constexpr int kGatherWgs = 1536;   // workgroups the gather launch aims for (six per compute unit)
constexpr int kGatherChunkRows = 128;   // rows of a chunk at most
// Image tokens whose destinations a workgroup of the gather holds in LDS.  (4096 keep all threads of the narrowest planes in long chunks busy,
// but are longer in the making than the rows are in coming: 2 x 16384 -> 5000 rows of 2 KB, twice, 51.2 -> 56.5 us, 8 x 9000 -> 3000
// rows of 7 KB and twice 64 bytes 162.9 -> 168.4.)
constexpr int kGatherTable = 1024;
static_assert(kGatherRows <= kGatherChunkRows && kGatherChunkRows <= kGatherTable, "a workgroup takes at least one chunk");
// Chunks of rows to a workgroup of the gather: as many as its threads hold, of no more tokens than its table does.
__host__ __device__ inline int gather_chunks(const PlaneDev &p, int rows_per_chunk) {
    const int most = kGatherTable / rows_per_chunk, fit = 256 >> p.tpr_log2;
    return fit < most ? fit : most;
}
constexpr long long kGatherCached = 256ll << 20;       // bytes of source rows that the memory-side cache can hold


constexpr int kRankTile = 8192;   // keys staged in LDS per step of the rank kernel (32 KB)
constexpr int kRankBlock = 64;    // tokens ranked by one workgroup (one per lane; the 16 waves split the keys)

// What is ranked: descending 32-bit keys of the n tokens of a sequence, ties by ascending index.
//   ByScore   the scores; rank[j] is the result
//   ByOwner   (similarity merge) the tokens that joined dominant position p get key ~p, the dominant ones 0, so that the
//             order is (owner, index) with the dominant tokens behind; order, owner and assign are the result
template <class KEY>
struct RankArgs {
    KEY key;
    int32_t *rank;                  // [B, n]
    unsigned long long *sorted;     // [B, n_blocks, 1024]  (long sequences)
    int32_t *kept;                  // [B, ceil(n / 64)]  tokens of every 64 with rank < n_kept, or null
    int n_kept;
    int n, n_blocks;
    int parts;                      // workgroups that share a token's searches
    int rank_wgs;                   // workgroups of the launch that rank; the rest take rows of `norm`
    NormJob norm;
};

struct ByScore {
    const float *score;      // [B, n]
    __device__ __forceinline__ uint32_t at(int b, int n, int i) const { return score_key(score[(long long)b * n + i]); }
    static constexpr bool kOrder = false;
    __device__ __forceinline__ void put(int, int, int, int) const {}
};

struct ByOwner {
    OwnerJob o;
    __device__ __forceinline__ uint32_t at(int b, int n, int i) const {
        const int d = o.dom_of[(long long)b * n + i];
        return d >= 0 ? 0u : ~(uint32_t)o.joined(b, d);
    }
    static constexpr bool kOrder = true;
    __device__ __forceinline__ void put(int b, int n, int j, int place) const {
        const int d = o.dom_of[(long long)b * n + j];
        const int pos = d >= 0 ? d : o.joined(b, d);
        o.assign[(long long)b * n + j] = pos;
        o.order[(long long)b * n + place] = j;
        o.owner[(long long)b * n + place] = pos;
    }
};

// 1 / |row| of 16 rows (one per wave).  The job rides along in a ranking launch: it needs nothing from the ranks and
// streams from memory while the ranking workgroups count.
__device__ __forceinline__ void norm_rows(const NormJob &w, int wg, int b) {
    const int lane = threadIdx.x & 63, j = wg * 16 + (threadIdx.x >> 6);
    if (j >= w.n) return;
    const char *row = w.src + (long long)b * w.stride_b + (long long)j * w.row_bytes;
    const int units = w.row_bytes / 16;
    float s = 0.f;
    for (int u0 = 0; u0 < units; u0 += 8 * 64) {
        uint4 v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int u = u0 + 64 * x + lane;
            v[x] = u < units ? *reinterpret_cast<const uint4 *>(row + 16ll * u) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const uint32_t d[4] = {v[x].x, v[x].y, v[x].z, v[x].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (w.dtype == LVLM_BF16) {
                    const float lo = __uint_as_float(d[i] << 16), hi = __uint_as_float(d[i] & 0xffff0000u);
                    s = fmaf(lo, lo, s);
                    s = fmaf(hi, hi, s);
                } else {
                    const float e = __uint_as_float(d[i]);
                    s = fmaf(e, e, s);
                }
            }
        }
    }
    s = wave_sum(s);
    if (lane == 0) w.inv_norm[(long long)b * w.n + j] = s > 0.f ? 1.0f / sqrtf(s) : 1.0f;
}

// The ranks of one wave's 64 tokens, j = 64 m + lane (lanes past the last token are not here), and how many of them are kept.
template <class KEY>
__device__ __forceinline__ void done(const RankArgs<KEY> &a, int b, int j, int rank) {
    if constexpr (KEY::kOrder) {
        a.key.put(b, a.n, j, rank);
    } else {
        a.rank[(long long)b * a.n + j] = rank;
        if (a.kept) {
            const unsigned long long bal = __ballot(rank < a.n_kept);
            if ((j & 63) == 0) a.kept[(long long)b * ((a.n + 63) / 64) + j / 64] = __popcll(bal);
        }
    }
}

// rank[j] = #{i : key_i > key_j, or key_i == key_j and i < j}.  A workgroup ranks 64 tokens: every wave
// holds the same 64 tokens (one per lane) and counts over its own sixteenth of the staged keys, read
// from LDS as broadcast 128-bit words; the sixteen counts are added through LDS.
template <class KEY>
__global__ __launch_bounds__(1024) void rank_kernel(RankArgs<KEY> a) {
    __shared__ __attribute__((aligned(16))) uint32_t keys[kRankTile];
    __shared__ int cnt_lds[16][kRankBlock];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.y;
    if ((int)blockIdx.x >= a.rank_wgs) {
        norm_rows(a.norm, blockIdx.x - a.rank_wgs, b);
        return;
    }
    const int j0 = blockIdx.x * kRankBlock;
    const int j = j0 + lane;
    const uint32_t kj = j < a.n ? a.key.at(b, a.n, j) : 0u;
    int cnt = 0;
    for (int t0 = 0; t0 < a.n; t0 += kRankTile) {
        const int tile_n = min(kRankTile, a.n - t0);
        const int share = ((tile_n + 15) / 16 + 3) & ~3;          // keys per wave, a multiple of 4
        __syncthreads();
        for (int x = tid; x < 16 * share && x < kRankTile; x += 1024) {
            const int i = t0 + x;
            // Padding sits above every real index, so it only ever meets the ">" rule (or the full
            // rule with i > j): the lowest key can never precede anything.
            keys[x] = i < a.n ? a.key.at(b, a.n, i) : 0u;
        }
        __syncthreads();
        const int x_lo = wave * share, x_hi = min(kRankTile, x_lo + share);
        // Groups of four keys: entirely below the block (i < j: ">=" precedes), entirely above
        // (i > j: only ">" precedes), or overlapping the block's own indices (full rule).
        const int below_end = min(x_hi, max(x_lo, (j0 - t0) & ~3));
        const int above_beg = max(x_lo, min(x_hi, (j0 + kRankBlock - t0 + 3) & ~3));
#pragma unroll 8
        for (int x = x_lo; x < below_end; x += 4) {
            const uint4 k4 = *reinterpret_cast<const uint4 *>(&keys[x]);
            cnt += (k4.x >= kj) + (k4.y >= kj) + (k4.z >= kj) + (k4.w >= kj);
        }
#pragma unroll 4
        for (int x = below_end; x < above_beg; x += 4) {
            const uint4 k4 = *reinterpret_cast<const uint4 *>(&keys[x]);
            const int i = t0 + x;
            cnt += ((k4.x > kj) | ((k4.x == kj) & (i < j))) + ((k4.y > kj) | ((k4.y == kj) & (i + 1 < j))) +
                   ((k4.z > kj) | ((k4.z == kj) & (i + 2 < j))) + ((k4.w > kj) | ((k4.w == kj) & (i + 3 < j)));
        }
#pragma unroll 8
        for (int x = above_beg; x < x_hi; x += 4) {
            const uint4 k4 = *reinterpret_cast<const uint4 *>(&keys[x]);
            cnt += (k4.x > kj) + (k4.y > kj) + (k4.z > kj) + (k4.w > kj);
        }
    }
    cnt_lds[wave][lane] = cnt;
    __syncthreads();
    if (wave == 0 && j < a.n) {
        int tot = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) tot += cnt_lds[w][lane];
        done(a, b, j, tot);
    }
}

// ---- ranks of long sequences: sorted blocks + binary searches ------------------------------------
// Counting costs n^2 comparisons; from kSortMinTokens tokens on the ranks come in two launches instead.
// A token's place in the order is told by one 64-bit word, key in the high half and inverted index in the low
// half: i precedes j  <=>  word_i > word_j (higher key, or the same key and the lower index).
//   rank_block_kernel   every block of 1024 tokens is sorted by counting WITHIN the block (1024 comparisons per
//                       token, spread over all workgroups): a token's word goes to its place in the block's
//                       descending order; places past the last token of a partly filled block hold 0 (below every word)
//   rank_search_kernel  a token's rank = over all sorted blocks, the number of words above its own, each found by
//                       a binary search (11 probes) in LDS; a workgroup stages eight or sixteen blocks at a time, and its
//                       waves search them for 64 to 256 tokens
//   rank_finish_kernel  (the longest sequences) what is made of a rank that several workgroups have added up
constexpr int kSortBlock = 1024;
constexpr int kSortMinTokens = 4096;

__device__ __forceinline__ unsigned long long order_word(uint32_t key, int idx) {
    return ((unsigned long long)key << 32) | (unsigned long long)(0xffffffffu - (uint32_t)idx);
}

// 64 tokens per workgroup (one per lane, the same in all 16 waves); wave w counts over words 64 w .. 64 w + 63 of
// the tokens' own block, read from LDS as broadcast 128-bit pairs.
template <class KEY>
__global__ __launch_bounds__(1024) void rank_block_kernel(RankArgs<KEY> a) {
    __shared__ __attribute__((aligned(16))) unsigned long long words[kSortBlock];
    __shared__ int cnt_lds[16][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.y;
    if ((int)blockIdx.x >= a.rank_wgs) {
        norm_rows(a.norm, blockIdx.x - a.rank_wgs, b);
        return;
    }
    const int j0 = blockIdx.x * 64, j = j0 + lane;
    const int blk = j0 / kSortBlock, r0 = blk * kSortBlock;
    unsigned long long *out = a.sorted + ((long long)b * a.n_blocks + blk) * kSortBlock;
    if (j0 >= a.n) {                              // nothing but padding here (uniform over the workgroup)
        if (wave == 0) out[j - r0] = 0ull;
        return;
    }
    {
        const int i = r0 + tid;
        words[tid] = i < a.n ? order_word(a.key.at(b, a.n, i), i) : 0ull;
    }
    const unsigned long long mine = j < a.n ? order_word(a.key.at(b, a.n, j), j) : 0ull;
    __syncthreads();
    int cnt = 0;
#pragma unroll 8
    for (int x = 64 * wave; x < 64 * wave + 64; x += 2) {
        const ulonglong2 w2 = *reinterpret_cast<const ulonglong2 *>(&words[x]);
        cnt += (w2.x > mine) + (w2.y > mine);
    }
    cnt_lds[wave][lane] = cnt;
    __syncthreads();
    if (wave == 0) {
        int place = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) place += cnt_lds[w][lane];
        // tokens past the end fill the places past the last token (the real ones take 0 .. count-1 between them)
        if (j < a.n) {
            out[place] = mine;
            if (a.parts > 1) a.rank[(long long)b * a.n + j] = 0;      // the searches add to it
        } else {
            out[j - r0] = 0ull;
        }
    }
}

// A workgroup searches S staged blocks (S x 8 KB) for TG times 64 tokens, and goes on to the next S or, with `parts`, leaves them to
// another workgroup.  Its time is what it stages, at a compute unit's L2 bandwidth, and eleven dependent LDS probes for every round;
// S = 8 leaves room for a second workgroup whose searches cover the staging (rank_search_form has the rule).
template <class KEY, int TG, int S>
__global__ __launch_bounds__(1024, S > 8 ? 4 : 8) void rank_search_kernel(RankArgs<KEY> a) {
    constexpr int WPG = 16 / TG, CH = S / WPG;             // waves per 64 tokens; blocks a wave searches side by side
    static_assert(CH >= 1 && CH * WPG == S, "every wave has blocks to search");
    __shared__ __attribute__((aligned(16))) unsigned long long words[S * kSortBlock];
    __shared__ int above[16][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), first = wave / TG;
    const int b = blockIdx.y;
    const int j = (blockIdx.x * TG + wave % TG) * 64 + lane;
    const unsigned long long mine = j < a.n ? order_word(a.key.at(b, a.n, j), j) : ~0ull;
    const uint4 *src = reinterpret_cast<const uint4 *>(a.sorted + (long long)b * a.n_blocks * kSortBlock);
    int cnt = 0;
    for (int g0 = S * blockIdx.z; g0 < a.n_blocks; g0 += S * a.parts) {
        const int nb = min(S, a.n_blocks - g0);
        const int units = nb * (kSortBlock / 2);                       // 16-byte units to stage
        if (g0 >= S * a.parts) __syncthreads();                        // the blocks before have been searched
#pragma unroll
        for (int x = 0; x < S * (kSortBlock / 2) / 1024; ++x)          // (places past the last block do not count)
            reinterpret_cast<uint4 *>(words)[1024 * x + tid] = src[(long long)g0 * (kSortBlock / 2) + min(1024 * x + tid, units - 1)];
        __syncthreads();
        if (first < nb) {
            // words above `mine` in each of the wave's blocks: they descend, so that is the first place whose word is not above it
            const unsigned long long *const blk = words + first * kSortBlock;
            int pos[CH];
#pragma unroll
            for (int x = 0; x < CH; ++x) pos[x] = 0;
#pragma unroll
            for (int step = kSortBlock / 2; step >= 1; step >>= 1)
#pragma unroll
                for (int x = 0; x < CH; ++x) pos[x] += blk[x * WPG * kSortBlock + pos[x] + step - 1] > mine ? step : 0;
#pragma unroll
            for (int x = 0; x < CH; ++x)
                if (first + x * WPG < nb) cnt += pos[x] + (blk[x * WPG * kSortBlock + pos[x]] > mine ? 1 : 0);      // place 1023 itself
        }
    }
    above[wave][lane] = cnt;
    __syncthreads();
    if (wave < TG && j < a.n) {
        int rank = 0;
#pragma unroll
        for (int w = 0; w < WPG; ++w) rank += above[w * TG + wave][lane];
        if (a.parts > 1) atomicAdd(&a.rank[(long long)b * a.n + j], rank);
        else done(a, b, j, rank);
    }
}

template <class KEY>
__global__ __launch_bounds__(256) void rank_finish_kernel(RankArgs<KEY> a) {
    const int j = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
    if (j < a.n) done(a, b, j, a.rank[(long long)b * a.n + j]);
}


// ---- gather -----------------------------------------------------------------

struct GatherArgs {
    PlaneDev plane[LVLM_MAX_PLANES];
    const int32_t *rank;     // [B, n_img], null: identity (nothing removed)
    const int32_t *kept;     // [B, ceil(n_img / 64)]  how many of every 64 tokens are kept
    int32_t *keep_idx;       // [B, n_keep-1] or null
    int32_t *merged_idx;     // [B, r+1] or null
    const float *w;          // rank -> weight table, or null for the linear table
    float lin_scale;         // 1 / (m (m+1) / 2)
    float *partial;          // [B][n_planes][n_sub_max][max_row_elems]
    int B, N, img_begin, n_img, n_keep, n_planes;
    int rows_per_sub, n_sub_max, max_row_elems;
};

// Where the image tokens of a workgroup's rows go, and with what weight they are merged.
struct GatherTable {
    int code[kGatherTable];      // >= 0: row inside the new image span; -1: most important merged token; -2: any other merged token
    float wgt[kGatherTable];     // merge weight (0 for kept tokens)
};

// Tokens [lo, hi) of a sequence, 64 of them (aligned) to a wave at a time: kept tokens stay in index order, so a token's row is the
// number of kept ones before it -- those of the 64s in front, which the ranking has counted, and those of its own.  It is a
// chain of one load and a reduction, beside the workgroup's first rows on their way; as a launch of its own, with destination and weight
// of every token through memory, it took 2.3 to 4.8 us of a
// call (whole calls, the search of long sequences above included: 16384 -> 5091 rows of 12 KB 78.0 -> 69.0 us, 4626 -> 2313 of 10 KB
// 31.0 -> 26.9, 7 x 465 -> 144 of 8 KB and twice 2 KB 25.6 -> 23.4, 514 -> 359 of 10 KB 15.6 -> 15.1).  `list`: the index lists are written too.
__device__ __forceinline__ void gather_table(const GatherArgs &a, int b, int lo, int hi, bool list, GatherTable &t) {
    const int lane = threadIdx.x & 63, n_unmerged = a.n_keep - 1, m = a.n_img - n_unmerged;
    const int32_t *rank = a.rank + (long long)b * a.n_img, *kept = a.kept + (long long)b * ((a.n_img + 63) / 64);
    for (int blk = lo / 64 + (threadIdx.x >> 6); 64 * blk < hi; blk += blockDim.x >> 6) {
        const int j = 64 * blk + lane;
        const int rk = j < a.n_img ? rank[j] : INT_MAX;
        uint32_t before = 0;
#pragma unroll 4
        for (int i = lane; i < blk; i += 64) before += kept[i];
        before = wave_reduce_u32(before, [](uint32_t x, uint32_t y) { return x + y; });
        const unsigned long long bal = __ballot(rk < n_unmerged);
        if (j < lo || j >= hi) continue;
        if (rk < n_unmerged) {
            const int p = (int)before + __popcll(bal & ((1ull << lane) - 1ull));
            t.code[j - lo] = p;
            t.wgt[j - lo] = 0.f;
            if (list && a.keep_idx) a.keep_idx[(long long)b * n_unmerged + p] = j;
        } else {
            const int k = rk - n_unmerged;
            t.code[j - lo] = k == 0 ? -1 : -2;
            t.wgt[j - lo] = a.w ? a.w[k] : (float)(m - k) * a.lin_scale;
            if (list && a.merged_idx) a.merged_idx[(long long)b * m + k] = j;
        }
    }
}

// One thread group walks `rows_per_sub` consecutive source rows of one plane, one unit column per thread.
// The loop is free of data-dependent branches before its stores: the rows of a batch are loaded unconditionally (indices
// clamped into range), so the loads of many rows are in flight at once; then kept rows are stored and merged ones are
// multiplied by their weights and accumulated.
template <int DT, int UB, int TEAMS, bool ONCE>
__device__ __forceinline__ void gather_plane(const GatherArgs &a, const PlaneDev &p, int pi, int b, float (*other)[256],
                                             GatherTable &table) {
    using U = typename Unit<UB>::type;
    constexpr int RB = kGatherRows;
    const int tid = threadIdx.x;
    const int tpr = 1 << p.tpr_log2;
    const int chunks = gather_chunks(p, a.rows_per_sub);  // of rows, per workgroup
    const int team = tid >> 8;                            // a chunk's batches of rows go to the teams in turn
    const int group = (tid & 255) >> p.tpr_log2;
    const int sub = blockIdx.x * chunks + group;
    const int row_units = p.row_bytes / UB;
    if ((int)blockIdx.x * chunks >= p.n_sub || (int)blockIdx.y >= p.col_blocks) return;      // uniform
    const int unit_raw = blockIdx.y * 256 + (tid & (tpr - 1));
    const bool active = unit_raw < row_units;
    const int unit = active ? unit_raw : row_units - 1;
    const int r = a.n_img - a.n_keep;
    const char *src = p.src + (long long)b * p.src_stride_b + (long long)unit * UB;
    char *dst = p.dst + (long long)b * p.dst_stride_b + (long long)unit * UB;
    const int n_lo = group < chunks ? min(a.N, sub * a.rows_per_sub) : a.N;
    const int n_hi = min(a.N, n_lo + a.rows_per_sub);     // (a chunk past the last one has no rows)
    if (a.rank == nullptr) {
        // nothing is removed (kernel-uniform case): plain row copy
        if (active) {
#pragma unroll 4
            for (int n = n_lo + team; n < n_hi; n += TEAMS)
                *reinterpret_cast<U *>(dst + (long long)n * p.row_bytes) =
                    *reinterpret_cast<const U *>(src + (long long)n * p.row_bytes);
        }
        return;
    }
    const bool weighted = p.rule == LVLM_RULE_WEIGHTED;             // uniform per plane
    const int new_row = a.img_begin + a.n_keep - 1;

    U val[RB];
    auto load = [&](int n0) {
#pragma unroll
        for (int x = 0; x < RB; ++x) {
            const U *at = reinterpret_cast<const U *>(src + (long long)min(n0 + x, n_hi - 1) * p.row_bytes);
            val[x] = ONCE ? load_once(at) : *at;
        }
    };
    int n0 = n_lo + team * RB;
    load(n0);
    // image tokens of the workgroup's rows, no more than chunks * rows_per_sub <= kGatherTable of them
    const int row0 = blockIdx.x * chunks * a.rows_per_sub;
    const int lo = max(row0 - a.img_begin, 0);
    gather_table(a, b, lo, min(row0 + chunks * a.rows_per_sub - a.img_begin, a.n_img), pi == 0 && blockIdx.y == 0, table);
    __syncthreads();

    Acc<DT, UB> acc;
#pragma unroll
    for (int i = 0; i < Acc<DT, UB>::NE; ++i) acc.v[i] = 0.f;

    while (n0 < n_hi) {
#pragma unroll
        for (int x = 0; x < RB; ++x) {
            const int n = n0 + x;
            const bool valid = active && n < n_hi;
            const bool in_img = n >= a.img_begin && n < a.img_begin + a.n_img;
            const int at = min(max(n - a.img_begin - lo, 0), kGatherTable - 1);
            const int code = table.code[at];
            int dest = n < a.img_begin ? n : n - r;                  // rows outside the image span
            if (in_img) dest = code >= 0 ? a.img_begin + code : (code == -1 && !weighted ? new_row : -1);
            if (valid && dest >= 0) *reinterpret_cast<U *>(dst + (long long)dest * p.row_bytes) = val[x];
            // Only the rows of P_merged enter the sum (a kept or text row must not, whatever it holds: 0 * inf
            // would poison the merged token).  A row is shared by whole waves for all but the narrowest planes,
            // so the test is uniform there.
            if constexpr (DT != LVLM_I32) {
                if (weighted && valid && in_img && code < 0) accumulate<DT, UB>(acc, val[x], table.wgt[at]);
            }
        }
        n0 += TEAMS * RB;
        if (n0 < n_hi) load(n0);
    }
    if constexpr (DT != LVLM_I32) {
        if (!weighted) return;                                       // uniform
        constexpr int NE = Acc<DT, UB>::NE;
        if constexpr (TEAMS > 1) {
            if (team) {
#pragma unroll
                for (int i = 0; i < NE; ++i) other[i][tid & 255] = acc.v[i];
            }
            __syncthreads();
            if (team) return;
#pragma unroll
            for (int i = 0; i < NE; ++i) acc.v[i] += other[i][tid];
        }
        if (active && group < chunks && sub < p.n_sub) {
            float *out = a.partial + (((long long)b * a.n_planes + pi) * a.n_sub_max + sub) * a.max_row_elems +
                         (long long)unit * NE;
#pragma unroll
            for (int i = 0; i < NE; ++i) out[i] = acc.v[i];
        }
    }
}

// What bounds it: HBM.  A thread keeps the eight loads of a batch in flight and then waits for them, so the chip is kept
// busy by the workgroups resident beside each other.  A chunk's batches go to two teams of 256 threads where it has two or more.  That
// puts no more loads in flight (84 registers: two such workgroups, 16 waves, on a compute unit against five of one team, 20), but a
// chunk is done in half the time and two fifths as many are under way: one team with chunks of half the rows gains as much here
// (16384 -> 5091 rows of 12 KB: 53.6 us, two teams 49.0, half the rows 47.4) and pays for twice the partial sums in the fold.
// One team -> two, whole calls: 16384 -> 5091 rows of 12 KB 90.4 -> 83 us, 8 x 3000 -> 1000 rows of 12 KB in three planes 119 ->
// 112, 2 x 10000 -> 5000 rows of 7 KB 79 -> 70; of 120 shapes beyond the line 7 % faster on average (with the index lists and the
// fold), nine slower by more than 1 %: chunks of 16 rows of planes of several widths (at worst 5 x 769 -> 76 rows of 14 KB and 2 KB
// 29.3 -> 32.0) and rows of 512 bytes (4 x 10000 -> 3100, 63.2 -> 66.7).  Chunks too short for two batches keep one team (2048 ->
// 1000 rows of 7 KB 22.9 -> 26.4 us with two).
// ONCE: loads past the caches, for planes that outgrow the 256 MB cache in front of the memory: they would only push each
// other out of it (305 MB: the call 112 -> 100 us; 353 MB: 150 -> 129); smaller ones may still lie there since they were
// written (64 MB 39 -> 45 us, 203 MB 83 -> 85 with such loads).
template <int TEAMS, bool ONCE>
__global__ __launch_bounds__(256 * TEAMS) void gather_kernel(GatherArgs a) {
    __shared__ float other[TEAMS > 1 ? 8 : 1][256];       // the second team's sums
    __shared__ GatherTable table;
    const int pi = blockIdx.z / a.B, b = blockIdx.z % a.B;
    // (selected by comparison: indexing the argument array with a run-time value would copy it to scratch)
    PlaneDev p = a.plane[0];
#pragma unroll
    for (int i = 1; i < LVLM_MAX_PLANES; ++i)
        if (pi == i) p = a.plane[i];
    if (p.dtype == LVLM_BF16) {
        if (p.unit_bytes == 16) gather_plane<LVLM_BF16, 16, TEAMS, ONCE>(a, p, pi, b, other, table);
        else if (p.unit_bytes == 4) gather_plane<LVLM_BF16, 4, TEAMS, ONCE>(a, p, pi, b, other, table);
        else gather_plane<LVLM_BF16, 2, TEAMS, ONCE>(a, p, pi, b, other, table);
    } else if (p.dtype == LVLM_F32) {
        if (p.unit_bytes == 16) gather_plane<LVLM_F32, 16, TEAMS, ONCE>(a, p, pi, b, other, table);
        else gather_plane<LVLM_F32, 4, TEAMS, ONCE>(a, p, pi, b, other, table);
    } else {
        if (p.unit_bytes == 16) gather_plane<LVLM_I32, 16, TEAMS, ONCE>(a, p, pi, b, other, table);
        else gather_plane<LVLM_I32, 4, TEAMS, ONCE>(a, p, pi, b, other, table);
    }
}

// P_new[c] = sum of the chunks' partial sums, rounded once.  A workgroup owns S columns; its S thread
// rows each add a contiguous share of the chunks (independent loads, unrolled), then the shares are
// added in order -- a fixed summation tree, so the result is reproducible.
// S = 32 shortens the chain where the chunks are many and the workgroups few (413 chunks of 6144 columns 6.5 -> 4.7 us, 360 of 2 x
// 3584 5.2 -> 4.6); with fewer chunks the larger workgroups cost what it gives (266 of 3584 3.9 -> 4.4), with more than a turn of
// them they cost more (16 x 5120 columns 6.5 -> 11.2).
template <int S>
__global__ __launch_bounds__(S * S) void finalize_kernel(GatherArgs a) {
    __shared__ float share[S][S + 1];
    const int pi = blockIdx.y / a.B, b = blockIdx.y % a.B;
    const PlaneDev &p = a.plane[pi];
    if (p.rule != LVLM_RULE_WEIGHTED) return;
    const int col = threadIdx.x % S, grp = threadIdx.x / S;
    const int c = blockIdx.x * S + col;
    if ((int)blockIdx.x * S >= p.row_elems) return;
    const int per = (p.n_sub + S - 1) / S;
    const int i_lo = grp * per, i_hi = min(p.n_sub, i_lo + per);
    float s = 0.f;
    if (c < p.row_elems) {
        const float *part = a.partial + ((long long)b * a.n_planes + pi) * a.n_sub_max * a.max_row_elems + c;
#pragma unroll 8
        for (int i = i_lo; i < i_hi; ++i) s += part[(long long)i * a.max_row_elems];
    }
    share[grp][col] = s;
    __syncthreads();
    if (grp == 0 && c < p.row_elems) {
        float t = 0.f;
#pragma unroll
        for (int g2 = 0; g2 < S; ++g2) t += share[g2][col];
        char *dst = p.dst + (long long)b * p.dst_stride_b + (long long)(a.img_begin + a.n_keep - 1) * p.row_bytes;
        if (p.dtype == LVLM_BF16)
            reinterpret_cast<uint16_t *>(dst)[c] = f32_to_bf16(t);
        else
            reinterpret_cast<float *>(dst)[c] = t;
    }
}

}  // namespace

size_t rank_scratch_bytes(int n, int B) {
    if (n < kSortMinTokens) return 0;
    return (size_t)B * ((n + kSortBlock - 1) / kSortBlock) * kSortBlock * sizeof(unsigned long long);
}

namespace {
template <class KEY>
void launch_rank_by(const Prof &prof, const KEY &key, int32_t *rank, int n, int B, void *scratch, const NormJob *norm,
                    int32_t *kept = nullptr, int n_kept = 0) {
    hipStream_t stream = prof.stream;
    RankArgs<KEY> a{};
    a.key = key;
    a.rank = rank;
    a.n = n;
    a.kept = kept;
    a.n_kept = n_kept;
    int norm_wgs = 0;
    if (norm) {
        a.norm = *norm;
        norm_wgs = (norm->n + 15) / 16;
    }
    if (scratch && n >= kSortMinTokens) {
        a.sorted = static_cast<unsigned long long *>(scratch);
        a.n_blocks = (n + kSortBlock - 1) / kSortBlock;
        a.rank_wgs = a.n_blocks * (kSortBlock / 64);
        const SearchForm f = rank_search_form(n, B);
        a.parts = f.parts;
        LVLM_LAUNCH(prof, rank_block_kernel<KEY>, dim3(a.rank_wgs + norm_wgs, B), dim3(1024), 0, stream, a);
#define LVLM_SEARCH(TG, S) \
    LVLM_LAUNCH(prof, (rank_search_kernel<KEY, TG, S>), dim3((n + 64 * TG - 1) / (64 * TG), B, a.parts), dim3(1024), 0, stream, a)
        if (f.groups == 1) LVLM_SEARCH(1, 16);
        else if (f.groups == 2) LVLM_SEARCH(2, 8);
        else LVLM_SEARCH(4, 8);
#undef LVLM_SEARCH
        if (a.parts > 1) LVLM_LAUNCH(prof, rank_finish_kernel<KEY>, dim3((n + 255) / 256, B), dim3(256), 0, stream, a);
        return;
    }
    a.rank_wgs = (n + kRankBlock - 1) / kRankBlock;
    LVLM_LAUNCH(prof, rank_kernel<KEY>, dim3(a.rank_wgs + norm_wgs, B), dim3(1024), 0, stream, a);
}
}  // namespace

void launch_rank(const Prof &prof, const float *score, int32_t *rank, int n, int B, void *scratch, const NormJob *norm,
                 int32_t *kept, int n_kept) {
    launch_rank_by(prof, ByScore{score}, rank, n, B, scratch, norm, kept, n_kept);
}

void launch_owner_order(const Prof &prof, const OwnerJob &owners, int32_t *rank, int n, int B, void *scratch) {
    launch_rank_by(prof, ByOwner{owners}, rank, n, B, scratch, nullptr);
}

MergeWs merge_ws(const lvlm_merge_desc &d, const lvlm_plane *planes) {
    MergeWs w{};
    w.n_split = 1;
    // gather kernel: rows per partial sum
    int max_elems = 1;
    long long units = 0;
    for (int i = 0; i < d.n_planes; ++i) {
        if (planes[i].row_elems > max_elems) max_elems = planes[i].row_elems;
        units += ((long long)planes[i].row_elems * elem_bytes(planes[i].dtype) + 4095) / 4096;
    }
    // about six workgroups per CU (a workgroup waits out the memory latency of every batch of rows, so the
    // overlap comes from its neighbours); longer chunks would mean fewer partial sums to write and re-read
    long long rows = (long long)d.N * d.B * (units ? units : 1) / kGatherWgs;
    rows = rows / 4 * 4;
    w.rows_per_chunk = (int)(rows < kGatherRows ? kGatherRows : (rows > kGatherChunkRows ? kGatherChunkRows : rows));
    w.n_chunk = (d.N + w.rows_per_chunk - 1) / w.rows_per_chunk;
    w.max_row_elems = max_elems;
    w.rank_part = 0;
    w.kept = align_up(w.rank_part + (size_t)d.B * w.n_split * d.n_img * sizeof(int32_t), 256);
    w.partial = align_up(w.kept + (size_t)d.B * ((d.n_img + 63) / 64) * sizeof(int32_t), 256);
    w.sorted = align_up(w.partial + (size_t)d.B * d.n_planes * w.n_chunk * max_elems * sizeof(float), 256);
    w.total = align_up(w.sorted + rank_scratch_bytes(d.n_img, d.B), 256);
    return w;
}

hipError_t launch_merge(const Prof &prof, const lvlm_merge_desc &d, const MergeWs &w, char *ws,
                        const float *score_mean, const float *wtab, const lvlm_plane *planes, int32_t *keep_idx,
                        int32_t *merged_idx) {
    hipStream_t stream = prof.stream;
    const int r = d.n_img - d.n_keep;
    GatherArgs g{};
    g.B = d.B; g.N = d.N; g.img_begin = d.img_begin; g.n_img = d.n_img; g.n_keep = d.n_keep;
    g.n_planes = d.n_planes;
    g.rows_per_sub = w.rows_per_chunk;
    g.n_sub_max = w.n_chunk;
    g.max_row_elems = w.max_row_elems;
    g.partial = reinterpret_cast<float *>(ws + w.partial);
    const double m = (double)r + 1.0;
    int32_t *rank = reinterpret_cast<int32_t *>(ws + w.rank_part), *kept = reinterpret_cast<int32_t *>(ws + w.kept);
    g.rank = r > 0 ? rank : nullptr;
    g.kept = kept;
    g.keep_idx = keep_idx;
    g.merged_idx = merged_idx;
    g.w = wtab;
    g.lin_scale = (float)(1.0 / (m * (m + 1.0) / 2.0));

    int grid_x = 1, grid_y = 1;
    bool any_weighted = false;
    long long source_bytes = 0;
    for (int i = 0; i < d.n_planes; ++i) {
        PlaneDev &p = g.plane[i];
        p = make_plane_dev(planes[i]);
        p.n_sub = w.n_chunk;
        const int groups = gather_chunks(p, w.rows_per_chunk);
        const int gx = (p.n_sub + groups - 1) / groups;
        if (gx > grid_x) grid_x = gx;
        if (p.col_blocks > grid_y) grid_y = p.col_blocks;
        any_weighted |= p.rule == LVLM_RULE_WEIGHTED;
        source_bytes += (long long)d.B * d.N * p.row_bytes;
    }

    if (r > 0) {
        prof.begin("merge_rank");
        launch_rank(prof, score_mean, rank, d.n_img, d.B, ws + w.sorted, nullptr, kept, d.n_keep - 1);
        prof.end();
    }
    prof.begin("merge_gather");
    const dim3 gather_grid(grid_x, grid_y, d.B * d.n_planes);
    if (w.rows_per_chunk < 2 * kGatherRows) LVLM_LAUNCH(prof, (gather_kernel<1, false>), gather_grid, dim3(256), 0, stream, g);
    else if (source_bytes <= kGatherCached) LVLM_LAUNCH(prof, (gather_kernel<2, false>), gather_grid, dim3(512), 0, stream, g);
    else LVLM_LAUNCH(prof, (gather_kernel<2, true>), gather_grid, dim3(512), 0, stream, g);
    prof.end();
    if (r > 0 && any_weighted) {
        prof.begin("merge_finalize");
        const dim3 wide((w.max_row_elems + 31) / 32, d.B * d.n_planes);
        if (w.n_chunk >= 320 && (long long)wide.x * wide.y <= 512)
            LVLM_LAUNCH(prof, finalize_kernel<32>, wide, dim3(1024), 0, stream, g);
        else
            LVLM_LAUNCH(prof, finalize_kernel<16>, dim3((w.max_row_elems + 15) / 16, d.B * d.n_planes), dim3(256), 0, stream, g);
        prof.end();
    }
    return hipGetLastError();
}

}  // namespace lvlm
