// Step 3b -- similarity merge (named by the benchmark spec; the paper itself merges by rank weights and
// avoids clustering, Sec. 3.2.1 par. 3).  The dominant tokens are the n_keep highest-scoring ones; every
// other token joins the dominant token it is most similar to (cosine of the rows of plane 0) and each
// dominant token becomes the size-weighted mean of its cluster.
//
//   rank_kernel (merge.hip)  ranks by score -> dominant = rank < n_keep; in the same launch 1 / |row| of every image token
//   sim_index_kernel         positions of dominant tokens, list of the others (both ascending)
//   sim_gemm_kernel          the one dense contraction of the path: (dominant x others) dot products on
//                            the matrix cores, with the arg-max over the dominant axis taken in the epilogue (nothing
//                            of the similarity matrix is stored): one 64-bit atomic maximum per other token and tile of
//                            (cosine, lower position first), so the result does not depend on who comes first
//   rank_kernel              tokens ordered by (dominant position joined, index): each cluster is a contiguous,
//                            index-ordered segment, so the sums below run in a fixed order
//   sim_merge_kernel         one workgroup per dominant token: size-weighted mean of its cluster; further workgroups
//                            copy the rows outside the image span
#include <limits.h>

#include "common.h"
#include "mma.h"
#include "planes.h"

namespace lvlm {
namespace {

struct SimArgs {
    PlaneDev plane[LVLM_MAX_PLANES];
    const float *size_in;   // [B, n] or null (all ones)
    float *size_out;        // [B, n_keep] or null
    int32_t *rank;          // [B, n]
    int32_t *dom_of;        // [B, n]  p >= 0: dominant position; -(q+1): q-th other token
    int32_t *keep_idx;      // [B, n_keep]
    int32_t *rest_idx;      // [B, r]
    float *inv_norm;        // [B, n]
    unsigned long long *best;   // [B, r]  (key of the cosine, ~dominant position)
    int32_t *assign;        // [B, n]
    int32_t *order;         // [B, n]   other tokens by (assignment, index), then the dominant ones
    int32_t *owner;         // [B, n]   assignment of order[s]
    int B, N, img_begin, n, n_keep, r, n_planes;
};

// ---- dominant positions and the list of the other tokens, both in ascending index ----
// One workgroup per 4096 tokens of a sequence (thread t holds four of them); it counts the dominant tokens in front of
// its chunk itself, all loads in flight together, so the chunks need nothing from each other.
constexpr int kSimChunk = 4096;
__global__ __launch_bounds__(1024) void sim_index_kernel(SimArgs a) {
    __shared__ int wave_tot[16], wave_before[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.y, s0 = blockIdx.x * kSimChunk, j0 = s0 + 4 * tid;
    const int32_t *rank = a.rank + (long long)b * a.n;
    bool dom[4];
    int cnt = 0, before = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        dom[e] = j0 + e < a.n && rank[min(j0 + e, a.n - 1)] < a.n_keep;
        cnt += dom[e];
    }
#pragma unroll 4
    for (int i = tid; i < s0; i += 1024) before += rank[i] < a.n_keep;
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
        before += __shfl_xor(before, o);
    }
    if (lane == 63) wave_tot[wave] = incl;
    if (lane == 0) wave_before[wave] = before;
    __syncthreads();
    int p = incl - cnt;
#pragma unroll
    for (int w = 0; w < 16; ++w) p += wave_before[w] + (w < wave ? wave_tot[w] : 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = j0 + e;
        if (j >= a.n) continue;
        if (dom[e]) {
            a.dom_of[(long long)b * a.n + j] = p;
            a.keep_idx[(long long)b * a.n_keep + p] = j;
            ++p;
        } else {
            const int q = j - p;              // tokens before j that are not dominant
            a.dom_of[(long long)b * a.n + j] = -(q + 1);
            a.rest_idx[(long long)b * a.r + q] = j;
            a.best[(long long)b * a.r + q] = 0ull;
        }
    }
}

// ---- dot products dominant x others on the matrix cores, arg-max over the dominant axis ----
// Workgroup tile: TM dominant rows x TN other rows, NWN x NWM waves, each owning TR x TC tiles of 32 x 32.
// Two shapes are built: 256 x 256 with eight waves of 128 x 64 (large problems: per tile product it moves
// a third less through LDS than the small shape, and half as much from L2) and 128 x 128 with four waves of
// 64 x 64 (more workgroups when the problem is small).  Rows are gathered by index; the contraction runs
// over 128-byte slices of the rows, double buffered in LDS with the next slice's global loads in flight
// (named scalars: they are carried around the loop).  One slice is eight 16-byte units per row and every
// thread stages four units of the dominant and four of the other rows.
//
// Tiles are numbered block by block (blocks of GN x GM tiles, ragged at the edges, batch rows one after the
// other) and handed out in runs of GN * GM consecutive numbers, run j to XCD j % 8 (workgroups reach the
// XCDs round-robin by id).  The workgroups resident on an XCD at the same time are then neighbours that
// sweep the contraction axis together: a row slice fetched into that XCD's L2 serves up to GM (dominant
// rows) or GN (other rows) of them, and every XCD gets the same number of tiles to within one run.
constexpr int kSimGN = 8, kSimGM = 4;

template <int DT, int NWN, int NWM, int TR, int TC, bool RAGGED>
__global__ __launch_bounds__(64 * NWN * NWM) void sim_gemm_kernel(SimArgs a) {
    constexpr int NT = 64 * NWN * NWM;
    constexpr int TM = NWN * TR * 32, TN = NWM * TC * 32;
    constexpr int SB = 128;              // bytes of one slice of a row
    constexpr int PITCH = SB + 16;       // slice + 16 bytes: spreads the rows over the LDS banks
    constexpr int RPI = NT / 8;          // rows one load instruction of the workgroup covers
    constexpr int UA = TM / RPI, UB = TN / RPI;      // staging units per thread: rows srow + RPI j of each operand
    __shared__ __attribute__((aligned(16))) char a_lds[2][TM * PITCH];
    __shared__ __attribute__((aligned(16))) char b_lds[2][TN * PITCH];
    __shared__ float invn[TM];
    __shared__ float bv[NWN][TN];
    __shared__ int bi[NWN][TN];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hf = lane >> 5, l32 = lane & 31;
    const int wn = wave % NWN, wm = __builtin_amdgcn_readfirstlane(wave / NWN);
    // tile of this workgroup
    const int NBt = (a.n_keep + TM - 1) / TM, MBt = (a.r + TN - 1) / TN;
    constexpr int RUN = kSimGN * kSimGM;
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    int t = ((seq / RUN) * 8 + xcd) * RUN + seq % RUN;
    if (t >= a.B * NBt * MBt) return;
    const int b = t / (NBt * MBt);
    t -= b * NBt * MBt;
    const int gm = (MBt + kSimGM - 1) / kSimGM, gn = (NBt + kSimGN - 1) / kSimGN;
    const int bj = min(t / (NBt * kSimGM), gm - 1);              // row of blocks; its height (the last may be lower)
    t -= bj * NBt * kSimGM;
    const int bh = min(kSimGM, MBt - bj * kSimGM);
    const int bi_ = min(t / (kSimGN * bh), gn - 1);              // block in that row; its width
    t -= bi_ * kSimGN * bh;
    const int bw = min(kSimGN, NBt - bi_ * kSimGN);
    const int nb = bi_ * kSimGN + t % bw, mb = bj * kSimGM + t / bw;

    const PlaneDev &p = a.plane[0];
    const int32_t *keep = a.keep_idx + (long long)b * a.n_keep;
    const int32_t *rest = a.rest_idx + (long long)b * a.r;
    const int srow = tid >> 3, su = tid & 7;        // staging: rows srow + RPI j (j < 4), unit su of the slice
    // Addresses are a uniform base (batch row, slice) plus a per-thread 32-bit byte offset (row, unit) that
    // never changes: the slice loop then needs no vector instruction per load -- on this chip matrix and
    // vector instructions do not overlap, so every one of them is time taken from the matrix cores.  The
    // offsets fit: the image rows of one batch row span less than 2 GiB (checked on the host).
    const char *img = p.src + (long long)b * p.src_stride_b + (long long)a.img_begin * p.row_bytes;
    // (named scalars below, not arrays: values carried around the slice loop must stay in registers)
    static_assert(UA <= 8 && UB <= 8, "staging registers are written out for up to eight units");
#define LVLM_SIM8(M) M(0) M(1) M(2) M(3) M(4) M(5) M(6) M(7)
#define LVLM_DECL(j)                                                                                        \
    const unsigned oa##j = j < UA ? keep[min(nb * TM + srow + RPI * j, a.n_keep - 1)] * p.row_bytes + 16 * su : 0; \
    const unsigned ob##j = j < UB ? rest[min(mb * TN + srow + RPI * j, a.r - 1)] * p.row_bytes + 16 * su : 0;      \
    uint4 sa##j, sb##j;      /* written by load before store reads them */
    LVLM_SIM8(LVLM_DECL)
#undef LVLM_DECL
    for (int i = tid; i < TM; i += NT) invn[i] = a.inv_norm[(long long)b * a.n + keep[min(nb * TM + i, a.n_keep - 1)]];
    const int nk = (p.row_bytes + SB - 1) / SB;      // the last slice may be partial: zero-filled

    // RAGGED: rows that are not a whole number of slices; units of the last slice beyond the row read as zero
    auto load = [&](int k) {
        const char *base = img + SB * k;             // uniform
        const bool in = !RAGGED || p.row_bytes - SB * k - 16 * su >= 16;
        const uint4 z = make_uint4(0, 0, 0, 0);
#define LVLM_LD(j)                                                                              \
        if constexpr (j < UA) sa##j = in ? *reinterpret_cast<const uint4 *>(base + oa##j) : z;  \
        if constexpr (j < UB) sb##j = in ? *reinterpret_cast<const uint4 *>(base + ob##j) : z;
        LVLM_SIM8(LVLM_LD)
#undef LVLM_LD
    };
    auto store = [&](int buf) {
        char *da = &a_lds[buf][srow * PITCH + 16 * su], *db = &b_lds[buf][srow * PITCH + 16 * su];
#define LVLM_ST(j)                                                                      \
        if constexpr (j < UA) *reinterpret_cast<uint4 *>(da + j * RPI * PITCH) = sa##j;  \
        if constexpr (j < UB) *reinterpret_cast<uint4 *>(db + j * RPI * PITCH) = sb##j;
        LVLM_SIM8(LVLM_ST)
#undef LVLM_ST
    };

    f32x16 acc[TR][TC];
#pragma unroll
    for (int nd = 0; nd < TR; ++nd)
#pragma unroll
        for (int nr = 0; nr < TC; ++nr)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nd][nr][r] = 0.f;

    load(0);
    store(0);
    load(min(1, nk - 1));
    __syncthreads();
    for (int k = 0; k < nk; ++k) {
        store((k + 1) & 1);                      // slice k+1 (a harmless repeat after the last one)
        load(min(k + 2, nk - 1));
        const int buf = k & 1;
        const char *ar = &a_lds[buf][(wn * TR * 32 + l32) * PITCH + (SB / 2) * hf];
        const char *br = &b_lds[buf][(wm * TC * 32 + l32) * PITCH + (SB / 2) * hf];
        // one contraction step (16 bytes per lane and tile row) at a time: TR + TC operand words, TR x TC products
#pragma unroll
        for (int i = 0; i < SB / 32; ++i) {
            uint4 fa[TR], fb[TC];
#pragma unroll
            for (int t = 0; t < TR; ++t) fa[t] = *reinterpret_cast<const uint4 *>(ar + t * 32 * PITCH + 16 * i);
#pragma unroll
            for (int t = 0; t < TC; ++t) fb[t] = *reinterpret_cast<const uint4 *>(br + t * 32 * PITCH + 16 * i);
#pragma unroll
            for (int nd = 0; nd < TR; ++nd)
#pragma unroll
                for (int nr = 0; nr < TC; ++nr) {
                    if constexpr (DT == LVLM_BF16) {
                        mfma_one<DT>(acc[nd][nr], fa[nd], fb[nr], 0);      // rows = dominant, cols = others
                    } else {
#pragma unroll
                        for (int cpt = 0; cpt < 4; ++cpt) mfma_one<DT>(acc[nd][nr], fa[nd], fb[nr], cpt);
                    }
                }
        }
        __syncthreads();
    }

    // arg-max over the dominant rows: lane-local over its TR x 16 registers, then the other lane half, then
    // the NWN waves that share the columns.  Larger cosine wins; equal cosines go to the lower position.
#pragma unroll
    for (int nr = 0; nr < TC; ++nr) {
        float best_v = -INFINITY;
        int best_i = INT_MAX;
#pragma unroll
        for (int nd = 0; nd < TR; ++nd) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int il = wn * TR * 32 + nd * 32 + acc_row(r, hf);
                const int gi = nb * TM + il;
                const float v = acc[nd][nr][r] * invn[il];
                if (gi < a.n_keep && (v > best_v || (v == best_v && gi < best_i))) {
                    best_v = v;
                    best_i = gi;
                }
            }
        }
        const float ov = __shfl_xor(best_v, 32);
        const int oi = __shfl_xor(best_i, 32);
        if (ov > best_v || (ov == best_v && oi < best_i)) {
            best_v = ov;
            best_i = oi;
        }
        if (hf == 0) {
            bv[wn][wm * TC * 32 + nr * 32 + l32] = best_v;
            bi[wn][wm * TC * 32 + nr * 32 + l32] = best_i;
        }
    }
    __syncthreads();
    for (int i = tid; i < TN; i += NT) {
        const int q = mb * TN + i;
        if (q < a.r) {
            float v = bv[0][i];
            int ix = bi[0][i];
#pragma unroll
            for (int w = 1; w < NWN; ++w)
                if (bv[w][i] > v || (bv[w][i] == v && bi[w][i] < ix)) {
                    v = bv[w][i];
                    ix = bi[w][i];
                }
            if (ix != INT_MAX)
                atomicMax(&a.best[(long long)b * a.r + q],
                          ((unsigned long long)score_key(v) << 32) | (unsigned long long)(0xffffffffu - (uint32_t)ix));
        }
    }
#undef LVLM_SIM8
}

// ---- size-weighted mean of each cluster ----
template <int DT, int UB>
__device__ __forceinline__ void store_mean(char *dst, const Acc<DT, UB> &acc, float inv_tot) {
    if constexpr (DT == LVLM_BF16 && UB == 16) {
        uint4 u;
        u.x = (uint32_t)f32_to_bf16(acc.v[0] * inv_tot) | ((uint32_t)f32_to_bf16(acc.v[1] * inv_tot) << 16);
        u.y = (uint32_t)f32_to_bf16(acc.v[2] * inv_tot) | ((uint32_t)f32_to_bf16(acc.v[3] * inv_tot) << 16);
        u.z = (uint32_t)f32_to_bf16(acc.v[4] * inv_tot) | ((uint32_t)f32_to_bf16(acc.v[5] * inv_tot) << 16);
        u.w = (uint32_t)f32_to_bf16(acc.v[6] * inv_tot) | ((uint32_t)f32_to_bf16(acc.v[7] * inv_tot) << 16);
        *reinterpret_cast<uint4 *>(dst) = u;
    } else if constexpr (DT == LVLM_BF16 && UB == 4) {
        *reinterpret_cast<uint32_t *>(dst) =
            (uint32_t)f32_to_bf16(acc.v[0] * inv_tot) | ((uint32_t)f32_to_bf16(acc.v[1] * inv_tot) << 16);
    } else if constexpr (DT == LVLM_BF16 && UB == 2) {
        *reinterpret_cast<uint16_t *>(dst) = f32_to_bf16(acc.v[0] * inv_tot);
    } else if constexpr (DT == LVLM_F32 && UB == 16) {
        *reinterpret_cast<float4 *>(dst) =
            make_float4(acc.v[0] * inv_tot, acc.v[1] * inv_tot, acc.v[2] * inv_tot, acc.v[3] * inv_tot);
    } else if constexpr (DT == LVLM_F32 && UB == 4) {
        *reinterpret_cast<float *>(dst) = acc.v[0] * inv_tot;
    }
}

// Units unit0, unit0 + 256, ... of one plane's row of dominant position i (token ji), NU at a time.  `members` holds the
// cluster's first 64 other tokens, one per lane; up to four of their rows are in flight together.
template <int DT, int UB, int NU>
__device__ __forceinline__ void merge_plane(const SimArgs &a, const PlaneDev &p, int b, int i, int ji, int lo, int n_mem,
                                            int members) {
    using U = typename Unit<UB>::type;
    const int units = p.row_bytes / UB;
    const char *img0 = p.src + (long long)b * p.src_stride_b + (long long)a.img_begin * p.row_bytes;
    char *dst0 = p.dst + (long long)b * p.dst_stride_b + (long long)(a.img_begin + i) * p.row_bytes;
    const bool weighted = p.rule == LVLM_RULE_WEIGHTED && DT != LVLM_I32;
    const float *size = a.size_in ? a.size_in + (long long)b * a.n : nullptr;
    // whole waves in and out of the loop: lanes without a unit still hand out member indices
    for (int w0 = threadIdx.x & ~63; w0 < units; w0 += 256 * NU) {
        const int u0 = w0 + (threadIdx.x & 63);
        int off[NU];                            // byte offset of the unit in a row (a repeat past the end, not stored)
#pragma unroll
        for (int x = 0; x < NU; ++x) off[x] = min(u0 + 256 * x, units - 1) * UB;
        U own[NU];
#pragma unroll
        for (int x = 0; x < NU; ++x) own[x] = *reinterpret_cast<const U *>(img0 + (long long)ji * p.row_bytes + off[x]);
        if (!weighted) {
#pragma unroll
            for (int x = 0; x < NU; ++x)
                if (u0 + 256 * x < units) *reinterpret_cast<U *>(dst0 + off[x]) = own[x];
            continue;
        }
        if constexpr (DT != LVLM_I32) {
            Acc<DT, UB> acc[NU];
            float tot = size ? size[ji] : 1.0f;
#pragma unroll
            for (int x = 0; x < NU; ++x) {
#pragma unroll
                for (int e = 0; e < Acc<DT, UB>::NE; ++e) acc[x].v[e] = 0.f;
                accumulate<DT, UB>(acc[x], own[x], tot);
            }
            int mem = members;
            for (int s0 = 0; s0 < n_mem; s0 += 4) {          // cluster members in ascending index
                if ((s0 & 63) == 0 && s0 > 0) mem = a.order[(long long)b * a.n + min(lo + s0 + (int)(threadIdx.x & 63), a.n - 1)];
                U val[4][NU];
                float w[4];
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const int t = __builtin_amdgcn_readlane(mem, (min(s0 + y, n_mem - 1)) & 63);
                    w[y] = size ? size[t] : 1.0f;
#pragma unroll
                    for (int x = 0; x < NU; ++x) val[y][x] = *reinterpret_cast<const U *>(img0 + (long long)t * p.row_bytes + off[x]);
                }
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    if (s0 + y >= n_mem) break;
#pragma unroll
                    for (int x = 0; x < NU; ++x) accumulate<DT, UB>(acc[x], val[y][x], w[y]);
                    tot += w[y];
                }
            }
#pragma unroll
            for (int x = 0; x < NU; ++x)
                if (u0 + 256 * x < units) store_mean<DT, UB>(dst0 + off[x], acc[x], 1.0f / tot);
            if (size && a.size_out && threadIdx.x == 0 && u0 == 0) a.size_out[(long long)b * a.n_keep + i] = tot;
        }
    }
}

// One row of every plane from its old place to its new one.
__device__ __forceinline__ void copy_row(const SimArgs &a, int b, int from, int to) {
    for (int pi = 0; pi < a.n_planes; ++pi) {
        const PlaneDev &p = a.plane[pi];
        const char *s = p.src + (long long)b * p.src_stride_b + (long long)from * p.row_bytes;
        char *d = p.dst + (long long)b * p.dst_stride_b + (long long)to * p.row_bytes;
        for (int byte = threadIdx.x * p.unit_bytes; byte < p.row_bytes; byte += 256 * p.unit_bytes) {
            if (p.unit_bytes == 16) *reinterpret_cast<uint4 *>(d + byte) = *reinterpret_cast<const uint4 *>(s + byte);
            else if (p.unit_bytes == 4) *reinterpret_cast<uint32_t *>(d + byte) = *reinterpret_cast<const uint32_t *>(s + byte);
            else *reinterpret_cast<uint16_t *>(d + byte) = *reinterpret_cast<const uint16_t *>(s + byte);
        }
    }
}

// nothing removed: every row stays where it is
__global__ __launch_bounds__(256) void sim_copy_kernel(SimArgs a) { copy_row(a, blockIdx.y, blockIdx.x, blockIdx.x); }

// One workgroup per dominant position, every plane and column in it; workgroups past them copy the rows outside the
// image span.  The tokens assigned to position i form the
// segment [lo, lo + n) of the sorted order; its two ends are found by all waves at once, 64 probes of the owners a
// round (two rounds up to 4096 other tokens, three up to 262144) instead of one thread's bisection, whose chain of some
// 20 pairs of dependent loads per workgroup was the time of the kernel.  Bound by memory: 8 x 1263 clusters of 4096 bf16
// channels (213 MB) 72 -> 33 us.
__global__ __launch_bounds__(256) void sim_merge_kernel(SimArgs a) {
    const int i = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63;
    if (i >= a.n_keep) {
        const int o = i - a.n_keep;                  // o-th row outside the image span
        copy_row(a, b, o < a.img_begin ? o : o + a.n, o < a.img_begin ? o : o + a.n_keep);
        return;
    }
    const int32_t *order = a.order + (long long)b * a.n, *owner = a.owner + (long long)b * a.n;
    const int ji = a.keep_idx[(long long)b * a.n_keep + i];
    // owners below i, and below i + 1, among the r other tokens: each lies in a range [base, base + len)
    int lo = 0, hi = 0, len_lo = a.r, len_hi = a.r;
    while (len_lo > 0 || len_hi > 0) {
        const int st_lo = (len_lo + 65) / 65, st_hi = (len_hi + 65) / 65;      // probes base + step * (lane + 1) - 1
        const int p_lo = lo + st_lo * (lane + 1) - 1, p_hi = hi + st_hi * (lane + 1) - 1;
        const int o_lo = owner[min(p_lo, a.n - 1)], o_hi = owner[min(p_hi, a.n - 1)];
        const int c_lo = __popcll(__ballot(len_lo > 0 && st_lo * (lane + 1) <= len_lo && o_lo < i));
        const int c_hi = __popcll(__ballot(len_hi > 0 && st_hi * (lane + 1) <= len_hi && o_hi < i + 1));
        // c probes are below: the end lies in the step behind the last of them, whose own last place is no candidate
        const int rest_lo = len_lo - c_lo * st_lo, rest_hi = len_hi - c_hi * st_hi;
        lo += c_lo * st_lo;
        hi += c_hi * st_hi;
        len_lo = max(0, min(st_lo - 1, rest_lo));
        len_hi = max(0, min(st_hi - 1, rest_hi));
    }
    const int n_mem = hi - lo;
    const int members = order[min(lo + lane, a.n - 1)];
    // sizes of all-ones clusters are written here (the weighted path writes them when sizes are given)
    if (threadIdx.x == 0 && a.size_out && a.size_in == nullptr) a.size_out[(long long)b * a.n_keep + i] = (float)(1 + n_mem);
    for (int pi = 0; pi < a.n_planes; ++pi) {
        const PlaneDev &p = a.plane[pi];
        if (p.dtype == LVLM_BF16) {
            if (p.unit_bytes == 16) merge_plane<LVLM_BF16, 16, 2>(a, p, b, i, ji, lo, n_mem, members);
            else if (p.unit_bytes == 4) merge_plane<LVLM_BF16, 4, 1>(a, p, b, i, ji, lo, n_mem, members);
            else merge_plane<LVLM_BF16, 2, 1>(a, p, b, i, ji, lo, n_mem, members);
        } else if (p.dtype == LVLM_F32) {
            if (p.unit_bytes == 16) merge_plane<LVLM_F32, 16, 2>(a, p, b, i, ji, lo, n_mem, members);
            else merge_plane<LVLM_F32, 4, 1>(a, p, b, i, ji, lo, n_mem, members);
        } else {
            if (p.unit_bytes == 16) merge_plane<LVLM_I32, 16, 1>(a, p, b, i, ji, lo, n_mem, members);
            else merge_plane<LVLM_I32, 4, 1>(a, p, b, i, ji, lo, n_mem, members);
        }
    }
}

// nothing removed: every token is its own cluster
__global__ __launch_bounds__(256) void sim_identity_kernel(SimArgs a) {
    const int j = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
    if (j >= a.n) return;
    if (a.keep_idx) a.keep_idx[(long long)b * a.n + j] = j;
    if (a.assign) a.assign[(long long)b * a.n + j] = j;
    if (a.size_out) a.size_out[(long long)b * a.n + j] = a.size_in ? a.size_in[(long long)b * a.n + j] : 1.0f;
}

}  // namespace

SimWs sim_ws(const lvlm_merge_desc &d) {
    SimWs w{};
    const size_t n = (size_t)d.B * d.n_img;
    const int r = d.n_img - d.n_keep;
    // the large tile shape once it still gives every CU two workgroups
    w.tile = ((long long)d.B * ((d.n_keep + 255) / 256) * ((r + 255) / 256) >= 512) ? 256 : 128;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    w.rank = take(n * 4);
    w.dom_of = take(n * 4);
    w.keep_idx = take((size_t)d.B * d.n_keep * 4);
    w.rest_idx = take((size_t)d.B * (r > 0 ? r : 1) * 4);
    w.inv_norm = take(n * 4);
    w.best = take((size_t)d.B * (r > 0 ? r : 1) * 8);
    w.assign = take(n * 4);
    w.rank2 = take(n * 4);
    w.order = take(n * 4);
    w.owner = take(n * 4);
    w.sorted = take(rank_scratch_bytes(d.n_img, d.B));     // sorted blocks of the two rankings, used in turn
    w.total = off;
    return w;
}

hipError_t launch_merge_similar(const Prof &prof, const lvlm_merge_desc &d, const SimWs &w, char *ws,
                                const float *score_mean, const lvlm_plane *planes, const float *size_in,
                                float *size_out, int32_t *keep_idx, int32_t *assign) {
    hipStream_t stream = prof.stream;
    const int r = d.n_img - d.n_keep;
    SimArgs a{};
    for (int i = 0; i < d.n_planes; ++i) a.plane[i] = make_plane_dev(planes[i]);
    a.size_in = size_in;
    a.size_out = size_out;
    a.rank = reinterpret_cast<int32_t *>(ws + w.rank);
    a.dom_of = reinterpret_cast<int32_t *>(ws + w.dom_of);
    a.keep_idx = keep_idx ? keep_idx : reinterpret_cast<int32_t *>(ws + w.keep_idx);
    a.rest_idx = reinterpret_cast<int32_t *>(ws + w.rest_idx);
    a.inv_norm = reinterpret_cast<float *>(ws + w.inv_norm);
    a.best = reinterpret_cast<unsigned long long *>(ws + w.best);
    a.assign = assign ? assign : reinterpret_cast<int32_t *>(ws + w.assign);
    a.order = reinterpret_cast<int32_t *>(ws + w.order);
    a.owner = reinterpret_cast<int32_t *>(ws + w.owner);
    a.B = d.B; a.N = d.N; a.img_begin = d.img_begin; a.n = d.n_img; a.n_keep = d.n_keep; a.r = r;
    a.n_planes = d.n_planes;

    if (r == 0) {
        a.keep_idx = keep_idx;
        a.assign = assign;
        prof.begin("sim_copy");
        LVLM_LAUNCH(prof, sim_copy_kernel, dim3(d.N, d.B), dim3(256), 0, stream, a);
        prof.end();
        if (keep_idx || assign || size_out)
            LVLM_LAUNCH(prof, sim_identity_kernel, dim3((d.n_img + 255) / 256, d.B), dim3(256), 0, stream, a);
        return hipGetLastError();
    }

    NormJob norm{};
    norm.src = a.plane[0].src + (long long)d.img_begin * a.plane[0].row_bytes;
    norm.stride_b = a.plane[0].src_stride_b;
    norm.inv_norm = a.inv_norm;
    norm.row_bytes = a.plane[0].row_bytes; norm.dtype = planes[0].dtype; norm.n = d.n_img;
    prof.begin("sim_rank");
    launch_rank(prof, score_mean, a.rank, d.n_img, d.B, ws + w.sorted, &norm);
    prof.end();
    prof.begin("sim_index");
    LVLM_LAUNCH(prof, sim_index_kernel, dim3((d.n_img + kSimChunk - 1) / kSimChunk, d.B), dim3(1024), 0, stream, a);
    prof.end();
    prof.begin("sim_gemm");
    {
        const long long tiles = (long long)d.B * ((d.n_keep + w.tile - 1) / w.tile) * ((r + w.tile - 1) / w.tile);
        constexpr int run = kSimGN * kSimGM;
        const dim3 ggrid((unsigned)(((tiles + run - 1) / run + 7) / 8 * 8 * run));
        const bool bf = planes[0].dtype == LVLM_BF16;
        const bool ragged = (planes[0].row_elems * (bf ? 2 : 4)) % 128 != 0;
#define LVLM_GEMM(DT, NWN, NWM, TR, TC)                                                                              \
    if (ragged)                                                                                                      \
        LVLM_LAUNCH(prof, (sim_gemm_kernel<DT, NWN, NWM, TR, TC, true>), ggrid, dim3(64 * NWN * NWM), 0, stream, a);  \
    else                                                                                                             \
        LVLM_LAUNCH(prof, (sim_gemm_kernel<DT, NWN, NWM, TR, TC, false>), ggrid, dim3(64 * NWN * NWM), 0, stream, a)
        if (w.tile == 256) {
            if (bf) { LVLM_GEMM(LVLM_BF16, 2, 4, 4, 2); } else { LVLM_GEMM(LVLM_F32, 2, 4, 4, 2); }
        } else {
            if (bf) { LVLM_GEMM(LVLM_BF16, 2, 2, 2, 2); } else { LVLM_GEMM(LVLM_F32, 2, 2, 2, 2); }
        }
#undef LVLM_GEMM
    }
    prof.end();
    OwnerJob oj{};
    oj.dom_of = a.dom_of; oj.best = a.best; oj.order = a.order; oj.owner = a.owner; oj.assign = a.assign; oj.r = r;
    prof.begin("sim_order");
    launch_owner_order(prof, oj, reinterpret_cast<int32_t *>(ws + w.rank2), d.n_img, d.B, ws + w.sorted);
    prof.end();
    prof.begin("sim_merge");
    LVLM_LAUNCH(prof, sim_merge_kernel, dim3(d.n_keep + d.N - d.n_img, d.B), dim3(256), 0, stream, a);
    prof.end();
    return hipGetLastError();
}

}  // namespace lvlm
