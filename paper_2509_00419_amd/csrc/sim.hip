// Step 3b -- similarity merge (named by the benchmark spec; the paper itself merges by rank weights and
// avoids clustering, Sec. 3.2.1 par. 3).  The dominant tokens are the n_keep highest-scoring ones; every
// other token joins the dominant token it is most similar to (cosine of the rows of plane 0) and each
// dominant token becomes the size-weighted mean of its cluster.
//
//   rank_kernel (merge.hip)  ranks by score -> dominant = rank < n_keep; in the same launch 1 / |row| of every image token, where
//                            the product does not do that
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
    float *inv_norm;        // [B, n], or null: the product takes the norms itself
    unsigned long long *best;   // [B, r]  (key of the cosine, ~dominant position)
    int32_t *assign;        // [B, n]
    int32_t *order;         // [B, n]   other tokens by (assignment, index), then the dominant ones
    int32_t *owner;         // [B, n]   assignment of order[s]
    int B, N, img_begin, n, n_keep, r, n_planes;
    bool sizes_apart;       // sizes are given and no weighted plane's means would write size_out
    int run;                // consecutive tiles of the similarity product an XCD takes at a time
};

// ---- dominant positions and the list of the other tokens, both in ascending index ----
// One workgroup per 1024 tokens of a sequence, one per thread; it counts the dominant tokens in front of
// its chunk itself, four of a thread's loads in flight together, so the chunks need nothing from each other.
constexpr int kSimChunk = 1024;
__global__ __launch_bounds__(1024) void sim_index_kernel(SimArgs a) {
    __shared__ __attribute__((aligned(16))) int wave_dom[16], wave_before[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.y, s0 = blockIdx.x * kSimChunk, j = s0 + tid;
    const int32_t *rank = a.rank + (long long)b * a.n;
    const bool dom = j < a.n && rank[min(j, a.n - 1)] < a.n_keep;
    uint32_t before = 0;
#pragma unroll 4
    for (int i = tid; i < s0; i += 1024) before += rank[i] < a.n_keep;
    const unsigned long long bal = __ballot(dom);
    before = wave_reduce_u32(before, [](uint32_t x, uint32_t y) { return x + y; });
    if (lane == 0) {
        wave_dom[wave] = __popcll(bal);
        wave_before[wave] = (int)before;
    }
    __syncthreads();
    int p = __popcll(bal & ((1ull << lane) - 1ull));
#pragma unroll
    for (int w = 0; w < 16; ++w) p += wave_before[w] + (w < wave ? wave_dom[w] : 0);
    if (j >= a.n) return;
    if (dom) {
        a.dom_of[(long long)b * a.n + j] = p;
        a.keep_idx[(long long)b * a.n_keep + p] = j;
    } else {
        const int q = j - p;                  // tokens before j that are not dominant
        a.dom_of[(long long)b * a.n + j] = -(q + 1);
        a.rest_idx[(long long)b * a.r + q] = j;
        a.best[(long long)b * a.r + q] = 0ull;
    }
}

// ---- dot products dominant x others on the matrix cores, arg-max over the dominant axis ----
// Workgroup tile: TM dominant rows x TN other rows, each wave 32 TR x 32 TC of it.  Rows are gathered by index; the
// contraction runs over 128-byte slices of the rows, which go from memory straight into a ring of LDS buffers (the
// direct loads need no staging registers and no LDS store instructions).  One wait and one barrier per slice: a
// wave waits for its own share of slice k, the barrier makes that everybody's share and at the same time frees
// the buffer of slice k-1 for slice k + RING - 1.  The direct loads are written out as assembly because the compiler,
// which cannot tell the ring's buffers apart, would wait for all of them before every LDS read; the waits that take
// its place are counted by hand: every wave issues the same number of loads for every slice (repeats of the last
// one past the end).
// A direct load fills 1024 consecutive LDS bytes lane by lane, so rows cannot be padded apart; instead the
// eight 16-byte units of row R lie in the order u ^ (R / 2 % 8), chosen by the address each lane reads from: the sixteen
// lanes an LDS read serves at a time then hit sixteen different bank groups (no conflicts counted).
// What bounds a workgroup is the time a slice takes to arrive, so there are four forms:
//   up to 288 tiles of 64 x 64: these, on four waves with a ring of four.  A workgroup takes in half the rows of a larger tile, and
//       more of them do (276 x 300 tokens of 3584 channels 9 -> 25 tiles, the whole call 43.3 -> 32.5 us; 4 x 270 x 630 of 6144 60 -> 200
//       tiles, 73 -> 56; of 43 shapes up to 288 tiles all gain, 4 to 36 %; 441 tiles are even, 768 lose 14 %; slices of 256 and 512
//       bytes and a ring of eight give nothing)
//   more, but up to 256 tiles of 128 x 128 (one per compute unit): a ring of four slices, eight waves, the loads of a slice spread
//       over the products (a compute unit takes 16 cycles per direct load: all of a slice's at once hold the products up)
//   more, but up to 256 tiles of 128 x 192 or 192 x 128: these, with a ring of three.  A unit then has one tile and a half to do
//       instead of up to two, and takes in 320 rows for it instead of 512 (8 x 1263 x 529 of 4096 channels: 400 -> 240 tiles, 61 ->
//       52 us, the whole call 133 -> 123; of 54 shapes of 260 to 400 tiles all gain, 3 % at 1024 channels to 13 % at 4096; from
//       257 of the larger tiles on the second turn costs 20 to 30 %)
//   more: 128 x 128, a ring of two and four waves, so that two workgroups share a compute unit and cover each other's waits;
//       the loads go out first
// (At 8 x 1263 x 529 of 4096 the loads alone take 38 us of the 52, the products alone 45, LDS reads and barriers alone 28; the
// reads of a slice beside the products of the one before, and four waves of 64 x 96, gave nothing.)
// (wider slices than 64 bytes: half a cache line each time fetched every line twice.  256 x 128 and 256 x 256 tiles, which
// load less per product, leave the last turn of workgroups emptier and came out even or behind.)
// Measured (staging through registers and LDS stores, with the 128- and 256-row tiles it had -> this): 300 x 276 tokens of
// 3584 channels 45 -> 28 us; 8 x 1263 x 529 of 4096 79 -> 59 us (its rows alone, once from memory: 22 us); 5091 x 11293
// of 6144 700 -> 650 us = 1085 TFLOP/s.
//
// Tiles are numbered block by block (blocks of GN x GM tiles, ragged at the edges, batch rows one after the
// other) and handed out in runs of consecutive numbers, run j to XCD j % 8 (workgroups reach the
// XCDs round-robin by id).  The workgroups resident on an XCD at the same time are then neighbours that
// sweep the contraction axis together: a row slice fetched into that XCD's L2 serves up to GM (dominant
// rows) or GN (other rows) of them.  A run is an eighth of the tiles where that is what an XCD can hold at a time (64):
// every XCD gets one stretch and fetches few rows that another one fetches too; else GN * GM.
constexpr int kSimGN = 8, kSimGM = 4;

// Adds the squares of a unit's elements to s, one after the other.
template <int DT>
__device__ __forceinline__ void squares(const uint4 &u, float &s) {
    const uint32_t d[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (DT == LVLM_BF16) {
            const float lo = __uint_as_float(d[i] << 16), hi = __uint_as_float(d[i] & 0xffff0000u);
            s = fmaf(lo, lo, s);
            s = fmaf(hi, hi, s);
        } else {
            s = fmaf(__uint_as_float(d[i]), __uint_as_float(d[i]), s);
        }
    }
}

__device__ __attribute__((aligned(16))) const uint32_t kSimZero[4] = {0, 0, 0, 0};     // what lies beyond the end of a row

template <int DT, int TM, int TN, int NWN, int NWM, int RING, bool NORMS, bool RAGGED>
__global__ __launch_bounds__(64 * NWN * NWM) void sim_gemm_kernel(SimArgs a) {
    constexpr int NW = NWN * NWM, NT = 64 * NW;
    constexpr int TR = TM / NWN / 32, TC = TN / NWM / 32;
    constexpr int SB = 128;              // bytes of one slice of a row
    constexpr int UPS = SB / 16, RPL = 64 / UPS;     // 16-byte units of a row's slice, rows per direct load
    constexpr int SLOT = (TM + TN) * SB; // the dominant rows, then the others
    constexpr int DPW = (TM + TN) / RPL / NW;        // direct loads per wave and slice
    __shared__ __attribute__((aligned(1024))) char ring[RING * SLOT];
    __shared__ float invn[TM];
    __shared__ float bv[NWN][TN];
    __shared__ int bi[NWN][TN];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hf = lane >> 5, l32 = lane & 31;
    const int wn = wave % NWN, wm = wave / NWN;
    // tile of this workgroup
    const int NBt = (a.n_keep + TM - 1) / TM, MBt = (a.r + TN - 1) / TN;
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    int t = ((seq / a.run) * 8 + xcd) * a.run + seq % a.run;
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
    // Direct load x of this wave: rows 8 (wave DPW + x) .. + 7 of the slot, lane -> row lane / 8, place lane % 8.
    // Addresses are a uniform base (batch row, slice) plus a per-thread 32-bit byte offset (row, unit) that never
    // changes.  The offsets fit: the image rows of one batch row span less than 2 GiB (checked on the host).
    const char *img = p.src + (long long)b * p.src_stride_b + (long long)a.img_begin * p.row_bytes;
    auto place = [](int row) { return (row >> 1) & 7; };
    // (rows 8 (wave DPW + x) ..: the place depends on bit 3 of a row's number, so an even DPW leaves the wave out of it)
    auto unit_of = [&](int x) { return (lane % UPS) ^ place(RPL * (DPW % 2 ? wave + x : x) + lane / UPS); };
    unsigned off[DPW];
#pragma unroll
    for (int x = 0; x < DPW; ++x) {
        const int R = RPL * (wave * DPW + x) + lane / UPS;
        const int row = R < TM ? keep[min(nb * TM + R, a.n_keep - 1)] : rest[min(mb * TN + R - TM, a.r - 1)];
        off[x] = (unsigned)row * (unsigned)p.row_bytes + 16 * unit_of(x);
    }
    if constexpr (!NORMS)
        for (int i = tid; i < TM; i += NT) invn[i] = a.inv_norm[(long long)b * a.n + keep[min(nb * TM + i, a.n_keep - 1)]];
    const int nk = (p.row_bytes + SB - 1) / SB;      // the last slice may be partial: zero-filled
    const unsigned ring0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)ring + 1024 * DPW * wave;
    // direct loads [lo, hi) of slice k (the last slice again past the end) into slot k % RING
    auto fetch = [&](int k, int lo, int hi) {
        const char *base = img + SB * min(k, nk - 1);             // uniform
        const unsigned dst = ring0 + (unsigned)(k % RING) * SLOT;
#pragma unroll
        for (int x = 0; x < DPW; ++x) {
            if (x < lo || x >= hi) continue;
            if constexpr (RAGGED) {
                const bool in = p.row_bytes - SB * min(k, nk - 1) - 16 * unit_of(x) >= 16;
                const char *src = in ? base + off[x] : reinterpret_cast<const char *>(kSimZero);
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(dst + 1024 * x)
                             : "memory", "m0");
            } else {
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off[x]), "s"(base),
                             "s"(dst + 1024 * x)
                             : "memory", "m0");
            }
        }
    };

    f32x16 acc[TR][TC];
#pragma unroll
    for (int nd = 0; nd < TR; ++nd)
#pragma unroll
        for (int nr = 0; nr < TC; ++nr)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nd][nr][r] = 0.f;

#pragma unroll
    for (int k = 0; k < RING - 1; ++k) fetch(k, 0, DPW);
    // contraction step i of lane half hf takes unit NS hf + i of a row's slice
    constexpr int NS = UPS / 2;
    // NORMS: squares of the dominant rows, NU units of a slice to a thread, always of the same rows, and a sum for every slice of eight:
    // the sums that a wave with a row to itself would have in its 64 lanes (norm_rows), so that both ways give the same bits
    constexpr int NU = TM * UPS / NT, PH = NORMS ? 8 : 1;
    static_assert(NU >= 1 && NU <= NS && NU * NT == TM * UPS, "at most one unit per contraction step");
    float sq[PH][NU];
#pragma unroll
    for (int ph = 0; ph < PH; ++ph)
#pragma unroll
        for (int x = 0; x < NU; ++x) sq[ph][x] = 0.f;
    int uo[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) uo[i] = l32 * SB + 16 * ((NS * hf + i) ^ place(l32));
    const char *const ar = ring + wn * (TR * 32 * SB), *const br = ring + TM * SB + wm * (TC * 32 * SB);
    // One slice, k, its squares added to SQ.  All but the RING - 2 youngest slices' loads of this wave have landed at the wait: slice k is
    // complete when everybody is at the barrier, and this wave's reads of slice k - 1 are back, whose slot is written next.  The squares go
    // behind the products (rows = dominant, columns = others): those do not wait for the units, which arrive last.
    // (A macro: one loop for both, or a lambda, moves the scalar arithmetic of the addresses in front of a slice's first products -- without
    // norms, fp32 rows of 20 KB, 83.3 -> 86 us.)
#define LVLM_SIM_SLICE(SQ) \
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(DPW * (RING - 2)) : "memory");                       \
    if constexpr (RING == 2) fetch(k + RING - 1, 0, DPW);                                                                 \
    const int at = (k % RING) * SLOT;                                                                                     \
    uint4 fa[NS][TR], fb[NS][TC];                                                                                         \
    _Pragma("unroll")                                                                                                     \
    for (int i = 0; i < NS; ++i) {                                                                                        \
        _Pragma("unroll")                                                                                                 \
        for (int t2 = 0; t2 < TR; ++t2) fa[i][t2] = *reinterpret_cast<const uint4 *>(ar + at + uo[i] + t2 * 32 * SB);     \
        _Pragma("unroll")                                                                                                 \
        for (int t2 = 0; t2 < TC; ++t2) fb[i][t2] = *reinterpret_cast<const uint4 *>(br + at + uo[i] + t2 * 32 * SB);     \
    }                                                                                                                     \
    uint4 own[NU];                                                                                                        \
    if constexpr (NORMS) {                                                                                                \
        _Pragma("unroll")                                                                                                 \
        for (int x = 0; x < NU; ++x) own[x] = *reinterpret_cast<const uint4 *>(ring + at + 16 * (tid + NT * x));          \
    }                                                                                                                     \
    if constexpr (RING > 2) __builtin_amdgcn_sched_barrier(0);                                                            \
    _Pragma("unroll")                                                                                                     \
    for (int i = 0; i < NS; ++i) {                                                                                        \
        _Pragma("unroll")                                                                                                 \
        for (int nd = 0; nd < TR; ++nd)                                                                                   \
            _Pragma("unroll")                                                                                             \
            for (int nr = 0; nr < TC; ++nr) {                                                                             \
                if constexpr (DT == LVLM_BF16) {                                                                          \
                    mfma_one<DT>(acc[nd][nr], fa[i][nd], fb[i][nr], 0);                                                   \
                } else {                                                                                                  \
                    _Pragma("unroll")                                                                                     \
                    for (int cpt = 0; cpt < 4; ++cpt) mfma_one<DT>(acc[nd][nr], fa[i][nd], fb[i][nr], cpt);               \
                }                                                                                                         \
            }                                                                                                             \
        if constexpr (NORMS)                                                                                              \
            if (i >= NS - NU) squares<DT>(own[i - (NS - NU)], SQ[i - (NS - NU)]);                                         \
        if constexpr (RING > 2) {                                                                                         \
            __builtin_amdgcn_sched_barrier(0);                                                                            \
            fetch(k + RING - 1, DPW * i / NS, DPW * (i + 1) / NS);                                                        \
            __builtin_amdgcn_sched_barrier(0);                                                                            \
        }                                                                                                                 \
    }
    if constexpr (NORMS) {
        for (int k0 = 0; k0 < nk; k0 += PH) {
#pragma unroll
            for (int ph = 0; ph < PH; ++ph) {
                const int k = k0 + ph;
                if (k >= nk) break;
                LVLM_SIM_SLICE(sq[ph])
            }
        }
    } else {
        for (int k = 0; k < nk; ++k) {
            LVLM_SIM_SLICE(sq[0])
        }
    }
#undef LVLM_SIM_SLICE
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // no load may land after the workgroup has left its LDS
    if constexpr (NORMS) {
        // wave_sum's order: the eight units of a slice (they lie permuted by an exclusive or, which this tree does not see), then the slices
#pragma unroll
        for (int x = 0; x < NU; ++x) {
            float t[8];
#pragma unroll
            for (int ph = 0; ph < 8; ++ph) {
                t[ph] = sq[ph][x];
                t[ph] += dpp_quad1(t[ph]);
                t[ph] += dpp_quad2(t[ph]);
                t[ph] += dpp_half_mirror(t[ph]);
            }
            const float s = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
            if (tid % UPS == 0) invn[(tid + NT * x) / UPS] = s > 0.f ? 1.0f / sqrtf(s) : 1.0f;
        }
    }
    __syncthreads();

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

// One plane's row of dominant position i (token ji), 256 NU units a turn, thread t taking units t, t + 256, ... of it; the
// workgroups of a cluster (gridDim.z) take the turns of all planes in rotation, and this one lets `wait` of them pass.  `members` holds the
// cluster's first 64 other tokens, one per lane; up to four of their rows are in flight together.
template <int DT, int UB, int NU, bool SHARED>
__device__ __forceinline__ void merge_plane(const SimArgs &a, const PlaneDev &p, int b, int i, int ji, int lo, int n_mem,
                                            int members, int &wait) {
    using U = typename Unit<UB>::type;
    const int units = p.row_bytes / UB;
    const char *img0 = p.src + (long long)b * p.src_stride_b + (long long)a.img_begin * p.row_bytes;
    char *dst0 = p.dst + (long long)b * p.dst_stride_b + (long long)(a.img_begin + i) * p.row_bytes;
    const bool weighted = p.rule == LVLM_RULE_WEIGHTED && DT != LVLM_I32;
    const float *size = a.size_in ? a.size_in + (long long)b * a.n : nullptr;
    // whole waves in and out of the loop: lanes without a unit still hand out member indices
    for (int t0 = 0; t0 < units; t0 += 256 * NU) {
        if constexpr (SHARED) {
            if (wait > 0) {
                --wait;
                continue;
            }
            wait = gridDim.z - 1;
        }
        const int w0 = t0 + (threadIdx.x & ~63);
        if (w0 >= units) continue;
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
            if (size && a.size_out && threadIdx.x == 0 && u0 == 0) a.size_out[(long long)b * a.n_keep + i] = tot;   // (every such plane the same)
        }
    }
}

// Size of the cluster of token ji: its own and its members' sizes added in ascending index, the order of the weighted means
// (one wave, 64 members a round).
__device__ __forceinline__ float cluster_size(const SimArgs &a, int b, int ji, int lo, int n_mem, int members) {
    const float *size = a.size_in + (long long)b * a.n;
    const int lane = threadIdx.x & 63;
    float tot = size[ji];
    for (int s0 = 0; s0 < n_mem; s0 += 64) {
        const int mem = s0 ? a.order[(long long)b * a.n + min(lo + s0 + lane, a.n - 1)] : members;
        const float w = size[mem];
        const int cnt = min(64, n_mem - s0);
        for (int t = 0; t < cnt; ++t) tot += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), t));
    }
    return tot;
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

// (1792 tokens -> n_keep, eight planes of 4096 and seven times 1024 channels; all of a cluster in one workgroup -> shared: 1 cluster
// 2964 -> 430 us, 8 clusters 464 -> 103, 64 clusters 123 -> 65 us)
constexpr int kSimMergeWgs = 512;

// nothing removed: every row stays where it is
__global__ __launch_bounds__(256) void sim_copy_kernel(SimArgs a) { copy_row(a, blockIdx.y, blockIdx.x, blockIdx.x); }

// One workgroup per dominant position, every plane and column in it, or (SHARED) gridDim.z of them; workgroups past
// them copy the rows outside the image span.  The tokens assigned to position i form the
// segment [lo, lo + n) of the sorted order; its two ends are found by all waves at once, 64 probes of the owners a
// round (two rounds up to 4096 other tokens, three up to 262144) instead of one thread's bisection, whose chain of some
// 20 pairs of dependent loads per workgroup was the time of the kernel.  Bound by memory: 8 x 1263 clusters of 4096 bf16
// channels (213 MB) 72 -> 33 us.
template <bool SHARED>
__global__ __launch_bounds__(256) void sim_merge_kernel(SimArgs a) {
    const int i = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63;
    if (i >= a.n_keep) {
        if (SHARED && blockIdx.z) return;
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
    // sizes of all-ones clusters are written here (the weighted means write them when sizes are given)
    if (threadIdx.x == 0 && a.size_out && a.size_in == nullptr) a.size_out[(long long)b * a.n_keep + i] = (float)(1 + n_mem);
    if constexpr (SHARED) {
        // (a call whose planes are all only kept takes this form: in the other the code alone cost 2 % of the launch)
        if (a.sizes_apart && blockIdx.z == 0 && threadIdx.x < 64) {
            const float tot = cluster_size(a, b, ji, lo, n_mem, members);
            if (lane == 0) a.size_out[(long long)b * a.n_keep + i] = tot;
        }
    }
    int wait = blockIdx.z;
    for (int pi = 0; pi < a.n_planes; ++pi) {
        const PlaneDev &p = a.plane[pi];
        if (p.dtype == LVLM_BF16) {
            if (p.unit_bytes == 16) merge_plane<LVLM_BF16, 16, 2, SHARED>(a, p, b, i, ji, lo, n_mem, members, wait);
            else if (p.unit_bytes == 4) merge_plane<LVLM_BF16, 4, 1, SHARED>(a, p, b, i, ji, lo, n_mem, members, wait);
            else merge_plane<LVLM_BF16, 2, 1, SHARED>(a, p, b, i, ji, lo, n_mem, members, wait);
        } else if (p.dtype == LVLM_F32) {
            if (p.unit_bytes == 16) merge_plane<LVLM_F32, 16, 2, SHARED>(a, p, b, i, ji, lo, n_mem, members, wait);
            else merge_plane<LVLM_F32, 4, 1, SHARED>(a, p, b, i, ji, lo, n_mem, members, wait);
        } else {
            if (p.unit_bytes == 16) merge_plane<LVLM_I32, 16, 1, SHARED>(a, p, b, i, ji, lo, n_mem, members, wait);
            else merge_plane<LVLM_I32, 4, 1, SHARED>(a, p, b, i, ji, lo, n_mem, members, wait);
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
    w.rank2 = take(rank_search_form(d.n_img, d.B).parts > 1 ? n * 4 : 0);     // (the order by owner needs ranks only where searches add up in them)
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
    a.best = reinterpret_cast<unsigned long long *>(ws + w.best);
    a.assign = assign ? assign : reinterpret_cast<int32_t *>(ws + w.assign);
    a.order = reinterpret_cast<int32_t *>(ws + w.order);
    a.owner = reinterpret_cast<int32_t *>(ws + w.owner);
    a.B = d.B; a.N = d.N; a.img_begin = d.img_begin; a.n = d.n_img; a.n_keep = d.n_keep; a.r = r;
    a.n_planes = d.n_planes;
    a.sizes_apart = size_in && size_out;
    for (int i = 0; i < d.n_planes; ++i)
        if (a.plane[i].rule == LVLM_RULE_WEIGHTED && a.plane[i].dtype != LVLM_I32) a.sizes_apart = false;

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

    auto tiles_of = [&](int tm, int tn) { return (long long)d.B * ((d.n_keep + tm - 1) / tm) * ((r + tn - 1) / tn); };
    int tm = 128, tn = 128;
    if (tiles_of(64, 64) <= 288) tm = tn = 64;
    else if (tiles_of(128, 128) > 256) {
        if (tiles_of(128, 192) <= 256) tn = 192;
        else if (tiles_of(192, 128) <= 256) tm = 192;
    }
    const long long tiles = tiles_of(tm, tn);
    // Who takes the norms; either way gives the same bits.  In the product they cost every tile its dominant rows' squares again, and LDS
    // reads, which are what bounds a slice; beside the ranking, on workgroups of 16 rows, they cost the launch a pass over all rows,
    // little of it while the launch is one turn of the chip: two workgroups fit a compute unit, but share its loads.  Beside the
    // ranking -> in the product, whole calls, us (bf16 unless said; 130 shapes of 150 to 1400 such workgroups timed both ways):
    //   64 x 64 tiles: in it when the launch would have more than 256 workgroups (16 x 256 rows of 12 KB 62.8 -> 57.9, 9 x 460 64.5 -> 59.8,
    //       20 x 400 of 10 KB 71.6 -> 62.3, 13 x 400 of 1 KB in fp32 34.7 -> 32.9; with fewer 4 x 576 of 12 KB 51.9 -> 53.5, 3 x 800 of
    //       7 KB 38.4 -> 40.1; even from 216 to 256)
    //   128 x 128, a ring of four: when it would have more than 512 (7 x 1733 of 7 KB 93.4 -> 89.0, 6 x 1100 of 12 KB 92.4 -> 87.0; with
    //       fewer 1 x 2600 of 12 KB 76.1 -> 84.5, 1 x 4000 96.9 -> 99.3; from 370 to 512 within 4 % either way)
    //   128 x 192: always (8 x 1792 of 8 KB 123.2 -> 118.5, 1 x 4500 of 12 KB 113.7 -> 109.7); 192 x 128: never (their squares' sums and
    //       the products' do not fit the registers: 1 x 10560 of 12 KB 171 -> 187), nor a ring of two, whose workgroups would no longer
    //       share a compute unit (9 x 2034 of 10 KB 188 -> 249)
    const long long beside_wgs = (long long)d.B * ((d.n_img + 63) / 64 + (d.n_img + 15) / 16);
    const bool beside = tm == 64 ? beside_wgs <= 256 : tn == 192 ? false : tm == 192 || tiles > 256 || beside_wgs <= 512;
    NormJob norm{};
    if (beside) {
        a.inv_norm = reinterpret_cast<float *>(ws + w.inv_norm);
        norm.src = a.plane[0].src + (long long)d.img_begin * a.plane[0].row_bytes;
        norm.stride_b = a.plane[0].src_stride_b;
        norm.inv_norm = a.inv_norm;
        norm.row_bytes = a.plane[0].row_bytes; norm.dtype = planes[0].dtype; norm.n = d.n_img;
    }
    prof.begin("sim_rank");
    launch_rank(prof, score_mean, a.rank, d.n_img, d.B, ws + w.sorted, beside ? &norm : nullptr);
    prof.end();
    prof.begin("sim_index");
    LVLM_LAUNCH(prof, sim_index_kernel, dim3((d.n_img + kSimChunk - 1) / kSimChunk, d.B), dim3(1024), 0, stream, a);
    prof.end();
    prof.begin("sim_gemm");
    {
        const long long per_xcd = (tiles + 7) / 8;
        a.run = (int)(per_xcd <= 64 ? per_xcd : kSimGN * kSimGM);
        const dim3 ggrid((unsigned)(((tiles + a.run - 1) / a.run + 7) / 8 * 8 * a.run));
        const bool bf = planes[0].dtype == LVLM_BF16;
        const bool ragged = (planes[0].row_elems * (bf ? 2 : 4)) % 128 != 0;
#define LVLM_GEMM_OF(DT, RAGGED, NORMS, TM, TN, NWN, NWM, RING) \
    LVLM_LAUNCH(prof, (sim_gemm_kernel<DT, TM, TN, NWN, NWM, RING, NORMS, RAGGED>), ggrid, dim3(64 * NWN * NWM), 0, stream, a)
#define LVLM_GEMM(...)                                                                                                      \
    if (bf && ragged) LVLM_GEMM_OF(LVLM_BF16, true, __VA_ARGS__);                                                          \
    else if (bf) LVLM_GEMM_OF(LVLM_BF16, false, __VA_ARGS__);                                                              \
    else if (ragged) LVLM_GEMM_OF(LVLM_F32, true, __VA_ARGS__);                                                            \
    else LVLM_GEMM_OF(LVLM_F32, false, __VA_ARGS__)
        if (tm == 64 && beside) { LVLM_GEMM(false, 64, 64, 2, 2, 4); }
        else if (tm == 64) { LVLM_GEMM(true, 64, 64, 2, 2, 4); }
        else if (tn == 192) { LVLM_GEMM(true, 128, 192, 4, 2, 3); }
        else if (tm == 192) { LVLM_GEMM(false, 192, 128, 2, 4, 3); }
        else if (tiles <= 256 && beside) { LVLM_GEMM(false, 128, 128, 2, 4, 4); }
        else if (tiles <= 256) { LVLM_GEMM(true, 128, 128, 2, 4, 4); }
        else { LVLM_GEMM(false, 128, 128, 2, 2, 2); }
#undef LVLM_GEMM_OF
#undef LVLM_GEMM
    }
    prof.end();
    OwnerJob oj{};
    oj.dom_of = a.dom_of; oj.best = a.best; oj.order = a.order; oj.owner = a.owner; oj.assign = a.assign; oj.r = r;
    prof.begin("sim_order");
    launch_owner_order(prof, oj, reinterpret_cast<int32_t *>(ws + w.rank2), d.n_img, d.B, ws + w.sorted);
    prof.end();
    prof.begin("sim_merge");
    // Few clusters are large ones, and a workgroup's time is its chain of members, once per turn (plane, 512 units of it): the turns
    // go to workgroups of their own until kSimMergeWgs of them walk a chain.
    long long turns = 0;
    for (int i = 0; i < d.n_planes; ++i) {
        const PlaneDev &p = a.plane[i];
        const int units = p.row_bytes / p.unit_bytes, per_turn = 256 * (p.unit_bytes == 16 && p.dtype != LVLM_I32 ? 2 : 1);
        turns += (units + per_turn - 1) / per_turn;
    }
    const long long clusters = (long long)d.n_keep * d.B;
    long long share = kSimMergeWgs / clusters;
    share = share < 1 ? 1 : (share > turns ? turns : share);
    const dim3 mgrid(d.n_keep + d.N - d.n_img, d.B, (unsigned)share);
    if (share > 1 || a.sizes_apart) LVLM_LAUNCH(prof, sim_merge_kernel<true>, mgrid, dim3(256), 0, stream, a);
    else LVLM_LAUNCH(prof, sim_merge_kernel<false>, mgrid, dim3(256), 0, stream, a);
    prof.end();
    return hipGetLastError();
}

}  // namespace lvlm
