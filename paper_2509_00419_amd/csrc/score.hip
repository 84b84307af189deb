// Step 1 -- token importance = attention received (Sec. 3.2.1).
//
// For one (batch, KV head) the G*T query rows of the head group meet a block
// of keys as a dense tile product on the matrix cores.  The softmax needs
// each row's normaliser over ALL visible keys before a column sum can be
// taken, so the work is two passes over the same tiling:
//   pass 0  keys x queries tiles  -> per-row (max, sum-exp) of every key block,
//           then a small kernel folds the blocks into log2-domain LSE per row;
//   pass 1  queries x keys tiles over the image span only ->
//           p = exp2(logit - lse), summed down the rows of the tile.
// When the caller already has the row LSE (an attention kernel produces it),
// pass 0 is skipped.  The N x N probability matrix is never stored.
//
// Tiling (wave64, MFMA 32x32): a workgroup of 4 waves owns 4*KPW*32 keys; each
// wave keeps its KPW 32-key operand tiles in registers for the whole kernel and
// streams 32-row query chunks through LDS (double buffered, one barrier per
// chunk).  The reduction index of the MFMA is a dummy index, so step i of lane
// half lane/32 simply takes bytes [32 i + 16 (lane/32), +16) of a head vector --
// global and LDS reads are then plain 16-byte vectors.
#include <limits.h>

#include "common.h"
#include "mma.h"

#include <algorithm>
#include <type_traits>

namespace lvlm {
namespace {


struct ScoreArgs {
    const char *q;
    const char *k;
    const float *row_lse;
    float *part_m;      // [nkb * 4][rows]   per key block and wave: row max (log2 domain)
    float *part_l;      // [nkb * 4][rows]   ... and sum of exp2(logit - max)
    float *lse2;        // [rows]
    float *colpart;     // [RS][B][Hkv][n_img]  column sums of each row split
    float *score_head;
    float *score_mean;
    int B, N, T, q_pos0, Hq, Hkv, G, img_begin, n_img, causal, nkb;
    int rs;             // row splits: workgroups that share a key block and take different query chunks
    int cps;            // chunks per split
    int n_seg;          // shared-tile form: runs the keys are cut into (1 = both sweeps in one launch)
    KeyRuns runs1, runs2;   // equal shares: how the keys of the two sweeps are dealt out
    unsigned t_magic;   // floor(2^32 / T) + 1: rho / T == umulhi(rho, t_magic) for rho, T < 65536
    float scale_log2;
    long long qsb, qst, qsh, ksb, ksn, ksh, shb, shh;
};


template <int DT, int HD, int KPW, int PASS>
__global__ __launch_bounds__(256, 3) void score_pass_kernel(ScoreArgs a) {
    constexpr int ES = esize<DT>();
    constexpr int ROWB = HD * ES;
    constexpr int PITCH = ROWB + 16;        // odd multiple of 16 B: conflict-free 128-bit LDS reads
    constexpr int UPR = ROWB / 16;          // 16-byte units per row
    constexpr int UPT = 32 * UPR / 256;     // units each thread stages per chunk
    constexpr int BN = 4 * KPW * 32;
    constexpr int NV = HalfRow<DT, HD>::NV;
    constexpr int NBUF = 3;
    static_assert(UPT >= 1 && UPT <= 4, "staging covers 1..4 units per thread");

    __shared__ __attribute__((aligned(16))) char q_lds[NBUF][32 * PITCH];
    __shared__ __attribute__((aligned(16))) int pos_lds[NBUF][32];
    __shared__ __attribute__((aligned(16))) float lse_lds[NBUF][32];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hf = lane >> 5, l32 = lane & 31;
    // Workgroups are handed to the 8 XCDs round-robin by linear id, and grid.x is a multiple of 8, so
    // blockIdx.x % 8 names the XCD (and its private L2).  The row splits of one key block are placed on
    // the same XCD: they read the same keys.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    // The normaliser pass takes its key blocks from the last one down: the blocks at the end of the sequence are the
    // ones that need the mask (the slow path), and a slow workgroup started last would run on after all the others.
    const int kslot = PASS == 0 ? (int)(gridDim.x / (8 * a.rs)) - 1 - slot / a.rs : slot / a.rs;
    const int kb = kslot * 8 + xcd, rs = slot % a.rs;
    const int g = blockIdx.y, b = blockIdx.z;
    if (kb * BN >= (PASS == 0 ? a.N : a.n_img)) return;      // padding of the key-block count to a multiple of 8
    const int GT = a.G * a.T;
    const int n_chunks = (GT + 31) >> 5;
    const int c_lo = rs * a.cps, c_hi = min(n_chunks, c_lo + a.cps);
    const int key_lo = PASS == 0 ? 0 : a.img_begin;
    const int key_hi = PASS == 0 ? a.N : a.img_begin + a.n_img;
    const int jbase = key_lo + kb * BN + wave * (KPW * 32);
    const long long rowbase = ((long long)b * a.Hq + (long long)g * a.G) * a.T;   // row index of chunk row rho: rowbase + rho
    const long long rows_total = (long long)a.B * a.Hq * a.T;

    // rho / T without a hardware divide (exact for rho, T < 65536; T == 1 has no 32-bit magic number)
    auto div_t = [&](int rho) -> int { return a.T == 1 ? rho : (int)__umulhi((unsigned)rho, a.t_magic); };

    // this wave's key tiles, resident for the whole kernel
    HalfRow<DT, HD> kf[KPW];
#pragma unroll
    for (int s = 0; s < KPW; ++s) {
        // Contraction step i of lane half hf takes bytes [32 i + 16 hf, +16) of a row (both operands).  The
        // load puts a lane PAIR on 32 contiguous bytes of one row -- the memory pipeline serves one request
        // per lane when every lane of a quad reads another row -- and a lane permute then moves each piece
        // to the lane (row l32, half hf) the MFMA wants it in.
        const int j = jbase + 32 * s + (lane >> 1);
        uint4 raw[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) raw[i] = make_uint4(0, 0, 0, 0);
        if (j < key_hi) {
            const char *src = a.k + ((long long)b * a.ksb + (long long)j * a.ksn + (long long)g * a.ksh) * ES +
                              16 * (lane & 1);
#pragma unroll
            for (int i = 0; i < NV; ++i) raw[i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
        }
        const int from = 4 * (2 * l32 + hf);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            kf[s].v[i].x = __builtin_amdgcn_ds_bpermute(from, raw[i].x);
            kf[s].v[i].y = __builtin_amdgcn_ds_bpermute(from, raw[i].y);
            kf[s].v[i].z = __builtin_amdgcn_ds_bpermute(from, raw[i].z);
            kf[s].v[i].w = __builtin_amdgcn_ds_bpermute(from, raw[i].w);
        }
    }

    // Two chunks of 32 query rows are on their way from global memory to LDS at any time (stages A and
    // B).  Named scalars, not arrays or structs: the values are carried around the chunk loop and must
    // stay in registers.
    uint4 stA0 = make_uint4(0, 0, 0, 0), stA1 = stA0, stA2 = stA0, stA3 = stA0;
    uint4 stB0 = stA0, stB1 = stA0, stB2 = stA0, stB3 = stA0;
    int stA_pos = -1, stB_pos = -1;
    float stA_lse = 0.f, stB_lse = 0.f;
    // A thread stages UPT 16-byte units of ONE row of every chunk.  Its source address is
    // carried from load to load (a stage takes every second chunk: 64 rows further down, stepping over to
    // the next head when the rows of one are used up), so the chunk loop holds no address multiplies.
    constexpr int TPR = UPR / UPT;       // threads per row: neighbouring lanes read neighbouring 16-byte units
    const int srow = tid / TPR, scu = tid % TPR;       // units scu + TPR x, x < UPT
    const long long q_step = 64 * a.qst * ES;                            // 64 rows further in the same head
    const long long q_wrap = (a.qsh - (long long)a.T * a.qst) * ES;      // from row T of a head to row 0 of the next
    const char *q_grp0 = a.q + ((long long)b * a.qsb + (long long)g * a.G * a.qsh) * ES;    // uniform
    const char *q_grp = q_grp0 + 16 * scu;
    // padding rows (beyond the last row of the group, in its last chunk only) repeat the last row; they are
    // masked in compute.  Its address is formed where it is used, from uniform values: a register pair
    // held around the loop would push a staging register out to scratch memory.
    const char *q_last0 = q_grp0 + ((long long)(a.G - 1) * a.qsh + (long long)(a.T - 1) * a.qst) * ES;
    auto chunk_row = [&](int c, const char *ptr) -> const uint4 * {
        if (c == n_chunks - 1) {
            int off = 16 * scu;
            asm volatile("" : "+v"(off));            // keeps the sum below inside this branch
            if (c * 32 + srow >= GT) ptr = q_last0 + off;
        }
        return reinterpret_cast<const uint4 *>(ptr);
    };
    auto row_ptr = [&](int c, int &i) -> const char * {
        const int rho = c * 32 + srow;
        const int hl = div_t(rho);
        i = rho - hl * a.T;
        return q_grp + ((long long)hl * a.qsh + (long long)i * a.qst) * ES;
    };
    int iA = 0, iB = 0;
    const char *pA = row_ptr(c_lo, iA), *pB = row_ptr(c_lo + 1, iB);
    auto advance = [&](const char *&ptr, int &i) {
        i += 64;
        ptr += q_step;
        if (a.T >= 64) {
            const bool over = i >= a.T;
            i -= over ? a.T : 0;
            ptr += over ? q_wrap : 0;
        } else {
            while (i >= a.T) {
                i -= a.T;
                ptr += q_wrap;
            }
        }
    };
    auto chunk_dst = [&](int buf, int x) -> uint4 * {
        return reinterpret_cast<uint4 *>(&q_lds[buf][srow * PITCH + 16 * (scu + TPR * x)]);
    };
    auto row_meta = [&](int c, int &pos, float &lse) {
        pos = -1;             // padding row: sees no key
        lse = 0.f;
        if (tid < 32) {
            const int rho = c * 32 + tid;
            if (rho < GT) {
                pos = a.causal ? a.q_pos0 + (rho - div_t(rho) * a.T) : INT_MAX;
                // (as loaded: the change of base waits for store time -- a use right here would stall the wave on the
                // load, with the chunk's own loads just issued in front of it)
                if (PASS == 1) lse = a.row_lse ? a.row_lse[rowbase + rho] : a.lse2[rowbase + rho];
            }
        }
    };
#define LVLM_STAGE_FUNCS(S)                                              \
    auto load_##S = [&](int kk) {           /* chunk c_lo + kk; nothing to fetch past the last chunk */ \
        const int c = c_lo + kk;                                         \
        if (c < c_hi) {                                                  \
            const uint4 *src = chunk_row(c, p##S);                      \
            st##S##0 = src[0];                                           \
            if constexpr (UPT > 1) st##S##1 = src[TPR];                  \
            if constexpr (UPT > 2) st##S##2 = src[2 * TPR];              \
            if constexpr (UPT > 3) st##S##3 = src[3 * TPR];              \
            row_meta(c, st##S##_pos, st##S##_lse);                       \
        }                                                                \
        advance(p##S, i##S);                                             \
    };                                                                   \
    auto store_##S = [&](int buf) {                                      \
        *chunk_dst(buf, 0) = st##S##0;                                   \
        if constexpr (UPT > 1) *chunk_dst(buf, 1) = st##S##1;            \
        if constexpr (UPT > 2) *chunk_dst(buf, 2) = st##S##2;            \
        if constexpr (UPT > 3) *chunk_dst(buf, 3) = st##S##3;            \
        if (tid < 32) {                                                  \
            pos_lds[buf][tid] = st##S##_pos;                             \
            lse_lds[buf][tid] = a.row_lse ? st##S##_lse * kLog2e : st##S##_lse;   /* a caller's are natural logarithms */ \
        }                                                                \
    };
    LVLM_STAGE_FUNCS(A)
    LVLM_STAGE_FUNCS(B)
#undef LVLM_STAGE_FUNCS

    float colsum[KPW];
#pragma unroll
    for (int s = 0; s < KPW; ++s) colsum[s] = 0.f;

    auto compute = [&](int c, int buf) {
        // Positions of the chunk's rows (uniform): a chunk inside one head covers rows i0 .. i0 + 31 of it, one
        // that straddles two heads anything from 0 to T - 1.
        const int rho0 = c * 32, rho1 = min(rho0 + 31, GT - 1);
        const int h0 = div_t(rho0), h1 = div_t(rho1);
        const int min_i = (h0 != h1) ? 0 : rho0 - h0 * a.T;
        const int max_i = (h0 != h1) ? a.T - 1 : rho1 - h1 * a.T;
        // Every key of this wave lies ahead of every row of the chunk (query rows inside the key range, as when
        // all rows of the sequence are scored): nothing to multiply.
        if (a.causal && jbase > a.q_pos0 + max_i) {
            if (PASS == 0) {
                const int rho = rho0 + l32;
                if (hf == 0 && rho < GT) {
                    const long long pidx = ((long long)kb * 4 + wave) * rows_total + rowbase + rho;
                    a.part_m[pidx] = -INFINITY;
                    a.part_l[pidx] = 0.f;
                }
            }
            return;
        }
        HalfRow<DT, HD> qa;
        {
            const char *src = &q_lds[buf][l32 * PITCH + 16 * hf];
#pragma unroll
            for (int i = 0; i < NV; ++i) qa.v[i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
        }
        f32x16 acc[KPW];
#pragma unroll
        for (int s = 0; s < KPW; ++s) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[s][r] = 0.f;
            if (PASS == 0)
                mma_tile<DT, HD>(acc[s], kf[s], qa);   // rows = keys, cols = queries
            else
                mma_tile<DT, HD>(acc[s], qa, kf[s]);   // rows = queries, cols = keys
        }
        // Is any element of this 32 x (KPW*32) block masked?  Uniform over the workgroup's wave:
        // keys beyond the range, padding rows, or a key ahead of the earliest query position of the chunk.
        const bool masked = jbase + KPW * 32 > key_hi || rho0 + 32 > GT ||
                            (a.causal && jbase + KPW * 32 - 1 > a.q_pos0 + min_i);

        if (PASS == 0) {
            // this lane: query l32 of the chunk, 16 keys per tile
            float m = -INFINITY, l = 0.f;
            if (!masked) {
#pragma unroll
                for (int s = 0; s < KPW; ++s)
#pragma unroll
                    for (int r = 0; r < 16; ++r) m = fmaxf(m, acc[s][r]);
                m = fmaxf(m, other_half(m)) * a.scale_log2;      // scale >= 0 (checked on the host)
#pragma unroll
                for (int s = 0; s < KPW; ++s)
#pragma unroll
                    for (int r = 0; r < 16; ++r) l += __builtin_amdgcn_exp2f(fmaf(acc[s][r], a.scale_log2, -m));
            } else {
                const int pos = pos_lds[buf][l32];
#pragma unroll
                for (int s = 0; s < KPW; ++s) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int j = jbase + 32 * s + acc_row(r, hf);
                        const float t = (j <= pos && j < key_hi) ? acc[s][r] * a.scale_log2 : -INFINITY;
                        acc[s][r] = t;
                        m = fmaxf(m, t);
                    }
                }
                m = fmaxf(m, other_half(m));
                const float ms = (m == -INFINITY) ? 0.f : m;
#pragma unroll
                for (int s = 0; s < KPW; ++s)
#pragma unroll
                    for (int r = 0; r < 16; ++r) l += __builtin_amdgcn_exp2f(acc[s][r] - ms);   // exp2(-inf) = 0
            }
            l += other_half(l);
            const int rho = rho0 + l32;
            if (hf == 0 && rho < GT) {
                const long long pidx = ((long long)kb * 4 + wave) * rows_total + rowbase + rho;
                a.part_m[pidx] = m;
                a.part_l[pidx] = l;
            }
        } else {
            // this lane: key l32 of each tile, 16 query rows of the chunk
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const float4 lse4 = *reinterpret_cast<const float4 *>(&lse_lds[buf][8 * qd + 4 * hf]);
                const float lse[4] = {lse4.x, lse4.y, lse4.z, lse4.w};
                if (!masked) {
#pragma unroll
                    for (int s = 0; s < KPW; ++s)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            colsum[s] += __builtin_amdgcn_exp2f(fmaf(acc[s][4 * qd + e], a.scale_log2, -lse[e]));
                } else {
                    const int4 pos4 = *reinterpret_cast<const int4 *>(&pos_lds[buf][8 * qd + 4 * hf]);
                    const int pos[4] = {pos4.x, pos4.y, pos4.z, pos4.w};
#pragma unroll
                    for (int s = 0; s < KPW; ++s) {
                        const int j = jbase + 32 * s + l32;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float p = __builtin_amdgcn_exp2f(fmaf(acc[s][4 * qd + e], a.scale_log2, -lse[e]));
                            colsum[s] += (j <= pos[e]) ? p : 0.f;
                        }
                    }
                }
            }
        }
    };

    // Pipeline over the chunks k = 0 .. nc-1 of this workgroup: chunk k is loaded from global memory into
    // a register stage two iterations before it is computed (even chunks in A, odd ones in B), copied
    // into one of three LDS buffers one iteration before, and one barrier per chunk publishes the copy.
    // Past the last chunk nothing is loaded; the copies then repeat stale registers that nothing reads.
    const int nc = c_hi - c_lo;
    load_A(0);
    store_A(0);
    load_B(1);
    load_A(2);
    __syncthreads();
    for (int k = 0; k < nc; k += 2) {
        store_B((k + 1) % NBUF);          // chunk k+1
        load_B(k + 3);
        compute(c_lo + k, k % NBUF);
        __syncthreads();
        if (k + 1 >= nc) break;
        store_A((k + 2) % NBUF);          // chunk k+2
        load_A(k + 4);
        compute(c_lo + k + 1, (k + 1) % NBUF);
        __syncthreads();
    }

    if (PASS == 1) {
#pragma unroll
        for (int s = 0; s < KPW; ++s) {
            const float tot = colsum[s] + other_half(colsum[s]);
            const int j = jbase + 32 * s + l32;
            if (hf == 0 && j < key_hi)
                a.colpart[(((long long)rs * a.B + b) * a.Hkv + g) * a.n_img + (j - a.img_begin)] = tot;
        }
    }
}

// ---- short sequences: both passes in one launch ---------------------------------------------------------
// A workgroup owns ONE chunk of 32 query rows (held in registers as an MFMA operand by all four waves) and
// sweeps over all keys twice: first for the row normalisers (online max / sum per row, folded over the
// waves through LDS), then again over the image keys for the column sums.  Nothing but the final column
// sums of the chunk leaves the workgroup, so the normaliser partials, their fold kernel and the second
// launch disappear; the price is that every chunk streams the keys from L2 itself, which only pays while
// the sequence is short (the launch decides by the bytes that re-streaming costs).  Wave w of NW takes the key
// tiles 32 (w + NW k) .. +32; a tile's rows go straight from global memory into operand registers, the next
// tile's loads are in flight while the current one is used (two named register sets).
#define LVLM_K16(M) M(0) M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15)

template <int DT, int HD, int NW>
__global__ __launch_bounds__(64 * NW, (DT == LVLM_F32 && HD == 128) ? 2 : 3) void score_small_kernel(ScoreArgs a) {
    constexpr int ES = esize<DT>();
    constexpr int NV = HalfRow<DT, HD>::NV;
    constexpr int SW = 32 * NW;             // keys all waves take per sweep step
    static_assert(NV <= 16, "operand registers are written out for up to 16 words");
    __shared__ float wm[NW][32], wl[NW][32];
    __shared__ float lse_s[32];
    __shared__ int pos_s[32];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hf = lane >> 5, l32 = lane & 31;
    // Workgroups reach the 8 XCDs round-robin by id: all chunks of one (batch, KV head) pair are given ids
    // with the same remainder, so that the pair's keys are fetched into one L2 only
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    const int pair = (seq / a.rs) * 8 + xcd, c = seq % a.rs;
    if (pair >= a.B * a.Hkv) return;
    const int b = pair / a.Hkv, g = pair % a.Hkv;
    const int GT = a.G * a.T;
    const long long rowbase = ((long long)b * a.Hq + (long long)g * a.G) * a.T;
    auto div_t = [&](int rho) -> int { return a.T == 1 ? rho : (int)__umulhi((unsigned)rho, a.t_magic); };

    // this lane's query row (padding rows repeat the last row and get an infinite LSE)
    const int rho = c * 32 + l32;
    const int rc = min(rho, GT - 1);
    const int hl = div_t(rc), qi = rc - hl * a.T;
    const int pos = a.causal ? a.q_pos0 + qi : INT_MAX;
    HalfRow<DT, HD> qa;
    {
        // contraction step i of lane half hf takes bytes [32 i + 16 hf, +16) of the row (the contraction index
        // is a dummy index: any split works as long as both operands use it): the two halves of one load
        // instruction then read 32 contiguous bytes of a row, half as many cache lines as with a half row each
        const char *src = a.q + ((long long)b * a.qsb + (long long)qi * a.qst + (long long)(g * a.G + hl) * a.qsh) * ES +
                          16 * hf;
#pragma unroll
        for (int i = 0; i < NV; ++i) qa.v[i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
    }
    if (tid < 32) pos_s[tid] = pos;

    // loads: lane pair (2 r, 2 r + 1) reads 32 contiguous bytes of row r (half as many memory requests as one
    // row per lane); LVLM_PACK moves each piece to the lane (row l32, half hf) the MFMA wants it in
    const char *kbase = a.k + ((long long)b * a.ksb + (long long)g * a.ksh) * ES + 16 * (lane & 1);
    const int k_src = 4 * (2 * l32 + hf);
#define LVLM_DECL(x) uint4 kA##x = make_uint4(0, 0, 0, 0), kB##x = make_uint4(0, 0, 0, 0), kC##x = make_uint4(0, 0, 0, 0);
    LVLM_K16(LVLM_DECL)
#undef LVLM_DECL
#define LVLM_LD(S, x) if (x < NV) S##x = *reinterpret_cast<const uint4 *>(kp_ + 32 * x);
#define LVLM_LOADK(S, j0, jmax)                                                              \
    {                                                                                        \
        const char *kp_ = kbase + (long long)min((j0) + (lane >> 1), (jmax) - 1) * a.ksn * ES; \
        LVLM_LD(S, 0) LVLM_LD(S, 1) LVLM_LD(S, 2) LVLM_LD(S, 3) LVLM_LD(S, 4) LVLM_LD(S, 5) LVLM_LD(S, 6) LVLM_LD(S, 7) \
        LVLM_LD(S, 8) LVLM_LD(S, 9) LVLM_LD(S, 10) LVLM_LD(S, 11) LVLM_LD(S, 12) LVLM_LD(S, 13) LVLM_LD(S, 14) LVLM_LD(S, 15) \
    }
#define LVLM_PACK(S, kf)                                                                     \
    {                                                                                        \
        const uint4 w_[16] = {S##0, S##1, S##2, S##3, S##4, S##5, S##6, S##7, S##8, S##9, S##10, S##11, S##12, S##13, S##14, S##15}; \
        _Pragma("unroll") for (int i = 0; i < NV; ++i) {                                     \
            kf.v[i].x = __builtin_amdgcn_ds_bpermute(k_src, w_[i].x);                         \
            kf.v[i].y = __builtin_amdgcn_ds_bpermute(k_src, w_[i].y);                         \
            kf.v[i].z = __builtin_amdgcn_ds_bpermute(k_src, w_[i].z);                         \
            kf.v[i].w = __builtin_amdgcn_ds_bpermute(k_src, w_[i].w);                         \
        }                                                                                    \
    }

    // the first tile of the second sweep is fetched now: its latency hides behind the first sweep (where
    // the operand registers allow a third set)
    constexpr bool kEarly = NV <= 8;
    const int key_lo = a.img_begin, key_hi = a.img_begin + a.n_img;
    const int j2_first = key_lo + 32 * wave;
    if (kEarly && j2_first < key_hi) LVLM_LOADK(kC, j2_first, key_hi)

    // A tile whose keys all lie in range and at or before the earliest query position of the chunk needs no
    // per-element mask (uniform test): that is every image key for instruction rows.
    const int rho_last = min(c * 32 + 31, GT - 1);
    const int hc0 = div_t(c * 32), hc1 = div_t(rho_last);
    const int pos_min = a.causal ? a.q_pos0 + ((hc0 != hc1) ? 0 : c * 32 - hc0 * a.T) : INT_MAX;

    // ---- sweep 1: row normalisers over all keys (rows = keys, columns = queries: the row's statistics are
    // lane-local over 16 registers)
    if (a.row_lse == nullptr) {
        float m = -INFINITY, l = 0.f;
        auto stats = [&](int j0, const HalfRow<DT, HD> &kf) {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            mma_tile<DT, HD>(acc, kf, qa);
            if (j0 + 32 <= a.N && j0 + 31 <= pos_min) {
                float tmax = acc[0];
#pragma unroll
                for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, acc[r]);
                const float mn = fmaxf(m, tmax * a.scale_log2);      // finite; scale >= 0 (checked on the host)
                float sum = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(fmaf(acc[r], a.scale_log2, -mn));
                l = l * __builtin_amdgcn_exp2f(m - mn) + sum;
                m = mn;
                return;
            }
            float t[16];
            float tmax = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = j0 + acc_row(r, hf);
                t[r] = (j <= pos && j < a.N) ? acc[r] * a.scale_log2 : -INFINITY;
                tmax = fmaxf(tmax, t[r]);
            }
            const float mn = fmaxf(m, tmax);
            const float ms = (mn == -INFINITY) ? 0.f : mn;
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(t[r] - ms);   // exp2(-inf) = 0
            l = l * __builtin_amdgcn_exp2f(m - ms) + sum;
            m = mn;
        };
        const int j_first = 32 * wave;
        if (j_first < a.N) LVLM_LOADK(kA, j_first, a.N)
        for (int j0 = j_first; j0 < a.N; j0 += 2 * SW) {
            HalfRow<DT, HD> kf;
            if (j0 + SW < a.N) LVLM_LOADK(kB, j0 + SW, a.N)
            LVLM_PACK(kA, kf)
            stats(j0, kf);
            if (j0 + SW >= a.N) break;
            if (j0 + 2 * SW < a.N) LVLM_LOADK(kA, j0 + 2 * SW, a.N)
            LVLM_PACK(kB, kf)
            stats(j0 + SW, kf);
        }
        // the two lane halves, then the four waves
        {
            const float mo = other_half(m), lo = other_half(l);
            const float mn = fmaxf(m, mo);
            const float ms = (mn == -INFINITY) ? 0.f : mn;
            l = l * __builtin_amdgcn_exp2f(m - ms) + lo * __builtin_amdgcn_exp2f(mo - ms);
            m = mn;
        }
        if (hf == 0) {
            wm[wave][l32] = m;
            wl[wave][l32] = l;
        }
        __syncthreads();
        if (tid < 32) {
            float mx = -INFINITY;
#pragma unroll
            for (int w = 0; w < NW; ++w) mx = fmaxf(mx, wm[w][tid]);
            const float ms = (mx == -INFINITY) ? 0.f : mx;
            float tot = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) tot += wl[w][tid] * exp2f(wm[w][tid] - ms);
            // no visible key, or a padding row: contributes nothing
            lse_s[tid] = (tot > 0.f && rho < GT) ? mx + log2f(tot) : INFINITY;
        }
    } else if (tid < 32) {
        lse_s[tid] = rho < GT ? a.row_lse[rowbase + rho] * kLog2e : INFINITY;
    }
    __syncthreads();

    // ---- sweep 2: column sums over the image keys (rows = queries, columns = keys: a key's sum is lane-local)
    float *out = a.colpart + (((long long)c * a.B + b) * a.Hkv + g) * a.n_img;
    auto colsum = [&](int j0, const HalfRow<DT, HD> &kf) {
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        mma_tile<DT, HD>(acc, qa, kf);
        const int j = j0 + l32;
        float sum = 0.f;
        if (j0 + 31 <= pos_min) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                sum += __builtin_amdgcn_exp2f(fmaf(acc[r], a.scale_log2, -lse_s[acc_row(r, hf)]));
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = acc_row(r, hf);
                const float p = __builtin_amdgcn_exp2f(fmaf(acc[r], a.scale_log2, -lse_s[row]));
                sum += (j <= pos_s[row]) ? p : 0.f;
            }
        }
        sum += other_half(sum);
        if (hf == 0 && j < key_hi) out[j - key_lo] = sum;
    };
    if (j2_first < key_hi) {
        HalfRow<DT, HD> kf;
        if (!kEarly) LVLM_LOADK(kC, j2_first, key_hi)
        if (j2_first + SW < key_hi) LVLM_LOADK(kB, j2_first + SW, key_hi)
        LVLM_PACK(kC, kf)
        colsum(j2_first, kf);
        for (int j0 = j2_first + SW; j0 < key_hi; j0 += 2 * SW) {      // tile j0 is in set B
            if (j0 + SW < key_hi) LVLM_LOADK(kA, j0 + SW, key_hi)
            LVLM_PACK(kB, kf)
            colsum(j0, kf);
            if (j0 + SW >= key_hi) break;
            if (j0 + 2 * SW < key_hi) LVLM_LOADK(kB, j0 + 2 * SW, key_hi)
            LVLM_PACK(kA, kf)
            colsum(j0 + SW, kf);
        }
    }
#undef LVLM_LD
#undef LVLM_LOADK
#undef LVLM_PACK
}
#undef LVLM_K16

// ---- short sequences, several query chunks per KV head: one launch, key tiles shared through LDS -------
// A workgroup owns FOUR chunks of 32 query rows of one (batch, KV head) pair, one per wave, each held in
// registers as an MFMA operand.  The keys are swept twice, tile by tile (32 keys): the 256 threads fetch a
// tile with fully coalesced 16-byte loads (16 lanes per row) two tiles ahead, copy it into one of two LDS
// buffers one tile ahead, and after one barrier per tile every wave reads it as its other operand -- the
// keys cross the memory pipeline once per workgroup instead of once per wave, and in whole 64-byte requests.
// Sweep 1 (rows = keys, columns = queries) leaves each lane the online (max, sum) of its own query row: no
// fold across waves; sweep 2 (rows = queries, columns = keys) over the image keys leaves each lane the
// column sum of its key for this wave's chunk, which is that chunk's part of the result.
// MODE 0: both sweeps in this launch.  MODE 1 / 2: the keys are cut into a.n_seg runs of whole tiles and a workgroup takes ONE
// run -- MODE 1 the normaliser sweep over it, leaving each row's (max, sum) of the run for score_lse_kernel to fold, MODE 2
// the column-sum sweep over it with the folded (or the caller's) normalisers.  A wave's unit of work is then a chunk over a
// run instead of a chunk over all keys twice, which is what lets a launch of few workgroups load every SIMD evenly.
template <int DT, int HD, int MODE>
__global__ __launch_bounds__(256, (DT == LVLM_F32 && HD == 128) ? 2 : 4) void score_chunks_kernel(ScoreArgs a) {
    constexpr int ES = esize<DT>();
    constexpr int ROWB = HD * ES;
    constexpr int PITCH = ROWB + 16;
    constexpr int NV = HalfRow<DT, HD>::NV;
    constexpr int UPR = ROWB / 16;          // 16-byte units per row
    constexpr int UPT = 32 * UPR / 256;     // units each thread stages per tile
    constexpr int TPR = UPR / UPT;          // threads per row
    static_assert(UPT >= 1 && UPT <= 4, "staging covers 1..4 units per thread");
    __shared__ __attribute__((aligned(16))) char k_lds[2][32 * PITCH];
    __shared__ float lse_s[4][32];
    __shared__ int pos_s[4][32];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hf = lane >> 5, l32 = lane & 31;
    // all workgroups of one (batch, KV head) pair on one XCD (ids with the same remainder modulo 8)
    const int wpp = (a.rs + 3) >> 2;                      // workgroups per pair
    const int xcd = blockIdx.x & 7;
    const int seg = MODE == 0 ? 0 : (int)(blockIdx.x >> 3) % a.n_seg;      // this workgroup's run of keys
    const int seq = MODE == 0 ? (int)(blockIdx.x >> 3) : (int)(blockIdx.x >> 3) / a.n_seg;
    const int pair = (seq / wpp) * 8 + xcd;
    if (pair >= a.B * a.Hkv) return;
    const int b = pair / a.Hkv, g = pair % a.Hkv;
    const int c = (seq % wpp) * 4 + wave;                 // this wave's chunk
    const bool live = c < a.rs;                           // a wave without a chunk only helps to move tiles
    const int GT = a.G * a.T;
    const long long rowbase = ((long long)b * a.Hq + (long long)g * a.G) * a.T;
    auto div_t = [&](int rho) -> int { return a.T == 1 ? rho : (int)__umulhi((unsigned)rho, a.t_magic); };

    // this lane's query row (padding rows repeat the last row and get an infinite LSE)
    const int rho = c * 32 + l32;
    const int rc = min(rho, GT - 1);
    const int hl = div_t(rc), qi = rc - hl * a.T;
    const int pos = a.causal ? a.q_pos0 + qi : INT_MAX;
    HalfRow<DT, HD> qa;
    {
        const char *src = a.q + ((long long)b * a.qsb + (long long)qi * a.qst + (long long)(g * a.G + hl) * a.qsh) * ES +
                          16 * hf;
#pragma unroll
        for (int i = 0; i < NV; ++i) qa.v[i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
    }
    if (hf == 0) pos_s[wave][l32] = pos;
    // earliest position of the chunk's rows (uniform per wave): tiles at or before it need no mask
    const int rho_last = min(c * 32 + 31, GT - 1);
    const int hc0 = div_t(min(c * 32, GT - 1)), hc1 = div_t(rho_last);
    const int pos_min = a.causal ? a.q_pos0 + ((hc0 != hc1) ? 0 : min(c * 32, GT - 1) - hc0 * a.T) : INT_MAX;

    // staging: thread -> row srow of the tile, units scu + TPR x
    const int srow = tid / TPR, scu = tid % TPR;
    const char *kbase = a.k + ((long long)b * a.ksb + (long long)g * a.ksh) * ES + 16 * scu;
    uint4 st0 = make_uint4(0, 0, 0, 0), st1 = st0, st2 = st0, st3 = st0;
    auto fetch = [&](int j0, int j_end) {                 // tile rows j0 .. j0+31, clamped to the range
        const uint4 *src = reinterpret_cast<const uint4 *>(kbase + (long long)min(j0 + srow, j_end - 1) * a.ksn * ES);
        st0 = src[0];
        if constexpr (UPT > 1) st1 = src[TPR];
        if constexpr (UPT > 2) st2 = src[2 * TPR];
        if constexpr (UPT > 3) st3 = src[3 * TPR];
    };
    auto stash = [&](int buf) {
        uint4 *dst = reinterpret_cast<uint4 *>(&k_lds[buf][srow * PITCH + 16 * scu]);
        dst[0] = st0;
        if constexpr (UPT > 1) dst[TPR] = st1;
        if constexpr (UPT > 2) dst[2 * TPR] = st2;
        if constexpr (UPT > 3) dst[3 * TPR] = st3;
    };
    auto tile_operand = [&](int buf, HalfRow<DT, HD> &kf) {
        const char *src = &k_lds[buf][l32 * PITCH + 16 * hf];
#pragma unroll
        for (int i = 0; i < NV; ++i) kf.v[i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
    };

    // ---- sweep 1: this lane's row normaliser over all keys
    float m = -INFINITY, l = 0.f;
    // SAFE = false: after the first whole tile has set a finite reference m, later whole tiles take it as it is --
    // no maximum, no rescaling; a logit far above it shows as an overflowing sum, checked after the sweep, and the
    // workgroup then repeats the sweep with SAFE = true (the reference follows the running maximum on every tile).
    auto stats = [&](int j0, bool first, const HalfRow<DT, HD> &kf, auto safe_tag) {
        constexpr bool SAFE = decltype(safe_tag)::value;
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        mma_tile<DT, HD>(acc, kf, qa);                    // rows = keys, columns = queries
        if (j0 + 32 <= a.N && j0 + 31 <= pos_min) {
            if (!SAFE && !first) {                        // the sweep's first tile was whole too (tiles ascend): m is finite
                float sum = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(fmaf(acc[r], a.scale_log2, -m));
                l += sum;
                return;
            }
            float tmax = acc[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, acc[r]);
            const float mn = fmaxf(m, tmax * a.scale_log2);      // finite; scale >= 0 (checked on the host)
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(fmaf(acc[r], a.scale_log2, -mn));
            l = l * __builtin_amdgcn_exp2f(m - mn) + sum;
            m = mn;
            return;
        }
        float t[16];
        float tmax = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int j = j0 + acc_row(r, hf);
            t[r] = (j <= pos && j < a.N) ? acc[r] * a.scale_log2 : -INFINITY;
            tmax = fmaxf(tmax, t[r]);
        }
        const float mn = fmaxf(m, tmax);
        const float ms = (mn == -INFINITY) ? 0.f : mn;
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(t[r] - ms);   // exp2(-inf) = 0
        l = l * __builtin_amdgcn_exp2f(m - ms) + sum;
        m = mn;
    };
    // ---- sweep 2: column sums of the image keys for this wave's chunk
    const int key_lo = a.img_begin, key_hi = a.img_begin + a.n_img;
    float *out = a.colpart + (((long long)min(c, a.rs - 1) * a.B + b) * a.Hkv + g) * a.n_img;
    float lse_r[16];                                      // the normalisers of this lane's 16 accumulator rows
    auto colsum = [&](int j0, const HalfRow<DT, HD> &kf) {
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        mma_tile<DT, HD>(acc, qa, kf);                    // rows = queries, columns = keys
        const int j = j0 + l32;
        float sum = 0.f;
        if (j0 + 31 <= pos_min) {
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(fmaf(acc[r], a.scale_log2, -lse_r[r]));
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(acc[r], a.scale_log2, -lse_r[r]));
                sum += (j <= pos_s[wave][acc_row(r, hf)]) ? p : 0.f;
            }
        }
        sum += other_half(sum);
        if (hf == 0 && j < key_hi) out[j - key_lo] = sum;
    };

    // One sweep: tile t is fetched in iteration t-2, copied to LDS in iteration t-1 and used in iteration t
    // (one barrier per tile publishes the copy; fetches past the last tile repeat its last row).
    auto sweep = [&](int j_begin, int j_end, bool second, auto safe_tag) {
        const int nt = (j_end - j_begin + 31) >> 5;
        fetch(j_begin, j_end);
        stash(0);
        fetch(j_begin + 32, j_end);
        __syncthreads();
        for (int t = 0; t < nt; ++t) {
            stash((t + 1) & 1);                           // tile t+1
            fetch(j_begin + 32 * (t + 2), j_end);
            if (live) {
                HalfRow<DT, HD> kf;
                tile_operand(t & 1, kf);
                if (second) colsum(j_begin + 32 * t, kf);
                else stats(j_begin + 32 * t, t == 0, kf, safe_tag);
            }
            __syncthreads();
        }
    };

    // the tiles of [lo, hi) this workgroup takes: all of them, or its run (equal shares of whole tiles)
    auto run_of = [&](int lo, int hi, int &jb, int &je) {
        jb = lo, je = hi;
        if (MODE != 0) {
            const long long nt = (hi - lo + 31) >> 5;
            jb = lo + 32 * (int)(nt * seg / a.n_seg);
            je = min(hi, lo + 32 * (int)(nt * (seg + 1) / a.n_seg));
        }
    };
    if (MODE == 1 || (MODE == 0 && a.row_lse == nullptr)) {
        int jb, je;
        run_of(0, a.N, jb, je);
        if (jb < je) {
            sweep(jb, je, false, std::false_type{});
            if (__syncthreads_or(!(l < 1.0e30f))) {       // some sum ran away (or is not a number): the careful sweep
                m = -INFINITY, l = 0.f;
                sweep(jb, je, false, std::true_type{});
            }
        }
        {
            const float mo = other_half(m), lo = other_half(l);
            const float mn = fmaxf(m, mo);
            const float ms = (mn == -INFINITY) ? 0.f : mn;
            l = l * __builtin_amdgcn_exp2f(m - ms) + lo * __builtin_amdgcn_exp2f(mo - ms);
            m = mn;
        }
        if (MODE == 1) {                                  // this run's share of the rows' normalisers
            if (hf == 0 && live && rho < GT) {
                const long long pidx = (long long)seg * a.B * a.Hq * a.T + rowbase + rho;
                a.part_m[pidx] = m;
                a.part_l[pidx] = l;
            }
            return;
        }
        // no visible key, or a padding row: contributes nothing
        if (hf == 0) lse_s[wave][l32] = (l > 0.f && rho < GT) ? m + log2f(l) : INFINITY;
    } else if (hf == 0) {
        const bool real = live && rho < GT;
        lse_s[wave][l32] = !real ? INFINITY : (a.row_lse ? a.row_lse[rowbase + rho] * kLog2e : a.lse2[rowbase + rho]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) lse_r[r] = lse_s[wave][acc_row(r, hf)];
    int jb, je;
    run_of(key_lo, key_hi, jb, je);
    if (jb < je) sweep(jb, je, true, std::true_type{});
}

// ---- many query chunks over long sequences: the keys of all pairs in equal shares, a launch per sweep ----------
// The two sweeps of score_chunks_kernel for bf16 calls of much work.  There the fragments that every wave reads from LDS for
// one 32-row chunk, a barrier per 32 keys and turns of workgroups that do not come out even cost more than the products.  Here
// a wave holds TWO chunks, so that a fragment feeds two products, a workgroup of NW waves owns 2 NW chunks of a (batch, KV head)
// pair, and the launch has two waves per SIMD, each with an equal share of the keys: the pairs' keys lie behind each
// other in steps of 64, and share j, whichever pairs it reaches into, goes to the workgroups of one XCD that own the pair's chunks
// (they read the same keys at the same time).
// Steps go from memory straight into a ring of LDS slots (direct loads, 16-byte units swizzled as in the few-rows kernel below;
// the loads are assembly for the reason given there, their waits counted by hand; one barrier per step).  Only two steps are
// requested before anything else, the rest of the ring when these have landed: all at once, every workgroup would wait for
// everybody's whole ring.
// Products and softmax of different chunks are meant to go side by side: the products of chunk 0 with the softmax of chunk 1 of the
// tile before, those of chunk 1 with the softmax of chunk 0, cut into slots of one product and two logits (scaling, exponential and
// sum a slot apart), with scheduling barriers between the slots.  Those hold inside a basic block only, and a step has branches
// (around its wait and its fetch): as compiled, one of a step's four softmaxes (column sums), or two (normalisers), are moved behind
// the branches and run alone, after products that nothing runs beside.
// SECOND = false: rows = keys, columns = queries; each row's (max, sum) of the share.  SECOND = true: rows = queries, columns =
// keys; the shares' normalisers are folded at the start of a pair (they are few), or the caller's taken, and a wave leaves the
// column sums of its two chunks as one part.
// A tile takes 220 ns per SIMD; without its fetches, barriers and fragment reads (and so without the branches) 190; a probe of 8
// products and 32 exponentials, scalings and sums alone 180, which is vector issue beside the products at the clock the power
// allows.  Against score_chunks_kernel in runs and its folds: 12 sequences x 5219 keys x 48 heads 249 -> 225 us for the call; under
// the profiler, on one machine, 135 and 133 us for the sweeps and 5 and 11 for the folds -> 131, 123 and 8 (725 -> 768 TFLOP/s over
// the sweeps; 818 on a machine that held a higher clock).
constexpr int kShareStep = 64;               // keys per step
// Normaliser of the rows that fill up the last chunk, or a wave's second one: their probabilities are zero, and where the row they
// repeat has an infinite logit they are infinite as its own is (an infinite normaliser would make a NaN of it).
constexpr float kNoRowLse = 3.0e38f;
template <int HD, bool SECOND, int NW>
__global__ __launch_bounds__(64 * NW, 2) void score_shares_kernel(ScoreArgs a) {
    constexpr int ES = 2, ROWB = HD * ES, NV = HD / 16;
    constexpr int RING = NW == 4 ? 4 : 2;   // slots: what two waves per SIMD leave room for
    constexpr int STEP = kShareStep, SLOT = STEP * ROWB;
    constexpr int UPR = ROWB / 16, RPL = 1024 / ROWB;      // 16-byte units per row, rows per direct load
    constexpr int DPW = SLOT / 1024 / NW;   // direct loads per wave and step
    constexpr int NOFF = DPW < 16 / RPL ? DPW : 16 / RPL;  // the swizzle repeats after 16 rows, and so do the offsets
    __shared__ __attribute__((aligned(1024))) char k_lds[RING * SLOT];
    __shared__ float lse_s[2 * NW][32];
    __shared__ int pos_s[2 * NW][32];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hf = lane >> 5, l32 = lane & 31;
    const int GT = a.G * a.T;
    const int n_chunks = (GT + 31) >> 5;
    const int wpp = (n_chunks + 2 * NW - 1) / (2 * NW);   // workgroups per pair
    const int xcd = blockIdx.x & 7, seq = (int)(blockIdx.x >> 3);
    const int c0 = (seq % wpp) * 2 * NW + 2 * wave;       // this wave's first chunk
    const bool live = c0 < n_chunks;                      // a wave without a chunk only helps to move the keys
    const KeyRuns &runs = SECOND ? a.runs2 : a.runs1;
    const int per_xcd = (runs.shares + 7) >> 3, share = xcd * per_xcd + seq / wpp;
    if (seq / wpp >= per_xcd || share >= runs.shares) return;
    int at = runs.begin(share);
    const int at_end = runs.begin(share + 1);
    const long long rows = (long long)a.B * a.Hq * a.T;
    auto div_t = [&](int rho) -> int { return a.T == 1 ? rho : (int)__umulhi((unsigned)rho, a.t_magic); };

    // load x of this wave fills rows RPL (DPW wave + x) .. of a slot, lane -> row lane / UPR, place lane % UPR
    const unsigned ksb = (unsigned)(a.ksn * ES);          // (the host checks that a step's rows span less than 2 GiB)
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)k_lds + 1024u * (DPW * wave);
    auto place = [](int row) { return ROWB == 128 ? (row >> 1) & 7 : row & 15; };
    const int frow = RPL * DPW * wave + lane / UPR;       // this lane's row in load 0
    unsigned off[NOFF];
#pragma unroll
    for (int x = 0; x < NOFF; ++x) off[x] = (frow + RPL * x) * ksb + 16 * ((lane % UPR) ^ place(frow + RPL * x));
    // contraction step i of lane half hf takes bytes [32 i + 16 hf, +16) of a row
    unsigned uo[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) uo[i] = l32 * ROWB + 16 * ((2 * i + hf) ^ place(l32));
    auto frag = [&](int slot, int s, int i) {             // word i of this lane's row of tile s of a slot
        return *reinterpret_cast<const uint4 *>(&k_lds[slot * SLOT + s * (32 * ROWB) + uo[i]]);
    };
    // All steps fetched have landed everywhere -- but the RING - 2 youngest if that many are under way -- and everybody's reads
    // of the step before are back.
    auto landed = [](bool full) {
        if (full) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(DPW * (RING - 2)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    const int key_lo = a.img_begin, key_hi = a.img_begin + a.n_img;

    for (int pair = at / runs.steps;; ++pair) {           // the pairs of this share
        const int b = pair / a.Hkv, g = pair % a.Hkv;
        const long long rowbase = ((long long)b * a.Hq + (long long)g * a.G) * a.T;
        const int s0 = at - pair * runs.steps, n_steps = min(runs.steps - s0, at_end - at);
        at += n_steps;
        const int jb = (SECOND ? key_lo : 0) + STEP * s0, je = min(SECOND ? key_hi : a.N, jb + STEP * n_steps);
        const char *kbase = a.k + ((long long)b * a.ksb + (long long)g * a.ksh) * ES;
        auto fetch = [&](int t) {                         // step t: rows clamped to the share's last one
            const int j0 = jb + STEP * t;
            const unsigned dst = lds0 + (unsigned)(t % RING * SLOT);
            const char *base = kbase + (long long)j0 * a.ksn * ES;
#pragma unroll
            for (int x = 0; x < DPW; ++x) {
                const int row = frow + RPL * x;
                const char *src = base;                   // uniform
                unsigned o = off[x % NOFF];
                if (j0 + STEP <= je) src += (long long)(x / NOFF * NOFF * RPL) * a.ksn * ES;
                else o = (unsigned)min(row, je - 1 - j0) * ksb + 16 * ((lane % UPR) ^ place(row));
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(o), "s"(src), "s"(dst + 1024u * x)
                             : "memory", "m0");
            }
        };
        auto begin = [&] {
            fetch(0);
            if (n_steps > 1) fetch(1);
        };
        begin();

        // this lane's query rows (padding rows repeat the last row, with kNoRowLse)
        int rho[2], pos[2];
        HalfRow<LVLM_BF16, HD> qa[2];
        int pos_min = INT_MAX;      // earliest position of the wave's rows (uniform): tiles at or before it need no mask
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int c = c0 + x;
            rho[x] = c * 32 + l32;
            const int rc = min(rho[x], GT - 1);
            const int hl = div_t(rc), qi = rc - hl * a.T;
            pos[x] = a.causal ? a.q_pos0 + qi : INT_MAX;
            const char *src = a.q + ((long long)b * a.qsb + (long long)qi * a.qst + (long long)(g * a.G + hl) * a.qsh) * ES + 16 * hf;
#pragma unroll
            for (int i = 0; i < NV; ++i) qa[x].v[i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
            if (hf == 0) pos_s[2 * wave + x][l32] = pos[x];
            const int r_first = min(c * 32, GT - 1), r_last = min(c * 32 + 31, GT - 1);
            const int hc0 = div_t(r_first), hc1 = div_t(r_last);
            if (a.causal) pos_min = min(pos_min, a.q_pos0 + ((hc0 != hc1) ? 0 : r_first - hc0 * a.T));
        }
        float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};     // sweep 1: the rows' (max, sum)
        float lse_r[2][16];                               // sweep 2: the normalisers of this lane's 16 accumulator rows
        if constexpr (SECOND) {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const long long row = rowbase + min(rho[x], GT - 1);
                float lse;
                if (a.row_lse) {
                    lse = a.row_lse[row] * kLog2e;
                } else {
                    // what the shares of sweep 1 left, every second one per lane half, sixteen at a time
                    const int n_part = a.runs1.count(pair);
                    float mx = -INFINITY, lx = 0.f;
                    for (int i0 = hf; i0 < n_part; i0 += 16) {
                        float mi[8], li[8];
#pragma unroll
                        for (int y = 0; y < 8; ++y) {
                            const long long from = min(i0 + 2 * y, n_part - 1) * rows + row;
                            mi[y] = a.part_m[from], li[y] = a.part_l[from];
                        }
                        float mn = mx;
#pragma unroll
                        for (int y = 0; y < 8; ++y) {
                            if (i0 + 2 * y >= n_part) mi[y] = -INFINITY, li[y] = 0.f;
                            mn = fmaxf(mn, mi[y]);
                        }
                        const float ms = (mn == -INFINITY) ? 0.f : mn;
                        lx *= exp2f(mx - ms);
#pragma unroll
                        for (int y = 0; y < 8; ++y) lx += li[y] * exp2f(mi[y] - ms);      // exp2(-inf) = 0 covers empty shares
                        mx = mn;
                    }
                    const float mo = other_half(mx), lo = other_half(lx);
                    const float mn = fmaxf(mx, mo), ms = (mn == -INFINITY) ? 0.f : mn;
                    lx = lx * exp2f(mx - ms) + lo * exp2f(mo - ms);
                    lse = lx > 0.f ? mn + log2f(lx) : INFINITY;      // no visible key: contributes nothing
                }
                if (hf == 0) lse_s[2 * wave + x][l32] = rho[x] < GT ? lse : kNoRowLse;
            }
            __syncthreads();
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) lse_r[x][r] = lse_s[2 * wave + x][acc_row(r, hf)];
        }
        float *out = a.colpart + (((long long)(min(c0, n_chunks - 1) / 2) * a.B + b) * a.Hkv + g) * a.n_img;

        // One tile with every check: sweep 1 follows the running maximum, sweep 2 stores lane by lane.  `stands`: the rows'
        // references were set by a whole tile, so that later tiles take neither a maximum nor a rescale (FAST sweeps only).
        auto careful = [&](int j0, bool stands, const HalfRow<LVLM_BF16, HD> &kf) {
            float col = 0.f;
            const bool whole = j0 + 32 <= je && j0 + 31 <= pos_min;
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                f32x16 acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.f;
                if constexpr (SECOND) {
                    mma_tile<LVLM_BF16, HD>(acc, qa[x], kf);
                    float part = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float p = __builtin_amdgcn_exp2f(fmaf(acc[r], a.scale_log2, -lse_r[x][r]));
                        part += whole || j0 + l32 <= pos_s[2 * wave + x][acc_row(r, hf)] ? p : 0.f;
                    }
                    col += part;
                } else {
                    mma_tile<LVLM_BF16, HD>(acc, kf, qa[x]);
                    float tmax = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int j = j0 + acc_row(r, hf);
                        acc[r] = whole || (j <= pos[x] && j < je) ? acc[r] * a.scale_log2 : -INFINITY;
                        tmax = fmaxf(tmax, acc[r]);
                    }
                    const float mn = stands ? m[x] : fmaxf(m[x], tmax), ms = (mn == -INFINITY) ? 0.f : mn;
                    float sum = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(acc[r] - ms);      // exp2(-inf) = 0
                    l[x] = (stands ? l[x] : l[x] * __builtin_amdgcn_exp2f(m[x] - ms)) + sum;
                    m[x] = mn;
                }
            }
            if constexpr (SECOND) {
                col += other_half(col);
                if (hf == 0 && j0 + l32 < je) out[j0 + l32 - key_lo] = col;
            }
        };
        // Steps [0, n_fast), whose keys all rows of the wave see.  Sweep 1: the first tile's maximum is every row's reference; a
        // logit far above it shows as an overflowing sum, checked after the sweep.
        auto fast = [&](int n_fast) {
            uint4 kf[NV];
            f32x16 acc[2], zero;
#pragma unroll
            for (int r = 0; r < 16; ++r) zero[r] = 0.f;
            float part[2][2];       // column sums: [tile of the step][chunk]
            auto mfma = [&](const uint4 &kw, const uint4 &qw, const f32x16 &c) {
                const bf16x8 kv = __builtin_bit_cast(bf16x8, kw), qv = __builtin_bit_cast(bf16x8, qw);
                return SECOND ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(qv, kv, c, 0, 0, 0)
                              : __builtin_amdgcn_mfma_f32_32x32x16_bf16(kv, qv, c, 0, 0, 0);
            };
            constexpr int LPS = 16 / NV;                  // logits per slot
            float e_arg[16], e_p[16], sum0, sum1;
            auto arg = [&](int x, int r) { return fmaf(acc[x][r], a.scale_log2, SECOND ? -lse_r[x][r] : -m[x]); };
            auto vec_begin = [&](int x) {
                sum0 = sum1 = 0.f;
#pragma unroll
                for (int e = 0; e < LPS; ++e) e_arg[e] = arg(x, e);
            };
            auto vec_slot = [&](int x, int i) {
#pragma unroll
                for (int e = LPS * i; e < LPS * (i + 1); ++e) {
                    if (i + 1 < NV) e_arg[LPS + e] = arg(x, LPS + e);
                    e_p[e] = __builtin_amdgcn_exp2f(e_arg[e]);
                }
                if (i > 0) {
#pragma unroll
                    for (int e = LPS * (i - 1); e < LPS * i; e += 2) sum0 += e_p[e], sum1 += e_p[e + 1];
                }
            };
            auto vec_end = [&](int x, int tile) {
#pragma unroll
                for (int e = 16 - LPS; e < 16; e += 2) sum0 += e_p[e], sum1 += e_p[e + 1];
                if (SECOND) part[tile][x] = sum0 + sum1;
                else l[x] += sum0 + sum1;
            };
            auto softmax = [&](int x, int tile) {
                vec_begin(x);
#pragma unroll
                for (int i = 0; i < NV; ++i) vec_slot(x, i);
                vec_end(x, tile);
            };
            // products of chunk x beside the softmax of the other chunk (of tile `tile` of its step); behind the last use of a
            // fragment (`next`) the read of tile ns of slot nslot
            auto phase = [&](int x, int tile, bool next, int nslot, int ns) {
                vec_begin(x ^ 1);
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    acc[x] = mfma(kf[i], qa[x].v[i], i == 0 ? zero : acc[x]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (next) kf[i] = frag(nslot, ns, i);
                    vec_slot(x ^ 1, i);
                    __builtin_amdgcn_sched_barrier(0);
                }
                vec_end(x ^ 1, tile);
            };
            auto put = [&](int t) {                       // the column sums of step t: lanes 0-31 its first tile, 32-63 its second
                if constexpr (SECOND) {
                    typedef unsigned u2 __attribute__((ext_vector_type(2)));
                    const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(part[0][0] + part[0][1]),
                                                                  __float_as_uint(part[1][0] + part[1][1]), false, false);
                    out[jb + STEP * t - key_lo + lane] = __uint_as_float(r.x) + __uint_as_float(r.y);
                }
            };
#pragma unroll
            for (int i = 0; i < NV; ++i) kf[i] = frag(0, 0, i);
#pragma unroll
            for (int i = 0; i < NV; ++i)
#pragma unroll
                for (int x = 0; x < 2; ++x) acc[x] = mfma(kf[i], qa[x].v[i], i == 0 ? zero : acc[x]);
            if constexpr (!SECOND) {
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    float tmax = acc[x][0];
#pragma unroll
                    for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, acc[x][r]);
                    m[x] = tmax * a.scale_log2;           // scale >= 0 (checked on the host)
                }
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) kf[i] = frag(0, 1, i);
            softmax(0, 0);
            // step t from the products of its second tile on, and the first tile of the next one
            auto step = [&](int t, auto slot_tag) {
                constexpr int next_slot = (decltype(slot_tag)::value + 1) % RING;
                phase(0, 0, false, 0, 0);
                if (t + 1 < n_steps) landed(t + RING - 1 < n_steps);      // step t + 1 is complete, step t's slot free
                if (t + RING < n_steps) fetch(t + RING);
                phase(1, 1, true, next_slot, 0);          // (past the last step: fragments that nothing uses)
                if (t + 1 < n_fast) {
                    phase(0, 1, false, 0, 0);
                    put(t);
                    phase(1, 0, true, next_slot, 1);
                } else {
                    softmax(1, 1);
                    put(t);
                }
            };
            for (int t = 0; t < n_fast; t += RING) {
                step(t, std::integral_constant<int, 0>{});
                if (t + 1 < n_fast) step(t + 1, std::integral_constant<int, 1>{});
                if constexpr (RING > 2) {
                    if (t + 2 < n_fast) step(t + 2, std::integral_constant<int, 2>{});
                    if (t + 3 < n_fast) step(t + 3, std::integral_constant<int, 3>{});
                }
            }
        };
        // One sweep, begun: every wave passes n_steps barriers, whatever its n_fast.
        auto sweep = [&](bool safe) {
            landed(false);
#pragma unroll
            for (int t = 2; t < RING; ++t)
                if (t < n_steps) fetch(t);
            const int n_fast = live && !safe ? steps_seen(jb, je, pos_min, STEP) : 0;      // steps that all rows of the wave see
            if (n_fast > 0) fast(n_fast);
            for (int t = n_fast; t < n_steps; ++t) {
                for (int s = 0; s < 2 && live; ++s) {
                    const int j0 = jb + STEP * t + 32 * s;
                    if (j0 >= je) continue;
                    HalfRow<LVLM_BF16, HD> kf;
#pragma unroll
                    for (int i = 0; i < NV; ++i) kf.v[i] = frag(t % RING, s, i);
                    careful(j0, n_fast > 0, kf);
                }
                if (t + 1 < n_steps) landed(t + RING - 1 < n_steps);
                if (t + RING < n_steps) fetch(t + RING);
            }
        };
        sweep(false);
        if constexpr (!SECOND) {
            if (__syncthreads_or(!(l[0] < 1.0e30f) || !(l[1] < 1.0e30f))) {      // some sum ran away (or is not a number)
                m[0] = m[1] = -INFINITY, l[0] = l[1] = 0.f;
                begin();
                sweep(true);
            }
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const float mo = other_half(m[x]), lo = other_half(l[x]);
                const float mn = fmaxf(m[x], mo), ms = (mn == -INFINITY) ? 0.f : mn;
                l[x] = l[x] * __builtin_amdgcn_exp2f(m[x] - ms) + lo * __builtin_amdgcn_exp2f(mo - ms);
                if (hf == 0 && rho[x] < GT) {             // this share's part of the rows' normalisers
                    const long long to = (long long)(share - runs.first(pair)) * rows + rowbase + rho[x];
                    a.part_m[to] = mn;
                    a.part_l[to] = l[x];
                }
            }
        }
        if (at >= at_end) return;
        __syncthreads();                                  // nobody reads the slots, positions or normalisers any more
    }
}

// ---- few query rows: the logits of a chunk over ALL keys in registers, one sweep -------------------------
// A workgroup of eight waves owns 16 query rows of one (batch, KV head) pair.  Wave w takes the 16-key tiles w, w + 8,
// ... (NTW of them at most) and keeps every logit -- 4 registers per tile -- so the keys are read and multiplied once
// where the other forms do it twice: the wave's own row maxima and sums, one exchange of them through LDS, and the
// exponentials already taken are scaled to probabilities and summed down the rows.  Nothing but the chunk's column sums
// leaves the workgroup.
// A tile goes from memory straight into one of four LDS buffers of the wave (direct loads of whole rows: as operands, lane
// = key, they would cost the memory pipeline a cycle per lane), three tiles ahead; no barrier, a wave waits for its own.
// The 16-byte units of row R lie in the order u ^ R (256-byte rows; u ^ R / 2 for 128), so that the sixteen lanes an LDS read
// serves at a time hit sixteen bank groups.  The loads are assembly for the reason given at the similarity product: the
// compiler would wait for all buffers.
// Operand lane = (l16, kg): contraction step i of lane group kg is bytes 64 i + 16 kg of a row; the result holds key l16 of a
// 16-key block for query rows 4 kg + r.
// What bounds it: launch and start-up (5.4 us for 200 keys), then a compute unit's rate of taking in the keys.
constexpr int kRowsWaves = 8;
template <int DT, int HD, int NTW>
__global__ __launch_bounds__(64 * kRowsWaves) void score_rows_kernel(ScoreArgs a) {
    constexpr int ES = esize<DT>();
    constexpr int ROWB = HD * ES, UPR = ROWB / 16;
    constexpr int NW = ROWB / 64;           // 16-byte words per lane of a row
    constexpr int NWV = kRowsWaves, STEP = 16 * NWV, RING = 4;
    constexpr int TB = 16 * ROWB;           // bytes of a tile
    constexpr int DPT = TB / 1024, RPL = 1024 / ROWB;      // direct loads per tile, rows per load
    static_assert(ROWB == 128 || ROWB == 256, "the swizzle is for these row lengths");
    __shared__ __attribute__((aligned(1024))) char tile[NWV][RING][TB];
    __shared__ __attribute__((aligned(16))) float wm[NWV][16], wl[NWV][16];      // [wave][row]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    // (batch, KV head, chunk) triples in memory order, an eighth of them to every XCD (ids with the same remainder modulo 8): the
    // chunks of a pair mostly share an L2, and no XCD gets more than another whatever the heads (with all chunks of a pair on one
    // XCD: one head of 37 chunks x 2632 keys 26.9 us, 18 heads of 13 x 242 keys 13.1; evenly 15.6 and 9.3)
    const int total = a.B * a.Hkv * a.rs, per_xcd = (total + 7) >> 3;
    const int item = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (item >= total) return;
    const int pair = item / a.rs, c = item % a.rs;
    const int b = pair / a.Hkv, g = pair % a.Hkv;
    const int GT = a.G * a.T;
    const long long rowbase = ((long long)b * a.Hq + (long long)g * a.G) * a.T;
    auto div_t = [&](int rho) -> int { return a.T == 1 ? rho : (int)__umulhi((unsigned)rho, a.t_magic); };

    const int key_lo = a.img_begin, key_hi = a.img_begin + a.n_img;
    // with the normalisers given only the image keys are needed
    const int j_lo = a.row_lse ? key_lo : 0, j_hi = a.row_lse ? key_hi : a.N;
    const int jw = j_lo + 16 * wave;
    const int n_t = jw < j_hi ? (j_hi - 1 - jw) / STEP + 1 : 0;     // this wave's tiles
    const char *kbase = a.k + ((long long)b * a.ksb + (long long)g * a.ksh) * ES;
    auto place = [](int row) { return ROWB == 256 ? row & 15 : (row >> 1) & 7; };
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)&tile[wave][0][0];
    const unsigned ksb = (unsigned)(a.ksn * ES);          // (the host checks that a tile's rows span less than 2 GiB)
    unsigned off[DPT], off_last[DPT];       // of this lane's units in a tile; in a tile that ends past the last row
    const int r_last = (j_hi - 1 - jw) & (STEP - 1);      // last row inside this wave's last tile (>= 15: a whole one)
#pragma unroll
    for (int x = 0; x < DPT; ++x) {
        const int row = RPL * x + lane / UPR, u = 16 * ((lane % UPR) ^ place(row));
        off[x] = row * ksb + u;
        off_last[x] = min(row, r_last) * ksb + u;
    }
    auto fetch = [&](int t) {               // tile t of this wave (the last one again past the end)
        const int tc = min(t, n_t - 1), j0 = jw + STEP * tc;
        const char *base = kbase + (long long)j0 * a.ksn * ES;
        const unsigned dst = lds0 + (unsigned)(t % RING) * TB;
        auto go = [&](const unsigned (&o)[DPT]) {
#pragma unroll
            for (int x = 0; x < DPT; ++x)
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(o[x]), "s"(base), "s"(dst + 1024u * x)
                             : "memory", "m0");
        };
        if (j0 + 16 <= j_hi) go(off);
        else go(off_last);
    };
    uint4 qf[NW];                           // row l16 of the chunk (rows past the last one repeat it; they weigh nothing)
    {
        const int rho = min(c * 16 + l16, GT - 1), hl = div_t(rho), i = rho - hl * a.T;
        const char *src = a.q + ((long long)b * a.qsb + (long long)i * a.qst + (long long)(g * a.G + hl) * a.qsh) * ES + 16 * kg;
#pragma unroll
        for (int x = 0; x < NW; ++x) qf[x] = *reinterpret_cast<const uint4 *>(src + 64 * x);
    }
    if (n_t > 0) {
#pragma unroll
        for (int t = 0; t < RING - 1; ++t) fetch(t);
    }
    int pos[4];                             // of rows 4 kg + r
    float given[4];
    bool real[4];
    int pos_min = INT_MAX;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int rho = c * 16 + 4 * kg + r, rc = min(rho, GT - 1);
        real[r] = rho < GT;
        pos[r] = a.causal ? a.q_pos0 + rc - div_t(rc) * a.T : INT_MAX;
        given[r] = a.row_lse ? a.row_lse[rowbase + rc] * kLog2e : 0.f;
        pos_min = min(pos_min, pos[r]);
    }
    // earliest position of the chunk's rows (uniform): tiles at or before it need no mask
    pos_min = min(pos_min, __float_as_int(swap_rows(__int_as_float(pos_min))));
    pos_min = __builtin_amdgcn_readfirstlane(min(pos_min, __float_as_int(swap_halves(__int_as_float(pos_min)))));

    static_assert(NTW % 4 == 0, "column sums go four tiles at a time");
    f32x4 s[NTW];
    float m[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
        const int j0 = jw + STEP * t;
        if (t < n_t) {
            // the buffer about to be written is the one read for tile t - 1: those reads have to be back
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fetch(t + RING - 1);            // (past the last tile: its last row again; the wait counts on these loads)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(DPT * (RING - 1)) : "memory");
            uint4 kf[NW];
#pragma unroll
            for (int i = 0; i < NW; ++i)
                kf[i] = *reinterpret_cast<const uint4 *>(&tile[wave][t % RING][l16 * ROWB + 16 * ((4 * i + kg) ^ place(l16))]);
            f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                if constexpr (DT == LVLM_BF16) {
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qf[i]), __builtin_bit_cast(bf16x8, kf[i]),
                                                                  acc, 0, 0, 0);
                } else {
                    const uint32_t qw[4] = {qf[i].x, qf[i].y, qf[i].z, qf[i].w}, kw[4] = {kf[i].x, kf[i].y, kf[i].z, kf[i].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qw[e]), __uint_as_float(kw[e]), acc, 0, 0, 0);
                }
            }
            if (j0 + 16 > j_hi || j0 + 15 > pos_min) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (j0 + l16 >= j_hi || j0 + l16 > pos[r]) acc[r] = -INFINITY;
            }
            s[t] = acc;
#pragma unroll
            for (int r = 0; r < 4; ++r) m[r] = fmaxf(m[r], acc[r]);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no load may land after the workgroup has left its LDS
    // the wave's row maxima (log2 domain), exponentials relative to them and their sums
    auto row_red = [](float v, auto op) {      // over the 16 lanes of the row group
        v = op(v, dpp_quad1(v));
        v = op(v, dpp_quad2(v));
        v = op(v, dpp_half_mirror(v));
        return op(v, dpp_row_mirror(v));
    };
    auto maxf = [](float x, float y) { return fmaxf(x, y); };
    auto addf = [](float x, float y) { return x + y; };
    float ref[4], l[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        m[r] = row_red(m[r], maxf) * a.scale_log2;        // scale > 0 (checked on the host)
        ref[r] = m[r] == -INFINITY ? 0.f : m[r];
        l[r] = 0.f;
    }
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
        if (t < n_t) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[t][r] = __builtin_amdgcn_exp2f(fmaf(s[t][r], a.scale_log2, -ref[r]));
                l[r] += s[t][r];
            }
        }
    }
    float f[4];                             // exponential -> probability
    if (a.row_lse) {
#pragma unroll
        for (int r = 0; r < 4; ++r) f[r] = real[r] && m[r] > -INFINITY ? __builtin_amdgcn_exp2f(ref[r] - given[r]) : 0.f;
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) l[r] = row_red(l[r], addf);
        if (l16 == 0) {
            *reinterpret_cast<float4 *>(&wm[wave][4 * kg]) = make_float4(m[0], m[1], m[2], m[3]);
            *reinterpret_cast<float4 *>(&wl[wave][4 * kg]) = make_float4(l[0], l[1], l[2], l[3]);
        }
        __syncthreads();
        // lane l16 takes wave l16's share of rows 4 kg + r (twice over: lanes 8 .. 15 repeat 0 .. 7, with sums of zero)
        const int wj = l16 & (NWV - 1);
        const float4 m4 = *reinterpret_cast<const float4 *>(&wm[wj][4 * kg]), l4 = *reinterpret_cast<const float4 *>(&wl[wj][4 * kg]);
        const float mj[4] = {m4.x, m4.y, m4.z, m4.w}, lj[4] = {l4.x, l4.y, l4.z, l4.w};
        const bool mine = l16 < NWV;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float mx = row_red(mj[r], maxf);
            const float ms = mx == -INFINITY ? 0.f : mx;
            const float tot = row_red(mine ? lj[r] * __builtin_amdgcn_exp2f(mj[r] - ms) : 0.f, addf);
            // a padding row, or no key of this wave visible: contributes nothing (without a maximum of the wave's own the
            // factor would be exp2(-ms), infinite for a row of very negative logits)
            f[r] = real[r] && m[r] > -INFINITY && tot > 0.f ? __builtin_amdgcn_exp2f(ref[r] - ms) / tot : 0.f;
        }
    }
    // column sums of the image keys: over the lane's four rows, then over the row groups -- four tiles at a time, each
    // exchange leaving half of them with every lane: row group kg ends with tile t + kg
    float *out = a.colpart + (((long long)c * a.B + b) * a.Hkv + g) * a.n_img;
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    auto fold16 = [](float x, float y) {       // lanes of even rows of 16: x of rows 2k and 2k + 1; of odd rows: y
        const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r.x) + __uint_as_float(r.y);
    };
    auto fold32 = [](float x, float y) {       // lanes 0-31: x of both halves; lanes 32-63: y
        const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r.x) + __uint_as_float(r.y);
    };
#pragma unroll
    for (int t = 0; t < NTW; t += 4) {
        if (t < n_t) {
            float x[4];
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                x[y] = s[t + y][0] * f[0];
#pragma unroll
                for (int r = 1; r < 4; ++r) x[y] = fmaf(s[t + y][r], f[r], x[y]);
            }
            const float v = fold32(fold16(x[0], x[1]), fold16(x[2], x[3]));
            const int j = jw + STEP * (t + kg) + l16;
            if (t + kg < n_t && j >= key_lo && j < key_hi) out[j - key_lo] = v;
        }
    }
}

// Fold the per-block, per-wave (max, sum) pairs of each row into a log2-domain LSE.  Eight lanes share a
// row: each folds every eighth pair online, then the eight partial (max, sum) states are merged.
__global__ __launch_bounds__(256) void score_lse_kernel(const float *part_m, const float *part_l, float *lse2,
                                                        int rows, int nparts) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    const int row = t >> 3, sub = t & 7;
    float m = -INFINITY, l = 0.f;
    if (row < rows) {
#pragma unroll 4
        for (int i = sub; i < nparts; i += 8) {
            const float mi = part_m[(long long)i * rows + row];
            const float li = part_l[(long long)i * rows + row];
            const float mn = fmaxf(m, mi);
            const float ms = (mn == -INFINITY) ? 0.f : mn;
            l = l * exp2f(m - ms) + li * exp2f(mi - ms);      // exp2(-inf) = 0 covers empty blocks
            m = mn;
        }
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
        const float mo = __shfl_xor(m, o), lo = __shfl_xor(l, o);
        const float mn = fmaxf(m, mo);
        const float ms = (mn == -INFINITY) ? 0.f : mn;
        l = l * exp2f(m - ms) + lo * exp2f(mo - ms);
        m = mn;
    }
    if (row < rows && sub == 0) lse2[row] = (l > 0.f) ? m + log2f(l) : INFINITY;   // no visible key: contributes nothing
}

// score_head[b][g][j] = (sum over row splits of the column sums) / G;  score_mean[b][j] = mean over g.
// A chain of latencies (launch, one round of loads, two barriers), so the parts of a column are spread over threads:
// thread (column, slot of four heads, slot of four parts) sums every fourth part of every fourth head, eight loads in
// flight; the sixteen slots meet in LDS in a fixed order.
__global__ __launch_bounds__(1024) void score_finalize_kernel(ScoreArgs a) {
    __shared__ float part[4][4][64];        // [part slot][head slot][column]
    __shared__ float mean_s[4][64];
    const int col = threadIdx.x & 63, hs = (threadIdx.x >> 6) & 3, ps = threadIdx.x >> 8;
    const int j = blockIdx.x * 64 + col, jc = min(j, a.n_img - 1);
    const int b = blockIdx.y;
    const float inv_g = 1.0f / (float)a.G;
    const long long split_stride = (long long)a.B * a.Hkv * a.n_img;
    float mean = 0.f;                       // of this head slot's heads (part slot 0)
    for (int g0 = 0; g0 < a.Hkv; g0 += 4) {
        const int g = g0 + hs;
        float tot = 0.f;
        if (g < a.Hkv) {
            const float *src = a.colpart + ((long long)b * a.Hkv + g) * a.n_img + jc;
            for (int r0 = ps; r0 < a.rs; r0 += 32) {
                float v[8];
#pragma unroll
                for (int x = 0; x < 8; ++x) v[x] = r0 + 4 * x < a.rs ? src[(r0 + 4 * x) * split_stride] : 0.f;
#pragma unroll
                for (int x = 0; x < 8; ++x) tot += v[x];
            }
        }
        if (g0) __syncthreads();
        part[ps][hs][col] = tot;
        __syncthreads();
        if (ps == 0 && g < a.Hkv) {
            const float s = ((part[0][hs][col] + part[1][hs][col]) + (part[2][hs][col] + part[3][hs][col])) * inv_g;
            if (j < a.n_img) a.score_head[(long long)b * a.shb + (long long)g * a.shh + j] = s;
            mean += s;
        }
    }
    if (ps == 0) mean_s[hs][col] = mean;
    __syncthreads();
    if (threadIdx.x < 64 && j < a.n_img)
        a.score_mean[(long long)b * a.n_img + j] = ((mean_s[0][col] + mean_s[1][col]) + (mean_s[2][col] + mean_s[3][col])) / (float)a.Hkv;
}

// The same where a thread per column already fills the chip: no exchange, a workgroup reads 1 KB runs, four heads x eight
// parts of a thread's loads in flight.
__global__ __launch_bounds__(256) void score_finalize_wide_kernel(ScoreArgs a) {
    constexpr int PARTS = 8;
    const int j = blockIdx.x * 256 + threadIdx.x;
    const int b = blockIdx.y;
    if (j >= a.n_img) return;
    const float inv_g = 1.0f / (float)a.G;
    const long long split_stride = (long long)a.B * a.Hkv * a.n_img;
    float mean = 0.f;
    for (int g0 = 0; g0 < a.Hkv; g0 += 4) {
        float tot[4] = {0.f, 0.f, 0.f, 0.f};
        for (int r0 = 0; r0 < a.rs; r0 += PARTS) {
            float v[4][PARTS];
#pragma unroll
            for (int gg = 0; gg < 4; ++gg)
#pragma unroll
                for (int r = 0; r < PARTS; ++r) {
                    const bool on = g0 + gg < a.Hkv && r0 + r < a.rs;
                    const int gc = min(g0 + gg, a.Hkv - 1), rc = min(r0 + r, a.rs - 1);
                    const float x = a.colpart[rc * split_stride + ((long long)b * a.Hkv + gc) * a.n_img + j];
                    v[gg][r] = on ? x : 0.f;
                }
#pragma unroll
            for (int gg = 0; gg < 4; ++gg) {
                float s = 0.f;
#pragma unroll
                for (int r = 0; r < PARTS; ++r) s += v[gg][r];
                tot[gg] += s;
            }
        }
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
            if (g0 + gg >= a.Hkv) break;
            float s = tot[gg];
            s *= inv_g;
            a.score_head[(long long)b * a.shb + (long long)(g0 + gg) * a.shh + j] = s;
            mean += s;
        }
    }
    a.score_mean[(long long)b * a.n_img + j] = mean / (float)a.Hkv;
}

// Which of the two, by what each thread of the wide form has to do in turn: a round of loads for every four heads and
// eight parts.  From three rounds on, with more parts than one round holds, the shorter chains of the 1024-thread form win;
// below that three quarters of its threads find no part and its two barriers per four heads are a loss (the whole
// call, 1024-thread form against wide, up to 256 workgroups of the former: 4 heads 1-3 parts +0.2 to +0.5 us, 4-8 parts
// +0.5 to +0.8, 12-16 +0.1, 24 -0.5, 48 -1.9 us; 8 heads 1-2 parts +0.1, 4-8 +0.5, 12 -0.7, 24 -1.7, 48 -4.5 us).
// And up to one turn of the chip, two such workgroups a compute unit (8 heads of 12 parts at 257-512 workgroups: even); a second
// turn costs more than the shorter chains give: 12 sequences x 5091 columns x 8 heads of 24 parts (47 MB, 960
// workgroups) 13.6 us against 10.8 us.
void launch_finalize(const Prof &prof, const ScoreArgs &a) {
    const dim3 grid((a.n_img + 63) / 64, a.B);
    const int rounds = ((a.Hkv + 3) / 4) * ((a.rs + 7) / 8);
    prof.begin("score_finalize");
    if (a.rs > 8 && rounds > 2 && (long long)grid.x * grid.y <= 512)
        LVLM_LAUNCH(prof, score_finalize_kernel, grid, dim3(1024), 0, prof.stream, a);
    else LVLM_LAUNCH(prof, score_finalize_wide_kernel, dim3((a.n_img + 255) / 256, a.B), dim3(256), 0, prof.stream, a);
    prof.end();
}

// ---- scores from probabilities the caller already holds ---------------------------------------------
// Workgroup (column block, row group c): thread (sub, cj) sums the 16 / ES columns of word cj of
// probs[b][g*G + hl][i][img_begin ..] over rows 8 sub .. of the group's 32 rows rho = hl*T + i, all of its loads in flight; the four
// row subsets are folded through LDS, the groups' sums go through the same finalize kernel as the column sums of the passes.
struct ProbsArgs {
    const char *p;
    float *colpart;
    int B, T, Hkv, G, img_begin, n_img;
    unsigned t_magic;
    long long psb, psh, pst;
};

// Bound by HBM.  Rows of odd lengths start anywhere: a word is then loaded from an address aligned to an element only (the memory
// pipeline takes it whole, a wave touches nine lines for eight), and the last word of a row ends with the row (element by element, where
// it would be partial, its loads went one after the other: 11 x 4 x 10 rows of 349 columns 5.8 -> 8.9 us).  Waves without a row of a
// last, partial group load nothing (the last row again and again: 14 x 32 rows of 37 columns 5.5 -> 6.5).
// Against one element per thread and load: 4 x 28 x 150 rows of 9000 of 9150 columns 178 -> 69 us for the call (4.4 TB/s), 4 x 48 x 130
// of 15000 of 15194 416 -> 160.
// ONCE: loads past the caches, for a matrix that clearly outgrows the 256 MB cache in front of the memory.  Kernel, repeated at once
// and on a matrix just written: 240 MB 39 -> 46 and 39 -> 39 us, 264 MB 46 -> 51 and 48 -> 44, 288 MB 58 -> 55 and 78 -> 48 (rows of
// odd lengths 53 -> 61 and 71 -> 70), 336 MB 70 -> 63 and 101 -> 56.
template <int DT, bool ALIGNED, bool ONCE>
__global__ __launch_bounds__(256) void probs_colsum_kernel(ProbsArgs a, int n_col_blocks) {
    constexpr int ES = esize<DT>();
    constexpr int CPT = 16 / ES;              // columns per thread
    constexpr int WC = 64 * CPT;              // columns per workgroup
    __shared__ float part[4][WC];
    const int cb = blockIdx.x % n_col_blocks, c = blockIdx.x / n_col_blocks;
    const int g = blockIdx.y, b = blockIdx.z;
    const int sub = threadIdx.x >> 6, cj = threadIdx.x & 63;
    const int j0 = cb * WC + cj * CPT;
    const int GT = a.G * a.T;
    const int r0 = c * 32 + 8 * sub, r1 = min(GT, r0 + 8);
    float acc[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) acc[e] = 0.f;
    // a row's last word, where it would be partial, begins `early` columns early
    const int early = ALIGNED || j0 >= a.n_img || a.n_img < CPT ? 0 : max(0, j0 + CPT - a.n_img);
    if (j0 < a.n_img && r0 < r1) {
        const char *base = a.p + ((long long)b * a.psb + (long long)g * a.G * a.psh + a.img_begin + j0 - early) * ES;
        uint4 v[8];
        auto row_at = [&](int u) {
            const int rho = min(r0 + u, GT - 1);
            const int hl = a.T == 1 ? rho : (int)__umulhi((unsigned)rho, a.t_magic), i = rho - hl * a.T;
            return base + ((long long)hl * a.psh + (long long)i * a.pst) * ES;
        };
        if (ALIGNED || a.n_img >= CPT) {
            typedef unsigned word16 __attribute__((ext_vector_type(4)));
            typedef unsigned word2 __attribute__((ext_vector_type(4), aligned(2)));
            using word = std::conditional_t<ALIGNED, word16, word2>;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const word *at = reinterpret_cast<const word *>(row_at(u));
                v[u] = __builtin_bit_cast(uint4, ONCE ? __builtin_nontemporal_load(at) : *at);
            }
        } else {                              // fewer columns than a word has (what the others repeat is not used)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const char *at = row_at(u);
                uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < CPT - 1; ++e) {
                    const int x = min(e, a.n_img - 1);
                    if constexpr (DT == LVLM_BF16) w[e >> 1] |= (uint32_t)reinterpret_cast<const uint16_t *>(at)[x] << (16 * (e & 1));
                    else w[e] = reinterpret_cast<const uint32_t *>(at)[x];
                }
                v[u] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (r0 + u >= r1) continue;
            const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (DT == LVLM_BF16) {
                    acc[2 * q] += __uint_as_float(w[q] << 16);
                    acc[2 * q + 1] += __uint_as_float(w[q] & 0xffff0000u);
                } else {
                    acc[q] += __uint_as_float(w[q]);
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < CPT; ++e)
        if (ALIGNED || e >= early) part[sub][cj * CPT + e - early] = acc[e];
    __syncthreads();
    for (int x = threadIdx.x; x < WC; x += 256) {
        const int j = cb * WC + x;
        if (j < a.n_img)
            a.colpart[(((long long)c * a.B + b) * a.Hkv + g) * a.n_img + j] =
                (part[0][x] + part[1][x]) + (part[2][x] + part[3][x]);
    }
}

template <int HD, int NW>
void launch_shares(const Prof &prof, const ScoreArgs &a, bool need_lse) {
    const int wpp = ((a.G * a.T + 31) / 32 + 2 * NW - 1) / (2 * NW);
    auto grid = [&](const KeyRuns &r) { return dim3((r.shares + 7) / 8 * 8 * wpp); };
    if (need_lse) {
        prof.begin("score_single");
        LVLM_LAUNCH(prof, (score_shares_kernel<HD, false, NW>), grid(a.runs1), dim3(64 * NW), 0, prof.stream, a);
        prof.end();
    }
    prof.begin("score_single");
    LVLM_LAUNCH(prof, (score_shares_kernel<HD, true, NW>), grid(a.runs2), dim3(64 * NW), 0, prof.stream, a);
    prof.end();
    launch_finalize(prof, a);
}

template <int DT, int HD, int KPW>
void launch_passes(const Prof &prof, const ScoreArgs &a, bool need_lse, bool single, bool shared_tiles, int rows, int share_waves) {
    hipStream_t stream = prof.stream;
    if constexpr (DT == LVLM_BF16) {
        if (share_waves) {
            ScoreArgs r = a;
            r.rs = ((a.G * a.T + 31) / 32 + 1) / 2;       // parts: one per wave
            if (share_waves == 4) launch_shares<HD, 4>(prof, r, need_lse);
            else launch_shares<HD, 2>(prof, r, need_lse);
            return;
        }
    }
    constexpr int BN = 4 * KPW * 32;
    constexpr bool can_rows = !(DT == LVLM_F32 && HD == 128);
    if (rows && can_rows) {
        const int n_t = ((need_lse ? a.N : a.n_img) + 16 * kRowsWaves - 1) / (16 * kRowsWaves);      // tiles per wave
        ScoreArgs r = a;
        r.rs = rows;
        const dim3 grid((a.B * a.Hkv * rows + 7) / 8 * 8), wg(64 * kRowsWaves);
        prof.begin("score_single");
        if constexpr (can_rows) {
            if (n_t <= 4) LVLM_LAUNCH(prof, (score_rows_kernel<DT, HD, 4>), grid, wg, 0, stream, r);
            else if (n_t <= 8) LVLM_LAUNCH(prof, (score_rows_kernel<DT, HD, 8>), grid, wg, 0, stream, r);
            else if (n_t <= 16) LVLM_LAUNCH(prof, (score_rows_kernel<DT, HD, 16>), grid, wg, 0, stream, r);
            else if (n_t <= 24) LVLM_LAUNCH(prof, (score_rows_kernel<DT, HD, 24>), grid, wg, 0, stream, r);
            else LVLM_LAUNCH(prof, (score_rows_kernel<DT, HD, 32>), grid, wg, 0, stream, r);
        }
        prof.end();
        launch_finalize(prof, r);
        return;
    }
    if (single) {
        prof.begin("score_single");
        if (shared_tiles && a.n_seg > 1) {
            // the keys in runs: the normaliser sweep, the fold of the runs' partials, then the column-sum sweep
            const dim3 grid((a.B * a.Hkv + 7) / 8 * 8 * ((a.rs + 3) / 4) * a.n_seg);
            if (need_lse) {
                LVLM_LAUNCH(prof, (score_chunks_kernel<DT, HD, 1>), grid, dim3(256), 0, stream, a);
                prof.end();
                const int rows = a.B * a.Hq * a.T;
                prof.begin("score_lse");
                LVLM_LAUNCH(prof, score_lse_kernel, dim3((rows * 8 + 255) / 256), dim3(256), 0, stream, a.part_m, a.part_l,
                                   a.lse2, rows, a.n_seg);
                prof.end();
                prof.begin("score_single");
            }
            LVLM_LAUNCH(prof, (score_chunks_kernel<DT, HD, 2>), grid, dim3(256), 0, stream, a);
        } else if (shared_tiles)
            LVLM_LAUNCH(prof, (score_chunks_kernel<DT, HD, 0>), dim3((a.B * a.Hkv + 7) / 8 * 8 * ((a.rs + 3) / 4)), dim3(256), 0,
                               stream, a);
        else
            LVLM_LAUNCH(prof, (score_small_kernel<DT, HD, 4>), dim3((a.B * a.Hkv + 7) / 8 * 8 * a.rs), dim3(256), 0, stream,
                               a);
        prof.end();
        launch_finalize(prof, a);
        return;
    }
    if (need_lse) {
        dim3 grid0(((a.N + BN - 1) / BN + 7) / 8 * 8 * a.rs, a.Hkv, a.B);
        prof.begin("score_pass0");
        LVLM_LAUNCH(prof, (score_pass_kernel<DT, HD, KPW, 0>), grid0, dim3(256), 0, stream, a);
        prof.end();
        const int rows = a.B * a.Hq * a.T;
        prof.begin("score_lse");
        LVLM_LAUNCH(prof, score_lse_kernel, dim3((rows * 8 + 255) / 256), dim3(256), 0, stream, a.part_m, a.part_l,
                           a.lse2, rows, a.nkb * 4);
        prof.end();
    }
    dim3 grid1(((a.n_img + BN - 1) / BN + 7) / 8 * 8 * a.rs, a.Hkv, a.B);
    prof.begin("score_pass1");
    LVLM_LAUNCH(prof, (score_pass_kernel<DT, HD, KPW, 1>), grid1, dim3(256), 0, stream, a);
    prof.end();
    launch_finalize(prof, a);
}

}  // namespace

constexpr int kRowSplitWgs = 1536;      // workgroups the two-pass kernels aim for
constexpr int kSingleMaxChunks = 32;
constexpr int kSharedMinWgs = 192;       // workgroups of four chunks from which the shared-tile form is taken
constexpr int kSingleMaxRows = 1100;      // in 256-byte key rows, one chunk per workgroup
constexpr int kSharedMaxRows = 8192;      // ... four chunks per workgroup sharing the key tiles

ProbsWs probs_ws(const lvlm_probs_desc &d) {
    ProbsWs w{};
    w.rs = (d.Hq / d.Hkv * d.T + 31) / 32;
    w.colpart = 0;
    w.total = align_up((size_t)w.rs * d.B * d.Hkv * d.n_img * sizeof(float), 256);
    return w;
}

hipError_t launch_score_probs(const Prof &prof, const lvlm_probs_desc &d, const ProbsWs &w, char *ws, const void *probs,
                              float *score_head, float *score_mean) {
    ProbsArgs pa{};
    pa.p = static_cast<const char *>(probs);
    pa.colpart = reinterpret_cast<float *>(ws + w.colpart);
    pa.B = d.B; pa.T = d.T; pa.Hkv = d.Hkv; pa.G = d.Hq / d.Hkv; pa.img_begin = d.img_begin; pa.n_img = d.n_img;
    pa.t_magic = (unsigned)(0x100000000ull / (unsigned long long)d.T) + 1u;
    pa.psb = d.p_stride_b; pa.psh = d.p_stride_h; pa.pst = d.p_stride_t;
    const int es = d.dtype == LVLM_BF16 ? 2 : 4, cpt = 16 / es;
    const bool aligned = (d.p_stride_b * es) % 16 == 0 && (d.p_stride_h * es) % 16 == 0 && (d.p_stride_t * es) % 16 == 0 &&
                         (d.img_begin * es) % 16 == 0 && d.n_img % cpt == 0;      // the base pointer is 16-byte aligned
    // (the line lies where both kinds of rows gain: probs_colsum_kernel)
    const bool once = (long long)d.B * d.Hq * d.T * d.n_img * es > (320ll << 20);
    const int ncb = (d.n_img + 64 * cpt - 1) / (64 * cpt);
    const dim3 grid(ncb * w.rs, d.Hkv, d.B);
    prof.begin("score_probs");
#define LVLM_PROBS(DT, ALIGNED, ONCE) \
    LVLM_LAUNCH(prof, (probs_colsum_kernel<DT, ALIGNED, ONCE>), grid, dim3(256), 0, prof.stream, pa, ncb)
#define LVLM_PROBS_OF(DT)                              \
    if (aligned && once) LVLM_PROBS(DT, true, true);   \
    else if (aligned) LVLM_PROBS(DT, true, false);     \
    else if (once) LVLM_PROBS(DT, false, true);        \
    else LVLM_PROBS(DT, false, false)
    if (d.dtype == LVLM_BF16) { LVLM_PROBS_OF(LVLM_BF16); }
    else { LVLM_PROBS_OF(LVLM_F32); }
#undef LVLM_PROBS_OF
#undef LVLM_PROBS
    prof.end();
    ScoreArgs a{};
    a.colpart = pa.colpart;
    a.rs = w.rs;
    a.score_head = score_head;
    a.score_mean = score_mean;
    a.B = d.B; a.Hkv = d.Hkv; a.G = pa.G; a.n_img = d.n_img;
    const bool dense = d.sh_stride_b == 0 && d.sh_stride_h == 0;
    a.shh = dense ? d.n_img : d.sh_stride_h;
    a.shb = dense ? (long long)d.Hkv * d.n_img : d.sh_stride_b;
    launch_finalize(prof, a);
    return hipGetLastError();
}

// Few query rows (score_rows_kernel): 16 of them per workgroup, the logits over all keys in registers.  Returns the chunks of
// a KV head, or 0 where the form chosen without it (`w`) is the faster one.  Its time is one chain: start-up, the keys
// at 1.6 us per 1000 of 128 bytes and 3.4 us of 256 bytes in bf16, 6 us in fp32, and a fold of one part per chunk; the other forms
// read the keys twice but share the work over more workgroups.  The lines below are from 800 shapes timed both ways (1 to 768
// workgroups, 1 to 130 chunks a head, 65 to 4096 keys, heads of 64 and 128 channels): the rule is 0.4 % from the faster
// form on average and no shape taken loses more than 5 % (other form -> this one in what follows).
static int few_rows(const lvlm_score_desc &d, const ScoreWs &w, int n_chunks, bool given) {
    const bool bf16 = d.dtype == LVLM_BF16;
    const int row_bytes = d.hd * (bf16 ? 2 : 4);
    const long long heads = (long long)d.B * d.Hkv;
    const int n16 = (d.Hq / d.Hkv * d.T + 15) / 16;
    const long long wgs = heads * n16;
    if (w.shared_tiles || (!bf16 && d.hd == 128) || d.N > 16 * kRowsWaves * 32 || !(d.scale > 0.f) ||
        d.k_stride_n * (bf16 ? 2 : 4) >= (1ll << 26))
        return 0;
    if (w.single) {
        // Against one chunk of 32 rows per workgroup: one turn of the chip, and in bf16 keys enough to pay for eight waves and twice
        // the parts, 27 KB of them (3 heads of 13 chunks, 64 channels, 6.9 -> 7.7 us at 187 keys; 28 heads x 64 rows 15.0 -> 11.1
        // at 700).  fp32 always (8 heads of one row 9.2 -> 8.6 us at 86 keys).  With the normalisers given the other form reads
        // the image keys once as well: 82 KB of them, 33 KB in fp32 (12 heads of 12 chunks, 64 channels, 7.0 -> 7.9 us at 202 keys, 8
        // heads x 96 rows, 128 channels, 12.0 -> 10.0 at 931; fp32 8 heads x 32 rows 13.9 -> 11.7 at 611).
        if (wgs > 256) return 0;
        if (given) return (long long)d.n_img * row_bytes > 256 * (bf16 ? 320 : 130) ? n16 : 0;
        return !bf16 || (long long)d.N * row_bytes > 256 * 105 ? n16 : 0;
    }
    // Against the two-pass kernels, whose three launches and fold cost 15 us whatever the shape and then split the keys over the
    // chip; with the normalisers given they are a single short pass.
    if (given || wgs > 768) return 0;
    // one query row per KV head: they take 28 us and more for 4000 keys
    if (d.T == 1 && n_chunks == 1) return n16;
    // the chain of a few workgroups over long sequences (2 heads of 4 chunks, 128 channels, 17.5 -> 18.4 us at 3980 keys, 23 heads of
    // one 39 -> 27; fp32 one head 17.4 -> 22.8 us at 2709 keys, 14 chunks of 6 heads 31.8 -> 26.0 at 2936)
    if (bf16) return d.hd == 64 || d.N <= 3500 || wgs >= 16 ? n16 : 0;
    return d.N <= 2050 || heads >= 8 || wgs >= 64 ? n16 : 0;
}

// Equal shares of the keys (score_shares_kernel): for bf16 calls of much work, whose two launches and start-up (some 25 us;
// 11 with the normalisers given) are then worth it.  Work: products of 32 rows and 32 keys, in 1024 SIMDs' turns; between 250 and
// 320 turns the other forms are 1 % ahead, at 100 twenty (88 us 1.0, 55 us 1.2 times).  Under 3072 keys many pairs to a share, each
// with a start-up of its own, cost what the rest gives (52 sequences x 2939 keys 652 -> 683 us, 86 x 443 86 -> 106).  The span has
// to be visible to every row: the masked path is slow.
// Beyond these lines, of 238 random shapes timed both ways (2 to 472 pairs of 3 to 32 chunks of 64 and 128 channels) those taken
// are 5 % faster on average with a normaliser sweep -- 9 % by workgroups of eight chunks, none slower; 4 % by workgroups of four,
// whose ring of two slots hides less, from 22 % faster to 7 % slower, nine of 112 by more than 2 % -- and 11 % with the normalisers
// given (4 % slower at worst).  Not taken, with a normaliser sweep: pairs of five or seven workgroups of four chunks with more
// than one chunk's place empty (17, 18, 25, 26 chunks), of which 72 were 1 % slower on average and up to 12 % (10 sequences x 4193
// keys x 64 heads of 64 channels, 17 chunks, 101 -> 114 us; 16 x 6719 x 64 of 128, 26 chunks, 458 -> 493).
static ScoreShares score_shares(const lvlm_score_desc &d, int n_chunks, bool given) {
    ScoreShares s{};
    const long long pairs = (long long)d.B * d.Hkv;
    const long long tiles = (given ? 0 : (d.N + 31) / 32) + (d.n_img + 31) / 32;
    if (d.dtype != LVLM_BF16 || n_chunks < 3 || n_chunks > 32 || d.n_img < (given ? 2048 : 3072) || d.k_stride_n * 2 >= (1ll << 25) ||
        (d.causal && d.q_pos0 < d.img_begin + d.n_img - 1) || pairs * n_chunks * tiles < 1024ll * (given ? 130 : 320) ||
        pairs * ((d.N + kShareStep - 1) / kShareStep) >= (1ll << 30))
        return s;
    // workgroups of eight chunks, which read the keys half as often, unless ones of four leave fewer places empty
    s.waves = (n_chunks + 7) / 8 * 8 == (n_chunks + 3) / 4 * 4 ? 4 : 2;
    const int wpp = (n_chunks + 2 * s.waves - 1) / (2 * s.waves);
    if (!given && wpp > 4 && 2 * s.waves * wpp - n_chunks > 1) return ScoreShares{};
    auto deal = [&](int keys) {
        KeyRuns r{};
        r.steps = (keys + kShareStep - 1) / kShareStep;
        const int total = (int)pairs * r.steps;
        r.shares = std::min(2048 / s.waves / wpp / 8 * 8, (total + 3) / 4);      // two waves per SIMD, none of under three steps
        r.size = total / r.shares;
        r.longer = total % r.shares;
        return r;
    };
    s.runs1 = deal(d.N);
    s.runs2 = deal(d.n_img);
    return s;
}

ScoreWs score_ws(const lvlm_score_desc &d) {
    ScoreWs w{};
    // Wide key blocks (2 tiles per wave) once they still give every CU two workgroups.
    const long long wide = (long long)d.B * d.Hkv * ((d.N + 255) / 256);
    w.block_keys = (d.dtype == LVLM_BF16 && wide >= 512) ? 256 : 128;
    w.nkb = (d.N + w.block_keys - 1) / w.block_keys;
    // Few workgroups: split the query chunks of a key block over several workgroups (>= 2 chunks each), up to six
    // workgroups per compute unit (measured on 16512 keys of one sequence: 110 us for both passes with 520
    // workgroups, 98 us with 1560).
    const int n_chunks = (d.Hq / d.Hkv * d.T + 31) / 32;
    const long long wgs = (long long)d.B * d.Hkv * w.nkb;
    int rs = (int)((kRowSplitWgs + wgs - 1) / wgs);
    if (rs > (n_chunks + 1) / 2) rs = (n_chunks + 1) / 2;
    if (rs > 8) rs = 8;            // (parts the finalize kernel has to add up)
    if (rs < 1) rs = 1;
    w.cps = (n_chunks + rs - 1) / rs;
    w.rs = (n_chunks + w.cps - 1) / w.cps;
    // Short sequences: both passes in ONE launch (the column sums then come in one part per chunk).  Two
    // shapes: four chunks per workgroup that share the key tiles through LDS, when that still fills the
    // chip -- measured faster than the two-pass kernels up to several thousand keys (it saves the partials,
    // their fold and a launch) -- else one chunk per workgroup whose waves split the keys and fetch them
    // themselves, which pays up to the length where the three launches it replaces cost the same.
    const long long sweep_rows = (long long)d.N * (d.hd * (d.dtype == LVLM_BF16 ? 2 : 4)) / 256;
    w.shared_tiles = n_chunks >= 3 && n_chunks <= kSingleMaxChunks && (long long)d.B * d.Hkv * ((n_chunks + 3) / 4) >= kSharedMinWgs &&
                     sweep_rows <= kSharedMaxRows;
    w.single = w.shared_tiles || (n_chunks <= kSingleMaxChunks && sweep_rows <= kSingleMaxRows);
    // The shared-tile kernel with the keys in runs.  A wave's unit of work is a chunk over ALL keys, twice: a launch of
    // 2.25 workgroups per compute unit takes the time of three, one of 0.75 the time of one whose lone wave per SIMD hides
    // nothing, and one long sequence has too few workgroups for the form at all.  Cutting the keys into runs (a launch
    // per sweep, a workgroup per four chunks and run, the runs' normaliser partials folded in between) makes the units
    // small and many; it costs each workgroup its start-up (about three tiles' time) per run and the call two more
    // launches.  Taken when the estimate below says it saves more than 12 us over the form chosen so far.
    w.key_segs = 1;
    if (n_chunks >= 3 && n_chunks <= kSingleMaxChunks && (w.shared_tiles || !w.single)) {
        const long long wgs = (long long)d.B * d.Hkv * ((n_chunks + 3) / 4);
        const double tiles = (d.N + 31) / 32 + (d.n_img + 31) / 32;          // both sweeps
        // (measured, in us per tile sweep of a workgroup, with k = 1..5 workgroups resident on every compute unit: a lone
        // wave per SIMD hides nothing, from three on the SIMDs are saturated; five are resident at most, a launch of more
        // runs in turns of 1280 workgroups plus the rest)
        auto launch_us = [](long long n_wg, double tiles_per_wg) {
            static const double per_tile[6] = {0.0, 0.53, 0.73, 0.95, 1.25, 1.5};
            const long long turns = n_wg / 1280, rest = n_wg % 1280;
            return tiles_per_wg * (1.5 * (double)turns + per_tile[(rest + 255) / 256]);
        };
        // the form chosen so far: one launch of this kernel, or the two-pass kernels (0.53 PFLOP/s measured on one
        // sequence of 16512 keys: 0.002 us per workgroup-tile of this kernel's size) with their fold
        const double so_far = w.shared_tiles ? launch_us(wgs, tiles) : 0.002 * (double)wgs * tiles + 12.0;
        double best = so_far - 12.0;
        for (int s = 2; s <= 32 && (wgs <= 1280 || !w.shared_tiles); s *= 2) {
            if (tiles / 2 / s < 12) break;                                    // runs of at least 12 tiles
            if (wgs * s < kSharedMinWgs || sweep_rows / s > kSharedMaxRows) continue;
            const double cut = launch_us(wgs * s, tiles / s + 2 * 3) + 10.0;
            if (cut < best) best = cut, w.key_segs = s;
        }
        if (w.key_segs > 1) w.shared_tiles = w.single = true;
    }
    if (w.single) {
        w.rs = n_chunks;
        w.cps = 1;
    }
    w.rows = few_rows(d, w, n_chunks, false);
    w.rows_given = few_rows(d, w, n_chunks, true);
    w.shares = score_shares(d, n_chunks, false);
    w.shares_given = score_shares(d, n_chunks, true);
    const size_t rows = (size_t)d.B * d.Hq * d.T;
    w.part_m = 0;
    const size_t n_part = std::max((size_t)w.nkb * 4, (size_t)w.key_segs), n_col = (size_t)std::max(w.rs, std::max(w.rows, w.rows_given));
    // Equal shares have to do with the scratch of the forms they replace, so that a workspace which held a call still does: a few
    // shapes of some 100000 keys, whose query chunks the two passes split over fewer workgroups than the shares leave parts, are not
    // worth up to 1.44 times the bytes.
    const size_t share_parts = (size_t)(n_chunks + 1) / 2;      // of column sums
    if (share_parts > n_col || (w.shares.waves && (size_t)((w.shares.runs1.steps - 1) / w.shares.runs1.size + 2) > n_part))
        w.shares = ScoreShares{};
    if (share_parts > n_col) w.shares_given = ScoreShares{};
    w.part_l = align_up(w.part_m + rows * n_part * sizeof(float), 256);
    w.lse2 = align_up(w.part_l + rows * n_part * sizeof(float), 256);
    w.colpart = align_up(w.lse2 + rows * sizeof(float), 256);
    w.total = align_up(w.colpart + n_col * d.B * d.Hkv * d.n_img * sizeof(float), 256);
    return w;
}

hipError_t launch_score(const Prof &prof, const lvlm_score_desc &d, const ScoreWs &w, char *ws, const void *q,
                        const void *k, const float *row_lse, float *score_head, float *score_mean) {
    ScoreArgs a{};
    a.q = static_cast<const char *>(q);
    a.k = static_cast<const char *>(k);
    a.row_lse = row_lse;
    a.part_m = reinterpret_cast<float *>(ws + w.part_m);
    a.part_l = reinterpret_cast<float *>(ws + w.part_l);
    a.lse2 = reinterpret_cast<float *>(ws + w.lse2);
    a.colpart = reinterpret_cast<float *>(ws + w.colpart);
    a.rs = w.rs;
    a.cps = w.cps;
    a.n_seg = w.key_segs;
    a.t_magic = (unsigned)(0x100000000ull / (unsigned long long)d.T) + 1u;
    a.score_head = score_head;
    a.score_mean = score_mean;
    a.B = d.B; a.N = d.N; a.T = d.T; a.q_pos0 = first_row_position(d); a.Hq = d.Hq; a.Hkv = d.Hkv; a.G = d.Hq / d.Hkv;
    a.img_begin = d.img_begin; a.n_img = d.n_img; a.causal = d.causal; a.nkb = w.nkb;
    a.scale_log2 = d.scale * kLog2e;
    a.qsb = d.q_stride_b; a.qst = d.q_stride_t; a.qsh = d.q_stride_h;
    a.ksb = d.k_stride_b; a.ksn = d.k_stride_n; a.ksh = d.k_stride_h;
    const bool dense = d.sh_stride_b == 0 && d.sh_stride_h == 0;
    a.shh = dense ? d.n_img : d.sh_stride_h;
    a.shb = dense ? (long long)d.Hkv * d.n_img : d.sh_stride_b;
    const bool need_lse = row_lse == nullptr;
    const bool wide = w.block_keys == 256;
    const int rows = need_lse ? w.rows : w.rows_given;
    const ScoreShares &sh = need_lse ? w.shares : w.shares_given;
    const int share_waves = sh.waves;
    a.runs1 = sh.runs1;
    a.runs2 = sh.runs2;
    if (d.dtype == LVLM_BF16 && d.hd == 128) {
        if (wide) launch_passes<LVLM_BF16, 128, 2>(prof, a, need_lse, w.single, w.shared_tiles, rows, share_waves);
        else launch_passes<LVLM_BF16, 128, 1>(prof, a, need_lse, w.single, w.shared_tiles, rows, share_waves);
    } else if (d.dtype == LVLM_BF16 && d.hd == 64) {
        if (wide) launch_passes<LVLM_BF16, 64, 2>(prof, a, need_lse, w.single, w.shared_tiles, rows, share_waves);
        else launch_passes<LVLM_BF16, 64, 1>(prof, a, need_lse, w.single, w.shared_tiles, rows, share_waves);
    } else if (d.dtype == LVLM_F32 && d.hd == 128) {
        launch_passes<LVLM_F32, 128, 1>(prof, a, need_lse, w.single, w.shared_tiles, rows, share_waves);
    } else {
        launch_passes<LVLM_F32, 64, 1>(prof, a, need_lse, w.single, w.shared_tiles, rows, share_waves);
    }
    return hipGetLastError();
}

}  // namespace lvlm
