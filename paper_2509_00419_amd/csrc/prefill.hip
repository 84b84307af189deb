// The layer's own prefill attention, leaving the row normalisers the token scores are computed from
// (Sec. 3.2.1: the scores are a by-product of the attention of the layer; Sec. 3.2.2: of its statistics).
//
// out[b,i,h,:] = sum_j softmax_j(scale q[b,i,h].k[b,j,g]) v[b,j,g,:], g = h / G, over the keys row i may
// see; row_lse[b,h,i] = natural-log sum-exp of the row's scaled logits.  The last T rows' normalisers are
// also left densely packed for the column-sum pass of the score kernels, which then needs no normaliser
// pass of its own.
#include "mma.h"
#include "prefill_rules.h"

#include <climits>
#include <type_traits>

namespace lvlm {
namespace {

struct PrefillArgs {
    const char *q, *k, *v;
    char *out;
    float *row_lse;     // [B][Hq][N]
    float *lse_t;       // [B][Hq][T] or null: the last T rows again
    int B, N, Hq, Hkv, G, causal, T;
    int nqb;            // query blocks per head
    int heads_per_xcd;  // ceil(B * Hq / 8)
    BlockDeal deal;
    float scale, scale_log2;
    long long qsb, qsn, qsh, ksb, ksn, ksh, vsb, vsn, vsh, osb, osn, osh;   // bytes
};

constexpr float kLazy = 8.f;    // SAFE sweep: log2 of how far the row maximum may run ahead of the reference before a rescale
constexpr float kRisk = 64.f;   // FAST sweep: ... before the workgroup takes the SAFE sweep

// max of a value and the one held by the lane 32 places away (the other half-wave): one lane-swap instruction
// instead of a trip through the LDS permute unit.  The swap exchanges lanes 32..63 of its first operand with
// lanes 0..31 of its second; with the same value in both, every lane ends up with the two halves' values.
__device__ __forceinline__ float half_max(float x) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const bf2 r = __builtin_convertvector(f2{lo, hi}, bf2);
    return __builtin_bit_cast(uint32_t, r);
}

// bf16, matrix cores.  A workgroup of two waves owns 128 query rows of one head, 64 per wave as two 32-row
// blocks held in registers as MFMA operands.  Keys and values go by in tiles of 32, K into LDS as it is (rows = keys),
// V turned around (rows = channels, 32 keys each) in registers on the way in; one barrier per tile.  Per tile and block:
// S^T = K Q^T (rows = keys, columns = queries), so a lane owns ONE query row and 16 of its logits -- the
// max and sum are lane-local but for one exchange with the other half-wave -- and the 16
// probabilities, rounded to bf16, are already laid out as the second operand of O^T += V^T P^T when the
// keys inside V^T's rows are stored in the order the accumulator registers hold them.  Both blocks of a wave
// use each K and V^T fragment read from LDS.
//
// There are two sweeps.  The FAST one fixes each row's reference maximum at the first tile (every row sees
// key 0 there) and never rescales: probabilities are exp2 of the distance to that reference, possibly far
// above 1, which fp32 sums and bf16 operands carry at unchanged relative precision.
// Should a logit rise more than 2^kRisk above its row's reference, the wave writes nothing and the workgroup does its
// block again in the SAFE sweep, the textbook online softmax, whose reference follows the running maximum (lazily, in
// steps of 2^kLazy) and rescales sums and accumulators when it moves.  Both are in one kernel, one behind the other in the
// same LDS: as a second kernel that looked through the marks of the first the SAFE sweep cost every call a launch (4 x 95 tokens,
// 40 heads 18.6 -> 16.5 us, 542 tokens 32.2 -> 30.1).

// Workgroup number -> (batch, head, query block); false: padding.  Numbers with the same remainder modulo 8 run on one
// XCD.  The B * Hq heads, in memory order (heads of one KV head next to each other), are dealt to the 8 XCDs in
// contiguous runs of equal length (+-1): heads that read the same keys and values mostly share an L2, and
// every XCD gets the same load whatever the head counts.  Within an XCD the longest blocks (latest rows)
// come first.
struct PrefillBlock {
    int b, h, g, q0;
};
__device__ __forceinline__ bool prefill_block(const PrefillArgs &a, int id, PrefillBlock &w) {
    const int xcd = id & 7, seq = id >> 3;
    const int NH = a.B * a.Hq;
    const int qb = a.nqb - 1 - seq / a.heads_per_xcd;
    const int head_first = (xcd * NH + 7) >> 3, head_end = ((xcd + 1) * NH + 7) >> 3;
    const int bh = head_first + seq % a.heads_per_xcd;
    if (bh >= head_end) return false;
    w.b = bh / a.Hq;
    w.h = bh % a.Hq;
    w.g = w.h / a.G;
    w.q0 = qb * 128;
    return true;
}

// Position of key kk of a tile inside a V^T row: accumulator register r of half hf holds key
// 8 (r / 4) + 4 hf + r % 4 of a 32-key tile, and the second product wants the 8 keys of registers
// 8 t .. 8 t + 7 in one 16-byte word: word index 2 t + hf, inside it 4 (r / 4 % 2) + r % 4.  Four keys
// 4 vkg .. 4 vkg + 3 stay together: they go to byte 32 (vkg / 4) + 16 (vkg % 2) + 8 (vkg / 2 % 2).
__device__ __forceinline__ int vt_offset(int vkg) { return 32 * (vkg >> 2) + 16 * (vkg & 1) + 8 * ((vkg >> 1) & 1); }
constexpr int kVtPitch = 80;            // V^T row: 32 keys x 2 bytes + 16
// channels 2m (low halves of word c) and 2m + 1 (high halves) of a 16-byte unit, four keys (rows v0 .. v3) each
__device__ __forceinline__ void vt_store(char *vd, int m, uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3) {
    uint2 lo, hi;
    lo.x = __builtin_amdgcn_perm(v1, v0, 0x05040100u);
    lo.y = __builtin_amdgcn_perm(v3, v2, 0x05040100u);
    hi.x = __builtin_amdgcn_perm(v1, v0, 0x07060302u);
    hi.y = __builtin_amdgcn_perm(v3, v2, 0x07060302u);
    *reinterpret_cast<uint2 *>(vd + (2 * m) * kVtPitch) = lo;
    *reinterpret_cast<uint2 *>(vd + (2 * m + 1) * kVtPitch) = hi;
}

// Did some probability of the wave's rows go beyond 2^kRisk (or to inf / NaN)?  Otherwise the sums stay below 2^kRisk
// times the row length.
__device__ __forceinline__ bool risky_sums(float l0, float l1) {
    const float limit = __builtin_amdgcn_exp2f(kRisk) * 65536.f;
    return __builtin_amdgcn_ballot_w64(!(l0 < limit) || !(l1 < limit)) != 0ull;
}

// Normalises and writes the 32-row block at row0: lane (query l32, half hf) holds channels 32 cb + 8 (r / 4) + 4 hf + r % 4.
// Stored from there, a wave's 64 lanes would write 16 bytes each of 32 rows at a time; put together in LDS (32 rows of
// HD * 2 + 16 bytes at io, the wave's own), whole rows leave (7 x 115 tokens, 48 heads 23.5 -> 21.2 us; 4 x 979, 32 heads
// 77.6 -> 72.1; 8 x 1888, 32 heads 351 -> 345; one sequence of 16512, 48 heads the same).
template <int HD>
__device__ __forceinline__ void prefill_write(const PrefillArgs &a, const PrefillBlock &w, char *io, int row0, int lane, float m_run,
                                              float l_run, const f32x16 (&oacc)[HD / 32]) {
    constexpr int P = HD * 2 + 16, UPR = HD / 8, RPI = 64 / UPR;    // row pitch; 16-byte units per row, rows per store
    if (row0 >= a.N) return;                // (uniform)
    const int hf = lane >> 5, l32 = lane & 31;
    const float l_tot = l_run + other_half(l_run);
    const float inv = 1.f / l_tot;
    wave_sync();                            // the wave's block before has been read (said behind the reads, it sends their rows through scratch)
#pragma unroll
    for (int cb = 0; cb < HD / 32; ++cb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            uint2 u;
            u.x = pack_bf16(oacc[cb][4 * r4 + 0] * inv, oacc[cb][4 * r4 + 1] * inv);
            u.y = pack_bf16(oacc[cb][4 * r4 + 2] * inv, oacc[cb][4 * r4 + 3] * inv);
            *reinterpret_cast<uint2 *>(io + l32 * P + 64 * cb + 16 * r4 + 8 * hf) = u;
        }
    wave_sync();                            // the rows are read by other lanes than wrote them
    const int row = row0 + l32;
    if (hf == 0 && row < a.N) {
        const float lse = m_run * a.scale + __logf(l_tot);
        a.row_lse[((long long)w.b * a.Hq + w.h) * a.N + row] = lse;
        if (a.lse_t && row >= a.N - a.T) a.lse_t[((long long)w.b * a.Hq + w.h) * a.T + (row - (a.N - a.T))] = lse;
    }
    const int r0 = lane / UPR, unit = 16 * (lane % UPR);
    const char *src = io + r0 * P + unit;
    uint4 u[32 / RPI];
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) u[i] = *reinterpret_cast<const uint4 *>(src + i * RPI * P);
    char *dst = a.out + (long long)w.b * a.osb + (long long)(row0 + r0) * a.osn + (long long)w.h * a.osh + unit;
    const long long step = RPI * a.osn;
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i, dst += step)
        if (row0 + r0 + i * RPI < a.N) *reinterpret_cast<uint4 *>(dst) = u[i];
}

template <int HD, bool SAFE>
__device__ __forceinline__ bool prefill_plain_block(const PrefillArgs &a, const PrefillBlock &w, char *k_mem, char *v_mem);

// The FAST kernel.  The matrix pipe and the vector ALUs of a SIMD work side by side when a wave has independent
// instructions for both (measured: 16 products with 4 fused multiply-adds or 2 exponentials behind each take the time
// of the products alone), and one tile's products and softmax, which depend on each other, are about equally long.
// So the loop is pipelined over three tiles: iteration t multiplies S(t+1) = K(t+1) Q and O += V(t-1) P(t-1)
// while it turns S(t) into P(t).  It is cut into 32 slots of one product and one lane's work on one logit, the logit's
// scaling, exponential and sum each a slot apart so that no slot waits for its own results; a scheduling barrier behind
// each keeps the compiler from drawing the pieces apart again.  The LDS fragments of the second product are
// read during the first, those of the next tile's first product during the second.  Staging (a ring of two K and two
// V^T tiles; K(t+3) and V(t) go to LDS and the next ones are requested) goes with the first product, so that the barrier
// at the end finds the LDS queue drained.  One wave per SIMD: the 128 output accumulators, two tiles of logits, the query
// operands and the fragments take 437 registers.
// The masks around the diagonal and at the end of the sequence are one compare and select per logit, in a second copy
// of the iteration that only the last (up to four) tiles of a workgroup run through.
// Addresses are a uniform base plus 32-bit offsets per thread (the host checks that a tile's rows span less than 2 GiB).
// What bounds it: the power the chip allows (16512 tokens: 5.8 M cycles, the products 57 % of them, at 1.79 of 2.4 GHz;
// the same call on zeros runs at 1390 TFLOP/s), then the masked tiles of short rows.  Measured against products and softmax
// in turn: 16512 tokens, 48 heads 3.92 -> 3.13 ms (855 -> 1070 TFLOP/s), 8 x 1888 tokens, 32 heads 353 -> 298 us,
// one sequence of 2176, 28 heads 90 -> 63 us.
__global__ __launch_bounds__(128, 1) void prefill_attn_bf16_kernel(PrefillArgs a) {
    constexpr int HD = 128;
    constexpr int ROWB = HD * 2;
    constexpr int KP = ROWB + 16;           // K tile pitch: odd multiple of 16 bytes
    constexpr int VP = kVtPitch;
    constexpr int NV = HD / 16;             // 16-byte words a lane holds of a row half = chunks of one product
    constexpr int NCB = HD / 32;            // blocks of 32 channels
    constexpr int KTPR = 128 / 32;          // threads per K row, four units each
    __shared__ __attribute__((aligned(16))) char k_lds[2][32 * KP];
    __shared__ __attribute__((aligned(16))) char v_lds[2][HD * VP];
    __shared__ int bail_s[2];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // uniform: conditions on it are scalar branches
    const int hf = lane >> 5, l32 = lane & 31;
    PrefillBlock w;
    if (!prefill_block(a, blockIdx.x, w)) return;     // padding
    const int wrow0 = w.q0 + 64 * wave;               // this wave's first row
    const int kmax = a.causal ? min(a.N, w.q0 + 128) : a.N;
    const int n_tiles = (kmax + 31) >> 5;
    const int j_last = (n_tiles - 1) << 5;

    // staging.  K: thread -> row krow, units kcu + KTPR x.  V: thread -> four keys 4 vkg .. 4 vkg + 3 of one
    // 16-byte unit vcu (8 channels).  In the last tile rows past the end repeat the last row (masked later).
    const int krow = tid / KTPR, kcu = tid % KTPR;
    const int vkg = tid & 7, vcu = tid >> 3;
    const unsigned ksn = (unsigned)a.ksn, vsn = (unsigned)a.vsn;
    const int r_last = a.N - 1 - j_last;
    const unsigned ko = krow * ksn + 16 * kcu, ko_e = min(krow, r_last) * ksn + 16 * kcu;
    unsigned vo[4], vo_e[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        vo[x] = (4 * vkg + x) * vsn + 16 * vcu;
        vo_e[x] = min(4 * vkg + x, r_last) * vsn + 16 * vcu;
    }
    const char *kbase = a.k + (long long)w.b * a.ksb + (long long)w.g * a.ksh;
    const char *vbase = a.v + (long long)w.b * a.vsb + (long long)w.g * a.vsh;
    auto k_unit = [&](int t, int x) {
        const int tc = min(t, n_tiles - 1);
        return *reinterpret_cast<const uint4 *>(kbase + (long long)(tc << 5) * a.ksn + (tc == n_tiles - 1 ? ko_e : ko) + 16 * KTPR * x);
    };
    auto v_unit = [&](int t, int x) {
        const int tc = min(t, n_tiles - 1);
        return *reinterpret_cast<const uint4 *>(vbase + (long long)(tc << 5) * a.vsn + (tc == n_tiles - 1 ? vo_e[x] : vo[x]));
    };
    char *const k_dst = &k_lds[0][krow * KP + 16 * kcu];
    char *const v_dst = &v_lds[0][(8 * vcu) * VP + vt_offset(vkg)];
    const char *const k_src = &k_lds[0][l32 * KP + 16 * hf];
    const char *const v_src = &v_lds[0][l32 * VP + 16 * hf];
    auto frag = [](const char *src) { return *reinterpret_cast<const uint4 *>(src); };

    // ---- the first tiles, all loads at once
    // (named registers: staging that is carried around the loop in arrays went to scratch memory)
    uint4 ks0 = k_unit(0, 0), ks1 = k_unit(0, 1), ks2 = k_unit(0, 2), ks3 = k_unit(0, 3);
    const uint4 t0 = k_unit(1, 0), t1 = k_unit(1, 1), t2 = k_unit(1, 2), t3 = k_unit(1, 3);
    uint4 qf[2][NV];                        // lane (row l32 of block x, half hf) holds bytes 16 hf + 32 i of its row
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const char *src = a.q + (long long)w.b * a.qsb + (long long)min(wrow0 + 32 * x + l32, a.N - 1) * a.qsn +
                          (long long)w.h * a.qsh + 16 * hf;
#pragma unroll
        for (int i = 0; i < NV; ++i) qf[x][i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
    }
    auto put_k = [&](char *dst, const uint4 &u0, const uint4 &u1, const uint4 &u2, const uint4 &u3) {
        *reinterpret_cast<uint4 *>(dst) = u0;
        *reinterpret_cast<uint4 *>(dst + 16 * KTPR) = u1;
        *reinterpret_cast<uint4 *>(dst + 32 * KTPR) = u2;
        *reinterpret_cast<uint4 *>(dst + 48 * KTPR) = u3;
    };
    put_k(k_dst, ks0, ks1, ks2, ks3);
    ks0 = k_unit(2, 0), ks1 = k_unit(2, 1), ks2 = k_unit(2, 2), ks3 = k_unit(2, 3);
    uint4 vs0 = v_unit(0, 0), vs1 = v_unit(0, 1), vs2 = v_unit(0, 2), vs3 = v_unit(0, 3);
    put_k(k_dst + 32 * KP, t0, t1, t2, t3);
    // V^T(-1) is zero: iteration 0 multiplies it with probabilities that are zero too
    for (int x = tid; x < HD * VP / 16; x += 128) *reinterpret_cast<uint4 *>(&v_lds[1][16 * x]) = make_uint4(0, 0, 0, 0);
    __syncthreads();

    f32x16 sa[2], sb[2];                    // logits of the even and the odd tiles
    uint32_t pa[2][8], pb[2][8];            // probabilities of the odd and the even tiles (of the tile before the logits)
    uint4 kf[NV], vf[NV];
    f32x16 oacc[2][NCB];
    float mb[2], m_run[2], l_run[2];
    auto mfma = [](const uint4 &x, const uint4 &y, const f32x16 &c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
    };
    auto quad = [](const uint32_t (&p)[8], int h) { return make_uint4(p[4 * h], p[4 * h + 1], p[4 * h + 2], p[4 * h + 3]); };
    // last visible key of this lane's row of block x, relative to key 4 hf of tile 0
    int lim0[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) lim0[x] = (a.causal ? min(wrow0 + 32 * x + l32, a.N - 1) : a.N - 1) - 4 * hf;
    auto hidden = [&](int r, int lim) { return 8 * (r >> 2) + (r & 3) > lim; };
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) kf[i] = frag(k_src + 32 * i);
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int x = 0; x < 2; ++x) sa[x] = mfma(kf[i], qf[x][i], i == 0 ? zero : sa[x]);
#pragma unroll
    for (int i = 0; i < NV; ++i) kf[i] = frag(k_src + 32 * KP + 32 * i);
    __syncthreads();
    put_k(k_dst, ks0, ks1, ks2, ks3);
    ks0 = k_unit(3, 0), ks1 = k_unit(3, 1), ks2 = k_unit(3, 2), ks3 = k_unit(3, 3);
    // the reference of every row: its maximum over the first tile (key 0 is visible to every row)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, hidden(r, lim0[x]) ? -INFINITY : sa[x][r]);
        m_run[x] = half_max(mx);
        mb[x] = -(m_run[x] * a.scale_log2);
        l_run[x] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) pa[x][i] = 0;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) oacc[x][cb] = zero;
    }
    __syncthreads();

    // iteration t: logits sin -> probabilities pout, products of the next logits into sout, probabilities pin of the
    // tile before into the output
    auto step = [&](int t, f32x16 (&sin)[2], f32x16 (&sout)[2], uint32_t (&pin)[2][8], uint32_t (&pout)[2][8], auto edge_tag) {
        constexpr bool EDGE = decltype(edge_tag)::value;
        const int buf = t & 1;
        const char *vr = v_src + (buf ^ 1) * (HD * VP), *kr = k_src + buf * (32 * KP);
        char *vw = v_dst + buf * (HD * VP), *kw = k_dst + (buf ^ 1) * (32 * KP);
        const int tk = min(t + 4, n_tiles - 1), tv = min(t + 1, n_tiles - 1);
        const char *kb = kbase + (long long)(tk << 5) * a.ksn, *vb = vbase + (long long)(tv << 5) * a.vsn;
        const unsigned ok = tk == n_tiles - 1 ? ko_e : ko;
        const int lim[2] = {lim0[0] - (t << 5), lim0[1] - (t << 5)};
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) asm volatile("" : "+a"(oacc[x][cb]));
        asm volatile("" : "+a"(sin[0]), "+a"(sin[1]));
        // softmax of logit el (block el / 16, register el % 16) in three stages, each a slot behind the one before
        // (a tile's probabilities are summed on their own and added to the row's sum once: one after the other into the
        // running sum, the small ones of a long row drop out of it -- 4e-6 of the sum at 16512 keys, against 2e-7 in rms)
        float e_arg[32], e_p[32], tile_sum[2];
        auto stage_arg = [&](int el) {
            float v = sin[el >> 4][el & 15];
            if constexpr (EDGE) v = hidden(el & 15, lim[el >> 4]) ? -INFINITY : v;
            e_arg[el] = fmaf(v, a.scale_log2, mb[el >> 4]);
        };
        auto stage_exp = [&](int el) { e_p[el] = __builtin_amdgcn_exp2f(e_arg[el]); };
        auto stage_sum = [&](int el) {
            const int x = el >> 4;
            tile_sum[x] = (el & 15) ? tile_sum[x] + e_p[el] : e_p[el];
            if ((el & 15) == 15) l_run[x] += tile_sum[x];
            if (el & 1) pout[el >> 4][(el & 15) >> 1] = pack_bf16(e_p[el - 1], e_p[el]);
        };
        stage_arg(0);
#pragma unroll
        for (int sl = 0; sl < 32; ++sl) {
            const int c = (sl >> 1) & 7, x = sl & 1;         // step of the product, block
            if (sl < 16) {
                sout[x] = mfma(kf[c], qf[x][c], c == 0 ? zero : sout[x]);
            } else {
                oacc[x][c >> 1] = mfma(vf[c], quad(pin[x], c & 1), oacc[x][c >> 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (sl < 16) {
                if (x == 0) vf[c] = frag(vr + (32 * (c >> 1)) * VP + 32 * (c & 1));
                // staging, behind the block-1 product of each step: K units in steps 0-3, V words in 4-7
#define LVLM_K_UNIT(u)                                                          \
    if (sl == 2 * u + 1) {                                                      \
        *reinterpret_cast<uint4 *>(kw + 16 * KTPR * u) = ks##u;                 \
        ks##u = *reinterpret_cast<const uint4 *>(kb + ok + 16 * KTPR * u);      \
    }
                LVLM_K_UNIT(0) LVLM_K_UNIT(1) LVLM_K_UNIT(2) LVLM_K_UNIT(3)
#undef LVLM_K_UNIT
                if (sl == 9) vt_store(vw, 0, vs0.x, vs1.x, vs2.x, vs3.x);
                if (sl == 11) vt_store(vw, 1, vs0.y, vs1.y, vs2.y, vs3.y);
                if (sl == 13) vt_store(vw, 2, vs0.z, vs1.z, vs2.z, vs3.z);
                if (sl == 15) vt_store(vw, 3, vs0.w, vs1.w, vs2.w, vs3.w);
            } else {
                if (sl < 24) kf[sl - 16] = frag(kr + 32 * (sl - 16));
                if (sl == 16) vs0 = *reinterpret_cast<const uint4 *>(vb + (tv == n_tiles - 1 ? vo_e[0] : vo[0]));
                if (sl == 17) vs1 = *reinterpret_cast<const uint4 *>(vb + (tv == n_tiles - 1 ? vo_e[1] : vo[1]));
                if (sl == 18) vs2 = *reinterpret_cast<const uint4 *>(vb + (tv == n_tiles - 1 ? vo_e[2] : vo[2]));
                if (sl == 19) vs3 = *reinterpret_cast<const uint4 *>(vb + (tv == n_tiles - 1 ? vo_e[3] : vo[3]));
            }
            if (sl < 31) stage_arg(sl + 1);
            stage_exp(sl);
            if (sl > 0) stage_sum(sl - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        stage_sum(31);
        __syncthreads();
    };
    // tiles [0, t_whole) are seen whole by every row of the workgroup
    const int t_whole = (a.causal ? min(w.q0, a.N) : a.N) >> 5;
    int t = 0;
    for (; t + 1 < t_whole; t += 2) {
        step(t, sa, sb, pa, pb, std::false_type{});
        step(t + 1, sb, sa, pb, pa, std::false_type{});
    }
    for (; t + 1 < n_tiles; t += 2) {
        step(t, sa, sb, pa, pb, std::true_type{});
        step(t + 1, sb, sa, pb, pa, std::true_type{});
    }
    if (t < n_tiles) {
        step(t, sa, sb, pa, pb, std::true_type{});
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int i = 0; i < 8; ++i) pa[x][i] = pb[x][i];
    }
    // the last tile's probabilities
    {
        const char *vr = v_src + ((n_tiles - 1) & 1) * (HD * VP);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const uint4 f = frag(vr + (32 * (i >> 1)) * VP + 32 * (i & 1));
#pragma unroll
            for (int x = 0; x < 2; ++x) oacc[x][i >> 1] = mfma(f, quad(pa[x], i & 1), oacc[x][i >> 1]);
        }
    }
    // A wave that sees the risk writes nothing, and the whole workgroup does its block again.
    const bool risky = risky_sums(l_run[0], l_run[1]);
    if (lane == 0) bail_s[wave] = risky;
    if (!risky)
#pragma unroll
        for (int x = 0; x < 2; ++x) prefill_write<HD>(a, w, k_lds[wave], wrow0 + 32 * x, lane, m_run[x], l_run[x], oacc[x]);
    __syncthreads();
    if (bail_s[0] | bail_s[1]) prefill_plain_block<HD, true>(a, w, &k_lds[0][0], &v_lds[0][0]);
}

// One tile after the other, products and softmax in turn: the SAFE sweep (a rescale touches everything in flight, so
// nothing is pipelined across tiles), and the FAST sweep for 64 channels, where the pipelined loop above has too few
// products per logit to hide the softmax behind and two waves per SIMD -- 253 of the 256 registers here, 300 there -- do
// better (2 x 4000 tokens, 32 heads: 185 us here, 221 us pipelined).  Returns whether a FAST sweep has to be done again.
template <int HD, bool SAFE>
__device__ __forceinline__ bool prefill_plain_block(const PrefillArgs &a, const PrefillBlock &w, char *k_mem, char *v_mem) {
    constexpr int ROWB = HD * 2;
    constexpr int KP = ROWB + 16;           // K tile pitch: odd multiple of 16 bytes
    constexpr int VP = kVtPitch;
    constexpr int NV = HD / 16;             // 16-byte words a lane holds of a row half
    constexpr int NCB = HD / 32;            // blocks of 32 channels
    constexpr int UPR = ROWB / 16;          // 16-byte units per row
    constexpr int KUPT = 32 * UPR / 128;    // K units per thread and tile
    constexpr int KTPR = UPR / KUPT;        // threads per K row
    char(*k_lds)[32 * KP] = reinterpret_cast<char(*)[32 * KP]>(k_mem);
    char(*v_lds)[HD * VP] = reinterpret_cast<char(*)[HD * VP]>(v_mem);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // uniform: conditions on it are scalar branches
    const int hf = lane >> 5, l32 = lane & 31;
    const int b = w.b, h = w.h, g = w.g, q0 = w.q0;
    const int wrow0 = q0 + 64 * wave;                 // this wave's first row
    const int kmax = a.causal ? min(a.N, q0 + 128) : a.N;
    const int n_tiles = (kmax + 31) >> 5;

    // staging.  K: thread -> row krow, units kcu + KTPR x.  V: thread -> four keys 4 vkg .. 4 vkg + 3 of one
    // 16-byte unit vcu (8 channels); HD = 64 needs only half the threads for V.
    const int krow = tid / KTPR, kcu = tid % KTPR;
    const char *kbase = a.k + (long long)b * a.ksb + (long long)g * a.ksh + 16 * kcu;
    const int vkg = tid & 7, vcu = tid >> 3;
    const bool v_on = vcu < UPR;
    const char *vbase = a.v + (long long)b * a.vsb + (long long)g * a.vsh + 16 * (v_on ? vcu : 0);
    // Named registers, not arrays (an indexed array that lives across the tile's arithmetic goes to scratch), and
    // written on EVERY tile (the last one fetches itself again): a value that may survive from the previous
    // tile is carried around the loop, and the compiler parks it in accumulation registers and copies it back.
    uint4 ks0 = make_uint4(0, 0, 0, 0), ks1 = ks0, ks2 = ks0, ks3 = ks0, vs0 = ks0, vs1 = ks0, vs2 = ks0, vs3 = ks0;
    const char *kthr = kbase + (long long)krow * a.ksn;           // this thread's row of tile 0
    const char *vthr = vbase + (long long)(4 * vkg) * a.vsn;
    auto fetch = [&](int j0) {
        if (j0 + 32 <= a.N) {                                     // whole tile: uniform offsets only
            const uint4 *src = reinterpret_cast<const uint4 *>(kthr + (long long)j0 * a.ksn);
            ks0 = src[0];
            if constexpr (KUPT > 1) ks1 = src[KTPR];
            if constexpr (KUPT > 2) ks2 = src[2 * KTPR];
            if constexpr (KUPT > 3) ks3 = src[3 * KTPR];
            if (v_on) {
                const char *vp = vthr + (long long)j0 * a.vsn;
                vs0 = *reinterpret_cast<const uint4 *>(vp);
                vs1 = *reinterpret_cast<const uint4 *>(vp + a.vsn);
                vs2 = *reinterpret_cast<const uint4 *>(vp + 2 * a.vsn);
                vs3 = *reinterpret_cast<const uint4 *>(vp + 3 * a.vsn);
            }
            return;
        }
        // the ragged last tile: rows past the end repeat the last row (masked later)
        const uint4 *src = reinterpret_cast<const uint4 *>(kbase + (long long)min(j0 + krow, a.N - 1) * a.ksn);
        ks0 = src[0];
        if constexpr (KUPT > 1) ks1 = src[KTPR];
        if constexpr (KUPT > 2) ks2 = src[2 * KTPR];
        if constexpr (KUPT > 3) ks3 = src[3 * KTPR];
        if (v_on) {
            const int jv = j0 + 4 * vkg;
            vs0 = *reinterpret_cast<const uint4 *>(vbase + (long long)min(jv + 0, a.N - 1) * a.vsn);
            vs1 = *reinterpret_cast<const uint4 *>(vbase + (long long)min(jv + 1, a.N - 1) * a.vsn);
            vs2 = *reinterpret_cast<const uint4 *>(vbase + (long long)min(jv + 2, a.N - 1) * a.vsn);
            vs3 = *reinterpret_cast<const uint4 *>(vbase + (long long)min(jv + 3, a.N - 1) * a.vsn);
        }
    };
    const int v_off = vt_offset(vkg);
    auto stash = [&](int buf) {
        uint4 *dst = reinterpret_cast<uint4 *>(&k_lds[buf][krow * KP + 16 * kcu]);
        dst[0] = ks0;
        if constexpr (KUPT > 1) dst[KTPR] = ks1;
        if constexpr (KUPT > 2) dst[2 * KTPR] = ks2;
        if constexpr (KUPT > 3) dst[3 * KTPR] = ks3;
        if (v_on) {
            char *vd = &v_lds[buf][(8 * vcu) * VP + v_off];
            vt_store(vd, 0, vs0.x, vs1.x, vs2.x, vs3.x);
            vt_store(vd, 1, vs0.y, vs1.y, vs2.y, vs3.y);
            vt_store(vd, 2, vs0.z, vs1.z, vs2.z, vs3.z);
            vt_store(vd, 3, vs0.w, vs1.w, vs2.w, vs3.w);
        }
    };

    float m_run[2], l_run[2];
    f32x16 oacc[2][NCB];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        m_run[x] = -INFINITY;
        l_run[x] = 0.f;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[x][cb][r] = 0.f;
    }
    fetch(0);
    // The operand loads go out after the first tile's: loads return in order, and the tile (mostly in L2) would
    // otherwise wait behind the operand rows (from memory) before it can go to LDS.
    // Query operands: lane (row l32 of block x, half hf) holds bytes 16 hf + 32 i of its row
    uint4 qf[2][NV];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int row = wrow0 + 32 * x + l32;
        const char *src = a.q + (long long)b * a.qsb + (long long)min(row, a.N - 1) * a.qsn + (long long)h * a.qsh + 16 * hf;
#pragma unroll
        for (int i = 0; i < NV; ++i) qf[x][i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
    }

    stash(0);
    __syncthreads();
    // One tile.  EDGE = false: every row of the workgroup sees the whole tile -- no masks, both blocks.  EDGE = true
    // (the up to four tiles around the diagonal, and a ragged last tile): per block the tile is seen whole, cut by
    // the diagonal (one fixed lane pattern, blocks and tiles being aligned alike), cut by the end of the sequence,
    // or not seen at all; a block that does not see it skips the logits and the softmax and multiplies zeros
    // into its accumulators (no branch around the instructions that update them: such a branch makes the
    // compiler copy all accumulators where its paths join).
    const int diag_lim = l32 - 4 * hf;       // register r of this lane holds a key past the diagonal iff 8 (r / 4) + r % 4 > diag_lim
    auto step = [&](int t, auto edge_tag) {
        constexpr bool EDGE = decltype(edge_tag)::value;
        const int j0 = t << 5, buf = t & 1;
        fetch(min(j0 + 32, (n_tiles - 1) << 5));
        // the output accumulators stay where the matrix instructions keep them
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) asm volatile("" : "+a"(oacc[x][cb]));
        uint4 pf[2][2];
        auto softmax = [&](int x, f32x16 &s) {
            // Key j0 is visible to every row of a block the tile reaches, so the first tile sets a finite reference.
            auto row_max = [&]() {
                float mx = s[0];
#pragma unroll
                for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
                return half_max(mx);
            };
            if constexpr (!SAFE) {
                // the reference is the first tile's maximum; later tiles need no maximum at all: a logit
                // far above the reference shows in the row sum (checked once, after the sweep)
                if (t == 0) m_run[x] = row_max();
            } else if (const float mx = row_max(); __builtin_amdgcn_ballot_w64((mx - m_run[x]) * a.scale_log2 > kLazy) != 0ull) {
                const float m_new = fmaxf(m_run[x], mx);
                const float alpha = __builtin_amdgcn_exp2f((m_run[x] - m_new) * a.scale_log2);   // first tile: 0
                l_run[x] *= alpha;
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[x][cb][r] *= alpha;
                m_run[x] = m_new;
            }
            const float mb = m_run[x] * a.scale_log2;
            float sum = 0.f;
            float p[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], a.scale_log2, -mb));
                sum += p[r];
            }
            l_run[x] += sum;
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
                pf[x][t2].x = pack_bf16(p[8 * t2 + 0], p[8 * t2 + 1]);
                pf[x][t2].y = pack_bf16(p[8 * t2 + 2], p[8 * t2 + 3]);
                pf[x][t2].z = pack_bf16(p[8 * t2 + 4], p[8 * t2 + 5]);
                pf[x][t2].w = pack_bf16(p[8 * t2 + 6], p[8 * t2 + 7]);
            }
        };
        const char *ksrc = &k_lds[buf][l32 * KP + 16 * hf];
        if constexpr (!EDGE) {
            f32x16 s0, s1;
#pragma unroll
            for (int r = 0; r < 16; ++r) s0[r] = 0.f, s1[r] = 0.f;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const uint4 kf = *reinterpret_cast<const uint4 *>(ksrc + 32 * i);
                const bf16x8 kb = __builtin_bit_cast(bf16x8, kf);
                s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb, __builtin_bit_cast(bf16x8, qf[0][i]), s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb, __builtin_bit_cast(bf16x8, qf[1][i]), s1, 0, 0, 0);
            }
            softmax(0, s0);
            softmax(1, s1);
        } else {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int blk0 = wrow0 + 32 * x;             // first row of the block
                if (a.causal && j0 > blk0) {                 // not seen at all
                    pf[x][0] = pf[x][1] = make_uint4(0, 0, 0, 0);
                    continue;
                }
                f32x16 s;
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const uint4 kf = *reinterpret_cast<const uint4 *>(ksrc + 32 * i);
                    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf),
                                                                __builtin_bit_cast(bf16x8, qf[x][i]), s, 0, 0, 0);
                }
                if (j0 + 32 > a.N) {                         // the ragged last tile: by key index
                    const int row = blk0 + l32;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int j = j0 + acc_row(r, hf);
                        if ((a.causal && j > row) || j >= a.N) s[r] = -INFINITY;
                    }
                } else if (a.causal && j0 == blk0) {         // the diagonal tile: a fixed pattern
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (8 * (r >> 2) + (r & 3) > diag_lim) s[r] = -INFINITY;
                }
                softmax(x, s);
            }
        }
        {
            const char *src = &v_lds[buf][l32 * VP + 16 * hf];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {
                    const uint4 vf = *reinterpret_cast<const uint4 *>(src + (32 * cb) * VP + 32 * t2);
                    const bf16x8 vb = __builtin_bit_cast(bf16x8, vf);
                    oacc[0][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb, __builtin_bit_cast(bf16x8, pf[0][t2]),
                                                                         oacc[0][cb], 0, 0, 0);
                    oacc[1][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb, __builtin_bit_cast(bf16x8, pf[1][t2]),
                                                                         oacc[1][cb], 0, 0, 0);
                }
            }
        }
        if (t + 1 < n_tiles) stash(buf ^ 1);
        __syncthreads();
    };
    // tiles [0, t_whole) are seen whole by every row of the workgroup
    const int t_whole = a.causal ? min(q0, a.N) >> 5 : a.N >> 5;
    for (int t = 0; t < t_whole; ++t) step(t, std::false_type{});
    for (int t = t_whole; t < n_tiles; ++t) step(t, std::true_type{});
    if (!SAFE && risky_sums(l_run[0], l_run[1])) return true;
#pragma unroll
    for (int x = 0; x < 2; ++x) prefill_write<HD>(a, w, k_lds[wave], wrow0 + 32 * x, lane, m_run[x], l_run[x], oacc[x]);
    return false;
}

__global__ __launch_bounds__(128, 1) void prefill_attn_d64_kernel(PrefillArgs a) {
    __shared__ __attribute__((aligned(16))) char k_lds[2][32 * (64 * 2 + 16)];
    __shared__ __attribute__((aligned(16))) char v_lds[2][64 * kVtPitch];
    __shared__ int bail_s[2];
    PrefillBlock w;
    if (!prefill_block(a, blockIdx.x, w)) return;     // padding
    const bool again = prefill_plain_block<64, false>(a, w, &k_lds[0][0], &v_lds[0][0]);
    if ((threadIdx.x & 63) == 0) bail_s[threadIdx.x >> 6] = again;
    __syncthreads();
    if (bail_s[0] | bail_s[1]) prefill_plain_block<64, true>(a, w, &k_lds[0][0], &v_lds[0][0]);
}

// The SAFE sweep alone: rows too far apart for the FAST kernels' 32-bit offsets.
template <int HD>
__global__ __launch_bounds__(128, 1) void prefill_attn_safe_kernel(PrefillArgs a) {
    __shared__ __attribute__((aligned(16))) char k_lds[2][32 * (HD * 2 + 16)];
    __shared__ __attribute__((aligned(16))) char v_lds[2][HD * kVtPitch];
    PrefillBlock w;
    if (prefill_block(a, blockIdx.x, w)) prefill_plain_block<HD, true>(a, w, &k_lds[0][0], &v_lds[0][0]);
}

// component c of a 16-byte word
__device__ __forceinline__ float word(const uint4 &v, int c) {
    return __uint_as_float(c == 0 ? v.x : c == 1 ? v.y : c == 2 ? v.z : v.w);
}

// fp32 (the small fp32 configuration), on the fp32 matrix instruction (16 x 16 x 4, exact fp32 products, fp32 sums).
// The instruction is slow (32 cycles for 2048 flops: 1024 cycles for the logits of 32 keys x 16 queries at 64
// channels, 1024 more for P V), so what bounds a small call is the length of one wave's chain of tiles, not memory.
// The keys are therefore split over the four waves of a workgroup, which owns QB blocks of 16 query rows of one head:
// wave w takes the 32-key tiles w, w + 4, ... with its own running maximum, sum and accumulators, and the four
// are folded through LDS at the end.  No tile is shared, so K and V go straight from memory (L2) into the operand
// registers and the loop has no barrier: the next tile's K is requested when the logits have consumed this one's, its
// V when the product has.
// Lane = (l16, kg).  S^T = K Q^T (rows = keys, columns = queries): contraction step (i, c) of lane group kg is channel
// 16 i + 4 kg + c for both operands, 16-byte loads of 64-byte pieces.  A lane then holds the logits of query l16 and
// keys 4 kg + r of each 16-key block, and the four keys of register r over the lane groups are one contraction step
// of O^T += V^T P^T as they stand; its other operand is V[that key][CPL l16 + cb], loaded as whole rows (16 lanes
// x CPL channels), output block cb then being the channels congruent to cb modulo CPL.
// Measured (4 heads, 64 channels; a wave per 32 rows walking all tiles, K and V shared through LDS -> this kernel):
// 640 tokens 57.1 -> 10.9 us, 2048 171 -> 50, 4200 347 -> 135 us (67 TFLOP/s), 16 sequences of 4200 1486 -> 1425 us
// (101 TFLOP/s of the 155 a large fp32 matrix product reaches).
struct F32Block {
    int b, h, qb;
};
// How a launch's blocks go out: the plain grid, dealt out, or dealt out an XCD's heads in groups.
enum { kPlain, kDealt, kGrouped };
template <int DEAL>
__device__ __forceinline__ bool dealt_to(const PrefillArgs &a, int n_blocks, F32Block &w) {
    int head;
    const bool any = dealt_block<DEAL == kGrouped>(a.deal, n_blocks, blockIdx.x, head, w.qb);
    w.b = head / a.Hq;
    w.h = head - w.b * a.Hq;
    return any;
}

template <int HD, int QB, int DEAL>
__global__ __launch_bounds__(256, 1) void prefill_attn_f32_kernel(PrefillArgs a) {
    constexpr int NW = HD / 16;             // 16-byte words of a row per lane
    constexpr int CPL = HD / 16;            // channels per lane
    constexpr int VW = CPL / 4;             // 16-byte words of a V row per lane
    constexpr int RP = HD + 4;              // LDS row pitch
    __shared__ __attribute__((aligned(16))) float wo[4][16 * QB][RP];
    __shared__ float wm[4][16 * QB], wl[4][16 * QB];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    F32Block blk{(int)blockIdx.z, (int)blockIdx.y, (int)(gridDim.x - 1 - blockIdx.x)};      // longest blocks first
    if constexpr (DEAL != kPlain)
        if (!dealt_to<DEAL>(a, (a.N + 16 * QB - 1) / (16 * QB), blk)) return;
    const int h = blk.h, b = blk.b, g = h / a.G;
    const int q0 = blk.qb * 16 * QB;
    const int kmax = a.causal ? min(a.N, q0 + 16 * QB) : a.N;
    const int n_tiles = (kmax + 31) >> 5;

    const char *kbase = a.k + (long long)b * a.ksb + (long long)g * a.ksh + 16 * kg;
    const char *vbase = a.v + (long long)b * a.vsb + (long long)g * a.vsh + 4 * CPL * l16;
    uint4 kf[2][NW], vf[8][VW];
    auto load_k = [&](int j0) {             // rows past the end repeat the last row (masked later)
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            const char *src = kbase + (long long)min(j0 + 16 * blk + l16, a.N - 1) * a.ksn;
#pragma unroll
            for (int i = 0; i < NW; ++i) kf[blk][i] = *reinterpret_cast<const uint4 *>(src + 64 * i);
        }
    };
    auto load_v = [&](int j0) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const char *src = vbase + (long long)min(j0 + 16 * (s >> 2) + 4 * kg + (s & 3), a.N - 1) * a.vsn;
#pragma unroll
            for (int i = 0; i < VW; ++i) vf[s][i] = *reinterpret_cast<const uint4 *>(src + 16 * i);
        }
    };
    if (wave < n_tiles) load_k(32 * wave);
    uint4 qf[QB][NW];
#pragma unroll
    for (int x = 0; x < QB; ++x) {
        const char *src = a.q + (long long)b * a.qsb + (long long)min(q0 + 16 * x + l16, a.N - 1) * a.qsn + (long long)h * a.qsh + 16 * kg;
#pragma unroll
        for (int i = 0; i < NW; ++i) qf[x][i] = *reinterpret_cast<const uint4 *>(src + 64 * i);
    }
    if (wave < n_tiles) load_v(32 * wave);

    float m_run[QB], l_run[QB];             // of query l16 of each block (l_run: this lane group's keys only)
    f32x4 oacc[QB][CPL];
#pragma unroll
    for (int x = 0; x < QB; ++x) {
        m_run[x] = -INFINITY;
        l_run[x] = 0.f;
#pragma unroll
        for (int cb = 0; cb < CPL; ++cb) oacc[x][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int t = wave; t < n_tiles; t += 4) {
        const int j0 = t << 5;
        f32x4 s[QB][2];
#pragma unroll
        for (int x = 0; x < QB; ++x) s[x][0] = s[x][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int x = 0; x < QB; ++x)
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk)
                        s[x][blk] = __builtin_amdgcn_mfma_f32_16x16x4f32(word(kf[blk][i], c), word(qf[x][i], c), s[x][blk], 0, 0, 0);
        const int j_next = t + 4 < n_tiles ? j0 + 128 : j0;       // (the last tile fetches itself again)
        load_k(j_next);
        const bool edge = (a.causal && j0 + 31 > q0) || j0 + 32 > a.N;
#pragma unroll
        for (int x = 0; x < QB; ++x) {
            if (edge) {
                const int lim = a.causal ? min(q0 + 16 * x + l16, a.N - 1) : a.N - 1;     // last visible key
#pragma unroll
                for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (j0 + 16 * blk + 4 * kg + r > lim) s[x][blk][r] = -INFINITY;
            }
            float mx = s[x][0][0];
#pragma unroll
            for (int r = 1; r < 8; ++r) mx = fmaxf(mx, s[x][r >> 2][r & 3]);
            mx = fmaxf(mx, other_row(mx));
            mx = fmaxf(mx, other_half(mx));
            const float m_new = fmaxf(m_run[x], mx);
            const float ref = m_new == -INFINITY ? 0.f : m_new;   // a wave's tiles may all lie past a row's diagonal
            const float alpha = __builtin_amdgcn_exp2f((m_run[x] - ref) * a.scale_log2);  // first tile: 0
            const float mb = ref * a.scale_log2;
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[x][r >> 2][r & 3], a.scale_log2, -mb));
                s[x][r >> 2][r & 3] = p;
                sum += p;
            }
            l_run[x] = l_run[x] * alpha + sum;
            m_run[x] = m_new;
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) oacc[x][cb] *= alpha;
        }
#pragma unroll
        for (int k8 = 0; k8 < 8; ++k8)
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb)
#pragma unroll
                for (int x = 0; x < QB; ++x)
                    oacc[x][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(word(vf[k8][cb >> 2], cb & 3), s[x][k8 >> 2][k8 & 3], oacc[x][cb], 0, 0, 0);
        load_v(j_next);
    }

    // ---- fold the four waves: register r of block cb is channel CPL (4 kg + r) + cb
#pragma unroll
    for (int x = 0; x < QB; ++x) {
        float l = l_run[x];
        l += other_row(l);
        l += other_half(l);
        const int row = 16 * x + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c4 = 0; c4 < VW; ++c4)
                *reinterpret_cast<float4 *>(&wo[wave][row][CPL * (4 * kg + r) + 4 * c4]) =
                    make_float4(oacc[x][4 * c4][r], oacc[x][4 * c4 + 1][r], oacc[x][4 * c4 + 2][r], oacc[x][4 * c4 + 3][r]);
        if (kg == 0) {
            wm[wave][row] = m_run[x];
            wl[wave][row] = l;
        }
    }
    __syncthreads();
    for (int u = tid; u < 16 * QB * (HD / 4); u += 256) {
        const int rr = u / (HD / 4), e = 4 * (u % (HD / 4)), row = q0 + rr;
        if (row >= a.N) break;
        const float mx = fmaxf(fmaxf(wm[0][rr], wm[1][rr]), fmaxf(wm[2][rr], wm[3][rr]));   // finite: wave 0 has tile 0
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        float l_tot = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float wgt = __builtin_amdgcn_exp2f((wm[w][rr] - mx) * a.scale_log2);
            const float4 v = *reinterpret_cast<const float4 *>(&wo[w][rr][e]);
            o.x = fmaf(v.x, wgt, o.x), o.y = fmaf(v.y, wgt, o.y), o.z = fmaf(v.z, wgt, o.z), o.w = fmaf(v.w, wgt, o.w);
            l_tot = fmaf(wl[w][rr], wgt, l_tot);
        }
        const float inv = 1.f / l_tot;
        char *dst = a.out + (long long)b * a.osb + (long long)row * a.osn + (long long)h * a.osh;
        *reinterpret_cast<float4 *>(dst + 4 * e) = make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
        if (e == 0) {
            const float lse = mx * a.scale + __logf(l_tot);
            a.row_lse[((long long)b * a.Hq + h) * a.N + row] = lse;
            if (a.lse_t && row >= a.N - a.T) a.lse_t[((long long)b * a.Hq + h) * a.T + (row - (a.N - a.T))] = lse;
        }
    }
}

// fp32 where whole turns of the chip share their tiles (f32_shares_tiles has the rule), on the fp32 matrix instruction of
// 32 x 32 x 2: the products of a 32 x 32 tile cost as much as above, but a K or V value read once serves 32 rows instead of 16 and the
// four waves of a workgroup read the same tile, so it is the matrix instructions that bound it and not the reading.
// A workgroup of four waves owns 128 query rows of one head, one 32-row block per wave, its rows held as an MFMA
// operand.  K and V tiles of 32 keys go through LDS as they are (rows = keys), fetched one tile ahead by the 256
// threads, one barrier per tile.  S^T = K Q^T (rows = keys, columns = queries): a lane owns one query row and 16
// of its logits; the textbook online softmax (the reference follows the running maximum, sums and accumulators
// are rescaled when it moves).  For O^T += V^T P^T the contraction of one instruction is two keys, one per
// half-wave: exactly the two keys the two halves hold in the same accumulator register, so register r of the
// probabilities is the second operand as it stands and the first is V[that key][channel] read from the tile.
template <int HD, int DEAL>
__global__ __launch_bounds__(256, 1) void prefill_attn_f32_shared_kernel(PrefillArgs a) {
    constexpr int ROWB = HD * 4;
    constexpr int KP = ROWB + 16;           // tile pitch: odd multiple of 16 bytes
    constexpr int NV = HalfRow<LVLM_F32, HD>::NV;
    constexpr int NCB = HD / 32;
    constexpr int UPR = ROWB / 16;          // 16-byte units per row
    constexpr int UPT = 32 * UPR / 256;     // units per thread and tile (2 or 4)
    constexpr int TPR = UPR / UPT;          // threads per row
    __shared__ __attribute__((aligned(16))) char k_lds[2][32 * KP];
    __shared__ __attribute__((aligned(16))) char v_lds[2][32 * KP];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hf = lane >> 5, l32 = lane & 31;
    F32Block blk{(int)blockIdx.z, (int)blockIdx.y, (int)(gridDim.x - 1 - blockIdx.x)};      // longest blocks first
    if constexpr (DEAL != kPlain)
        if (!dealt_to<DEAL>(a, a.nqb, blk)) return;
    const int h = blk.h, b = blk.b, g = h / a.G;
    const int q0 = blk.qb * 128, blk0 = q0 + 32 * wave;
    const int row = blk0 + l32;
    const int kmax = a.causal ? min(a.N, q0 + 128) : a.N;
    const int n_tiles = (kmax + 31) >> 5;

    HalfRow<LVLM_F32, HD> qa;               // lane (row l32, half hf): bytes 16 hf + 32 i of its row
    {
        const char *src = a.q + (long long)b * a.qsb + (long long)min(row, a.N - 1) * a.qsn + (long long)h * a.qsh + 16 * hf;
#pragma unroll
        for (int i = 0; i < NV; ++i) qa.v[i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
    }
    const int srow = tid / TPR, scu = tid % TPR;
    const char *kbase = a.k + (long long)b * a.ksb + (long long)g * a.ksh + 16 * scu;
    const char *vbase = a.v + (long long)b * a.vsb + (long long)g * a.vsh + 16 * scu;
    uint4 ks0 = make_uint4(0, 0, 0, 0), ks1 = ks0, ks2 = ks0, ks3 = ks0, vs0 = ks0, vs1 = ks0, vs2 = ks0, vs3 = ks0;
    auto fetch = [&](int j0) {              // rows past the end repeat the last row (masked later)
        const long long r = min(j0 + srow, a.N - 1);
        const uint4 *ksrc = reinterpret_cast<const uint4 *>(kbase + r * a.ksn);
        const uint4 *vsrc = reinterpret_cast<const uint4 *>(vbase + r * a.vsn);
        ks0 = ksrc[0], vs0 = vsrc[0];
        ks1 = ksrc[TPR], vs1 = vsrc[TPR];
        if constexpr (UPT > 2) {
            ks2 = ksrc[2 * TPR], vs2 = vsrc[2 * TPR];
            ks3 = ksrc[3 * TPR], vs3 = vsrc[3 * TPR];
        }
    };
    auto stash = [&](int buf) {
        uint4 *kd = reinterpret_cast<uint4 *>(&k_lds[buf][srow * KP + 16 * scu]);
        uint4 *vd = reinterpret_cast<uint4 *>(&v_lds[buf][srow * KP + 16 * scu]);
        kd[0] = ks0, vd[0] = vs0;
        kd[TPR] = ks1, vd[TPR] = vs1;
        if constexpr (UPT > 2) {
            kd[2 * TPR] = ks2, vd[2 * TPR] = vs2;
            kd[3 * TPR] = ks3, vd[3 * TPR] = vs3;
        }
    };

    float m_run = -INFINITY, l_run = 0.f;
    f32x16 oacc[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[cb][r] = 0.f;

    fetch(0);
    stash(0);
    __syncthreads();
    for (int t = 0; t < n_tiles; ++t) {
        const int j0 = t << 5, buf = t & 1;
        fetch(min(j0 + 32, (n_tiles - 1) << 5));
        if (!a.causal || j0 <= blk0 + 31) {                       // the block sees some key of the tile
            HalfRow<LVLM_F32, HD> kf;
            {
                const char *src = &k_lds[buf][l32 * KP + 16 * hf];
#pragma unroll
                for (int i = 0; i < NV; ++i) kf.v[i] = *reinterpret_cast<const uint4 *>(src + 32 * i);
            }
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.f;
            mma_tile<LVLM_F32, HD>(s, kf, qa);                    // rows = keys, columns = queries
            if ((a.causal && j0 + 31 > blk0) || j0 + 32 > a.N) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = j0 + acc_row(r, hf);
                    if ((a.causal && j > row) || j >= a.N) s[r] = -INFINITY;
                }
            }
            float mx = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
            mx = fmaxf(mx, other_half(mx));                       // finite: key j0 <= blk0 is visible to every row
            const float m_new = fmaxf(m_run, mx);
            const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * a.scale_log2);   // first tile: 0
            const float mb = m_new * a.scale_log2;
            float p[16], sum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], a.scale_log2, -mb));
                sum += p[r];
            }
            l_run = l_run * alpha + sum;
            m_run = m_new;
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[cb][r] *= alpha;
                // register r of the two half-waves: keys acc_row(r, 0) and acc_row(r, 1) -- the two keys one
                // instruction contracts
                const char *vsrc = &v_lds[buf][4 * (32 * cb + l32)];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float vv = *reinterpret_cast<const float *>(vsrc + acc_row(r, hf) * KP);
                    oacc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv, p[r], oacc[cb], 0, 0, 0);
                }
            }
        }
        if (t + 1 < n_tiles) stash(buf ^ 1);
        __syncthreads();
    }

    const float l_tot = l_run + other_half(l_run);
    if (row >= a.N) return;
    const float inv = 1.f / l_tot;
    // lane (query l32, half hf) holds channels 32 cb + 8 (r / 4) + 4 hf + r % 4
    float *dst = reinterpret_cast<float *>(a.out + (long long)b * a.osb + (long long)row * a.osn + (long long)h * a.osh) + 4 * hf;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
            *reinterpret_cast<float4 *>(dst + 32 * cb + 8 * r4) =
                make_float4(oacc[cb][4 * r4 + 0] * inv, oacc[cb][4 * r4 + 1] * inv, oacc[cb][4 * r4 + 2] * inv,
                            oacc[cb][4 * r4 + 3] * inv);
    if (hf == 0) {
        const float lse = m_run * a.scale + __logf(l_tot);
        a.row_lse[((long long)b * a.Hq + h) * a.N + row] = lse;
        if (a.lse_t && row >= a.N - a.T) a.lse_t[((long long)b * a.Hq + h) * a.T + (row - (a.N - a.T))] = lse;
    }
}

}  // namespace

PrefillWs prefill_ws(const lvlm_prefill_desc &d) {
    PrefillWs w{};
    w.lse_t = 0;
    w.score = align_up((size_t)d.B * d.Hq * (d.T > 0 ? d.T : 0) * sizeof(float), 256);
    w.total = w.score > 256 ? w.score : 256;        // (never none, so that every call asks for a workspace alike)
    if (d.T > 0) w.total += align_up(score_ws(prefill_score_desc(d)).total, 256);
    return w;
}

lvlm_score_desc prefill_score_desc(const lvlm_prefill_desc &d) {
    lvlm_score_desc s{};
    s.dtype = d.dtype; s.B = d.B; s.N = d.N; s.T = d.T; s.q_pos0 = d.N - d.T; s.Hq = d.Hq; s.Hkv = d.Hkv; s.hd = d.hd;
    s.img_begin = d.img_begin; s.n_img = d.n_img; s.causal = d.causal; s.scale = d.scale;
    s.q_stride_b = d.q_stride_b; s.q_stride_t = d.q_stride_n; s.q_stride_h = d.q_stride_h;
    s.k_stride_b = d.k_stride_b; s.k_stride_n = d.k_stride_n; s.k_stride_h = d.k_stride_h;
    s.sh_stride_b = d.sh_stride_b; s.sh_stride_h = d.sh_stride_h;
    return s;
}

hipError_t launch_prefill_attn(const Prof &prof, const lvlm_prefill_desc &d, const PrefillWs &w, char *ws, const void *q,
                               const void *k, const void *v, void *out, float *row_lse, float *score_head,
                               float *score_mean) {
    hipStream_t stream = prof.stream;
    const int es = d.dtype == LVLM_BF16 ? 2 : 4;
    PrefillArgs a{};
    a.q = static_cast<const char *>(q); a.k = static_cast<const char *>(k); a.v = static_cast<const char *>(v);
    a.out = static_cast<char *>(out);
    a.row_lse = row_lse;
    a.lse_t = d.T > 0 ? reinterpret_cast<float *>(ws + w.lse_t) : nullptr;
    a.B = d.B; a.N = d.N; a.Hq = d.Hq; a.Hkv = d.Hkv; a.G = d.Hq / d.Hkv; a.causal = d.causal; a.T = d.T;
    a.nqb = (d.N + 127) / 128;
    a.heads_per_xcd = (d.B * d.Hq + 7) / 8;
    a.scale = d.scale; a.scale_log2 = d.scale * kLog2e;
    a.qsb = d.q_stride_b * es; a.qsn = d.q_stride_n * es; a.qsh = d.q_stride_h * es;
    a.ksb = d.k_stride_b * es; a.ksn = d.k_stride_n * es; a.ksh = d.k_stride_h * es;
    a.vsb = d.v_stride_b * es; a.vsn = d.v_stride_n * es; a.vsh = d.v_stride_h * es;
    a.osb = d.o_stride_b * es; a.osn = d.o_stride_n * es; a.osh = d.o_stride_h * es;
    prof.begin("prefill_attn");
    if (d.dtype == LVLM_BF16) {
        const long long grid = (long long)a.heads_per_xcd * 8 * a.nqb;
        // the FAST kernels address a tile's rows by 32-bit offsets
        const bool fast = d.k_stride_n * es < (1ll << 26) && d.v_stride_n * es < (1ll << 26);
        const dim3 g((unsigned)grid);
        if (d.hd == 128) {
            if (fast) LVLM_LAUNCH(prof, prefill_attn_bf16_kernel, g, dim3(128), 0, stream, a);
            else LVLM_LAUNCH(prof, prefill_attn_safe_kernel<128>, g, dim3(128), 0, stream, a);
        } else {
            if (fast) LVLM_LAUNCH(prof, prefill_attn_d64_kernel, g, dim3(128), 0, stream, a);
            else LVLM_LAUNCH(prof, prefill_attn_safe_kernel<64>, g, dim3(128), 0, stream, a);
        }
    } else {
        const F32Form f = prefill_f32_form(d);
        a.deal = f.deal;
        const dim3 grid = f.dealt ? dim3(f.dealt) : dim3((unsigned)f.blocks, (unsigned)d.Hq, (unsigned)d.B);
#define LVLM_F32(KERNEL, ...)                                                                                              \
    if (d.hd == 128) LVLM_LAUNCH(prof, (KERNEL<128, __VA_ARGS__>), grid, dim3(256), 0, stream, a);                         \
    else LVLM_LAUNCH(prof, (KERNEL<64, __VA_ARGS__>), grid, dim3(256), 0, stream, a)
        if (f.shared && f.dealt) { LVLM_F32(prefill_attn_f32_shared_kernel, kDealt); }
        else if (f.shared) { LVLM_F32(prefill_attn_f32_shared_kernel, kPlain); }
        else if (f.two && f.grouped) { LVLM_F32(prefill_attn_f32_kernel, 2, kGrouped); }
        else if (f.two && f.dealt) { LVLM_F32(prefill_attn_f32_kernel, 2, kDealt); }
        else if (f.two) { LVLM_F32(prefill_attn_f32_kernel, 2, kPlain); }
        else if (f.grouped) { LVLM_F32(prefill_attn_f32_kernel, 1, kGrouped); }
        else if (f.dealt) { LVLM_F32(prefill_attn_f32_kernel, 1, kDealt); }
        else { LVLM_F32(prefill_attn_f32_kernel, 1, kPlain); }
#undef LVLM_F32
    }
    prof.end();
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || d.T <= 0) return e;
    // the scores of the last T rows from the normalisers just written: the column-sum pass alone
    const lvlm_score_desc sd = prefill_score_desc(d);
    const char *q_t = static_cast<const char *>(q) + (long long)(d.N - d.T) * d.q_stride_n * es;
    return launch_score(prof, sd, score_ws(sd), ws + w.score, q_t, k, a.lse_t, score_head, score_mean);
}

}  // namespace lvlm
