// Host rules of the fp32 prefill attention, and the arithmetic that host and kernels share.
#pragma once

#include "common.h"

namespace lvlm {

// ---- causal blocks dealt out to the compute units ----
// Workgroup number -> (head, block), for blocks that are on the chip beside each other: causal ones are as long as their
// last row, so what a compute unit is handed adds up to its time.  The eight XCDs -- workgroups with the same remainder -- get
// equally many heads, or parts of heads (every P-th block), neighbours in memory order; an XCD takes its parts' blocks longest first in
// turns of its 32 compute units, every other turn backwards: the unit with the longest block of one turn has the shortest of the next.
// Head by head instead, the first units had the longest block of every head (4 heads of 64 channels, 1503 tokens 42.1 -> 32.1 us, 2203
// 60.6 -> 43.5, 4103 138 -> 109; 16 x 4 heads, 1103 tokens 151 -> 137, 3603 1160 -> 1125).
// P is the one that leaves the fewest workgroups, idle ones among them: heads may be no multiple of eight, then the last XCD has fewer
// parts, and blocks none of P, then some parts have a block less.  (Always parts enough for eight equal shares: 577 heads of
// nine blocks 51 us, 44 so; 866 of two blocks, 128 channels, 378 -> 200.)  Of few levels parts mix up the order of lengths, and heads whole are
// preferred up to a fifteenth more workgroups (306 heads of four blocks, 128 channels 392 -> 288 us).
// An XCD works on as many parts at a time as have K and V of 6 MB between them, which its 4 MB L2 serves about as well as if they fitted: all of
// its heads side by side read K and V from memory once for every level (heads x tokens, all heads side by side -> in groups; the plain grid:
// 506 x 405 220 -> 178 us; 183, 234 x 988 466 -> 357; 371, of 128 channels 303 x 731 828 -> 692; 697.  3 MB and 9 MB: 0.6 % behind on
// average, at worst 7 and 14 %.)  The kernel that shares its tiles reads them an eighth as often, and groups only disturb its few levels (256
// heads x 500 95.6 -> 110).
// The plain grid stays for up to 256 blocks, one to a unit: nothing to level, and the divisions here are 0.4 us before the first load (154
// tokens 13.7 -> 14.2).  So it does up to 112 tokens, where no wave has more than one tile of 32 keys, but for more than 768 blocks of 64
// channels (three to a unit at once) of more than 64 tokens (plain -> dealt out, 64 channels: 122 heads x 61 tokens 6.4 -> 6.9, 121 x 88 7.7 ->
// 8.6, 394 x 112 24.6 -> 22.9; 128 channels: 180 x 106 31.9 -> 33.9).  Else, of some 400 shapes timed both ways, dealt out is 9 % faster on average
// and 2.5 % behind at worst (97 and 209 heads).
// The one grid dimension holds less than 2^32 threads: what does not fit it takes the plain grid too, whose three do.
struct BlockDeal {
    int heads, parts_log2, xcd_parts;      // parts of a head (log2), parts per XCD
    int group;                             // ... of which it takes so many at a time
};
// Returns the workgroups, or 0 for the plain grid.  rows: of a block.
inline unsigned deal_blocks(const lvlm_prefill_desc &d, int rows, BlockDeal &deal) {
    const long long heads = (long long)d.B * d.Hq, blocks = (d.N + rows - 1) / rows;
    deal = BlockDeal{};
    if (!d.causal || blocks <= 1 || blocks * heads <= 256) return 0;
    if (d.N <= 64 || (d.N <= 112 && (d.hd == 128 || blocks * heads <= 768))) return 0;
    long long grid = 0;
    for (int log2 = 0; log2 <= 3; ++log2) {
        const long long parts = ((heads << log2) + 7) / 8, levels = ((blocks - 1) >> log2) + 1, wgs = 8 * parts * levels;
        if (grid && (levels < 8 ? wgs * 16 >= grid * 15 : wgs >= grid)) continue;
        grid = wgs;
        deal = BlockDeal{(int)heads, log2, (int)parts, (int)parts};
    }
    const long long kv_bytes = 2ll * d.N * d.hd * sizeof(float), sharing = (long long)(d.Hq / d.Hkv) << deal.parts_log2;
    int group = 4;
    while (2 * group * kv_bytes <= sharing * (6 << 20)) group *= 2;
    if (rows < 128 && 2ll * deal.xcd_parts > 3ll * group) deal.group = group;      // (no small group left over)
    return grid * 256 < 1ll << 32 ? (unsigned)grid : 0;
}
// false: no block for this workgroup.  GROUPED: group < xcd_parts
template <bool GROUPED>
__host__ __device__ __forceinline__ bool dealt_block(const BlockDeal &deal, int n_blocks, unsigned wg, int &head, int &qb) {
    const int P = 1 << deal.parts_log2, xcd = wg & 7, seq = wg >> 3;
    const int levels = (n_blocks + P - 1) >> deal.parts_log2;
    int at = seq, first = 0, parts = deal.xcd_parts;
    if constexpr (GROUPED) {
        const int g = seq / (deal.group * levels);
        at = seq - g * deal.group * levels;
        first = g * deal.group;
        parts = min(deal.group, parts - first);
    }
    const int turn = at & ~31, last = min(turn + 31, parts * levels - 1);
    const int rank = (at & 32) ? turn + last - at : at;
    const int level = rank / parts, part = xcd * deal.xcd_parts + first + rank - level * parts;
    head = part >> deal.parts_log2;
    qb = n_blocks - 1 - ((level << deal.parts_log2) + (part & (P - 1)));
    return qb >= 0 && head < deal.heads;
}

// ---- the kernel that shares its tiles ----
// Whether the fp32 kernel that shares its tiles is the faster one, from 680 shapes timed both ways (1 to 960 heads, 20 to
// 4288 tokens).  It works in turns of 256 workgroups of 128 rows, each as long as its longest block: it needs turns that are
// nearly full.  Heads of 64 channels: where the four waves of the other kernel have equally many tiles (all but, of few
// blocks), it reads less per product -- 256 heads x 384 tokens 95 -> 64 us, 512 heads x 128 tokens 45 -> 28 us, but 128 heads x 800 causal 144 -> 167 us.  Of 128
// channels the other kernel is bound by reading K and V, and loses from three quarters of a turn on while the work is
// small: 256 heads x 128 tokens 57 -> 31 us, 512 heads x 256 290 -> 189 us, 384 of 94 tokens 57 -> 43 us.
// Causal blocks dealt out, beyond one turn, gain with their number (other kernel, dealt out too -> this one; before, with
// a head's blocks one after the other, four to a head came to the same compute units in every turn): 128 heads x 500 tokens
// 75.5 -> 66.7 us (91 before), 256 x 500 151 -> 109 (162), of 128 channels 448 x 512 591 -> 436 (625).  One turn of several blocks
// has nothing to level with and waits for the longest: 64 heads x 512 tokens 59.5 -> 45.4 us with the other kernel, 84 x 380 48.2 -> 39.7, of 128
// channels 56 x 500 110 -> 98, but 84 x 384 96.5 -> 89.4 with this one.  More than five blocks to a head stay with the other kernel: from 640 blocks on this one
// is faster (64 heads x 1400 tokens 193 -> 182 us, 64 x 3600 1070 -> 974; 40 x 1700 174 -> 184), but a row's sums are one chain here and four there:
// against 64 bits 9.0e-7 instead of 7.0e-7 (2-norm) at 3600 tokens.
inline bool f32_shares_tiles(const lvlm_prefill_desc &d) {
    const long long heads = (long long)d.B * d.Hq, nqb = (d.N + 127) / 128, wgs = heads * nqb;
    const int tiles = (d.N + 31) / 32, n16 = (d.N + 15) / 16;
    if (tiles < 2 && d.hd == 64) return false;
    if (d.causal && nqb > 5) return false;
    if (d.causal && wgs <= 256 && nqb > (d.hd == 64 ? 1 : 3)) return false;
    const double fill = (double)wgs / (double)((wgs + 255) / 256 * 256);
    // tiles a wave of the other kernel takes in turn, over its blocks of 16 rows; tiles a workgroup of this one takes
    long long in_turn = 0, shared = 0;
    if (d.causal) {
        for (int x = 0; x < n16; ++x) in_turn += ((x < n16 - 1 ? 16 * x + 16 : d.N) + 127) / 128;
        for (int x = 0; x < nqb; ++x) shared += (x < nqb - 1 ? 4 * (x + 1) : tiles);
    } else {
        in_turn = (long long)n16 * ((tiles + 3) / 4);
        shared = nqb * tiles;
    }
    if (d.hd == 64) return fill > 0.9 && (double)(4 * in_turn) > (nqb <= 3 ? 6.7 : 7.8) * (double)shared;
    return fill > 0.9 || (fill > (d.causal ? 0.78 : 0.71) && heads * in_turn <= 36 * 256);
}

// ---- the kernel a call takes ----
struct F32Form {
    bool shared;          // tiles shared by four waves of 32 rows, else blocks of 16 rows
    bool two;             // ... two of them per workgroup
    long long blocks;     // workgroups per head
    unsigned dealt;       // workgroups in all if the blocks are dealt out, else 0
    bool grouped;         // ... and an XCD's heads taken in groups
    BlockDeal deal;
};
inline F32Form prefill_f32_form(const lvlm_prefill_desc &d) {
    F32Form f{};
    f.shared = f32_shares_tiles(d);
    // Not shared: one block of 16 rows per workgroup; two (each K and V operand feeds two products, 64 bytes of L2 traffic per
    // product instead of 128) once that still leaves many rounds of the chip: it is 3-4 % faster from about
    // 16000 workgroups on and slower by up to 1.7 times below 4000
    const long long n16 = (d.N + 15) / 16;
    f.two = !f.shared && n16 * d.B * d.Hq >= 16384;
    const int rows = f.shared ? 128 : f.two ? 32 : 16;
    f.blocks = (d.N + rows - 1) / rows;
    f.dealt = deal_blocks(d, rows, f.deal);
    f.grouped = f.dealt && f.deal.group < f.deal.xcd_parts;
    return f;
}

}  // namespace lvlm
