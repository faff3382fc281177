// retopk_plan.h -- launch plans that are plain arithmetic on the host: how the work
// of a call is split over blocks.  No HIP in it, so that a CPU program can check
// the rules over whole ranges of sizes.  Not part of the public C ABI.
#pragma once

#include <stdint.h>

namespace retopk {

constexpr int kCUs = 256;             // compute units of the chip

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// Full (dense) attention: rows of a chunk, which one block takes
// ---------------------------------------------------------------------------

constexpr int kDenseRows = 1024;      // f32: most rows of a chunk (its scores sit in LDS)
constexpr int kDenseRowsMin = 256;    // a 32-row tile for each of a block's 8 waves
constexpr int kDenseRowsMax = 65536;  // no sum is a chain of more than about 130 flushes
constexpr int kDenseBlocks = 240;     // bf16 blocks of one round
constexpr int kDenseFill = 160;       // bf16 blocks that use up the HBM bandwidth together
constexpr int kDenseRounds = 16;      // rounds of blocks compared
constexpr int kDenseRoundBytes = 12 << 20;   // what HBM reads in the 2 us a round costs

// bf16 (k_dense_wave): whole 32-row tiles, in chunks that fill whole rounds of one
// block per CU (most builds hold one by their registers, and a few blocks past 256 start
// a second round: 128K rows of 8 groups take 99 us in 256 blocks, 111-131 in 264).  160
// blocks read at the full rate (16K rows of 72 groups: 109 us in 216 blocks, 112 in 504,
// 144 in 288), so where the whole chunks of one round are that many, that is the split.
// Otherwise (129-159 groups, more than 256, or chunks past kDenseRowsMax) it is the
// number of rounds with the least work, idle slots of the last round included, and the
// least starts, about 2 us a round (16K rows: 136 groups take 235 us in 136 blocks and
// 205 in 680, 264 groups 541 in 264 and 398 in 2112; the kernel before, in chunks of
// 1024 rows and two blocks a CU: 213 and 398), in chunks of at least two tiles a wave
// (600 rows of 320 groups: 34.7 us in one chunk a group, 38.0 in three of 256 rows).
inline int64_t dense_round_rows(int64_t len, int64_t chunks)
{
    const int64_t r = ceil_div(ceil_div(len, chunks), 32) * 32;
    return r < kDenseRowsMin ? kDenseRowsMin : r;
}

// The fewest rounds whose chunks stay within kDenseRowsMax rows.
inline int64_t dense_first_round(int64_t groups, int64_t len)
{
    return ceil_div(groups * ceil_div(len, kDenseRowsMax), kCUs);
}

// Chunks a group in one round: 240 blocks and not 256 where the groups allow it, the
// faster by 0.8 % (128K rows, 8 groups: 96.7 us in 240, 97.5 in 248).
inline int64_t dense_one_round(int64_t groups) { return (groups <= kDenseBlocks ? kDenseBlocks : kCUs) / groups; }

// Chunks that start j MiB apart, give or take j * 8 KiB, meet on the same memory
// channels, at the ends of the band above all (920 000 rows of one group of 8, d = 128:
// 101.5 and 100.0 us in chunks of 4064 and 4128 rows, 93.4 in 4032 and 4160; 1 840 000
// rows at d = 64: 103.2 and 102.8 us in 8128 and 8256, 89.9 in 8320), and inside it at
// d = 64 with several groups (224 000 rows of 8: 88-90 us, 86 outside).  At most 1.6 %
// more rows step over it.
inline bool dense_stride_collides(int64_t bytes)
{
    const int64_t j = (bytes + (1 << 19)) >> 20, off = bytes - (j << 20);
    return j > 0 && (off < 0 ? -off : off) <= j * 8192;
}

// Rows of a chunk of `groups` KV groups of len rows, d elements a row.
inline int dense_wave_rows(int64_t groups, int64_t len, int d)
{
    const int64_t one = dense_one_round(groups);
    int64_t r = one > 0 ? dense_round_rows(len, one) : 0;
    if (one * groups < kDenseFill || r > kDenseRowsMax) {
        const int64_t m0 = dense_first_round(groups, len), start = kDenseRoundBytes / (4 * d);
        int64_t best = -1;
        for (int64_t m = m0; m < m0 + kDenseRounds; ++m) {
            int64_t rows = dense_round_rows(len, kCUs * m / groups);
            if (rows < 2 * kDenseRowsMin) rows = 2 * kDenseRowsMin;
            const int64_t blocks = groups * ceil_div(len, rows), last = blocks % kCUs;
            const int64_t slots = blocks - last + (last == 0 || last > kDenseFill ? last : kDenseFill);
            // a block takes as long as its longest wave
            const int64_t cost = slots * ceil_div(rows, kDenseRowsMin) * kDenseRowsMin + ceil_div(blocks, kCUs) * start;
            if (best < 0 || cost < best) {
                best = cost;
                r = rows;
            }
        }
    }
    while (dense_stride_collides(r * d * 2)) r += 32;
    return (int)r;
}

// The most chunks a group dense_wave_rows gives any length up to max_len.
inline int64_t dense_wave_chunks(int64_t groups, int64_t max_len)
{
    const int64_t one = dense_one_round(groups);
    if (one * groups >= kDenseFill && max_len <= one * kDenseRowsMax) return one;
    const int64_t most = kCUs * (dense_first_round(groups, max_len) + kDenseRounds - 1) / groups;
    const int64_t fine = ceil_div(max_len, kDenseRowsMin);
    return most < fine ? most : fine;
}

// f32 (k_dense, up to two blocks a CU): the fewest rows with at most one block per CU, else
// whole chunks.  More blocks than CUs pay more for their reductions than they win (8
// groups of d = 128: 4K rows 18.2 us in 128 chunks of 256 rows, 27.3 in 32 of 1024; 16K
// rows 35.9 in 512 of 256, 31.7 in 256 of 512, 33.0 in 128 of 1024; 64K rows 110.7 in
// 1024 of 512, 103.4 in 512 of 1024).
inline int dense_f32_rows(int64_t groups, int64_t len)
{
    int r = kDenseRowsMin;
    while (r < kDenseRows && groups * ceil_div(len, r) > kCUs) r *= 2;
    return r;
}

// The most chunks a group dense_f32_rows gives any length up to max_len.
inline int64_t dense_f32_chunks(int64_t groups, int64_t max_len)
{
    const int64_t spread = ceil_div(kCUs, groups), most = ceil_div(max_len, kDenseRows);
    return spread > most ? spread : most;
}

// ---------------------------------------------------------------------------
// Batched prefill initialisation (bf16, retopk_prefill.hip)
// ---------------------------------------------------------------------------

constexpr int kPfThreads = 512;
constexpr int kPfWaveCols = 128;      // virtual queries held by one wave
constexpr int kPfMinList = 4096;      // smallest list capacity of a virtual head
// Device memory of the batched prefill (the lists or score rows of U positions of
// every head).  One workspace a device is kept between calls while it has handles:
// allocating it per call cost 0.45 ms of an 8.9 ms prefill at 128K, and 17 ms where
// other handles' memory came and went between the calls.  257 MiB hold 256 positions of
// 32 heads at K = 512 (32 KiB of list a virtual head and 8 bytes beside it), past which
// the key reads per launch are no longer what bounds it.
constexpr int64_t kPfWorkspaceBytes = (int64_t)257 << 20;
struct PrefillPlan {
    int64_t cap;               // list capacity of a virtual head
    int64_t rows16;            // rows of a score row: the prompt in whole tiles
    int64_t row_bytes;         // memory of a virtual head's list or score row
    int64_t positions;         // positions a launch takes
    bool lists;                // launches keep lists (prompts of 2 cap rows on), else score rows
    int64_t again_at, over_at; // offsets of the overflowed lists' bounds and of the words
    int64_t bytes;             // the whole workspace
};

// n positions of `heads` query heads, G to a KV group, of a prompt of prefill_len rows.
inline PrefillPlan prefill_plan(int64_t heads, int G, int64_t K, int64_t n, int64_t prefill_len)
{
    PrefillPlan p;
    // eight times K, four times what the bound is expected to leave
    p.cap = 8 * K > kPfMinList ? 8 * K : kPfMinList;
    p.rows16 = ceil_div(prefill_len, 16) * 16;
    // A list of cap ranks, which also holds its group maxima (at most 8 K floats), or a
    // score row of up to 2 cap rows; beside it the count and the bound.
    p.row_bytes = p.rows16 * 4 < p.cap * 8 ? p.rows16 * 4 : p.cap * 8;
    p.lists = p.rows16 >= 2 * p.cap;
    const int64_t per_u = heads * (p.row_bytes + 8);
    int64_t U = kPfWorkspaceBytes / per_u;
    // whole 128-query tiles where the budget allows
    int gcd = G, m = kPfWaveCols;
    while (m) {
        const int r = gcd % m;
        gcd = m;
        m = r;
    }
    const int64_t unit = kPfWaveCols / gcd;
    if (U >= unit) U -= U % unit;
    p.positions = U < 1 ? 1 : (U > n ? n : U);
    // the virtual heads' memory, then the bounds that every position's lists leave and
    // its overflow word
    p.again_at = ceil_div(per_u * p.positions, 256) * 256;
    p.over_at = p.again_at + n * heads * 8;
    p.bytes = p.over_at + n * 4;
    return p;
}

// Grid of k_pf_scan: blocks of wc * 128 virtual queries times a chunk of key rows.
struct PrefillGrid {
    int wc, col_blocks, chunks;
    int64_t chunk_rows;
};

// `cols` virtual queries per KV group over the rows of `groups` KV groups: as many waves
// side by side along the queries as there are 128-query tiles (up to the block's 8), and
// key chunks, no shorter than 512 rows, for whole rounds of blocks.  A CU holds one
// block (by its registers), a (KV group, chunk) pair's blocks run on one XCD of 32 CUs,
// and a few blocks too many cost a round (12/2 heads, 128K rows: 757 us in 258
// blocks of 43 chunks, 491 in 240 of 40).  Of 16 numbers of rounds the shortest
// counts; a block's start (its queries, 256 KB) costs as much as 170 rows (two rounds of
// half the rows took 4 % longer than one).
inline PrefillGrid prefill_grid(int64_t cols, int64_t groups, int64_t rows)
{
    constexpr int64_t kXcds = 8, kStartRows = 170, kRounds = 16;
    PrefillGrid g;
    const int64_t tiles = ceil_div(cols, kPfWaveCols);
    g.wc = 1;
    while (g.wc < kPfThreads / 64 && g.wc < tiles) g.wc *= 2;
    const int64_t cb = ceil_div(tiles, g.wc), most = ceil_div(rows, 512);
    g.col_blocks = (int)cb;
    const int64_t unit = 16 * (kPfThreads / 64 / g.wc);
    const int64_t slots = kCUs / kXcds;             // of an XCD
    const int64_t m0 = ceil_div(ceil_div(groups, kXcds) * cb, slots);
    int64_t best = -1;
    for (int64_t m = m0; m < m0 + kRounds; ++m) {
        int64_t n = slots * m / cb * kXcds / groups;
        if (n > most) n = most;
        const int64_t chunk = ceil_div(ceil_div(rows, n), unit) * unit;
        const int64_t pairs = groups * ceil_div(rows, chunk);
        const int64_t cost = ceil_div(ceil_div(pairs, kXcds) * cb, slots) * (chunk + kStartRows);
        if (best < 0 || cost < best) {
            best = cost;
            g.chunk_rows = chunk;
        }
    }
    g.chunks = (int)ceil_div(rows, g.chunk_rows);
    return g;
}

}  // namespace retopk
