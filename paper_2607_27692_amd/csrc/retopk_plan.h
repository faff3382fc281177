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

}  // namespace retopk
