// retopk_prefill.hip -- gfx950 kernels of the batched prefill initialisation
// (bf16): the Exact Top-K support of many prompt positions of every head at once
// (Sec. 3.3), each over its own causal prefix.
//
// The scores of Eq. 4 for U positions x G heads of a KV group (the group's
// "virtual queries", vq = u * G + j) against its keys are one matrix product of
// depth d on the matrix cores (v_mfma_f32_16x16x32_bf16).  Storing them would
// cost 4 bytes per (position, head, key), so the product runs twice instead and
// only entries that can be selected leave the chip:
//   k_pf_scan<BOUND>    over a sample of the key tiles: the maximum of each group
//                       of 4 * 2^lt sampled keys, per virtual query;
//   k_pf_bound          the K-th largest of those maxima: K distinct keys score
//                       at least that much, so it bounds the K-th largest score
//                       from below, whatever the scores are;
//   k_pf_scan<COLLECT>  over all keys: the entries at or above the bound, as
//                       ranks appended to the virtual head's list;
//   k_pf_select         the exact Top-K of each list, in index order (through an
//                       index bitmap), and the cache entry.
// For exchangeable keys the bound leaves about F * K entries (F: one key tile in
// F is sampled).  Keys whose high scores lie in long runs leave more, up to the
// list's capacity and past it, and so do thousands of equal scores.  The K-th
// largest entry of a full list, whichever entries it holds, bounds the head's K-th
// from below again, and more tightly: k_pf_select stores it, k_pf_raise makes it
// the head's bound, and k_pf_scan<RECOLLECT> collects the entries at or above it, by
// rank (score, then index), so that ties are cut too (512 positions of 32/8 heads at
// 128K, K = 512: keys with neighbour correlation 0.999 2.2 ms, 18.3 with score rows;
// half the keys one row 3.1 ms, 29.0; all of them 14.0 ms, 23.3).  Positions with a list
// that still overflows after a few such runs are scored with k_pf_scan<DENSE>, which
// stores every score row, and the same k_pf_select; so are prompts of fewer than two
// lists' rows.
#include "retopk_internal.h"
#include "retopk_device.h"

#include <cfloat>

namespace retopk {

namespace {

constexpr int kPfWaves = kPfThreads / 64;
constexpr int kPfQueue = 512;         // accumulator quads a wave queues in LDS
constexpr int kPfMaxima = 4;          // tile groups whose maxima a wave gathers in LDS
constexpr int kPfSelThreads = 256;    // k_pf_bound and k_pf_select blocks
constexpr int kPfBins = 1024;         // value-linear bins
constexpr int kPfTie = 64;            // entries of the last bin ranked by lane
constexpr int kPfSegBits = 131072;    // indices per bitmap pass

// A raw score below t by more than the rounding that can make two raw scores one scaled
// score, and finite where t is +inf.
__device__ __forceinline__ float raw_bound(float t)
{
    return t < FLT_MAX ? t - fabsf(t) * 1.0e-6f - 1.0e-37f : FLT_MAX;
}

// The larger of two finite scores, without the quieting that fmaxf does first.
__device__ __forceinline__ float fmax_nan(float x, float y) { return __builtin_elementwise_maximum(x, y); }

}  // namespace

// k_pf_scan: block = 8 waves, wc of them side by side along the virtual queries
// (128 each, whose vectors stay in 128 VGPRs for the whole block at d = 128) and
// wk_n = 8 / wc along the key tiles of the block's chunk.  Lane l supplies key row
// and query l % 16 for dims 8 (l / 16) .. + 7 of each 32-dim step and receives keys
// 4 (l / 16) .. + 3 of query l % 16.  Keys go through LDS in stages of 8 tiles, in
// the lane order of the MFMA operand (one 16-byte read a lane and step, without
// bank conflicts): each wave fetches one tile of the next stage into registers
// before it scores the current one and stores it to the other half afterwards, so
// that a stage costs one barrier and no load is waited for with an idle matrix
// core.  Blocks on the same chunk run on one XCD (equal blockIdx % 8) and share
// its keys through that L2.
// For 256 positions of 32 heads at 128K and K = 512 (1024 queries a group, 275 GFLOP
// over all keys): BOUND over half the keys 131 us, COLLECT 387 us, of which about
// 100 us append 1100 entries a virtual head (F = 1, a tighter bound from every key,
// costs another 130 us of BOUND; F = 4 twice the appends).  The matrix cores are busy
// 46 % and 32 % of that; a build without LDS staging (each wave loading its own
// tiles) took 292 and 442 us, and the kernel that stored every score and counted it
// in LDS histograms 2500 us for the same positions, its filter 1100 us.
template <int D, int MODE>
__global__ __launch_bounds__(kPfThreads, 2) void k_pf_scan(PfArgs a)
{
    constexpr int KS = D / 32, CT = kPfWaveCols / 16;
    constexpr bool LIST = MODE == PF_COLLECT || MODE == PF_RECOLLECT;
    __shared__ int s_vh[kPfWaves * kPfWaveCols];    // virtual head of a column, -1: padding
    __shared__ u32x4_t s_key[2][kPfWaves][KS][64];
    constexpr int CW = LIST ? kPfWaves : 1, CQ = LIST ? kPfQueue : 1;
    __shared__ f32x4_t s_qv[CW][CQ];                 // queued quads: raw scores of 4 keys
    __shared__ uint32_t s_qi[CW][CQ];                // their column << 24 | first key
    __shared__ uint32_t s_cur[CW][kPfWaveCols];
    __shared__ float s_thr[LIST ? kPfWaves * kPfWaveCols : 1];
    __shared__ float s_mx[MODE == PF_BOUND ? kPfWaves : 1][MODE == PF_BOUND ? kPfMaxima : 1][CT][64];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = a.wc, wk_n = kPfWaves / wc, wcol = wave & (wc - 1), wk = wave / wc;
    // the col_blocks blocks of a (KV group, key chunk) pair share blockIdx % 8
    const int j = (int)blockIdx.x;
    const int pair = (j & 7) + 8 * (j / (8 * a.col_blocks));
    const int cb = (j >> 3) % a.col_blocks;
    if (pair >= a.pairs) return;
    const int grp = pair / a.chunks, chunk = pair - grp * a.chunks;
    const int b = grp / a.Hkv, g = grp - b * a.Hkv;
    const int BH = a.B * a.Hq, nvq = a.G * a.U;
    const int vq0 = cb * wc * kPfWaveCols;

    // The key tiles of the waves at key position x: its iteration it covers rows
    // row_of(x, it) .. + 15, for it < n_it(x).
    const uint16_t *kbase = a.k + ((int64_t)b * a.Hkv + g) * a.max_len * D;
    const int64_t len_max = a.len0 + a.U - 1;
    int64_t k0 = 0;
    int span;                  // tile groups (BOUND) or tiles of the chunk
    if constexpr (MODE == PF_BOUND) {
        // tile groups, 2^lt tiles each, spread over the prefix (tiles
        // F * (r + n_groups * s)), all below the shortest prefix
        const int r1 = (chunk + 1) * a.chunk_groups < a.n_groups ? (chunk + 1) * a.chunk_groups : a.n_groups;
        span = r1 - chunk * a.chunk_groups;
    } else {
        k0 = (int64_t)chunk * a.chunk_rows;
        const int64_t k1 = k0 + a.chunk_rows < len_max ? k0 + a.chunk_rows : len_max;
        span = k0 < k1 ? (int)((k1 - k0 + 15) >> 4) : 0;
    }
    const int lt = MODE == PF_BOUND ? a.lt : 0;
    const int per = MODE == PF_BOUND ? a.chunk_groups / wk_n : 0;   // tile groups of a key position
    auto group0 = [&](int x) { return chunk * a.chunk_groups + x * per; };
    auto iters = [&](int x) {
        if constexpr (MODE == PF_BOUND) {
            const int n = span - x * per;
            return (n < 0 ? 0 : n < per ? n : per) << lt;
        } else {
            return x < span ? (span - x + wk_n - 1) / wk_n : 0;
        }
    };
    auto row_of = [&](int x, int it) -> int64_t {
        if constexpr (MODE == PF_BOUND) {
            const int r = group0(x) + (it >> lt), s = it & ((1 << lt) - 1);
            return ((int64_t)r + (int64_t)a.n_groups * s) * a.F * 16;
        } else {
            return k0 + ((int64_t)it * wk_n + x) * 16;
        }
    };
    // one wave of each SIMD's two goes first, so that their matrix and vector phases
    // alternate instead of coinciding (COLLECT of 256 positions at 128K: 398 -> 380 us)
    if (wave < kPfWaves / 2) __builtin_amdgcn_s_setprio(2);
    const int n_it = iters(wk);
    const int n_stage = (iters(0) + wc - 1) / wc;       // the longest sequence
    if (n_stage == 0) return;                           // block-uniform

    // The tile this wave fetches in a stage: iteration stage * wc + wave % wc of the
    // waves at key position wave / wc (rows past the last are clamped, not used).
    auto fetch = [&](u32x4_t (&kv)[KS], int stage) {
        int64_t r = row_of(wk, stage * wc + wcol) + col;
        r = r < len_max ? r : len_max - 1;
        const u32x4_t *rp = (const u32x4_t *)(kbase + r * D);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kv[ks] = rp[ks * 4 + kq];
    };
    u32x4_t nx[KS];
    fetch(nx, 0);
    for (int i = tid; i < wc * kPfWaveCols; i += kPfThreads) {
        const int vq = vq0 + i;
        s_vh[i] = vq < nvq ? (vq / a.G) * BH + b * a.Hq + g * a.G + vq % a.G : -1;
    }
    __syncthreads();
    const int cbase = wcol * kPfWaveCols;            // this wave's columns in s_vh
    bf16x8_t qb[CT][KS];
    float thr[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int vh = s_vh[cbase + ct * 16 + col];
        const int vhe = vh >= 0 ? vh : b * a.Hq + g * a.G;
        const int u = vhe / BH, bh = vhe - u * BH;
        const u32x4_t *qr = (const u32x4_t *)(a.q + (int64_t)bh * a.q_head_stride + (int64_t)u * D);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qb[ct][ks] = __builtin_bit_cast(bf16x8_t, qr[ks * 4 + kq]);
        thr[ct] = LIST && vh >= 0 ? a.thr[vh] : INFINITY;
        if (LIST) s_thr[cbase + ct * 16 + col] = thr[ct];   // same value from each wave and kq
    }

    // --- COLLECT, RECOLLECT: the wave's queue of entries and its append to the lists
    uint32_t qn = 0u;
    auto flush = [&]() {
        uint32_t *cur = s_cur[wave];
        cur[lane] = 0u;
        cur[lane + 64] = 0u;
        wave_lds_fence();
        // a quad's entries at or above its column's bound, as a bit mask
        auto passing = [&](uint32_t i, uint32_t &c, f32x4_t &v) {
            c = s_qi[wave][i] >> 24;
            v = s_qv[wave][i];
            if constexpr (MODE == PF_RECOLLECT) {
                const int vh = s_vh[cbase + c];
                const uint64_t least = vh >= 0 ? a.again[vh] : 0ull;
                const uint32_t row = s_qi[wave][i] & 0xFFFFFFu;
                uint32_t m = 0u;
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (least != 0ull && rank_of(v[x] * a.inv_sqrt_d, row + x) >= least) m |= 1u << x;
                return m;
            }
            const float t = s_thr[cbase + c];
            return (v[0] >= t ? 1u : 0u) | (v[1] >= t ? 2u : 0u) | (v[2] >= t ? 4u : 0u) | (v[3] >= t ? 8u : 0u);
        };
        for (uint32_t i = lane; i < qn; i += 64) {
            uint32_t c;
            f32x4_t v;
            const uint32_t m = passing(i, c, v);
            atomicAdd(&cur[c], (uint32_t)__popc(m));
        }
        wave_lds_fence();
        uint32_t base[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t c = cur[lane + 64 * h];
            const int vh = s_vh[cbase + lane + 64 * h];
            base[h] = c != 0u && vh >= 0 ? atomicAdd(&a.cnt[vh], c) : 0u;
        }
        cur[lane] = base[0];
        cur[lane + 64] = base[1];
        wave_lds_fence();
        for (uint32_t i = lane; i < qn; i += 64) {
            uint32_t c;
            f32x4_t v;
            const uint32_t m = passing(i, c, v), row = s_qi[wave][i] & 0xFFFFFFu;
            uint32_t at = atomicAdd(&cur[c], (uint32_t)__popc(m));
            const int vh = s_vh[cbase + c];
            uint64_t *list = a.list + (int64_t)(vh >= 0 ? vh : 0) * a.cap;
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if ((m >> x) & 1u) {
                    if (at < (uint32_t)a.cap && vh >= 0) list[at] = rank_of(v[x] * a.inv_sqrt_d, row + x);
                    ++at;
                }
        }
        wave_lds_fence();
        qn = 0u;
    };
    // Queues every quad of accumulators (4 keys of a column) whose largest reaches the
    // column's bound, without a branch; flush() sorts out which of the 4 do.
    auto collect = [&](const f32x4_t (&acc)[CT], uint32_t row) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            if (qn + 64u * (CT / 4) > (uint32_t)kPfQueue) flush();
#pragma unroll
            for (int c = 0; c < CT / 4; ++c) {
                const int ct = h * (CT / 4) + c;
                const f32x4_t x = acc[ct];
                const bool pass = fmax_nan(fmax_nan(x[0], x[1]), fmax_nan(x[2], x[3])) >= thr[ct];
                const uint64_t m = __ballot(pass);
                const uint32_t at = qn + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (pass) {
                    s_qv[wave][at] = x;
                    s_qi[wave][at] = (uint32_t)(ct * 16 + col) << 24 | (row + 4 * kq);
                }
                qn += (uint32_t)__popcll(m);
            }
        }
    };

    // --- BOUND: running maxima of the current tile group
    float mx[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) mx[ct] = -INFINITY;

    // Scores of the tile in kv; then kv takes the wave's next tile from LDS.
    auto score = [&](u32x4_t (&kv)[KS], int it, const u32x4_t (*next)[64]) {
        f32x4_t acc[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8_t, kv[ks]), qb[ct][ks], acc[ct], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);   // the MFMAs in this order, eight chains side by side
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kv[ks] = next[ks][lane];
        if constexpr (MODE == PF_BOUND) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                mx[ct] = fmax_nan(fmax_nan(mx[ct], fmax_nan(acc[ct][0], acc[ct][1])),
                                  fmax_nan(acc[ct][2], acc[ct][3]));
            if (((it + 1) & ((1 << lt) - 1)) == 0) {
                const int gi = it >> lt, slot = gi & (kPfMaxima - 1);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    s_mx[wave][slot][ct][lane] = mx[ct];
                    mx[ct] = -INFINITY;
                }
                if (slot == kPfMaxima - 1 || it + 1 == n_it) {
                    // 4 lanes a column, one tile group each: 64 bytes of a row of maxima
                    wave_lds_fence();
                    const int c4 = lane >> 2, s4 = lane & 3;
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        const float *src = &s_mx[wave][s4][ct][c4];
                        const int vh = s_vh[cbase + ct * 16 + c4];
                        if (vh >= 0 && s4 <= slot)
                            *(float4 *)(a.maxima + (int64_t)vh * 2 * a.cap + 4 * (group0(wk) + gi - slot + s4)) =
                                make_float4(src[0], src[16], src[32], src[48]);
                    }
                    wave_lds_fence();
                }
            }
        } else {
            const int64_t row = row_of(wk, it);
            if constexpr (LIST) {
                // past the shortest prefix of the launch a column's own limit counts
                if (row + 16 > a.len0) {
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        const int64_t clen = a.len0 + s_vh[cbase + ct * 16 + col] / BH;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (row + 4 * kq + i >= clen) acc[ct][i] = -INFINITY;
                    }
                }
                collect(acc, (uint32_t)row);
            } else {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const int vh = s_vh[cbase + ct * 16 + col];
                    // rows past a column's prefix are stored too (inside the row's
                    // stride) and never read
                    if (vh >= 0)
                        *(float4 *)(a.scores + (int64_t)vh * a.score_stride + row + 4 * kq) =
                            make_float4(acc[ct][0] * a.inv_sqrt_d, acc[ct][1] * a.inv_sqrt_d,
                                        acc[ct][2] * a.inv_sqrt_d, acc[ct][3] * a.inv_sqrt_d);
                }
            }
        }
    };
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s_key[0][wave][ks][lane] = nx[ks];
    __syncthreads();
    for (int st = 0; st < n_stage; ++st) {
        u32x4_t ny[KS];
        fetch(ny, st + 1 < n_stage ? st + 1 : st);
        const int it0 = st * wc, m = n_it - it0 < wc ? n_it - it0 : wc;
        const u32x4_t (*tile)[KS][64] = &s_key[st & 1][wk * wc];
        u32x4_t kv[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kv[ks] = tile[0][ks][lane];
        for (int i = 0; i < m; ++i) score(kv, it0 + i, tile[i + 1 < m ? i + 1 : i]);
        // the readers of the other half passed the previous barrier
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s_key[(st + 1) & 1][wave][ks][lane] = ny[ks];
        // The waves' queues fill alike: emptied here they hold up the barrier together,
        // and no key load in flight has to wait for the appends.
        if constexpr (LIST) {
            if (qn >= (uint32_t)kPfQueue * 3 / 8) flush();
        }
        __syncthreads();
    }
    if constexpr (LIST) {
        if (qn != 0u) flush();
    }
}

// k_pf_bound: per virtual head, a lower bound of its K-th largest raw score (q.k
// before the 1/sqrt d factor): the smallest of the maxima in the bins at or above
// the one that holds the K-th largest of them (value-linear bins, so at least K
// maxima are at or above it), less the rounding.  Clears the head's list.
template <int VPT>
__global__ __launch_bounds__(kPfSelThreads) void k_pf_bound(PfArgs a)
{
    constexpr int NT = kPfSelThreads, NW = NT / 64;
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kPfBins];
    __shared__ float s_red[NW];
    const int tid = threadIdx.x, vh = blockIdx.x, M = 4 * a.n_groups;
    const float *mx = a.maxima + (int64_t)vh * 2 * a.cap;
    for (int i = tid; i < kPfBins; i += NT) s_hist[i] = 0u;
    float x[VPT];              // loads in flight together; padded with the first
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int i = 0; i < VPT; ++i) x[i] = mx[tid + i * NT < M ? tid + i * NT : 0];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        lo = fminf(lo, x[i]);
        hi = fmaxf(hi, x[i]);
    }
    auto smaller = [](float x, float y) { return fminf(x, y); };
    lo = block_reduce<NT>(lo, s_red, smaller);
    hi = block_reduce<NT>(hi, s_red, [](float x, float y) { return fmaxf(x, y); });
    float t = lo;
    if (lo == -INFINITY) {
        // masked rows (scores of -inf) share the lowest bin and do not stretch the others
        lo = INFINITY;
#pragma unroll
        for (int i = 0; i < VPT; ++i) lo = fminf(lo, x[i] > -INFINITY ? x[i] : INFINITY);
        lo = block_reduce<NT>(lo, s_red, smaller);
    }
    const float range = hi - lo;
    if (range > 0.0f && range < 3.0e38f) {      // block-uniform
        const float scale = (float)(kPfBins - 1) / range;
        int bin[VPT];
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            bin[i] = min((int)fmaxf((x[i] - lo) * scale, 0.0f), kPfBins - 1);
            if (tid + i * NT < M) atomicAdd(&s_hist[bin[i]], 1u);
        }
        __syncthreads();
        uint32_t bstar, above, cnt;
        wave_find_bin<kPfBins>(s_hist, (uint32_t)a.K, bstar, above, cnt);
        t = INFINITY;
#pragma unroll
        for (int i = 0; i < VPT; ++i)
            if (bin[i] >= (int)bstar) t = fminf(t, x[i]);
        t = block_reduce<NT>(t, s_red, smaller);
    }
    if (tid == 0) {
        a.thr[vh] = raw_bound(t);
        a.cnt[vh] = 0u;
        a.overflow[vh / (a.B * a.Hq)] = 0u;
    }
}

// k_pf_raise: prepares k_pf_scan<RECOLLECT>, one thread per virtual head: the raw score
// that the stored rank implies as the bound of an overflowed list, which is cleared; no
// raw score for the others.
__global__ __launch_bounds__(kPfSelThreads) void k_pf_raise(PfArgs a)
{
    const int vh = blockIdx.x * kPfSelThreads + threadIdx.x, BH = a.B * a.Hq;
    if (vh >= BH * a.U) return;
    const uint64_t least = a.again[vh];
    const float s = key_score(rank_key(least));
    a.thr[vh] = least == 0ull ? INFINITY : raw_bound(s > -FLT_MAX ? s / a.inv_sqrt_d : -INFINITY);
    a.cnt[vh] = 0u;
    if (vh % BH == 0) a.overflow[vh / BH] = 0u;
}

// k_pf_select: one block per virtual head: the Top-K (Eq. 1) of its entries -- its
// list, or every score of its row (DENSE) -- written to the cache in index order
// with the normalised query.  Bins linear in the score locate the K-th largest
// entry in one bin, ranked exactly when it holds at most kPfTie entries; heavier
// ties take a radix select on the 64-bit ranks.  The selected indices pass through
// a bitmap, which orders them without a sort (a bitmap pass covers kPfSegBits
// rows).  Of a list that overflowed (cap >= 8 K entries) only the K-th largest entry is
// found, the bound of its next run.  A virtual head's list is about 1100 entries at K = 512, held in
// registers; longer ones are read three times, after the first from the caches.
// 22 KB of LDS a block keep seven blocks on a CU.
template <int D, bool DENSE>
__global__ __launch_bounds__(kPfSelThreads) void k_pf_select(PfArgs a)
{
    constexpr int NT = kPfSelThreads, NW = NT / 64;
    constexpr int EPT = 8;
    constexpr int WORDS = kPfSegBits / 32, WPT = WORDS / NT;   // 16 words per thread
    // word i sits at i + i / WPT, so that threads reading their WPT words side by
    // side hit different banks
    __shared__ uint32_t s_bits[WORDS + NT];
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kPfBins];
    __shared__ uint64_t s_tie[kPfTie];
    __shared__ uint64_t s_red64[NW];
    __shared__ uint32_t s_red[NW], s_redmin[NW];
    __shared__ uint32_t s_ntie;
    __shared__ float s_qbar[D];
    __shared__ double s_redd[NW];
    const int tid = threadIdx.x, lane = tid & 63, vh = blockIdx.x;
    const int BH = a.B * a.Hq, u = vh / BH, bh = vh - u * BH;
    const int64_t clen = a.len0 + u;
    const int K = a.K;
    const float *row = DENSE ? a.scores + (int64_t)vh * a.score_stride : nullptr;
    const uint64_t *list = DENSE ? nullptr : a.list + (int64_t)vh * a.cap;
    const uint32_t n_list = DENSE ? 0u : a.cnt[vh];
    const uint16_t *q = a.q + (int64_t)bh * a.q_head_stride + (int64_t)u * D;
    if (!DENSE && a.rerun && a.again[vh] == 0ull) return;      // selected before (block-uniform)
    const bool over = !DENSE && n_list > (uint32_t)a.cap;      // holds cap of its entries
    const int n = DENSE ? (int)clen : over ? a.cap : (int)n_list;
    auto get = [&](int j) -> uint64_t {
        if constexpr (DENSE) return rank_of(row[j], (uint32_t)j);
        else return list[j];
    };
    // calls f(entry) for every entry: from registers when they fit (EPT a thread, one
    // round trip), else re-read each time, four loads in flight per thread
    const bool held = n <= EPT * NT;
    uint64_t reg[EPT];
    if (held)
#pragma unroll
        for (int i = 0; i < EPT; ++i) reg[i] = get(tid + i * NT < n ? tid + i * NT : 0);
    auto each = [&](auto f) {
        if (held) {
#pragma unroll
            for (int i = 0; i < EPT; ++i)
                if (tid + i * NT < n) f(reg[i]);
            return;
        }
        for (int j0 = tid; j0 < n; j0 += 4 * NT) {
            uint64_t e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = get(j0 + i * NT < n ? j0 + i * NT : j0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (j0 + i * NT < n) f(e[i]);
        }
    };
    for (int i = tid; i < kPfBins; i += NT) s_hist[i] = 0u;
    if (tid == 0) s_ntie = 0u;
    block_qbar<uint16_t, D, NT>(q, s_qbar, s_redd);     // under the entries' latency

    uint64_t thr = 0ull;             // selected: the entries with rank >= thr
    if (n > K) {
        uint32_t kmax = 0u, kmin = ~0u;
        each([&](uint64_t e) {
            kmax = max(kmax, rank_key(e));
            kmin = min(kmin, rank_key(e));
        });
        kmax = wave_max_u32(kmax);
        kmin = ~wave_max_u32(~kmin);
        if (lane == 0) {
            s_red[tid >> 6] = kmax;
            s_redmin[tid >> 6] = kmin;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            kmax = max(kmax, s_red[i]);
            kmin = min(kmin, s_redmin[i]);
        }
        const float smin = key_score(kmin), smax = key_score(kmax);
        const float range = smax - smin;
        bool done = false;
        if (range > 0.0f && range < 3.0e38f) {
            const float scale = (float)(kPfBins - 1) / range;
            auto bin_of = [&](uint64_t e) {
                return (uint32_t)min(max((int)((key_score(rank_key(e)) - smin) * scale), 0), kPfBins - 1);
            };
            each([&](uint64_t e) { atomicAdd(&s_hist[bin_of(e)], 1u); });
            __syncthreads();
            uint32_t bstar, above, cnt;
            wave_find_bin<kPfBins>(s_hist, (uint32_t)K, bstar, above, cnt);
            if (cnt <= (uint32_t)kPfTie) {
                each([&](uint64_t e) {
                    if (bin_of(e) == bstar) s_tie[atomicAdd(&s_ntie, 1u)] = e;
                });
                __syncthreads();
                // every wave ranks the bin's entries: lane i holds entry i
                const uint64_t x = lane < (int)cnt ? s_tie[lane] : 0ull;
                uint32_t higher = 0u;
                for (int i = 0; i < (int)cnt; ++i) higher += s_tie[i] > x ? 1u : 0u;
                const uint64_t at = __ballot(lane < (int)cnt && higher == (uint32_t)K - above - 1u);
                const int src = __builtin_ctzll(at);
                thr = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), src) << 32) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, src);
                done = true;
            }
        }
        if (!done) {
            // radix select on the ranks (distinct), 10 bits at a time from the highest
            // bit in which they differ: the Top-K are the entries with
            // (rank & mask) >= prefix
            uint64_t rmax = 0ull, rmin = ~0ull;
            each([&](uint64_t e) {
                rmax = e > rmax ? e : rmax;
                rmin = e < rmin ? e : rmin;
            });
            rmax = block_reduce<NT>(rmax, s_red64, [](uint64_t x, uint64_t y) { return x > y ? x : y; });
            rmin = block_reduce<NT>(rmin, s_red64, [](uint64_t x, uint64_t y) { return x < y ? x : y; });
            const int hb = 63 - __clzll((long long)(rmax ^ rmin));
            uint64_t mask = hb < 63 ? ~0ull << (hb + 1) : 0ull, prefix = rmax & mask;
            uint32_t k_rem = (uint32_t)K;
            for (int top = hb; top >= 0; top -= 10) {
                const int width = top + 1 < 10 ? top + 1 : 10, sh = top + 1 - width;
                __syncthreads();
                for (int i = tid; i < kPfBins; i += NT) s_hist[i] = 0u;
                __syncthreads();
                each([&](uint64_t e) {
                    if ((e & mask) == prefix) atomicAdd(&s_hist[(uint32_t)(e >> sh) & ((1u << width) - 1u)], 1u);
                });
                __syncthreads();
                uint32_t digit, above, cnt;
                wave_find_bin<kPfBins>(s_hist, k_rem, digit, above, cnt);
                k_rem -= above;
                prefix |= (uint64_t)digit << sh;
                mask |= (uint64_t)((1u << width) - 1u) << sh;
                if (cnt == k_rem) break;         // block-uniform
            }
            thr = prefix;
        }
    }

    if constexpr (!DENSE) {
        if (tid == 0) a.again[vh] = over ? thr : 0ull;
        if (over) {                                            // block-uniform
            if (tid == 0) a.overflow[u] = 1u;
            return;
        }
    }
    const int64_t slot = (int64_t)bh * a.M + (a.insert_slot + u) % a.M;
    int32_t *dst = a.supp + slot * K;
    const int kn = n < K ? n : K;
    uint32_t done_before = 0u;
    for (int64_t seg = 0; seg < clen; seg += kPfSegBits) {
        const int nbits = (int)(clen - seg < kPfSegBits ? clen - seg : kPfSegBits);
        const int nth = (nbits + 32 * WPT - 1) / (32 * WPT);    // threads that own words
        __syncthreads();
        for (int i = tid; i < nth * (WPT + 1); i += NT) s_bits[i] = 0u;
        __syncthreads();
        each([&](uint64_t e) {
            const int64_t x = (int64_t)rank_index(e) - seg;
            if (e >= thr && x >= 0 && x < nbits) {
                const int wd = (int)(x >> 5);
                atomicOr(&s_bits[wd + wd / WPT], 1u << (x & 31));
            }
        });
        __syncthreads();
        uint32_t mine = 0u;
        if (tid < nth)
#pragma unroll
            for (int i = 0; i < WPT; ++i) mine += (uint32_t)__popc(s_bits[tid * (WPT + 1) + i]);
        uint32_t total;
        uint32_t pos = done_before + block_excl_scan<NT>(mine, s_red, &total);
        if (mine)
            for (int i = 0; i < WPT; ++i) {
                uint32_t bits = s_bits[tid * (WPT + 1) + i];
                while (bits) {
                    const int bit = __ffs(bits) - 1;
                    bits &= bits - 1u;
                    if (pos < (uint32_t)K) dst[pos] = (int32_t)(seg + ((int64_t)tid * WPT + i) * 32 + bit);
                    ++pos;
                }
            }
        done_before += total;
    }
    for (int t = kn + tid; t < K; t += NT) dst[t] = -1;
    if (tid == 0) a.supp_cnt[slot] = kn;
    for (int t = tid; t < D; t += NT) a.qbar[slot * D + t] = s_qbar[t];
}

void describe_prefill(int which, const PfArgs &a, KernelDesc *k)
{
    const bool d64 = a.D == 64;
    const unsigned vheads = (unsigned)((int64_t)a.B * a.Hq * a.U);
    const unsigned scan_blocks = (unsigned)((a.pairs + 7) / 8 * 8 * a.col_blocks);
    switch (which) {
    case PF_BOUND:
        *k = KernelDesc{d64 ? (const void *)&k_pf_scan<64, PF_BOUND> : (const void *)&k_pf_scan<128, PF_BOUND>,
                        dim3(scan_blocks), dim3(kPfThreads), 0u, 1};
        return;
    case PF_COLLECT:
        *k = KernelDesc{d64 ? (const void *)&k_pf_scan<64, PF_COLLECT> : (const void *)&k_pf_scan<128, PF_COLLECT>,
                        dim3(scan_blocks), dim3(kPfThreads), 0u, 1};
        return;
    case PF_RECOLLECT:
        *k = KernelDesc{d64 ? (const void *)&k_pf_scan<64, PF_RECOLLECT> : (const void *)&k_pf_scan<128, PF_RECOLLECT>,
                        dim3(scan_blocks), dim3(kPfThreads), 0u, 1};
        return;
    case PF_RAISE:
        *k = KernelDesc{(const void *)&k_pf_raise, dim3((vheads + kPfSelThreads - 1) / kPfSelThreads),
                        dim3(kPfSelThreads), 0u, 1};
        return;
    case PF_DENSE:
        *k = KernelDesc{d64 ? (const void *)&k_pf_scan<64, PF_DENSE> : (const void *)&k_pf_scan<128, PF_DENSE>,
                        dim3(scan_blocks), dim3(kPfThreads), 0u, 1};
        return;
    case PF_THRESHOLD:
        // fewer than 8 K maxima, or 8 192 of a short prefix
        *k = KernelDesc{4 * a.n_groups <= 16 * kPfSelThreads ? (const void *)&k_pf_bound<16>
                                                             : (const void *)&k_pf_bound<64>,
                        dim3(vheads), dim3(kPfSelThreads), 0u, 1};
        return;
    case PF_SELECT_LIST:
        *k = KernelDesc{d64 ? (const void *)&k_pf_select<64, false> : (const void *)&k_pf_select<128, false>,
                        dim3(vheads), dim3(kPfSelThreads), 0u, 1};
        return;
    default:
        *k = KernelDesc{d64 ? (const void *)&k_pf_select<64, true> : (const void *)&k_pf_select<128, true>,
                        dim3(vheads), dim3(kPfSelThreads), 0u, 1};
        return;
    }
}

}  // namespace retopk
