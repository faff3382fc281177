// retopk_device.h -- device helpers shared by the kernel files: score keys and
// ranks, cross-lane sums and scans, row geometry and dot products, the
// normalised query.  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace retopk {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
// 16 bytes as one register value (HIP's uint4 is a struct, whose arrays the compiler
// keeps in scratch memory where they live across a loop with a barrier in it).
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Scalar helpers
// ---------------------------------------------------------------------------

// Order-preserving image of an fp32 score (finite inputs); -0.0 maps like +0.0.
__device__ __forceinline__ uint32_t ord_key(float s)
{
    uint32_t u = __float_as_uint(s);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_score(uint32_t k)
{
    uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return __uint_as_float(u);
}

// Larger rank = higher score, or equal score and lower index.
__device__ __forceinline__ uint64_t rank_of(float s, uint32_t idx)
{
    return ((uint64_t)ord_key(s) << 32) | (uint64_t)(0xFFFFFFFFu - idx);
}
__device__ __forceinline__ uint32_t rank_index(uint64_t r) { return 0xFFFFFFFFu - (uint32_t)r; }
__device__ __forceinline__ uint32_t rank_key(uint64_t r) { return (uint32_t)(r >> 32); }

__device__ __forceinline__ float bf16_lo(uint32_t x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t x) { return __uint_as_float(x & 0xFFFF0000u); }

template <typename T> __device__ __forceinline__ double elem_f64(const T *p, int i);
template <> __device__ __forceinline__ double elem_f64<float>(const float *p, int i)
{
    return (double)p[i];
}
template <> __device__ __forceinline__ double elem_f64<uint16_t>(const uint16_t *p, int i)
{
    return (double)__uint_as_float((uint32_t)p[i] << 16);
}

// ---------------------------------------------------------------------------
// Cross-lane helpers (DPP inside a quad of lanes; shuffles elsewhere)
// ---------------------------------------------------------------------------

constexpr int kQuadXor1 = 0xB1;   // quad_perm:[1,0,3,2]
constexpr int kQuadXor2 = 0x4E;   // quad_perm:[2,3,0,1]
constexpr int kHalfMirror = 0x141; // row_half_mirror: lane i <-> 7 - i in each 8 lanes

template <int CTRL> __device__ __forceinline__ float dpp_f32(float x)
{
    return __builtin_bit_cast(float,
        __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

template <int CTRL> __device__ __forceinline__ double dpp_f64(double x)
{
    uint64_t u = __builtin_bit_cast(uint64_t, x);
    int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
}

// Sum over the 4 lanes of a quad; every lane of the quad gets the same value.
__device__ __forceinline__ float quad_sum(float x)
{
    x += dpp_f32<kQuadXor1>(x);
    x += dpp_f32<kQuadXor2>(x);
    return x;
}
__device__ __forceinline__ double quad_sum(double x)
{
    x += dpp_f64<kQuadXor1>(x);
    x += dpp_f64<kQuadXor2>(x);
    return x;
}

// Reductions over a wave: DPP inside each row of 16 lanes (quad swaps, half-row
// and row mirrors), then the four row results read as scalars.  Every lane gets
// the result.
__device__ __forceinline__ uint32_t row_max_u32(uint32_t x)
{
    x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kQuadXor1, 0xF, 0xF, true));
    x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kQuadXor2, 0xF, 0xF, true));
    x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kHalfMirror, 0xF, 0xF, true));
    x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x140, 0xF, 0xF, true));   // row_mirror
    return x;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x)
{
    x = row_max_u32(x);
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 0);
    const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 32);
    const uint32_t r3 = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
    return max(max(r0, r1), max(r2, r3));
}
__device__ __forceinline__ float wave_sum_f32(float x)
{
    x += dpp_f32<kQuadXor1>(x);
    x += dpp_f32<kQuadXor2>(x);
    x += dpp_f32<kHalfMirror>(x);
    x += dpp_f32<0x140>(x);   // row_mirror
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 48));
    return (r0 + r1) + (r2 + r3);
}

__device__ __forceinline__ double wave_max_f64(double x)
{
    x = fmax(x, dpp_f64<kQuadXor1>(x));
    x = fmax(x, dpp_f64<kQuadXor2>(x));
    x = fmax(x, dpp_f64<kHalfMirror>(x));
    x = fmax(x, dpp_f64<0x140>(x));   // row_mirror
    auto rl = [&](int l) {
        const uint64_t u = __builtin_bit_cast(uint64_t, x);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
        return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    };
    return fmax(fmax(rl(0), rl(16)), fmax(rl(32), rl(48)));
}

// x from lane (i + n) mod 16 of the same row of 16 lanes (DPP row_ror:n, 1..15).
__device__ __forceinline__ float row_ror_f32(float x, int n)
{
    int r;
    switch (n) {
    case 1: r = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x121, 0xF, 0xF, true); break;
    case 2: r = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x122, 0xF, 0xF, true); break;
    case 4: r = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x124, 0xF, 0xF, true); break;
    default: r = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x128, 0xF, 0xF, true); break;
    }
    return __builtin_bit_cast(float, r);
}

// gfx950 row swaps: permlane32_swap exchanges the first operand's upper 32 lanes with
// the second's lower 32, permlane16_swap the first's odd rows of 16 lanes with the
// second's even ones.  add32_f32(x, y): lanes 0-31 get the sum of x over lanes i and
// i ^ 32, lanes 32-63 that of y (add16_f32: even rows x, odd rows y, over i and i ^ 16);
// with x == y every lane gets the full sum.
__device__ __forceinline__ float add32_f32(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add16_f32(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The largest of x over lanes i, i ^ 16, i ^ 32 and i ^ 48.
__device__ __forceinline__ float max_rows_f32(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}

// Orders LDS accesses of the lanes of one wave (LDS runs them in program order; this
// keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Inclusive prefix sum over the 64 lanes of a wave: Hillis-Steele inside each row
// of 16 lanes (DPP row shifts, lanes shifted in from outside the row read 0), then
// the row totals carried across rows with the row broadcasts of lanes 15 and 31.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return x;
}

// Block reductions.  All threads must call them; every thread gets the same
// result (fixed combination order).  red: NT/64 scratch slots.
template <int NT, typename V, typename Op>
__device__ __forceinline__ V block_reduce(V v, V *red, Op op)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    V t = red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) t = op(t, red[w]);
    __syncthreads();
    return t;
}

// Exclusive prefix sum over the block; *total receives the block sum.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *red, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = wave_incl_scan(v);
    if (lane == 63) red[wave] = incl;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        uint32_t x = red[w];
        if (w < wave) before += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return before + incl - v;
}

// ---------------------------------------------------------------------------
// Row geometry.  A row of D elements of type T is split over the 4 lanes of a
// quad: lane p holds the 16-byte vectors s*4 + p, s = 0 .. NV-1.  One wave covers
// 16 rows per pass, and each load instruction reads 64 contiguous bytes per row.
// ---------------------------------------------------------------------------

template <typename T, int D> struct RowT {
    static constexpr int kBytes = D * (int)sizeof(T);
    static constexpr int kNV = kBytes / 64;
};

// Waves per SIMD that k_score is built for: 4 (two 512-thread blocks per CU), or
// 2 (256 registers a lane) where the group's query vectors and the two key rows a
// lane holds in flight would take more than 96 of 128 registers (G + 2 rows of
// kNV * 4 in the quad layout), or, in the octet layout of the fp32 8-head build,
// where the query vectors alone would take half of them (the bf16 8-head build
// holds D / 32 MFMA operands).
template <typename T, int D, int G>
constexpr int kGroupWaves = (G == 8 && sizeof(T) == 2) ? 4
                            : G == 8 ? (2 * G * RowT<T, D>::kNV > 64 ? 2 : 4)
                                     : ((G + 2) * RowT<T, D>::kNV * 4 > 96 ? 2 : 4);
// The same for k_dense (fp32), whose lanes also hold G value accumulators of 4 floats
// (the 8-head build takes its scores in the octet layout, its queries dead by the time
// the accumulators live).
template <int D, int G>
constexpr int kDenseWaves = G == 8 ? (16 * RowT<float, D>::kNV > 64 ? 2 : 4)
                                   : (G * 4 * (RowT<float, D>::kNV + 1) > 96 ? 2 : 4);

template <typename T> struct Dot;
template <> struct Dot<uint16_t> {
    // 8 bf16 products accumulated in fp32 with v_dot2_f32_bf16.
    static __device__ __forceinline__ float f(uint4 k, uint4 q, float acc)
    {
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k.x),
                                              __builtin_bit_cast(bf16x2_t, q.x), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k.y),
                                              __builtin_bit_cast(bf16x2_t, q.y), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k.z),
                                              __builtin_bit_cast(bf16x2_t, q.z), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k.w),
                                              __builtin_bit_cast(bf16x2_t, q.w), acc, false);
        return acc;
    }
    static __device__ __forceinline__ void axpy(uint4 v, float w, float *acc)
    {
        acc[0] += w * bf16_lo(v.x); acc[1] += w * bf16_hi(v.x);
        acc[2] += w * bf16_lo(v.y); acc[3] += w * bf16_hi(v.y);
        acc[4] += w * bf16_lo(v.z); acc[5] += w * bf16_hi(v.z);
        acc[6] += w * bf16_lo(v.w); acc[7] += w * bf16_hi(v.w);
    }
};
template <> struct Dot<float> {
    static __device__ __forceinline__ float f(uint4 k, uint4 q, float acc)
    {
        acc = fmaf(__uint_as_float(k.x), __uint_as_float(q.x), acc);
        acc = fmaf(__uint_as_float(k.y), __uint_as_float(q.y), acc);
        acc = fmaf(__uint_as_float(k.z), __uint_as_float(q.z), acc);
        acc = fmaf(__uint_as_float(k.w), __uint_as_float(q.w), acc);
        return acc;
    }
    static __device__ __forceinline__ void axpy(uint4 v, float w, float *acc)
    {
        acc[0] += w * __uint_as_float(v.x); acc[1] += w * __uint_as_float(v.y);
        acc[2] += w * __uint_as_float(v.z); acc[3] += w * __uint_as_float(v.w);
    }
};

// Reduce-scatter inside a quad: lane p of the quad holds partial sums a0..a3 of
// four dot products; on return it holds the full (4-lane) sum of dot product p.
// Two butterfly steps: at each one a lane keeps the half of its values whose
// index bit matches its own lane bit and sends the other half to its partner.
__device__ __forceinline__ float quad_transpose_sum(float a0, float a1, float a2, float a3, int p)
{
    const bool b0 = (p & 1) != 0, b1 = (p & 2) != 0;
    const float keep0 = b0 ? a1 : a0, send0 = b0 ? a0 : a1;
    const float keep1 = b0 ? a3 : a2, send1 = b0 ? a2 : a3;
    const float r0 = keep0 + dpp_f32<kQuadXor1>(send0);   // dot 0 + b0
    const float r1 = keep1 + dpp_f32<kQuadXor1>(send1);   // dot 2 + b0
    const float keep = b1 ? r1 : r0, send = b1 ? r0 : r1;
    return keep + dpp_f32<kQuadXor2>(send);                // dot 2*b1 + b0
}

// Full scores of a G-head group after each lane of a quad accumulated its quarter
// of every row: lane p returns the scores of heads p and p + 4 (when they exist).
template <int G>
__device__ __forceinline__ void group_scores(const float (&acc)[G], int p, float &s_lo, float &s_hi)
{
    if constexpr (G == 1) {
        s_lo = quad_sum(acc[0]);
        s_hi = 0.0f;
    } else if constexpr (G == 2) {
        const bool b0 = (p & 1) != 0;
        const float r = (b0 ? acc[1] : acc[0]) + dpp_f32<kQuadXor1>(b0 ? acc[0] : acc[1]);
        s_lo = r + dpp_f32<kQuadXor2>(r);
        s_hi = 0.0f;
    } else if constexpr (G == 4) {
        s_lo = quad_transpose_sum(acc[0], acc[1], acc[2], acc[3], p);
        s_hi = 0.0f;
    } else {
        s_lo = quad_transpose_sum(acc[0], acc[1], acc[2], acc[3], p);
        s_hi = quad_transpose_sum(acc[4], acc[5], acc[6], acc[7], p);
    }
}

// Reduce-scatter inside an octet of lanes (8 lanes per row, one per head of an
// 8-head group): lane o holds partial sums of the 8 dot products and returns the
// full (8-lane) sum of dot product o.  Three butterfly steps, as in
// quad_transpose_sum; the first pairs lane o with lane 7 - o (a DPP half-row
// mirror), whose bit 2 is the opposite of o's, which is all the step needs.
__device__ __forceinline__ float octet_transpose_sum(const float (&acc)[8], int o)
{
    const bool b2 = (o & 4) != 0, b1 = (o & 2) != 0, b0 = (o & 1) != 0;
    float h4[4], h2[2];
#pragma unroll
    for (int i = 0; i < 4; ++i)   // heads (o & 4) + i
        h4[i] = (b2 ? acc[i + 4] : acc[i]) + dpp_f32<kHalfMirror>(b2 ? acc[i] : acc[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i)   // heads (o & 6) + i
        h2[i] = (b1 ? h4[i + 2] : h4[i]) + dpp_f32<kQuadXor2>(b1 ? h4[i] : h4[i + 2]);
    return (b0 ? h2[1] : h2[0]) + dpp_f32<kQuadXor1>(b0 ? h2[0] : h2[1]);   // head o
}

// ---------------------------------------------------------------------------
// q_bar = fl32(q / ||q||_2), norm in float64 (Eq. 5, Eq. 6)
// ---------------------------------------------------------------------------

template <typename T, int D, int NT>
__device__ void block_qbar(const T *q, float *s_qbar, double *red)
{
    static_assert(NT >= D, "one thread per element");
    const int t = threadIdx.x;
    double x = t < D ? elem_f64<T>(q, t) : 0.0;
    double ss = block_reduce<NT>(x * x, red, [](double a, double b) { return a + b; });
    double nrm = sqrt(ss);
    if (t < D) s_qbar[t] = nrm > 0.0 ? (float)(x / nrm) : 0.0f;
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Histogram search by one wave
// ---------------------------------------------------------------------------

// The bin b* that holds the k-th largest of the entries counted in hist (nb bins,
// descending from bin nb - 1), the count above it and its own count, found by one
// wave (every wave gets the same result): lane l sums bins nb-1-BPL*l ..
// nb-BPL-BPL*l, a wave prefix sum finds the lane, that lane walks its bins.
template <int NB>
__device__ __forceinline__ void wave_find_bin(const uint32_t *hist, uint32_t k, uint32_t &bstar,
                                              uint32_t &above, uint32_t &cnt)
{
    constexpr int BPL = NB / 64;
    static_assert(BPL % 4 == 0, "whole 16-byte reads");
    const int lane = threadIdx.x & 63;
    uint32_t c[BPL], mine = 0u;
    const uint4 *hv = (const uint4 *)&hist[NB - BPL * (lane + 1)];
#pragma unroll
    for (int i = 0; i < BPL / 4; ++i) {
        const uint4 x = hv[i];
        c[BPL - 1 - 4 * i] = x.x;
        c[BPL - 2 - 4 * i] = x.y;
        c[BPL - 3 - 4 * i] = x.z;
        c[BPL - 4 - 4 * i] = x.w;
    }
#pragma unroll
    for (int i = 0; i < BPL; ++i) mine += c[i];
    const uint32_t inc = wave_incl_scan(mine);
    const uint64_t hit = __ballot(inc - mine < k && inc >= k);
    const int src = __builtin_ctzll(hit);   // k <= total: exactly one lane
    uint32_t bs = 0u, ab = 0u, cb = 0u, run = inc - mine;
#pragma unroll
    for (int i = 0; i < BPL; ++i) {
        if (run < k && run + c[i] >= k) {
            bs = (uint32_t)(NB - 1 - BPL * lane - i);
            ab = run;
            cb = c[i];
        }
        run += c[i];
    }
    bstar = (uint32_t)__builtin_amdgcn_readlane((int)bs, src);
    above = (uint32_t)__builtin_amdgcn_readlane((int)ab, src);
    cnt = (uint32_t)__builtin_amdgcn_readlane((int)cb, src);
}

}  // namespace retopk
