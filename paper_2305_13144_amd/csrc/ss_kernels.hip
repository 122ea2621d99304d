// gfx950 kernels of the decode path.  One wavefront = 64 lanes; matrix work uses
// v_mfma_f32_16x16x32_f16 (A: 16 rows x 32 k, B: 32 k x 16 cols, 8 halves per lane;
// D: lane holds rows 4*(lane/16)..+3 of column lane%16).
//
// Convention for every contraction here: the weight strip is the A operand (its 16 output
// columns become D's rows) and the activation strip is the B operand (its 16 token rows become
// D's columns), so a lane ends up with 4 consecutive output columns of one token row.
#include "ss_kernels.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ss_internal.h"

namespace ss {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));  // one 16-byte operand fragment

// ------------------------------------------------------------------------------------------ helpers
__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

__device__ __forceinline__ bf16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even (inputs are finite)
    return (bf16_t)(u >> 16);
}

// Both operands of every projection are IEEE half.  A bf16 weight keeps its exact value in that format (8
// significand bits fit in 11; see k_pack_weight for the two ends of the range).  An activation that feeds a
// projection is rounded to half once: 11 significand bits, where a bf16 operand would keep 8 - one such rounding
// per projection input, six per layer over 32+ layers, is the dominant term of the logit error, and at 8 bits it
// is as large as the whole tolerance.  Finite values saturate, like the key/value slots below; a NaN stays a NaN.
__device__ __forceinline__ f16_t f2h(float f)
{
    const float c = fminf(fmaxf(f, -65504.f), 65504.f);   // of a NaN and a number these return the number
    return __builtin_bit_cast(f16_t, (_Float16)(f != f ? f : c));
}

// Rotation of a pair of elements.  Which product of the sum is rounded first is written out: the compiler would choose by what is around
// it, and every kernel that rotates is to round alike (a prompt's keys and queries do not depend on whether q|k|v was cut in k-slices).
// In the difference it rounds the second product in all of them.
__device__ __forceinline__ float2 rotated(float a, float b, float cs, float sn)
{
    return make_float2(a * cs - b * sn, fmaf(b, cs, a * sn));
}

// Key/value slots are stored as IEEE half: the same 2 bytes per element as bf16 with three more
// significand bits; keys and values are projections of RMS-normalised activations, far inside its range.
__device__ __forceinline__ float kv2f(kv_t b) { return (float)__builtin_bit_cast(_Float16, b); }
// Saturating: a value beyond the half range is stored as the largest finite half, never as infinity (an infinite
// key would turn the softmax into NaN and the token choice into an arbitrary id).
__device__ __forceinline__ kv_t f2kv(float f)
{
    return __builtin_bit_cast(kv_t, (_Float16)fminf(fmaxf(f, -65504.f), 65504.f));
}

// Element (r, k) of a packed [rows, Kp] matrix.
__device__ __forceinline__ size_t pk_index(int r, int k, int Kp)
{
    return ((size_t)(r >> 4) * (size_t)(Kp >> 5) + (size_t)(k >> 5)) * 512u +
           (size_t)(((((k & 31) >> 3) << 4) + (r & 15)) * 8 + (k & 7));
}

// Output strips of q, k and v are packed in pairs: a head's strip i of its first half (elements 16i..16i+15) and its
// strip i of the second half are neighbours, so that the two elements of a rotation pair (e, e + hd/2) are in the same
// lane of whichever wave computes them, as gate and up are.  qkv_strip: natural strip -> packed strip; qkv_col: column of
// element e < hd/2 of a head in the projection's output (its partner follows 16 columns later).
__device__ __forceinline__ int qkv_strip(int strip, int head_strips)
{
    const int h = strip / head_strips, i = strip - h * head_strips, half = head_strips >> 1;
    return h * head_strips + (i < half ? 2 * i : 2 * (i - half) + 1);
}
__device__ __forceinline__ int qkv_col(int e) { return (e >> 4) * 32 + (e & 15); }

// v of another lane of the same row of 16 lanes (a DPP control), at the cost of a register move.
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int kDppRotate4 = 0x124, kDppRotate8 = 0x128;

// op(v, v of the lane M = 16 or 32 away), M being a bit of the lane's number: two rows or halves of the wave change places,
// which takes no trip through LDS as a general shuffle does (the norms and the decode attention are chains of such latencies:
// with general shuffles, decode of 7B, one row, 24 steps 64.3 ms instead of 63.5, 16 rows 79.6 / 78.9, 51 rows 58.4 / 57.8).
template <int M, typename Op>
__device__ __forceinline__ float across(float v, Op op)
{
    const unsigned u = (unsigned)__float_as_int(v);
    const auto r = M == 32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false) : __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return op(__int_as_float((int)r[0]), __int_as_float((int)r[1]));
}
struct Add { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct Max { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// Over the wave, in each lane: lanes 32, 16, 8, 4, 2 and 1 apart in turn (after a step the lanes that it joined are alike, so
// that a turn by 4 in a row of 16 does for 4 apart).
template <typename Op>
__device__ __forceinline__ float wave_all(float v, Op op)
{
    v = across<16>(across<32>(v, op), op);
    v = op(v, dpp<kDppRotate8>(v));
    v = op(v, dpp<kDppRotate4>(v));
    v = op(v, dpp<kDppXor2>(v));
    return op(v, dpp<kDppXor1>(v));
}
__device__ __forceinline__ float wave_sum(float v) { return wave_all(v, Add()); }
__device__ __forceinline__ float wave_max(float v) { return wave_all(v, Max()); }

// Sum over a group of 8 or 16 neighbouring lanes, in each of them.
template <int N>
__device__ __forceinline__ float group_sum(float v)
{
    static_assert(N == 8 || N == 16, "half a row or a row");
    v += dpp<kDppXor1>(v);
    v += dpp<kDppXor2>(v);
    v += dpp<kDppHalfMirror>(v);   // the lanes of four are alike by now
    if (N == 16) v += dpp<kDppMirror>(v);
    return v;
}

// ------------------------------------------------------------------------------------------ weight packing
// src is row-major [n_src, k] (bf16 bits or fp32, rounded to bf16 first); source row r lands in packed row
// (strip * blk_stride + blk_off) * 16 + r%16, where strip = r/16, or with head_strips > 0 (q, k, v) the place that
// qkv_strip gives it inside its head.  One thread moves 8 consecutive k.  The packed element is the bf16
// value written as IEEE half: the same number for 2^-17 <= |w| <= 65504 (half subnormals included); smaller
// magnitudes are rounded to a multiple of 2^-24 (an absolute error below 3e-8 per weight), larger ones saturate.
__global__ void k_pack_weight(const void* __restrict__ src, int src_f32, f16_t* __restrict__ dst, int n_src, int k,
                              int kp, int blk_stride, int blk_off, int head_strips)
{
    const int groups = k >> 3;
    const size_t total = (size_t)n_src * groups;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const int r = (int)(i / groups), kg = (int)(i % groups);
        bf16_t v[8];
        if (src_f32) {
            const float* sp = (const float*)src + (size_t)r * k + kg * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = f2bf(sp[e]);
        } else {
            const uint4 raw = *(const uint4*)((const bf16_t*)src + (size_t)r * k + kg * 8);
            *(uint4*)v = raw;
        }
        f16_t o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = f2h(bf2f(v[e]));
        const int strip = head_strips > 0 ? qkv_strip(r >> 4, head_strips) : r >> 4;
        const int rd = (strip * blk_stride + blk_off) * 16 + (r & 15);
        *(uint4*)(dst + pk_index(rd, kg * 8, kp)) = *(const uint4*)o;
    }
}

// ------------------------------------------------------------------------------------------ 12-bit weights
// A second copy of a weight matrix for the kernels that are bound by streaming it (decode batches), at 12 bits per
// weight instead of 16 and with exactly the same values.  A packed weight is a bf16 value written as IEEE half; below
// 0.25 in magnitude that is sign, 4 exponent bits (2^-17 .. 2^-3, code 0 = multiples of 2^-24 below) and 7 mantissa bits:
// eight times the weight, as a half, has bit 14 and bits 2..0 clear.  The kernels multiply with eight times the weight
// and scale their sums by 1/8, both exactly; sums of products round alike, but for the last bit of some that contain
// weights which are subnormal as halves.  A matrix with a value of 0.25 or more (or a NaN) has no such copy and is
// streamed as halves.
// Layout: [strip][group of 4 k-blocks][3 planes][lane] of 16 bytes, strips apart by narrow_strip: a lane's 4 operand fragments (4 dwords each) take
// 12 dwords, 3 per fragment, read as three fully coalesced 1 KiB loads.  Of a fragment's 4 dwords the first three are
// stored as they are, and the 8 clear bits of each hold a third of the fourth.
// Why: a decode step of few rows is a weight stream and its bytes are its time; the 15 vector instructions that open a
// fragment run beside it.  Measured alone and without gaps between strips, halves / 12 bits, 16 rows, 7B: q|k|v 18.7 / 14.3 us, gate|up 31.0 / 25.8, down
// 16.7 / 14.6, o 8.2 / 7.1, LM head 43.4 / 32.1; 13B gate|up 47.8 / 36.4.  With more row strips LDS reads and matrix work
// take over (64 rows: gate|up 32.0 / 30.5, 96 rows 37.3 / 36.4), so the copies are read up to kNarrowMaxRows rows.
constexpr unsigned kNarrowMask = 0xBFF8BFF8u;   // sign, exponent and mantissa bits of two halves
constexpr float kNarrowScale = 0.125f;

__global__ __launch_bounds__(256) void k_narrow_weight(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                       size_t n_groups, int strip_groups, int32_t* __restrict__ unfit)
{
    const size_t total = n_groups * 64;   // one thread per group of 4 k-blocks and lane
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const size_t g = i >> 6;
        const int lane = (int)(i & 63);
        unsigned o[12];
        bool bad = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x4 w = src[(g * 4 + q) * 64 + lane];
            unsigned f[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned lo = w[e] & 0xffffu, hi = w[e] >> 16;
                bad = bad || (lo & 0x7fffu) >= 0x3400u || (hi & 0x7fffu) >= 0x3400u;
                const _Float16 a = __builtin_bit_cast(_Float16, (unsigned short)lo) * (_Float16)8.f;
                const _Float16 b = __builtin_bit_cast(_Float16, (unsigned short)hi) * (_Float16)8.f;
                f[e] = (unsigned)__builtin_bit_cast(unsigned short, a) | ((unsigned)__builtin_bit_cast(unsigned short, b) << 16);
                bad = bad || (f[e] & ~kNarrowMask) != 0u;
            }
            // the fourth dword's bits 5..3, 8..6, 11..9 and 15, 13, 12 of each half: see narrow_frag
            o[3 * q] = f[0] | ((f[3] >> 3) & 0x00070007u) | ((f[3] >> 1) & 0x40004000u);
            o[3 * q + 1] = f[1] | ((f[3] >> 6) & 0x00070007u) | ((f[3] << 1) & 0x40004000u);
            o[3 * q + 2] = f[2] | ((f[3] >> 9) & 0x00070007u) | ((f[3] << 2) & 0x40004000u);
        }
        if (bad) *unfit = 1;
        if (!dst) continue;
        const size_t at = (g / strip_groups) * narrow_strip(strip_groups * 4) + (g % strip_groups) * 192 + lane;
#pragma unroll
        for (int p = 0; p < 3; ++p)
            dst[at + p * 64] = (u32x4){o[4 * p], o[4 * p + 1], o[4 * p + 2], o[4 * p + 3]};
    }
}

// Three stored dwords -> the four dwords of an operand fragment (eight times the weights).  15 vector instructions.
__device__ __forceinline__ u32x4 narrow_frag(unsigned a, unsigned b, unsigned c)
{
    unsigned d = (a << 3) & 0x00380038u;
    d |= (b << 6) & 0x01C001C0u;
    d |= (c << 9) & 0x0E000E00u;
    d |= (a << 1) & 0x80008000u;
    d |= (b >> 1) & 0x20002000u;
    d |= (c >> 2) & 0x10001000u;
    return (u32x4){a & kNarrowMask, b & kNarrowMask, c & kNarrowMask, d};
}

// Fragment q (0..3) of a lane's three 16-byte pieces of a group.
template <int Q>
__device__ __forceinline__ u32x4 narrow_group_frag(const u32x4 (&p)[3])
{
    return narrow_frag(p[(3 * Q) / 4][(3 * Q) % 4], p[(3 * Q + 1) / 4][(3 * Q + 1) % 4], p[(3 * Q + 2) / 4][(3 * Q + 2) % 4]);
}

__global__ void k_cast_rows(const void* __restrict__ src, int src_f32, bf16_t* __restrict__ dst, size_t count)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src_f32 ? f2bf(((const float*)src)[i]) : ((const bf16_t*)src)[i];
}

__global__ void k_fill_i32(int32_t* p, int32_t v, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// ------------------------------------------------------------------------------------------ embedding
__global__ __launch_bounds__(256) void k_embed(MbState st, const bf16_t* __restrict__ embed, float* __restrict__ x,
                                               int d)
{
    const int j = blockIdx.x;
    if (j >= *st.d_n) return;
    const bf16_t* e = embed + (size_t)st.tr_tok[j] * d;
    float* xr = x + (size_t)j * d;
    for (int c = threadIdx.x * 8; c < d; c += 256 * 8) {
        const uint4 raw = *(const uint4*)(e + c);
        const bf16_t* v = (const bf16_t*)&raw;
        float4 a = make_float4(bf2f(v[0]), bf2f(v[1]), bf2f(v[2]), bf2f(v[3]));
        float4 b = make_float4(bf2f(v[4]), bf2f(v[5]), bf2f(v[6]), bf2f(v[7]));
        *(float4*)(xr + c) = a;
        *(float4*)(xr + c + 4) = b;
    }
}

// ------------------------------------------------------------------------------------------ RMSNorm
// Row j (or sel[j]) of the residual stream: x += sum over k-slices of the previous projection's
// partial sums (written back when sel is null), then h = x * rsqrt(mean x^2 + eps) * w as packed halves.
// T threads per row, at most ITER float4 chunks per thread (T * ITER * 4 >= d, d <= 8192); the loads of all k-slices of a
// chunk are issued together (the slice loop is unrolled with a predicate), so a row costs about one
// memory round trip instead of one per slice.
constexpr int kNormMaxSplit = 8;
constexpr int kNormNarrowFrom = 384;   // token-rows from which a row gets 256 threads instead of 1024

// Written out: every kernel that norms rows is to round alike.
__device__ __forceinline__ float norm_squares(const float4& a) { return fmaf(a.w, a.w, fmaf(a.z, a.z, fmaf(a.x, a.x, a.y * a.y))); }

// Four elements of a row, normalised (r: the row's factor, wr: their gains), to `out`.
__device__ __forceinline__ void norm_store(f16_t* out, const float4& v, float r, const uint2& wr)
{
    const bf16_t* wv = (const bf16_t*)&wr;
    const f16_t o[4] = {f2h(v.x * r * bf2f(wv[0])), f2h(v.y * r * bf2f(wv[1])), f2h(v.z * r * bf2f(wv[2])), f2h(v.w * r * bf2f(wv[3]))};
    *(uint2*)out = *(const uint2*)o;
}

template <int T, int ITER>
__global__ __launch_bounds__(T) void k_rmsnorm(const int32_t* __restrict__ d_count, float* __restrict__ x,
                                                  const float* __restrict__ part, int ksplit, size_t part_stride,
                                                  const bf16_t* __restrict__ w, float eps,
                                                  const int32_t* __restrict__ sel, f16_t* __restrict__ h, int d,
                                                  int n_rows)
{
    // A packed row is pieces of 16 bytes, and 16 rows together fill whole lines.  With many rows the 16 rows of a strip
    // therefore go to workgroups of one die (ids are dealt to the 8 dies round-robin), whose L2 puts the lines
    // together; few rows gain nothing, their lines are read by all dies at once.  Per launch, 7B: 7200
    // token-rows 72 -> 52 us, 3000 28 -> 21, 12311 109 -> 77 (4 TB/s).
    const int b = blockIdx.x;
    const int j = T == 1024 ? b : ((b >> 7) * 8 + (b & 7)) * 16 + ((b >> 3) & 15);
    if (T != 1024 && j >= n_rows) return;   // the grid is whole groups of 8 strips
    // The row count, the row, its partial sums and the norm weights are all requested before anything waits:
    // the kernel is a chain of dependent round trips otherwise (count, then the row, then the weights), and its
    // whole cost is latency.  Rows at or beyond the count are loaded as well (the buffers are sized for the grid)
    // and dropped before the first store; with a selection list the index itself is only valid below the count.
    const int count = *d_count;
    int src = j;
    if (sel) {
        if (j >= count) return;
        src = sel[j];
    }
    float4 v[ITER];
    uint2 wr[ITER];
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int c = threadIdx.x * 4 + it * T * 4;
        if (c < d) {
            float4 a = *(const float4*)(x + (size_t)src * d + c);
            float4 p[kNormMaxSplit];
#pragma unroll
            for (int s = 0; s < kNormMaxSplit; ++s)
                p[s] = s < ksplit ? *(const float4*)(part + (size_t)s * part_stride + (size_t)src * d + c)
                                  : make_float4(0.f, 0.f, 0.f, 0.f);
            wr[it] = *(const uint2*)(w + c);
#pragma unroll
            for (int s = 0; s < kNormMaxSplit; ++s) { a.x += p[s].x; a.y += p[s].y; a.z += p[s].z; a.w += p[s].w; }
            v[it] = a;
            ss += norm_squares(a);
        }
    }
    if (j >= count) return;   // block-uniform
    if (ksplit > 0 && !sel) {
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int c = threadIdx.x * 4 + it * T * 4;
            if (c < d) *(float4*)(x + (size_t)src * d + c) = v[it];
        }
    }
    __shared__ float red[T / 64];
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < T / 64; ++i) tot += red[i];
    const float r = rsqrtf(tot / (float)d + eps);
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int c = threadIdx.x * 4 + it * T * 4;
        if (c < d) {
            const size_t at = pk_index(j, c, d);   // d is a multiple of 64: Kp == d
            norm_store(h + at, v[it], r, wr[it]);
        }
    }
}

// ------------------------------------------------------------------------------------------ skinny GEMM
// Up to 64 token rows (MT strips of 16); the whole cost is streaming the weights once from HBM.
// A workgroup of 4 wavefronts owns NB strips of 16 output columns and one outer k-slice; its waves cut
// that slice into 4 contiguous k-ranges, so every wave streams NB contiguous runs of 1 KiB operand
// blocks (non-temporal: each weight byte is used exactly once per step) and never waits for another
// wave until the end.  Loads are double-buffered in registers: while the MFMAs of KD k-blocks run, the
// next KD*NB KiB are already in flight.  The activation operands (MT per k-block) come from L2.
// At the end waves 1..3 hand their accumulators to wave 0 through LDS; wave 0 runs the epilogue.
__device__ __forceinline__ float silu_f(float z) { return z / (1.f + __expf(-z)); }

// WN: weights in the 12-bit form (KD = 4, one group per load; k-ranges are whole groups).
template <int MT, int NB, int KD, int WN>
struct SkinnyFrags {
    static_assert(!WN || KD == 4, "a 12-bit load covers 4 k-blocks");
    u32x4 w[NB][WN ? 3 : KD];
    u32x4 x[MT][KD];
};

// Loads for k-blocks kb..kb+KD-1; k-blocks at or beyond kend are clamped re-reads whose activation
// operands are zeroed in skinny_mma, so they add 0.
template <int MT, int NB, int KD, int WN>
__device__ __forceinline__ void skinny_load(SkinnyFrags<MT, NB, KD, WN>& f, const u32x4* __restrict__ Wl,
                                            const u32x4* __restrict__ Xl, int KB, int nb0, int nvalid, int kb,
                                            int kend)
{
    if (WN) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int nb = nb0 + (i < nvalid ? i : 0);
            const u32x4* g = Wl + nb * narrow_strip(KB) + (size_t)(kb >> 2) * 192;
#pragma unroll
            for (int p = 0; p < 3; ++p) f.w[i][p] = __builtin_nontemporal_load(g + p * 64);
        }
    }
#pragma unroll
    for (int q = 0; q < KD; ++q) {
        const int kk = min(kb + q, kend - 1);
        if (!WN) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int nb = nb0 + (i < nvalid ? i : 0);
                f.w[i][q] = __builtin_nontemporal_load(Wl + ((size_t)nb * KB + kk) * 64);
            }
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) f.x[m][q] = Xl[((size_t)m * KB + kk) * 64];
    }
}

template <int MT, int NB, int KD, int WN>
__device__ __forceinline__ void skinny_mma(const SkinnyFrags<MT, NB, KD, WN>& f, f32x4 (&acc)[NB][MT], int kb, int kend)
{
    if constexpr (WN) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const u32x4 w[4] = {narrow_group_frag<0>(f.w[i]), narrow_group_frag<1>(f.w[i]), narrow_group_frag<2>(f.w[i]),
                                narrow_group_frag<3>(f.w[i])};
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w[q]),
                                                                       __builtin_bit_cast(f16x8, f.x[m][q]), acc[i][m], 0, 0, 0);
        }
        return;
    } else {
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < KD; ++q) {
        const bool live = kb + q < kend;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const u32x4 xv = live ? f.x[m][q] : zero;
#pragma unroll
            for (int i = 0; i < NB; ++i)
                acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, f.w[i][q]),
                                                                   __builtin_bit_cast(f16x8, xv), acc[i][m], 0, 0, 0);
        }
    }
    }
}

template <int MT, int NB, int KD, int EPI, int WN>
__global__ __launch_bounds__(256) void k_gemm_skinny(GemmArgs a, int n_groups, int kb_per_slice)
{
    __shared__ f32x4 red[3][NB][MT][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ng = blockIdx.x % n_groups, ks = blockIdx.x / n_groups;
    const int KB = a.Kp >> 5, NBT = a.N >> 4;
    const int s0 = ks * kb_per_slice, s1 = min(KB, s0 + kb_per_slice);
    int per_wave = (max(s1 - s0, 0) + 3) >> 2;
    if (WN) per_wave = (per_wave + 3) & ~3;   // whole groups of 4 k-blocks (the slices are, too)
    const int kbeg = min(s1, s0 + wave * per_wave), kend = min(s1, kbeg + per_wave);
    const int nb0 = ng * NB;
    const int nvalid = min(NB, NBT - nb0);  // block-uniform

    f32x4 acc[NB][MT];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[i][m] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const u32x4* Wl = (const u32x4*)(WN ? a.Wn : a.W) + lane;
    const u32x4* Xl = (const u32x4*)a.X + lane;
    if (kbeg < kend) {
        SkinnyFrags<MT, NB, KD, WN> fa, fb;
        skinny_load(fa, Wl, Xl, KB, nb0, nvalid, kbeg, kend);
        // Loads past the wave's k-range are skipped rather than clamped: measured, the wasted re-reads of an
        // unconditional tail cost more (k-ranges are only 4-40 blocks) than the conservative load-counter waits
        // the branches cause; latency is hidden by the 12-20 resident waves per CU, not inside a wave.
        for (int kb = kbeg; kb < kend; kb += 2 * KD) {
            if (kb + KD < kend) skinny_load(fb, Wl, Xl, KB, nb0, nvalid, kb + KD, kend);
            skinny_mma(fa, acc, kb, kend);
            if (kb + 2 * KD < kend) skinny_load(fa, Wl, Xl, KB, nb0, nvalid, kb + 2 * KD, kend);
            if (kb + KD < kend) skinny_mma(fb, acc, kb + KD, kend);
        }
    }
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int m = 0; m < MT; ++m) red[wave - 1][i][m][lane] = acc[i][m];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[i][m] += red[w][i][m][lane];
    if (WN) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[i][m] *= kNarrowScale;
    }

    const int col4 = (lane >> 4) * 4;  // first of this lane's 4 consecutive output columns inside a strip
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = m * 16 + (lane & 15);
        if (row >= a.m_rows) continue;
        if (EPI == EPI_PARTIAL) {
            float* o = a.out + ((size_t)ks * a.m_stride + row) * a.N;
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (i < nvalid)
                    *(float4*)(o + (nb0 + i) * 16 + col4) =
                        make_float4(acc[i][m][0], acc[i][m][1], acc[i][m][2], acc[i][m][3]);
        } else {
            // strips alternate gate, up for the same 16 MLP columns
#pragma unroll
            for (int i = 0; i + 1 < NB; i += 2)
                if (i + 1 < nvalid) {
                    const int f = ((nb0 + i) >> 1) * 16 + col4;
                    f16_t o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = f2h(silu_f(acc[i][m][e]) * acc[i + 1][m][e]);
                    const size_t at = pk_index(row, f, a.kp_out);
                    *(uint2*)(a.out_packed + at) = *(const uint2*)o;
                }
        }
    }
}

// ------------------------------------------------------------------------------------------ sweep GEMM
// Up to 192 token rows (12 row strips), for projections large enough to give every compute unit one workgroup
// with several waves of work.  What bounds a weight stream on this chip is the number of bytes a compute unit can have in
// flight towards L2/HBM, and every byte requested through the vector memory path counts, also an activation
// operand that hits in L2: in the kernel above, where each wave fetches its own activation operands, those
// take a quarter of that budget (2 strips) or an eighth (4 strips).  Here the waves of a workgroup own
// different output strips and sweep the same k-range together, so an activation chunk (KC k-blocks,
// all row strips) is fetched once per workgroup, staged in LDS (double-buffered, one barrier per chunk) and
// read from there by every wave; one workgroup per compute unit means once per unit.  No wave shares an
// output with another: no reduction at the end, and the SwiGLU epilogue stays inside the wave that owns a
// gate strip and its up strip.  Weight loads run two chunks ahead in two named register slots; nothing in
// the loop is conditional, so the load counter waits are exact.  K-blocks beyond the k-slice and strips
// beyond the matrix read a block of zeros instead of weights (an L2 hit) and add 0.
// With KH = 2 two waves share a unit: wave 2u takes the first half of every chunk's k-blocks, wave 2u + 1 the second
// (each loads only its own weight blocks and reads only its own operands from LDS); the odd wave hands its
// accumulators to the even one through LDS at the end.  Used above 96 rows when a workgroup owns at most 4 units:
// there the matrix-core and LDS work per weight byte grows with the row strips, and 3 or 4 waves (one per SIMD,
// nothing to overlap their waits with) no longer keep up with the weight stream.
// With WN = 1 the weights come in the 12-bit form, one group of 4 k-blocks per wave and chunk.  A workgroup with at most
// 4 units then always runs two waves per unit on chunks of 8 k-blocks: 4 waves have too few of the shorter loads in
// flight (16 rows, one / two waves per unit: down 16.4 / 14.6 us, gate|up 26.7 / 25.8, o at 24 rows 8.5 / 7.4).
template <int NBW, int KQ, int WN>
struct SweepSlot {
    static_assert(!WN || KQ == 4, "a 12-bit group covers 4 k-blocks");
    u32x4 w[NBW][WN ? 3 : KQ];   // KQ = k-blocks of a chunk this wave handles
};

template <int NBW, int KQ, int WN>
__device__ __forceinline__ void sweep_load_w(SweepSlot<NBW, KQ, WN>& f, const u32x4* __restrict__ Wl,
                                             const u32x4* __restrict__ Zl, int KB, int nb0, int nvalid, int kb, int kend)
{
    if (WN) {   // slices are whole groups: a chunk is either inside or beyond
        const int kg = min(kb, kend - 4) >> 2;
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            const uintptr_t wp = (uintptr_t)(Wl + (nb0 + i) * narrow_strip(KB) + (size_t)kg * 192), zp = (uintptr_t)Zl;
            const uintptr_t mask = (kb < kend && i < nvalid) ? ~(uintptr_t)0 : (uintptr_t)0;
            const u32x4* g = (const u32x4*)(zp ^ ((wp ^ zp) & mask));
#pragma unroll
            for (int p = 0; p < 3; ++p) f.w[i][p] = __builtin_nontemporal_load(g + p * 64);
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < (WN ? 0 : KQ); ++q) {
        const bool live = kb + q < kend;
        const int kk = min(kb + q, kend - 1);
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            // weights or the zero block: selected by address arithmetic (a select between two pointers can be
            // compiled into a branch around the load)
            const uintptr_t wp = (uintptr_t)(Wl + ((size_t)(nb0 + i) * KB + kk) * 64), zp = (uintptr_t)Zl;
            const uintptr_t mask = (live && i < nvalid) ? ~(uintptr_t)0 : (uintptr_t)0;
            f.w[i][q] = __builtin_nontemporal_load((const u32x4*)(zp ^ ((wp ^ zp) & mask)));
        }
    }
}

// An activation chunk is KC*MT operand blocks of 64 x 16 bytes, block m*KC + q = row strip m, k-block q of
// the chunk.  Thread t of the workgroup moves pieces t, t + 64P, ...;
// indices past the end are clamped to the last piece (the same bytes written twice).
template <int P, int MT, int KC>
struct SweepStage {
    static constexpr int PIECES = KC * MT * 64;
    static constexpr int XI = (PIECES + 64 * P - 1) / (64 * P);
    u32x4 v[XI];
};

template <int P, int MT, int KC>
__device__ __forceinline__ void sweep_load_x(SweepStage<P, MT, KC>& xs, const u32x4* __restrict__ X, int KB, int kb,
                                             int kend)
{
#pragma unroll
    for (int i = 0; i < SweepStage<P, MT, KC>::XI; ++i) {
        const int piece = min((int)threadIdx.x + i * 64 * P, SweepStage<P, MT, KC>::PIECES - 1);
        const int b = piece >> 6, l = piece & 63;
        const int m = b / KC, q = b % KC;
        const int kk = min(kb + q, kend - 1);
        xs.v[i] = X[((size_t)m * KB + kk) * 64 + l];
    }
}

template <int P, int MT, int KC>
__device__ __forceinline__ void sweep_store_x(const SweepStage<P, MT, KC>& xs, u32x4* buf)
{
#pragma unroll
    for (int i = 0; i < SweepStage<P, MT, KC>::XI; ++i)
        buf[min((int)threadIdx.x + i * 64 * P, SweepStage<P, MT, KC>::PIECES - 1)] = xs.v[i];
}

// q0: first k-block of the chunk this wave handles (0, or KC/2 for the second wave of a pair).
template <int MT, int NBW, int KC, int KQ, int WN>
__device__ __forceinline__ void sweep_mma(const SweepSlot<NBW, KQ, WN>& f, const u32x4* buf, int lane, int q0,
                                          f32x4 (&acc)[NBW][MT])
{
    u32x4 wn[NBW][WN ? 4 : 1];
    if constexpr (WN) {
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            wn[i][0] = narrow_group_frag<0>(f.w[i]);
            wn[i][1] = narrow_group_frag<1>(f.w[i]);
            wn[i][2] = narrow_group_frag<2>(f.w[i]);
            wn[i][3] = narrow_group_frag<3>(f.w[i]);
        }
    }
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
        u32x4 xv[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) xv[m] = buf[(m * KC + q0 + q) * 64 + lane];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int i = 0; i < NBW; ++i)
                acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                    __builtin_bit_cast(f16x8, WN ? wn[i][WN ? q : 0] : f.w[i][WN ? 0 : q]),
                    __builtin_bit_cast(f16x8, xv[m]), acc[i][m], 0, 0, 0);
    }
}

// The k sweep of one wave.  ACTIVE = false is a wave without a unit (the workgroup got fewer than P): it only
// moves its share of the activation chunks and keeps the barriers; weight loads for it, even of the zero
// block, would take their share of the compute unit's memory requests.  The two variants are separate
// straight-line loops, chosen once per wave, because a load under a branch inside the loop would make
// every wait there cover all loads in flight.
template <bool ACTIVE, int P, int MT, int NBW, int KC, int KH, int WN>
__device__ __forceinline__ void sweep_run(u32x4* xl0, u32x4* xl1, f32x4 (&acc)[NBW][MT],
                                          const u32x4* __restrict__ Wl, const u32x4* __restrict__ Zl,
                                          const u32x4* __restrict__ X, int KB, int nb0, int nvalid, int s0, int s1,
                                          int C, int lane, int q0)
{
    constexpr int KQ = KC / KH;
    SweepSlot<NBW, KQ, WN> fa, fb;
    SweepStage<P, MT, KC> xs;
    sweep_load_x<P, MT, KC>(xs, X, KB, s0, s1);
    if (ACTIVE) sweep_load_w<NBW, KQ, WN>(fa, Wl, Zl, KB, nb0, nvalid, s0 + q0, s1);
    __builtin_amdgcn_sched_barrier(0);
    sweep_store_x<P, MT, KC>(xs, xl0);
    __builtin_amdgcn_sched_barrier(0);
    sweep_load_x<P, MT, KC>(xs, X, KB, s0 + KC, s1);
    if (ACTIVE) sweep_load_w<NBW, KQ, WN>(fb, Wl, Zl, KB, nb0, nvalid, s0 + KC + q0, s1);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // Two chunks per trip (slot fa with LDS buffer 0, slot fb with buffer 1).  Within a chunk: contract it,
    // write the next chunk's activations (loaded one chunk ago) into the other buffer, start the loads of
    // the chunk after that, barrier.  A buffer is rewritten one barrier after its last read.
    for (int c = 0; c < C; c += 2) {
        const int k2 = s0 + (c + 2) * KC, k3 = k2 + KC;
        if (ACTIVE) sweep_mma<MT, NBW, KC, KQ, WN>(fa, xl0, lane, q0, acc);
        __builtin_amdgcn_sched_barrier(0);
        sweep_store_x<P, MT, KC>(xs, xl1);
        __builtin_amdgcn_sched_barrier(0);
        sweep_load_x<P, MT, KC>(xs, X, KB, k2, s1);
        if (ACTIVE) sweep_load_w<NBW, KQ, WN>(fa, Wl, Zl, KB, nb0, nvalid, k2 + q0, s1);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        if (ACTIVE) sweep_mma<MT, NBW, KC, KQ, WN>(fb, xl1, lane, q0, acc);
        __builtin_amdgcn_sched_barrier(0);
        sweep_store_x<P, MT, KC>(xs, xl0);
        __builtin_amdgcn_sched_barrier(0);
        sweep_load_x<P, MT, KC>(xs, X, KB, k3, s1);
        if (ACTIVE) sweep_load_w<NBW, KQ, WN>(fb, Wl, Zl, KB, nb0, nvalid, k3 + q0, s1);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
    }
}

// Grid: n_gn workgroups per k-slice x ksplit; workgroup gn of a slice owns units [gn*n_units/n_gn,
// (gn+1)*n_units/n_gn) (a unit = NBW consecutive strips; at most P/KH of them, checked by the launcher), one per
// wave, or with KH = 2 one per pair of waves.
template <int P, int MT, int NBW, int EPI, int KH, int WN>
__global__ __launch_bounds__(64 * P) void k_gemm_sweep(GemmArgs a, int n_units, int n_gn, int kb_per_slice)
{
    // k-blocks per chunk: 4 (both staging buffers: 8 KiB per row strip, at most 96 KiB).
    // Measured: one strip 4 against 2 and 8, 5-8 strips 4 against 2: 4 is the fastest; 9-12 strips 4 against 2: 4 % faster.
    constexpr int KC = WN ? 4 * KH : 4;
    static_assert(KC % KH == 0, "a chunk's k-blocks split evenly between the waves of a unit");
    constexpr int STAGE = SweepStage<P, MT, KC>::PIECES;
    // two staging buffers; after the sweep the same memory carries the odd waves' accumulators (KH = 2)
    constexpr int RED = KH == 2 ? (P / 2) * NBW * MT * 64 : 0;
    __shared__ u32x4 xlds[2 * STAGE > RED ? 2 * STAGE : RED];
    u32x4* const xl0 = xlds;
    u32x4* const xl1 = xlds + STAGE;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gn = blockIdx.x % n_gn, ks = blockIdx.x / n_gn;
    const int KB = a.Kp >> 5, NBT = a.N >> 4;
    const int s0 = ks * kb_per_slice, s1 = min(KB, s0 + kb_per_slice);
    const int u0 = (int)((long long)gn * n_units / n_gn), u1 = (int)((long long)(gn + 1) * n_units / n_gn);
    const int slot = wave / KH;                   // unit slot of this wave inside the workgroup
    const int q0 = (wave % KH) * (KC / KH);       // first k-block of every chunk this wave handles
    const int unit = u0 + slot;
    const int nb0 = unit * NBW;
    const int nvalid = unit < u1 ? max(min(NBW, NBT - nb0), 0) : 0;
    const bool active = nvalid > 0;   // wave-uniform

    f32x4 acc[NBW][MT];
#pragma unroll
    for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[i][m] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const u32x4* Wl = (const u32x4*)(WN ? a.Wn : a.W) + lane;
    const u32x4* Zl = (const u32x4*)a.zero_blk + lane;
    const u32x4* X = (const u32x4*)a.X;
    const int C = (s1 - s0 + KC - 1) / KC;   // chunks of this slice: the same for every wave of the workgroup
    if (C > 0) {
        if (active)
            sweep_run<true, P, MT, NBW, KC, KH, WN>(xl0, xl1, acc, Wl, Zl, X, KB, nb0, nvalid, s0, s1, C, lane, q0);
        else
            sweep_run<false, P, MT, NBW, KC, KH, WN>(xl0, xl1, acc, Wl, Zl, X, KB, nb0, nvalid, s0, s1, C, lane, q0);
    }
    if (KH == 2) {
        // the odd wave of a pair hands its sums to the even one (the staging buffers are free after the last barrier
        // of the sweep; with no chunk at all nobody has touched them)
        f32x4* red = (f32x4*)xlds;
        if (active && (wave & 1)) {
#pragma unroll
            for (int i = 0; i < NBW; ++i)
#pragma unroll
                for (int m = 0; m < MT; ++m) red[((slot * NBW + i) * MT + m) * 64 + lane] = acc[i][m];
        }
        __syncthreads();
        if (wave & 1) return;
        if (active) {
#pragma unroll
            for (int i = 0; i < NBW; ++i)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[i][m] += red[((slot * NBW + i) * MT + m) * 64 + lane];
        }
    }
    if (!active) return;
    if (WN) {
#pragma unroll
        for (int i = 0; i < NBW; ++i)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[i][m] *= kNarrowScale;
    }

    const int col4 = (lane >> 4) * 4;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = m * 16 + (lane & 15);
        if (row >= a.m_rows) continue;
        if (EPI == EPI_PARTIAL) {
            float* o = a.out + ((size_t)ks * a.m_stride + row) * a.N;
#pragma unroll
            for (int i = 0; i < NBW; ++i)
                if (i < nvalid)
                    *(float4*)(o + (nb0 + i) * 16 + col4) =
                        make_float4(acc[i][m][0], acc[i][m][1], acc[i][m][2], acc[i][m][3]);
        } else {
#pragma unroll
            for (int i = 0; i + 1 < NBW; i += 2)
                if (i + 1 < nvalid) {
                    const int f = ((nb0 + i) >> 1) * 16 + col4;
                    f16_t o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = f2h(silu_f(acc[i][m][e]) * acc[i + 1][m][e]);
                    const size_t at = pk_index(row, f, a.kp_out);
                    *(uint2*)(a.out_packed + at) = *(const uint2*)o;
                }
        }
    }
}

// ------------------------------------------------------------------------------------------ GEMM of few rows
// Decode forwards of up to kFewRows rows that stream 12-bit weights.  So few rows' activations are small enough for every workgroup
// to hold all of them: it normalises the residual stream itself (every workgroup the same numbers), or has whole sums and
// adds them to the stream itself, so that no norm is launched, and reads them from LDS without a barrier in its loop.  The
// norm's trip to memory runs beside the weights' first ones.
// The numbers are those of the kernels above, bit for bit, so that a row gets the same whether other rows of its strip are alive
// or not: a unit's k-blocks are summed in the same chains (FewPlan), the chains added in the same order, and the sums of
// squares taken in the order of k_rmsnorm<1024, 2>.
// What bounds it: the weight stream, and per launch the trip to memory for the activations before the first product.  7B, one
// row, us per launch, before (norm + projection) / now: q|k|v 4.3 + 14.0 / 14.2, o 7.1 / 7.0, gate|up 4.3 + 24.4 / 24.3, down 13.4 / 14.2; a layer with its
// attention 72.7 / 65; decode of one row, 24 steps 59.3 -> 54.4 ms.  Four rows 74.8 -> 72.6: every workgroup reads and norms all of them, which more
// rows would not pay for (kFewRows).
template <int R, int NBW, int EPI, bool NORM, int PR = 1>
__global__ __launch_bounds__(64 * kFewWaves) void k_gemm_few(FewArgs a)
{
    constexpr int T = 64 * kFewWaves, VT = 1024 / T;   // VT: threads of the norm that a thread stands for
    extern __shared__ __attribute__((aligned(16))) char few_lds[];
    const int KB = a.Kp >> 5, xrow = a.Kp + 32;        // 64 bytes between rows: the rows' operand pieces are in different banks
    f16_t* const xs = (f16_t*)few_lds;                                     // [R][xrow]
    f32x4* const red = (f32x4*)(few_lds + (size_t)R * xrow * 2);           // [kFewWaves][NBW][64]
    float* const sq = (float*)(red + kFewWaves * NBW * 64);                // [R][16]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const FewPlan& p = a.plan;

    // activations on their way first, then the weights: what is used first returns first
    float4 v[NORM ? R : 1][VT][2];
    uint2 wr[VT][2];
    constexpr int NP = NORM ? 1 : PR * R;   // 16-byte pieces per thread: rows of up to PR * 4096 columns
    u32x4 piece[NP];
    const int n_pieces = NORM ? 0 : (a.Kp >> 3) * R;
    if (NORM) {
#pragma unroll
        for (int t = 0; t < VT; ++t)
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int c = (tid + t * T) * 4 + it * 4096;
                if (c < a.Kp) {
                    wr[t][it] = *(const uint2*)(a.gain + c);
#pragma unroll
                    for (int r = 0; r < R; ++r) v[NORM ? r : 0][t][it] = *(const float4*)(a.x + (size_t)r * a.Kp + c);
                }
            }
    } else {
        const __amdgpu_buffer_rsrc_t xsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.X, (short)0, KB * 1024, 0x00020000);
#pragma unroll
        for (int i = 0; i < NP; ++i) {   // beyond the last piece: beyond the buffer
            const int z = tid + i * T, r = z % R, kg = z / R;   // k-group kg of row r
            piece[i] = __builtin_amdgcn_raw_buffer_load_b128(xsrc, (kg >> 2) * 1024 + ((kg & 3) * 16 + r) * 16, 0, 0);
        }
    }

    const int slot = wave / p.items, item = wave - slot * p.items;
    const int unit = blockIdx.x * p.units_wg + slot;
    const bool active = slot < p.units_wg && unit < a.units;   // wave-uniform
    // this wave's chain: groups first, first + step, ... of 4 k-blocks, count of them
    const int slice = item / p.parts, part = item - slice * p.parts;
    const int s0 = slice * p.kb_slice, s1 = min(KB, s0 + p.kb_slice);
    const int G = max(s1 - s0, 0) >> 2;
    int first = s0 >> 2, step = 1, count = G, restart = 0;
    if (p.wave_kb) {   // contiguous quarters of the slice, whole groups: each a chain
        const int quarter = (((max(s1 - s0, 0) + 3) >> 2) + 3) >> 2;
        if (p.parts == 4) {
            first += min(G, part * quarter);
            count = min(G, (part + 1) * quarter) - min(G, part * quarter);
        } else {
            restart = quarter;
        }
    } else if (p.parts == 2) {   // groups in turn
        first += part;
        step = 2;
        count = (G - part + 1) >> 1;
    }
    if (!active) count = 0;
    const size_t strip_bytes = narrow_strip(KB) * 16;
    const __amdgpu_buffer_rsrc_t wsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)a.Wn + (active ? (size_t)unit * NBW : 0) * strip_bytes),
                                                                          (short)0, (int)(NBW * strip_bytes), 0x00020000);
    struct Slot {
        u32x4 w[NBW][3];
    } fa, fb;
    auto load = [&](Slot& f, int i) {   // past the chain's end: beyond the buffer, nothing is fetched
        const unsigned at = i < count ? (unsigned)((first + i * step) * 3072 + lane * 16) : 0xF0000000u;
#pragma unroll
        for (int n = 0; n < NBW; ++n)
#pragma unroll
            for (int z = 0; z < 3; ++z)
                f.w[n][z] = __builtin_amdgcn_raw_buffer_load_b128(wsrc, at + (unsigned)(z * 1024 + n * (int)strip_bytes), 0, 2);
    };
    load(fa, 0);
    load(fb, 1);
    __builtin_amdgcn_sched_barrier(0);

    float4 old = make_float4(0.f, 0.f, 0.f, 0.f);   // the residual stream at this lane's place
    const int col4 = (lane >> 4) * 4, row = lane & 15;
    if (NORM) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < VT; ++t) {
                float ss = 0.f;
#pragma unroll
                for (int it = 0; it < 2; ++it)
                    if ((tid + t * T) * 4 + it * 4096 < a.Kp) ss += norm_squares(v[NORM ? r : 0][t][it]);
                ss = wave_sum(ss);
                if (lane == 0) sq[r * 16 + t * kFewWaves + wave] = ss;
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float tot = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) tot += sq[r * 16 + i];
            const float f = rsqrtf(tot / (float)a.Kp + a.eps);
#pragma unroll
            for (int t = 0; t < VT; ++t)
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int c = (tid + t * T) * 4 + it * 4096;
                    if (c < a.Kp) norm_store(xs + r * xrow + c, v[NORM ? r : 0][t][it], f, wr[t][it]);
                }
        }
    } else {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int z = tid + i * T, r = z % R, kg = z / R;
            if (z < n_pieces) *(u32x4*)(xs + r * xrow + kg * 8) = piece[i];
        }
    }
    __syncthreads();

    f32x4 acc[NBW], tot[NBW];
#pragma unroll
    for (int n = 0; n < NBW; ++n) acc[n] = tot[n] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const f16_t* const xl = xs + min(row, R - 1) * xrow + (lane >> 4) * 8;
    int left = restart;
    auto use = [&](const Slot& f, int i) {
        const f16_t* xg = xl + (first + i * step) * 128;
        u32x4 xv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) xv[q] = *(const u32x4*)(xg + q * 32);
#pragma unroll
        for (int n = 0; n < NBW; ++n) {
            const u32x4 w[4] = {narrow_group_frag<0>(f.w[n]), narrow_group_frag<1>(f.w[n]), narrow_group_frag<2>(f.w[n]),
                                narrow_group_frag<3>(f.w[n])};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w[q]), __builtin_bit_cast(f16x8, xv[q]),
                                                                acc[n], 0, 0, 0);
        }
        if (restart > 0 && --left == 0) {   // the chain ends: the next one begins at zero
            left = restart;
#pragma unroll
            for (int n = 0; n < NBW; ++n) {
                tot[n] = tot[n] + acc[n];
                acc[n] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        }
    };
#pragma unroll 1
    for (int i = 0; i < count; i += 2) {
        use(fa, i);
        load(fa, i + 2);
        if (i + 1 < count) use(fb, i + 1);
        load(fb, i + 3);
    }
#pragma unroll
    for (int n = 0; n < NBW; ++n) red[(wave * NBW + n) * 64 + lane] = restart > 0 ? tot[n] + acc[n] : acc[n];
    const bool stores = active && item == 0 && row < R;
    if (EPI == EPI_RESIDUAL && stores) old = *(const float4*)(a.out + (size_t)row * a.N + unit * 16 + col4);
    __syncthreads();
    if (!stores) return;
    f32x4 sum[NBW];
#pragma unroll
    for (int n = 0; n < NBW; ++n) sum[n] = EPI == EPI_RESIDUAL ? (f32x4){old.x, old.y, old.z, old.w} : (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < p.items; i += p.parts)
#pragma unroll
        for (int n = 0; n < NBW; ++n) {
            f32x4 z = red[((wave + i) * NBW + n) * 64 + lane];
            for (int j = 1; j < p.parts; ++j) z += red[((wave + i + j) * NBW + n) * 64 + lane];
            z *= kNarrowScale;
            sum[n] = EPI == EPI_SWIGLU ? z : sum[n] + z;
        }
    if (EPI == EPI_SWIGLU) {
        const int f = unit * 16 + col4;
        f16_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = f2h(silu_f(sum[0][e]) * sum[NBW - 1][e]);
        *(uint2*)(a.out_packed + pk_index(row, f, a.kp_out)) = *(const uint2*)o;
    } else {
        *(float4*)(a.out + (size_t)row * a.N + unit * 16 + col4) = make_float4(sum[0][0], sum[0][1], sum[0][2], sum[0][3]);
    }
}

// ------------------------------------------------------------------------------------------ block GEMM
// Many token rows (prompt forwards; decode batches beyond sweep_rows): both operands go through LDS, so that every
// byte fetched from L2 feeds MS or NS strips instead of one wave's.  A workgroup computes MS*16 token rows x NS*16 output
// columns with WM x WN waves of (MS/WM) x (NS/WN) strips each.  A stage is one k-block of both tiles, MS + NS operand
// blocks of 1 KiB, copied from global memory straight into LDS (no registers, no address arithmetic per lane: a block is
// contiguous and lands in the order in which a wave reads it back, conflict-free).  ST stages form a ring; a stage is
// requested ST - 1 trips before it is read.  One trip: wait until the next stage has landed, barrier, then, spread over
// the matrix instructions of this trip, the copies of the stage ST ahead into the slot that the barrier has just freed
// and the LDS reads of the next trip's operands.
// What bounds it: the power the chip may take.  On random data the matrix instructions alone run at 2.0 PFLOP/s (the clock
// falls to 2.06 GHz), with the LDS reads beside them at 1.68, with the copies too at 1.33 to 1.38.  A trip (256 x 256 x 32)
// takes 1131 clocks (1249 before the reads were given out between the products and the copies' addresses cut to one
// addition), 1024 of them matrix work: with the order of the tiles, gate|up of 7B in a prompt forward of 12311 rows takes
// 1692 us instead of 1748 (1.31 PFLOP/s; launched alone, 1603).  Measured against the kernel it replaced (weights straight
// from L2 to registers, 64 or 128 rows per tile) before that, gate|up: 256 rows 73.7 -> 56.3 us, 494 123 -> 81, 995 216 ->
// 166, 3146 544 -> 488, 12311 1989 -> 1743; down 494 67 -> 49, 995 98 -> 87, 4200 504 -> 351.
// The copies are written in assembly because the compiler would wait for all of them before every LDS read: it counts
// only its own loads, and the waits here are written out.  They name no output register; waits that the compiler adds
// for loads of its own can only be too strict.
__device__ __forceinline__ void lds_copy_1k(unsigned slot, unsigned place, const void* base, unsigned lane_off)
{
    asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" ::"s"(slot), "s"(place), "v"(lane_off), "s"(base)
                 : "memory", "scc");
}

// At most N copies of this wave are still on their way, its LDS reads are done, and then so are every other wave's.  The
// builtin tells the compiler that the operands read before are in their registers (after a wait in assembly it would wait
// for each of them once more).
template <int N>
__device__ __forceinline__ void wait_copies_and_meet()
{
    static_assert(N < 64, "the counter has 6 bits");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));   // vmcnt(N) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// Unsliced launches finish their results themselves.  EPI_RESIDUAL adds the sums to the residual stream in place, EPI_QKV
// rotates q and k and puts q, k and v where the attention reads them, instead of writing fp32 sums for the next launch to
// read.  12311 token-rows, 7B, per layer: the rotation launch (184 us) is gone, the norms take 108 us instead of 167, o
// and down 716 instead of 680, q|k|v 1112 instead of 1097 (k_rope_append and the sums in the norm stay for sliced launches).
template <int MS, int NS, int WM, int WN, int ST, int EPI>
__global__ __launch_bounds__(64 * WM * WN, 2) void k_gemm_block(GemmArgs a, QkvOut qo, int kb_per_slice,
                                                                                  int n_ntiles, int n_mtiles)
{
    constexpr int W = WM * WN;                 // waves
    constexpr int RM = MS / WM, RN = NS / WN;  // strips per wave
    constexpr int SB = MS + NS;                // operand blocks of a stage
    constexpr int CP = (SB + W - 1) / W;       // copies per wave and stage (the same for all: the last block may go twice)
    static_assert(MS % WM == 0 && NS % WN == 0, "even shares");
    __shared__ u32x4 ring[ST][SB][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int KB = a.Kp >> 5, NBT = a.N >> 4, MBT = (a.m_rows + 15) >> 4;
    const int tiles = n_ntiles * n_mtiles, ks = blockIdx.x / tiles;
    const BlockPlace place_of = block_place(blockIdx.x % tiles, n_ntiles, n_mtiles, MS);
    const int nb0 = place_of.n_tile * NS, mb0 = place_of.m_tile * MS;
    const int s0 = ks * kb_per_slice, s1 = min(KB, s0 + kb_per_slice);
    const int trips = s1 - s0;

    f32x4 acc[RN][RM];
#pragma unroll
    for (int i = 0; i < RN; ++i)
#pragma unroll
        for (int m = 0; m < RM; ++m) acc[i][m] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // this wave copies blocks wave*CP .. +CP-1 of a stage: the first MS are activation strips, the others weight strips
    constexpr unsigned STAGE = SB * 1024;   // bytes
    const char* src[CP];
    unsigned place[CP];
    const unsigned ring0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)&ring[0][0][0];
#pragma unroll
    for (int c = 0; c < CP; ++c) {
        const int blk = min(wave * CP + c, SB - 1);
        const char* p = blk < MS ? (const char*)a.X + (size_t)min(mb0 + blk, MBT - 1) * KB * 1024
                                 : (const char*)a.W + (size_t)min(nb0 + blk - MS, NBT - 1) * KB * 1024;
        src[c] = p + (size_t)s0 * 1024;
        place[c] = ring0 + (unsigned)(blk * 1024);
    }
    // a lane's offset into the k-block of this trip, inside any strip; k-blocks beyond the slice: the last one once more, never used
    auto lane_off = [&](int trip) { return (unsigned)(min(trip, trips - 1) * 1024 + lane * 16); };
    u32x4 xf[2][RM], wf[2][RN];
    if (trips > 0) {
#pragma unroll
        for (int q = 0; q < ST; ++q)
#pragma unroll
            for (int c = 0; c < CP; ++c) lds_copy_1k(q * STAGE, place[c], src[c], lane_off(q));
        wait_copies_and_meet<(ST - 1) * CP>();
#pragma unroll
        for (int i = 0; i < RN; ++i) wf[0][i] = ring[0][MS + wn * RN + i][lane];
#pragma unroll
        for (int m = 0; m < RM; ++m) xf[0][m] = ring[0][wm * RM + m][lane];
        unsigned slot = 0;   // byte offset of this trip's stage
        auto trip = [&](int it, u32x4 (&xc)[RM], u32x4 (&wc)[RN], u32x4 (&xn)[RM], u32x4 (&wn_)[RN]) {
            // the operands of this trip are in registers; the next stage has landed, and this one's place is free
            wait_copies_and_meet<(ST - 2) * CP>();
            const unsigned at = lane_off(it + ST), free_slot = __builtin_amdgcn_readfirstlane(slot);
            slot = slot + STAGE == ST * STAGE ? 0u : slot + STAGE;
            const u32x4* st = (const u32x4*)((const char*)&ring[0][0][0] + slot) + lane;
            // In exactly this order: a product each with the reads of the next trip's operands until all are on their way
            // (the last ones would hold up the wait above otherwise), the copies evenly among the products (all at once
            // they hold up every wave of the workgroup behind the address unit).
            constexpr int R = RM + RN, E = RM * RN;
            static_assert(R <= E && CP <= E, "a product for each");
#pragma unroll
            for (int e = 0; e < E; ++e) {
                acc[e % RN][e / RN] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, wc[e % RN]),
                                                                             __builtin_bit_cast(f16x8, xc[e / RN]),
                                                                             acc[e % RN][e / RN], 0, 0, 0);
                if (e < RN) wn_[e < RN ? e : 0] = st[(MS + wn * RN + e) * 64];
                else if (e < R) xn[e >= RN && e < R ? e - RN : 0] = st[(wm * RM + e - RN) * 64];
#pragma unroll
                for (int c = 0; c < CP; ++c)
                    if (c * E / CP == e) lds_copy_1k(free_slot, place[c], src[c], at);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int it = 0;
        for (; it + 2 <= trips; it += 2) {
            trip(it, xf[0], wf[0], xf[1], wf[1]);
            trip(it + 1, xf[1], wf[1], xf[0], wf[0]);
        }
        if (it < trips) trip(it, xf[0], wf[0], xf[1], wf[1]);
        wait_copies_and_meet<0>();   // nothing may still be on its way into LDS when the workgroup ends
    }

    const int col4 = (lane >> 4) * 4;
    const int c0 = nb0 + wn * RN, r0 = mb0 + wm * RM;
#pragma unroll
    for (int m = 0; m < RM; ++m) {
        const int row = (r0 + m) * 16 + (lane & 15);
        if (row >= a.m_rows) continue;
        if (EPI == EPI_PARTIAL) {
            float* o = a.out + ((size_t)ks * a.m_stride + row) * a.N;
#pragma unroll
            for (int i = 0; i < RN; ++i)
                if (c0 + i < NBT)
                    *(float4*)(o + (c0 + i) * 16 + col4) = make_float4(acc[i][m][0], acc[i][m][1], acc[i][m][2], acc[i][m][3]);
        } else if (EPI == EPI_RESIDUAL) {
            float* o = a.out + (size_t)row * a.N;
#pragma unroll
            for (int i = 0; i < RN; ++i)
                if (c0 + i < NBT) {
                    float4* p = (float4*)(o + (c0 + i) * 16 + col4);
                    const float4 x = *p;
                    *p = make_float4(x.x + acc[i][m][0], x.y + acc[i][m][1], x.z + acc[i][m][2], x.w + acc[i][m][3]);
                }
        } else if (EPI == EPI_QKV) {
            const int mb_row = qo.st.tr_row[row], pos = qo.st.tr_pos[row];
            const int d = a.N / 3, half = qo.hd >> 1, hs = qo.hd >> 4, part_strips = d >> 4;
            const int64_t slab = qo.st.row_so[mb_row] * d;
            const int cap = qo.st.row_cap[mb_row];
#pragma unroll
            for (int i = 0; i + 1 < RN; i += 2)
                if (c0 + i + 1 < NBT) {
                    const int part = (c0 + i) / part_strips, strip = (c0 + i) - part * part_strips;   // wave-uniform
                    const int h = strip / hs, e = ((strip - h * hs) >> 1) * 16 + col4;
                    float x[4], y[4];   // elements e..e+3 and their partners
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        x[q] = acc[i][m][q];
                        y[q] = acc[i + 1][m][q];
                    }
                    if (part < 2) {
                        const float4 c4 = *(const float4*)(qo.rcos + (size_t)pos * half + e);
                        const float4 s4 = *(const float4*)(qo.rsin + (size_t)pos * half + e);
                        const float cs[4] = {c4.x, c4.y, c4.z, c4.w}, sn[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float2 r = rotated(x[q], y[q], cs[q], sn[q]);
                            x[q] = r.x;
                            y[q] = r.y;
                        }
                    }
                    if (part == 0) {
                        float* o = qo.qrot + (size_t)row * d + h * qo.hd + e;
                        *(float4*)o = make_float4(x[0], x[1], x[2], x[3]);
                        *(float4*)(o + half) = make_float4(y[0], y[1], y[2], y[3]);
                    } else {
                        kv_t* o = (part == 1 ? qo.kc : qo.vc) + slab + ((size_t)h * cap + pos) * qo.hd + e;
                        const kv_t xv[4] = {f2kv(x[0]), f2kv(x[1]), f2kv(x[2]), f2kv(x[3])};
                        const kv_t yv[4] = {f2kv(y[0]), f2kv(y[1]), f2kv(y[2]), f2kv(y[3])};
                        *(uint2*)o = *(const uint2*)xv;
                        *(uint2*)(o + half) = *(const uint2*)yv;
                    }
                }
        } else {
#pragma unroll
            for (int i = 0; i + 1 < RN; i += 2)
                if (c0 + i + 1 < NBT) {
                    const int f = ((c0 + i) >> 1) * 16 + col4;
                    f16_t o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = f2h(silu_f(acc[i][m][e]) * acc[i + 1][m][e]);
                    const size_t at = pk_index(row, f, a.kp_out);
                    *(uint2*)(a.out_packed + at) = *(const uint2*)o;
                }
        }
    }
}

// ------------------------------------------------------------------------------------------ RoPE + KV append
// Token-row j: sums the k-slices of its [q | k | v] projection, rotates q and k at the row's position
// (pairs e, e + hd/2; cos/sin from a table indexed [pos][e]), stores q as fp32 and k, v as IEEE half (kv_t) into the
// row's key/value slab: element (head h, slot s, e) of row i lives at so[i]*d + (h*cap[i] + s)*hd + e.
// One pair of elements per thread, 256 of them per workgroup: a prompt of a few dozen tokens is all latency, and a workgroup per row made a
// row's pieces wait for each other (47 token-rows, 7B: 9.6 -> 5.3 us; their prompt forward through 8 layers and the head 883 -> 843, 80 token-rows of 13B through 6 1005 -> 956).
__global__ __launch_bounds__(256) void k_rope_append(MbState st, const float* __restrict__ part, int ksplit,
                                                     size_t part_stride, float* __restrict__ qrot,
                                                     kv_t* __restrict__ kc, kv_t* __restrict__ vc,
                                                     const float* __restrict__ rcos, const float* __restrict__ rsin,
                                                     int d, int H, int hd)
{
    const int j = blockIdx.x, idx = blockIdx.y * 256 + threadIdx.x;
    const int count = *st.d_n;
    const int row = st.tr_row[j], pos = st.tr_pos[j];
    const int half = hd >> 1;
    if (j >= count || idx >= (d >> 1)) return;
    const size_t slab = (size_t)st.row_so[row] * d;
    const int cap = st.row_cap[row];
    const int h = idx / half, e = idx - h * half;
    const int c = h * hd + e;
    const float* p = part + (size_t)j * 3 * d + h * hd + qkv_col(e);
    float v[kNormMaxSplit][6];   // q, k, v of this element and of its partner; every slice's loads before the first sum
#pragma unroll
    for (int s = 0; s < kNormMaxSplit; ++s)
#pragma unroll
        for (int i = 0; i < 6; ++i) v[s][i] = s < ksplit ? p[s * part_stride + (i >> 1) * d + (i & 1) * 16] : 0.f;
    const float cs = rcos[(size_t)pos * half + e], sn = rsin[(size_t)pos * half + e];
    float t[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        t[i] = 0.f;
#pragma unroll
        for (int s = 0; s < kNormMaxSplit; ++s) t[i] += v[s][i];
    }
    const float2 q = rotated(t[0], t[1], cs, sn), k = rotated(t[2], t[3], cs, sn);
    qrot[(size_t)j * d + c] = q.x;
    qrot[(size_t)j * d + c + half] = q.y;
    const size_t o = slab + ((size_t)h * cap + pos) * hd + e;
    kc[o] = f2kv(k.x);
    kc[o + half] = f2kv(k.y);
    vc[o] = f2kv(t[4]);
    vc[o + half] = f2kv(t[5]);
}

// ------------------------------------------------------------------------------------------ attention
// One workgroup per (token-row, head): softmax(q.K^T / sqrt(hd)) V over the row's own slots 0..pos.
// Two passes, exactly the max-subtracted definition: scores to LDS, block max and sum, then the weighted
// sum of V.  A wave's load covers 64/LPK consecutive keys (LPK = hd/8 lanes of 16 bytes per key), so K
// and V are each streamed once, fully coalesced; a wave issues AU such loads before it consumes them, so
// a context of a few hundred slots costs two or three memory round trips, not one per load.
// Short contexts are bound by vector instructions (a load's share of the dot products and of the sums is some 60), so the
// loads of a group that lie beyond the context are left out of both passes.  Per layer, 7B: 163 rows
// 31.4 -> 27.1 us, 51 rows 15.7 -> 14.1, one row 8.1 -> 6.8 (contexts of 16 to 70).
constexpr int kAttnUnroll = 8, kAttnShort = 4;   // loads of a wave before it consumes them; where that many hold the whole context
// (row, head) pairs, and trips of all waves over the context, for which a load that lies wholly beyond the context is skipped by a branch
// instead of issued for nothing: some units have a pair more than others there, and what those issue is on the longest path; with more
// trips, or next to no or many pairs a unit, the branches cost more.  Microseconds a launch, lanes tested (the form before buffers) / all loads
// issued / skipped: 288 pairs (7B, 9 rows) at 140 slots 8.0 / 8.7 / 7.8, 250 slots 10.8 / 11.3 / 10.5, 520 slots 17.0 / 18.1 / 16.9, 700 slots (6
// trips) 21.4 / 19.6 / 20.8; 640 pairs (13B, 16 rows) at 110 slots 10.2 / 10.7 / 10.3; 32 pairs at 200 slots 6.1 / 5.9 / 6.3; 1536 at 330 51.9 / 51.6 / 52.6.
constexpr int kAttnTailFrom = 256, kAttnTailTo = 1024, kAttnTailTrips = 3;

// The slots are dealt to NW slices, one per wave, or NW / PW for each of PW waves: the sums are the same sums in the same order.
// A wave's loads then go to its slices in turn, so that the workgroup walks over the slots as with NW = PW (one slice after the
// other it asks for every second 4 KB at a time: 16 rows of 40 heads, context 1500, 174 us a layer instead of 165).
// SPLIT: the slots are a share of the row's; their sums, maximum and total go to `share` (see k_attention_join).
// TAIL: loads that lie wholly beyond the context are not issued.
template <int HD, int NW, int PW, bool SPLIT, int AU, bool TAIL>
__device__ __forceinline__ void attend(const float* __restrict__ qs, float* __restrict__ sc, float* __restrict__ red,
                                       float (*__restrict__ oacc)[HD], const kv_t* __restrict__ kbase,
                                       const kv_t* __restrict__ vbase, int ctx, f16_t* __restrict__ out, int out_r,
                                       int out_k0, int out_kp, float* __restrict__ share)
{
    constexpr int LPK = HD / 8;       // lanes per key
    constexpr int KPW = 64 / LPK;     // keys per wave load
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = lane % LPK, kin = lane / LPK;
    constexpr int R = NW / PW;        // slices per wave
    static_assert(NW % PW == 0 && AU % R == 0, "every load of a trip belongs to one slice");
    const float scale = rsqrtf((float)HD);
    // Slots beyond the context are beyond the buffer: they read as zeros, and nothing is fetched for them.  A fifth of the
    // instructions of loads that test each lane (and 12 registers less); where they issue, 8 loads for the few slots of a short context
    // would take that back, hence the form with kAttnShort.  Decode step of 7B per layer: 64 rows at context 1000 296 -> 291 us, 16 rows 127.2 -> 126.5, 3000
    // slots 209 -> 207, one row 1000 77.0 -> 75.6; 51 rows at 40 slots 105.1 -> 104.3.
    auto slots = [&](const kv_t* base) {
        const uint64_t at = (uint64_t)base;
        const uint64_t u = (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)at) |
                           (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32;
        return __builtin_amdgcn_make_buffer_rsrc((void*)u, (short)0, __builtin_amdgcn_readfirstlane(ctx) * HD * 2, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t ksrc = slots(kbase), vsrc = slots(vbase);
    const unsigned lane_at = (unsigned)(kin * HD + sub * 8) * 2;
    auto load = [&](__amdgpu_buffer_rsrc_t src, int first) {   // this lane's piece of the wave's keys from `first` on
        if (TAIL && first >= ctx) return make_uint4(0, 0, 0, 0);   // wave-uniform
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(src, lane_at + (unsigned)(first * HD * 2), 0, 0));
    };
    float q[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) q[e] = qs[sub * 8 + e];

    float mx = -3.0e38f;
    for (int c0 = wave * KPW; c0 < ctx; c0 += PW * KPW * AU) {
        uint4 raw[AU];
#pragma unroll
        for (int u = 0; u < AU; ++u) {
            raw[u] = load(ksrc, c0 + u * PW * KPW);
        }
#pragma unroll
        for (int u = 0; u < AU; ++u) {
            if (c0 + u * PW * KPW >= ctx) break;   // wave-uniform: nothing of this load is inside the context
            const int s = c0 + u * PW * KPW + kin;
            const kv_t* kv = (const kv_t*)&raw[u];
            float part = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) part += q[e] * kv2f(kv[e]);
            part = group_sum<LPK>(part) * scale;
            if (s < ctx) {
                if (sub == 0) sc[s] = part;
                mx = fmaxf(mx, part);
            }
        }
    }
    // the first chunk of V does not depend on the scores: get it moving before the reductions
    uint4 vraw[AU];
#pragma unroll
    for (int u = 0; u < AU; ++u) {
        vraw[u] = load(vsrc, wave * KPW + u * PW * KPW);
    }
    mx = wave_max(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = red[0];
#pragma unroll
    for (int w = 1; w < PW; ++w) mx = fmaxf(mx, red[w]);
    float sum[R] = {};
    for (int s0 = wave * 64 + lane; s0 < ctx; s0 += 64 * NW)
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int s = s0 + i * 64 * PW;
            if (i > 0 && s >= ctx) break;
            const float p = __expf(sc[s] - mx);
            sc[s] = p;
            sum[i] += p;
        }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        sum[i] = wave_sum(sum[i]);
        if (lane == 0) red[PW + wave + i * PW] = sum[i];
    }
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) tot += red[PW + w];
    const float inv = 1.f / tot;

    float o[R][8] = {};
    for (int c0 = wave * KPW; c0 < ctx; c0 += PW * KPW * AU) {
        uint4 raw[AU];
#pragma unroll
        for (int u = 0; u < AU; ++u) {
            if (c0 == wave * KPW)
                raw[u] = vraw[u];
            else
                raw[u] = load(vsrc, c0 + u * PW * KPW);
        }
#pragma unroll
        for (int u = 0; u < AU; ++u) {
            if (c0 + u * PW * KPW >= ctx) break;
            const int s = c0 + u * PW * KPW + kin;
            const float p = s < ctx ? sc[s] : 0.f;
            const kv_t* vv = (const kv_t*)&raw[u];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[u % R][e] += p * kv2f(vv[e]);
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (LPK == 8) o[i][e] += dpp<kDppRotate8>(o[i][e]);
            o[i][e] = across<32>(across<16>(o[i][e], Add()), Add());
        }
        if (kin == 0)
#pragma unroll
            for (int e = 0; e < 8; ++e) oacc[wave + i * PW][sub * 8 + e] = o[i][e];
    }
    __syncthreads();
    if (tid < HD / 4) {
        f16_t r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = tid * 4 + e;
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) t += oacc[w][c];
            if (SPLIT) share[c] = t;
            r[e] = f2h(t * inv);
        }
        if (SPLIT) {
            if (tid == 0) {
                share[HD] = mx;
                share[HD + 1] = tot;
            }
            return;
        }
        const size_t at = pk_index(out_r, out_k0 + tid * 4, out_kp);
        *(uint2*)(out + at) = *(const uint2*)r;
    }
}

// Prompt forwards: q was rotated and K, V put into their slots for every token-row before this runs.
// Causal attention of one (row, head, tile of 64 * QT queries) per workgroup; each of its 4 waves owns QT tiles of 16
// queries.  The row's keys and values are visited in tiles of 64 slots that are staged once in LDS for all queries
// (K as stored, V transposed), the next tile's global loads in flight while the current one is used.
// Both contractions run on the matrix cores in half precision, the cache's own format:
//   S^T = K Q^T   A = K tile (16 keys x 32 head elements), B = Q^T; q is carried as the sum of two halves (hi + lo), so
//                 the scores see q to ~22 bits (to 2^-25 where an element is below 1/8) like the decode kernel's fp32
//                 dot product.  The factor log2(e) / sqrt(hd) comes after the product, in the exponent's multiply-add:
//                 a q made smaller by it first would keep fewer bits;
//                 D: lane holds, for query lane%16, keys 4*(lane/16)..+3 of a 16-key tile.
//   O^T = V^T P^T two score tiles (32 keys) form one B operand as they lie in the registers: contraction slot
//                 8*(lane/16) + j is key 4*(lane/16) + j of the first tile for j < 4, of the second for j >= 4;
//                 V^T is staged in that slot order (vt_pos), so the A operand is one 16-byte LDS read;
//                 D: lane holds, for query lane%16, output elements 16t + 4*(lane/16)..+3.
// So a query's running maximum, sum and rescale factor stay in its own lanes: fp32 online softmax with no
// transposition of the probabilities.  Slots above a query's position are masked before the exponential; only tiles that
// reach past the wave's first query test for it, and the accumulators are rescaled only when some maximum has moved.
// What bounds it: matrix instructions and, as many cycles again, the vector work of the softmax.  With two query tiles a
// wave reads every staged operand for 32 queries; the loads of short rows are latency, and there one tile with
// one buffer leaves room for three workgroups per compute unit instead of two.
// Per layer, 7B, against 32-slot tiles with one query tile per wave and V transposed by 2-byte LDS writes: three prompts of
// about 2400 slots 945 -> 416 us, 256 prompts of 8 to 256 slots 301 -> 139 us, 16 of about 45 12.1 -> 10.0 us.
constexpr int kAttnTile = 64;        // slots per staged tile
constexpr int kAttnTallFrom = 256;   // longest row of the forward from which a wave owns two query tiles
// Place of a tile's slot in the staged V^T rows.
__device__ __forceinline__ int vt_pos(int k) { return (k & 32) + ((k >> 2) & 3) * 8 + ((k >> 4) & 1) * 4 + (k & 3); }

template <int HD, int QT, int NBUF>
__global__ __launch_bounds__(256, QT == 2 ? 2 : 3) void k_attention_prompt(MbState st, const float* __restrict__ qrot,
                                                                          const kv_t* __restrict__ kc,
                                                                          const kv_t* __restrict__ vc,
                                                                          f16_t* __restrict__ out, int d)
{
    constexpr int KT = kAttnTile;
    constexpr int KS = HD / 32;          // steps of the score contraction
    constexpr int ET = HD / 16;          // 16-element tiles of the output
    constexpr int OCT = HD / 8;          // 16-byte pieces per key
    constexpr int KROW = HD + 8;         // halves per staged key row (16 bytes of padding: conflict-free operand reads)
    constexpr int VROW = KT + 8;         // halves per row of the transposed value tile (likewise)
    constexpr int PPT = KT * OCT / 256;  // pieces per thread: PPT keys rows apart, and PPT neighbouring keys' values
    constexpr int NKG = KT / PPT;        // groups of neighbouring keys
    static_assert(PPT == 4 || PPT == 2, "head_dim 128 or 64");
    __shared__ __attribute__((aligned(16))) _Float16 k_lds[NBUF][KT * KROW];
    __shared__ __attribute__((aligned(16))) _Float16 v_lds[NBUF][HD * VROW];
    // heads are the fastest index: a multiple of 8 of them keeps each head's keys and values on one die; tiles of late
    // queries, which visit the most slots, come first
    const int h = blockIdx.x, row = blockIdx.y, qt = gridDim.z - 1 - blockIdx.z;
    const int p = st.row_plen[row];      // tokens of this row in the forward: positions 0..p-1
    const int q0 = qt * 64 * QT;
    if (q0 >= p) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ql = lane & 15, g = lane >> 4;
    const int j0 = st.row_j0[row];
    const size_t base = (size_t)st.row_so[row] * d + (size_t)h * st.row_cap[row] * HD;
    const u32x4* Kg = (const u32x4*)(kc + base);
    const u32x4* Vg = (const u32x4*)(vc + base);
    const int wave_first = q0 + wave * 16 * QT;
    const int wave_last = wave_first < p ? min(wave_first + 16 * QT - 1, p - 1) : -1;   // -1: no query, nothing to visit
    const int n_keys = min(p, q0 + 64 * QT);
    const int n_tiles = (n_keys + KT - 1) / KT;
    const float scale = rsqrtf((float)HD) * 1.44269504088896341f;   // of the scores, in units of log2: exp2 below

    u32x4 kreg[PPT], vreg[PPT];
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    auto load_tile = [&](int t) {
#pragma unroll
        for (int i = 0; i < PPT; ++i) {
            const int c = tid + i * 256;
            const int key = t * KT + c / OCT;
            const u32x4 kv = Kg[(size_t)min(key, n_keys - 1) * OCT + c % OCT];
            kreg[i] = key < n_keys ? kv : zero4;
        }
#pragma unroll
        for (int i = 0; i < PPT; ++i) {
            const int key = t * KT + (tid % NKG) * PPT + i;
            const u32x4 vv = Vg[(size_t)min(key, n_keys - 1) * OCT + tid / NKG];
            vreg[i] = key < n_keys ? vv : zero4;
        }
    };
    auto stage_tile = [&](int b) {   // K rows as stored, V transposed
#pragma unroll
        for (int i = 0; i < PPT; ++i) {
            const int c = tid + i * 256;
            *(u32x4*)&k_lds[b][(c / OCT) * KROW + (c % OCT) * 8] = kreg[i];
        }
        _Float16* vt = &v_lds[b][(tid / NKG) * 8 * VROW + vt_pos((tid % NKG) * PPT)];
        f16x8 v[PPT];
#pragma unroll
        for (int i = 0; i < PPT; ++i) v[i] = __builtin_bit_cast(f16x8, vreg[i]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (PPT == 4) {
                const f16x4 o = {v[0][e], v[1][e], v[PPT - 2][e], v[PPT - 1][e]};
                *(f16x4*)(vt + e * VROW) = o;
            } else {
                const f16x2 o = {v[0][e], v[1][e]};
                *(f16x2*)(vt + e * VROW) = o;
            }
        }
    };
    load_tile(0);

    // this lane's queries: head elements 32*ks + 8*g .. +7 for every step, split into two halves (queries past the row's
    // end repeat its last one, and are never stored)
    f16x8 qh[QT][KS], qlo[QT][KS];
    int qpos[QT];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        qpos[u] = min(wave_first + u * 16 + ql, p - 1);
        const float* qp = qrot + (size_t)(j0 + qpos[u]) * d + h * HD + 8 * g;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const float4 a = *(const float4*)(qp + 32 * ks), b = *(const float4*)(qp + 32 * ks + 4);
            const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const _Float16 hi = (_Float16)v[e];
                qh[u][ks][e] = hi;
                qlo[u][ks][e] = (_Float16)(v[e] - (float)hi);
            }
        }
    }
    f32x4 o[QT][ET];
    float m_run[QT], l_run[QT];   // m_run: before the factor; l_run: this lane's share of the sum, over its own slots
#pragma unroll
    for (int u = 0; u < QT; ++u) {
#pragma unroll
        for (int t = 0; t < ET; ++t) o[u][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
        m_run[u] = -3.0e38f;
        l_run[u] = 0.f;
    }

    auto use_tile = [&](int b, int k0, auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
        f32x4 s[QT][4];
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
#pragma unroll
            for (int u = 0; u < QT; ++u) s[u][kt] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (MASKED && k0 + kt * 16 > wave_last) continue;   // wave-uniform
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const f16x8 a = *(const f16x8*)&k_lds[b][(kt * 16 + ql) * KROW + ks * 32 + 8 * g];
#pragma unroll
                for (int u = 0; u < QT; ++u) {
                    s[u][kt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, qlo[u][ks], s[u][kt], 0, 0, 0);
                    s[u][kt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, qh[u][ks], s[u][kt], 0, 0, 0);
                }
            }
        }
        f16x8 pb[QT][2];
#pragma unroll
        for (int u = 0; u < QT; ++u) {
            float mt = -3.0e38f;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (MASKED && k0 + kt * 16 + 4 * g + i > qpos[u]) s[u][kt][i] = -3.0e38f;
                    mt = fmaxf(mt, s[u][kt][i]);
                }
            mt = across<32>(across<16>(mt, Max()), Max());
            if (__any(mt > m_run[u])) {
                const float m_new = fmaxf(m_run[u], mt);
                const float alpha = __builtin_amdgcn_exp2f((m_run[u] - m_new) * scale);
                m_run[u] = m_new;
                l_run[u] *= alpha;
#pragma unroll
                for (int tt = 0; tt < ET; ++tt) o[u][tt] *= alpha;
            }
            const float m_scaled = m_run[u] * scale;   // its rounding is a factor common to all of a query's slots
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float pv = __builtin_amdgcn_exp2f(fmaf(s[u][kt][i], scale, -m_scaled));   // masked: 0, some slot is not
                    l_run[u] += pv;
                    pb[u][kt >> 1][(kt & 1) * 4 + i] = (_Float16)pv;
                }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (MASKED && k0 + c * 32 > wave_last) continue;
#pragma unroll
            for (int tt = 0; tt < ET; ++tt) {
                const f16x8 av = *(const f16x8*)&v_lds[b][(tt * 16 + ql) * VROW + c * 32 + 8 * g];
#pragma unroll
                for (int u = 0; u < QT; ++u) o[u][tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, pb[u][c], o[u][tt], 0, 0, 0);
            }
        }
    };
    stage_tile(0);
    for (int t = 0; t < n_tiles; ++t) {
        const int b = NBUF == 2 ? t & 1 : 0;
        __syncthreads();
        if (t + 1 < n_tiles) load_tile(t + 1);
        const int k0 = t * KT;
        if (k0 <= wave_last) {   // wave-uniform: tiles wholly above this wave's queries are skipped
            if (k0 + KT - 1 <= wave_first) use_tile(b, k0, std::false_type{});
            else use_tile(b, k0, std::true_type{});
        }
        if (NBUF == 1) __syncthreads();   // with two buffers the next one was last read before this trip's barrier
        if (t + 1 < n_tiles) stage_tile(NBUF == 2 ? b ^ 1 : 0);
    }
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        float l = l_run[u];
        l = across<32>(across<16>(l, Add()), Add());
        if (wave_first + u * 16 + ql >= p) continue;
        const float inv = 1.f / l;
        const int j = j0 + qpos[u];
#pragma unroll
        for (int tt = 0; tt < ET; ++tt) {
            f16_t r[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = f2h(o[u][tt][e] * inv);
            const size_t at = pk_index(j, h * HD + tt * 16 + 4 * g, d);
            *(uint2*)(out + at) = *(const uint2*)r;
        }
    }
}

// Decode forwards: the (token-row, head) workgroup first finishes its own slice of the q|k|v projection
// (sums the k-slices, rotates q and k at the row's position, appends k and v to the row's slab), then
// attends.  Saves a launch and the round trip of q through HBM for every layer of every step.
// PW waves per workgroup: 8 (256 cache slots per round trip) when the grid is small enough for every workgroup to
// be resident with room to spare, 4 (128 slots) for larger batches, whose many workgroups already fill the chip, or 2, and 16
// (512 slots) when the micro-batch has less than one workgroup per compute unit and a context exceeds 256 slots: what a
// unit has in flight is then all that counts.
// SPLIT: the workgroups of a pair along z share out its slots (few pairs, long contexts: see attention_split); the one that holds
// the new slot appends it.
template <int HD, int NW, int PW, bool SPLIT>
__global__ __launch_bounds__(64 * PW) void k_attention_decode(MbState st, const float* __restrict__ part, int ksplit,
                                                          size_t part_stride, kv_t* __restrict__ kc,
                                                          kv_t* __restrict__ vc, const float* __restrict__ rcos,
                                                          const float* __restrict__ rsin, f16_t* __restrict__ out,
                                                          int d, float* __restrict__ shares)
{
    __shared__ float sc[kMaxPos];
    __shared__ float red[PW + NW];
    __shared__ float oacc[NW][HD];
    __shared__ float qs[HD];
    constexpr int HALF = HD / 2;
    const int j = blockIdx.x, h = blockIdx.y;
    // count, row and position are requested together (the tables are sized for the grid); only the loads that
    // are indexed by the row wait for the count check
    const int count = *st.d_n;
    const int row = st.tr_row[j], pos = st.tr_pos[j];
    if (j >= count) return;
    const size_t base = (size_t)st.row_so[row] * d + (size_t)h * st.row_cap[row] * HD;
    int begin = 0, slots = pos + 1;
    float* share = nullptr;
    if (SPLIT) {
        const int S = gridDim.z, per = ((pos + S) / S + 63) & ~63;
        begin = blockIdx.z * per;
        slots = min(pos + 1 - begin, per);
        share = shares + (((size_t)j * gridDim.y + h) * S + blockIdx.z) * (HD + 2);
        if (slots <= 0) {   // a shorter row than the micro-batch's longest
            if (threadIdx.x < HD + 2) share[threadIdx.x] = threadIdx.x == HD ? -3.0e38f : 0.f;
            return;
        }
    }
    auto finish = [&](int t) {
        const int which = t / HALF, e = t % HALF;   // 0 q, 1 k, 2 v
        if (which >= 3 || (SPLIT && which != 0 && begin + slots != pos + 1)) return;
        const float* p = part + (size_t)j * 3 * d + (size_t)which * d + h * HD + qkv_col(e);
        float pa[kNormMaxSplit], pb[kNormMaxSplit];   // every k-slice load issued before the first add
#pragma unroll
        for (int s = 0; s < kNormMaxSplit; ++s) {
            pa[s] = s < ksplit ? p[(size_t)s * part_stride] : 0.f;
            pb[s] = s < ksplit ? p[(size_t)s * part_stride + 16] : 0.f;
        }
        float a = 0.f, b = 0.f;
#pragma unroll
        for (int s = 0; s < kNormMaxSplit; ++s) {
            a += pa[s];
            b += pb[s];
        }
        if (which < 2) {
            const float cs = rcos[(size_t)pos * HALF + e], sn = rsin[(size_t)pos * HALF + e];
            const float2 r = rotated(a, b, cs, sn);
            a = r.x;
            b = r.y;
        }
        if (which == 0) {
            qs[e] = a;
            qs[e + HALF] = b;
        } else {
            kv_t* dst = (which == 1 ? kc : vc) + base + (size_t)pos * HD + e;
            dst[0] = f2kv(a);
            dst[HALF] = f2kv(b);
        }
    };
    finish(threadIdx.x);
    if (64 * PW < 3 * HALF) finish(threadIdx.x + 64 * PW);
    __syncthreads();   // the new key/value slot and q are visible to the whole workgroup
    const kv_t *kb = kc + base + (size_t)begin * HD, *vb = vc + base + (size_t)begin * HD;
    const int pairs = gridDim.x * gridDim.y, load_slots = PW * (512 / HD);   // slots of one load of every wave
    if (!SPLIT && slots <= kAttnShort * load_slots)
        attend<HD, NW, PW, SPLIT, kAttnShort, false>(qs, sc, red, oacc, kb, vb, slots, out, j, h * HD, d, share);
    else if (!SPLIT && NW <= 8 && pairs > kAttnTailFrom && pairs <= kAttnTailTo && slots <= kAttnTailTrips * kAttnUnroll * load_slots)
        attend<HD, NW, PW, SPLIT, kAttnUnroll, true>(qs, sc, red, oacc, kb, vb, slots, out, j, h * HD, d, share);
    else
        attend<HD, NW, PW, SPLIT, kAttnUnroll, false>(qs, sc, red, oacc, kb, vb, slots, out, j, h * HD, d, share);
}

// The shares of a pair's slots put together: one wave per pair, two elements a lane (HD 64: half the lanes).
template <int HD>
__global__ __launch_bounds__(64) void k_attention_join(MbState st, const float* __restrict__ shares, int S, f16_t* __restrict__ out, int d)
{
    const int j = blockIdx.x, h = blockIdx.y, e = threadIdx.x * 2;
    const int count = *st.d_n;
    if (e >= HD) return;
    const float* p = shares + ((size_t)j * gridDim.y + h) * S * (HD + 2);
    float2 o[kAttnMaxSplit];
    float m[kAttnMaxSplit], t[kAttnMaxSplit], top = -3.0e38f;
#pragma unroll
    for (int s = 0; s < kAttnMaxSplit; ++s) {   // all loads on their way together; beyond S the last one again, without weight
        const float* q = p + (size_t)min(s, S - 1) * (HD + 2);
        o[s] = *(const float2*)(q + e);
        m[s] = q[HD];
        t[s] = q[HD + 1];
    }
    if (j >= count) return;
#pragma unroll
    for (int s = 0; s < kAttnMaxSplit; ++s) top = fmaxf(top, m[s]);
    float all = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int s = 0; s < kAttnMaxSplit; ++s) {
        const float f = s < S ? __expf(m[s] - top) : 0.f;   // an empty share: its total and sums are 0
        all += f * t[s];
        o0 += f * o[s].x;
        o1 += f * o[s].y;
    }
    const float inv = 1.f / all;
    const f16_t r[2] = {f2h(o0 * inv), f2h(o1 * inv)};
    *(uint32_t*)(out + pk_index(j, h * HD + e, d)) = *(const uint32_t*)r;
}

// ------------------------------------------------------------------------------------------ a row's whole decode step
// Small models (row_step_plan): a decode step of 7 launches per layer is nothing but launches there, 3.4 us each for a few
// hundred kilobytes.  Here one workgroup takes one row through the whole step, embedding to logits and their argmax: rows
// need nothing from each other, so nothing but its own barriers is waited for.
// What bounds it: every workgroup reads all the weights, 64 bytes a clock from the L2 of its die (151 GB/s alone, 138 each
// for 256 workgroups; a launch that does nothing else takes 26 us for 3.6 MB), and the barriers' latencies, some 15 us in two
// layers.  So the loads go on over the barriers: there is one loop for all matrices, and the block that a wave has used
// last is replaced by the first one it needs of the next matrix.  (A loop per matrix is 5000 instructions, spills, and waits
// for everything at each end: 58 us.)  Tiny model, 16 rows, context 20: 63 us as 19 launches -> 48; 250 rows 103 -> 58.
// With a.steps a launch takes its rows to their ends, where those are known and nothing is sampled or polled (with compaction a
// row leaves at its own end, else all stay to the last one's): group of 16, 47 forwards, 2.83 -> 2.50 ms, the weights' first blocks
// wait in registers when a step begins.
// A wave owns pairs of output strips (the two halves of a head's strip, gate and up; two sums under way at once); the
// matrix instruction's activation operand is the row's vector for all of its 16 columns, so that every lane ends up with
// valid sums.  Rounding as in the other kernels: residual stream, sums, rotation and softmax in fp32; projection inputs,
// keys and values as halves, once each.
constexpr int kRowThreads = 64 * kRowWaves;
constexpr int kRowGroup = 8;   // k-blocks of both strips that a wave has in flight: 128 KiB for the workgroup

// Waits for this wave's LDS traffic and meets the others; loads from global memory stay on their way.
__device__ __forceinline__ void row_meet()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A group of a pair's k-blocks: scalar base and offsets (as plain loads the compiler keeps an address per load and lane).
// Past a strip's last k-block that one is read again and meets zeros; an odd last strip comes twice.
struct RowGroup {
    __amdgpu_buffer_rsrc_t rsrc;
    int at[2], left;
    __device__ __forceinline__ RowGroup(const f16_t* W, int KB, int strips, int pair, int g)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc((void*)W, (short)0, strips * KB * 1024, 0x00020000)),
          at{(2 * pair * KB + g * kRowGroup) * 1024, (min(2 * pair + 1, strips - 1) * KB + g * kRowGroup) * 1024},
          left(KB - g * kRowGroup)
    {
    }
    __device__ __forceinline__ u32x4 load(int i, int q) const
    {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (threadIdx.x & 63) * 16, at[i] + min(q, left - 1) * 1024, 0);
    }
};

__device__ __forceinline__ float pick4(const f32x4& v, int i) { return i < 2 ? (i == 0 ? v[0] : v[1]) : (i == 2 ? v[2] : v[3]); }

// hb <- the normalised residual row as halves; gain: this thread's norm weight (thread = column)
__device__ __forceinline__ void row_norm(const float* x, f16_t* hb, int d, float eps, bf16_t gain, int lane)
{
    float ss = 0.f;
    for (int c = lane; c < d; c += 64) ss += x[c] * x[c];   // every wave by itself: no barrier
    ss = group_sum<16>(ss);
    ss = across<32>(across<16>(ss, Add()), Add());
    const float r = rsqrtf(ss / (float)d + eps);
    if ((int)threadIdx.x < d) hb[threadIdx.x] = f2h(x[threadIdx.x] * r * bf2f(gain));
}

template <int HD>
__global__ __launch_bounds__(kRowThreads) void k_row_step(MbState st, RowStepArgs a)
{
    constexpr int HALF = HD / 2, PH = HD / 32;            // PH: pairs of strips per head
    constexpr int LPK = HD / 8, KPW = 64 / LPK, AU = 4;   // lanes per key, keys per wave load, loads in flight
    const int j = blockIdx.x;
    const int count = *st.d_n;
    const int row = st.tr_row[j], step0 = *st.d_step;
    int pos = st.tr_pos[j], tok = st.tr_tok[j];
    if (j >= count) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = a.d, H = a.H, dp = row_padded(d), fp = row_padded(a.Fp);
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float* x = (float*)lds;                 // [d] residual stream
    float* q = x + d;                       // [d] rotated query
    float* cs = q + d;                      // [HD] cosines, then sines of this position
    float* part = cs + HD;                  // [kRowWaves][HD + 4] attention: sums, maximum and total of every wave
    f16_t* hb = (f16_t*)(part + kRowWaves * (HD + 4));   // [dp] input of q|k|v, o, gate|up, head
    f16_t* act = hb + dp;                   // [fp] input of down
    f16_t* kn = act + fp;                   // [d], [d] this position's key and value
    f16_t* vn = kn + d;

    // Phase 4 * l + t: matrix t (q|k|v, o, gate|up, down) of layer l; the last one is the head.
    const int phases = 4 * a.n_layers + 1;
    auto weights = [&](int ph) {
        return ph == phases - 1 ? a.lm_head : a.layer[ph >> 2].w[ph & 3];
    };
    auto kblocks = [&](int ph) { return (ph & 3) == 3 ? a.Fp >> 5 : d >> 5; };
    auto strips_of = [&](int ph) {
        const int t = ph & 3;
        return ph == phases - 1 ? a.V >> 4 : t == 0 ? 3 * d >> 4 : t == 2 ? a.F >> 3 : d >> 4;
    };
    // of the phase to come; each phase looks the next one's up while it waits for its own operands
    // (looked up when it began, they kept every phase waiting 350 clocks: 16 rows 49.5 -> 49.1 us a step, their 48 tokens 2.25 -> 2.22 ms)
    const f16_t* W2 = weights(0);
    int KB2 = kblocks(0), strips2 = strips_of(0);
    u32x4 v[2][kRowGroup];
    {
        const RowGroup n(W2, KB2, strips2, min(wave, (strips2 >> 1) - 1), 0);
#pragma unroll
        for (int z = 0; z < kRowGroup; ++z) {
            v[0][z] = n.load(0, z);
            v[1][z] = n.load(1, z);
        }
    }
    bf16_t gain = tid < d ? a.layer[0].attn_norm[tid] : 0;
    for (int c = d + tid; c < dp; c += kRowThreads) hb[c] = 0;
    for (int c = a.F + tid; c < fp; c += kRowThreads) act[c] = 0;
    const int64_t so = st.row_so[row];
    const int cap = st.row_cap[row];
    const int sel = lane & 3, col = (lane >> 4) * 4 + sel;   // a strip's 16 columns: one each in the lanes below
    const bool owner = (lane & 15) < 4;
    // a head's earlier slots are shared out to P waves, and inside a wave to groups of LPK lanes
    const int P = kRowWaves / H, h = min(wave / P, H - 1), p = wave % P, sub = lane % LPK, kin = lane / LPK;
    const int limit = a.steps > 0 ? st.row_limit[row] : 0;
    kv_t* const kv0 = a.kv + so * d;
    const size_t kv_layer = 2 * a.kv_layer_stride;
    uint4 kr[AU], vr[AU];
    float best;   // the head's largest logit and its column
    int bi;

    for (int step = 0;; ++step) {
        if (tid < d) x[tid] = bf2f(a.embed[(size_t)tok * d + tid]);
        if (tid < HD) cs[tid] = tid < HALF ? a.rope_cos[(size_t)pos * HALF + tid] : a.rope_sin[(size_t)pos * HALF + tid - HALF];
        best = -3.4e38f;
        bi = 0x7fffffff;
        row_meet();
        for (int ph = 0; ph < phases; ++ph) {
            const int t = ph == phases - 1 ? 4 : ph & 3;
            kv_t* const kc = kv0 + (ph >> 2) * kv_layer;
            kv_t* const vc = kc + a.kv_layer_stride;
            const kv_t *kb = kc + (size_t)h * cap * HD + sub * 8, *vb = vc + (size_t)h * cap * HD + sub * 8;
            // the first slots of a layer are asked for before anything that they do not depend on
            auto slot = [&](int c0, int u) { return c0 + u * P * KPW + kin; };
            auto load_slots = [&](uint4 (&r)[AU], const kv_t* from, int c0) {
#pragma unroll
                for (int u = 0; u < AU; ++u) r[u] = *(const uint4*)(from + (size_t)min(slot(c0, u), pos - 1) * HD);
            };
            if (t == 0) {
                load_slots(kr, kb, p * KPW);
                load_slots(vr, vb, p * KPW);
            }
            if ((t & 1) == 0) {   // normalised input
                row_norm(x, hb, d, a.eps, gain, lane);
                if (tid < d)
                    gain = (t == 0 ? a.layer[ph >> 2].mlp_norm : t == 4 ? a.layer[0].attn_norm :
                            ph + 3 == phases ? a.final_norm :
                            a.layer[(ph >> 2) + 1].attn_norm)[tid];
                row_meet();
            }
            // This wave's pairs of the matrix times the vector at xb.  A block is replaced by its successor, the first ones of
            // the next matrix at the end, as soon as it is used: one unbroken row of loads, every wait for the oldest only.
            {
                const f16_t *const W = W2, *const xb = t == 3 ? act : hb;
                const int KB = KB2, strips = strips2, pairs = (strips + 1) >> 1;
                const int after = ph + 1 < phases ? ph + 1 : 0;
                W2 = weights(after);
                KB2 = kblocks(after);
                strips2 = strips_of(after);
                const int first2 = min(wave, ((strips2 + 1) >> 1) - 1);
                f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
                int pair = wave, g = 0;
                do {   // a wave without a pair holds the last one's first group, and drops it
                    f16x8 b[kRowGroup];
#pragma unroll
                    for (int z = 0; z < kRowGroup; ++z)
                        b[z] = *(const f16x8*)(xb + (g * kRowGroup + z) * 32 + (lane >> 4) * 8);
                    const int now = pair;
                    const bool whole = KB - g * kRowGroup <= kRowGroup;
                    pair += whole ? kRowWaves : 0;
                    g = whole ? 0 : g + 1;
                    const bool more = pair < pairs;
                    const RowGroup n(more ? W : W2, more ? KB : KB2, more ? strips : strips2, more ? pair : first2, g);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int z = 0; z < kRowGroup; ++z) {
                        a0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, v[0][z]), b[z], a0, 0, 0, 0);
                        a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, v[1][z]), b[z], a1, 0, 0, 0);
                        v[0][z] = n.load(0, z);
                        v[1][z] = n.load(1, z);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (!whole) continue;
                    float s0 = pick4(a0, sel), s1 = pick4(a1, sel);   // column `col` of either strip
                    a0 = a1 = (f32x4){0.f, 0.f, 0.f, 0.f};
                    if (now >= pairs) continue;
                    if (t == 4) {
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const float z = i ? s1 : s0;
                            const int c = now * 32 + i * 16 + col;
                            if (c >= a.V) continue;   // an odd last strip
                            if (owner && a.steps <= 0) a.logits[(size_t)j * a.V + c] = z;
                            if (z > best || (z == best && c < bi)) {   // lowest index on ties, as in k_argmax
                                best = z;
                                bi = c;
                            }
                        }
                    } else if (owner) {
                        if (t == 2) {
                            act[now * 16 + col] = f2h(silu_f(s0) * s1);
                        } else if (t != 0) {
                            x[now * 32 + col] += s0;
                            x[now * 32 + 16 + col] += s1;
                        } else {   // elements e and e + HD/2 of a head (see qkv_strip)
                            const int which = now / (d >> 5), r = now - which * (d >> 5), e = r / PH * HD + r % PH * 16 + col;
                            if (which < 2) {
                                const float2 r = rotated(s0, s1, cs[e % HD], cs[HALF + e % HD]);
                                s0 = r.x;
                                s1 = r.y;
                            }
                            if (which == 0) {
                                q[e] = s0;
                                q[e + HALF] = s1;
                            } else {
                                kv_t* n1 = (which == 1 ? kn : vn) + e;
                                n1[0] = f2kv(s0);
                                n1[HALF] = f2kv(s1);
                            }
                        }
                    }
                } while (pair < pairs || g != 0);
            }
            row_meet();
            if (t != 0) continue;
            // Attention: every wave keeps a softmax of its own; the slots before this one come from the cache, this one
            // from LDS.
            if (tid < d) {
                const size_t at = ((size_t)(tid / HD) * cap + pos) * HD + tid % HD;
                kc[at] = kn[tid];
                vc[at] = vn[tid];
            }
            if (wave < H * P) {
                const float scale = rsqrtf((float)HD);
                float qf[8], m = -3.0e38f, tot = 0.f, acc[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    qf[e] = q[h * HD + sub * 8 + e];
                    acc[e] = 0.f;
                }
                auto score = [&](const uint4& raw) {
                    const kv_t* k = (const kv_t*)&raw;
                    float s = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) s += qf[e] * kv2f(k[e]);
                    return group_sum<LPK>(s) * scale;
                };
                auto add = [&](float w, const uint4& raw) {
                    const kv_t* u = (const kv_t*)&raw;
                    tot += w;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] += w * kv2f(u[e]);
                };
                auto largest = [](float z) {   // of the wave's groups
                    if (LPK == 8) z = fmaxf(z, dpp<kDppRotate8>(z));
                    return across<32>(across<16>(z, Max()), Max());
                };
                if (p == 0) {   // this slot: the same in every group, counted in the first
                    m = score(*(const uint4*)(kn + h * HD + sub * 8));
                    add(kin == 0 ? 1.f : 0.f, *(const uint4*)(vn + h * HD + sub * 8));
                }
                for (int c0 = p * KPW; c0 < pos; c0 += P * KPW * AU) {   // wave-uniform
                    const int c1 = c0 + P * KPW * AU;
                    float s[AU], top = m;
#pragma unroll
                    for (int u = 0; u < AU; ++u) {
                        s[u] = slot(c0, u) < pos ? score(kr[u]) : -3.0e38f;
                        top = fmaxf(top, s[u]);
                    }
                    if (c1 < pos) load_slots(kr, kb, c1);
                    top = largest(top);
                    const float keep = __expf(m - top);
                    m = top;
                    tot *= keep;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] *= keep;
#pragma unroll
                    for (int u = 0; u < AU; ++u) add(slot(c0, u) < pos ? __expf(s[u] - m) : 0.f, vr[u]);
                    if (c1 < pos) load_slots(vr, vb, c1);
                }
                auto over_groups = [](float z) {
                    if (LPK == 8) z += dpp<kDppRotate8>(z);
                    return across<32>(across<16>(z, Add()), Add());
                };
                tot = over_groups(tot);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] = over_groups(acc[e]);
                float* w = part + wave * (HD + 4);
                if (kin == 0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) w[sub * 8 + e] = acc[e];
                    if (sub == 0) {
                        w[HD] = m;
                        w[HD + 1] = tot;
                    }
                }
            }
            row_meet();
            if (tid < d) {
                const float* w = part + tid / HD * P * (HD + 4);
                float m = -3.0e38f, tot = 0.f, sum = 0.f;
                for (int z = 0; z < P; ++z) m = fmaxf(m, w[z * (HD + 4) + HD]);
                for (int z = 0; z < P; ++z) {
                    const float f = __expf(w[z * (HD + 4) + HD] - m);
                    tot += f * w[z * (HD + 4) + HD + 1];
                    sum += f * w[z * (HD + 4) + tid % HD];
                }
                hb[tid] = f2h(sum / tot);
            }
            row_meet();
        }
        if (!a.am) return;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            const float ob = __shfl_xor(best, m, 64);
            const int oi = __shfl_xor(bi, m, 64);
            if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
        }
        float* const sb = part;
        int* const si = (int*)(part + kRowWaves);
        if (lane == 0) { sb[wave] = best; si[wave] = bi; }
        row_meet();
        best = sb[0];
        bi = si[0];
#pragma unroll
        for (int w = 1; w < kRowWaves; ++w)
            if (sb[w] > best || (sb[w] == best && si[w] < bi)) { best = sb[w]; bi = si[w]; }
        tok = (unsigned)bi < (unsigned)a.V ? bi : 0;
        if (a.steps <= 0) {
            if (tid == 0) a.am[j] = tok;
            return;
        }
        const int s = step0 + step;   // the number of this token
        if (tid == 0 && s < limit) st.out_tok[(size_t)row * st.max_new + s] = tok;
        if (step + 1 >= a.steps || (a.compact && s + 1 >= limit)) return;   // the same for the whole workgroup
        ++pos;
        // the key and value that this step stored are read by other waves in the next
        __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
        row_meet();
    }
}

// ------------------------------------------------------------------------------------------ argmax
// Greedy choice per selected row: index of the largest logit, lowest index on exact ties.
// 1024 threads per row, all of a thread's loads issued before the first compare.
__global__ __launch_bounds__(1024) void k_argmax(const float* __restrict__ logits, int vocab,
                                                 const int32_t* __restrict__ d_count, int32_t* __restrict__ am)
{
    const int j = blockIdx.x;
    if (j >= *d_count) return;
    const float* lg = logits + (size_t)j * vocab;
    float best = -3.4e38f;
    int bi = 0x7fffffff;
    for (int c0 = threadIdx.x * 4; c0 < vocab; c0 += 4096 * 4) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * 4096;
            v[u] = c < vocab ? *(const float4*)(lg + c) : make_float4(-3.4e38f, -3.4e38f, -3.4e38f, -3.4e38f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * 4096;
            const float vv[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c < vocab && (vv[e] > best || (vv[e] == best && c + e < bi))) { best = vv[e]; bi = c + e; }
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const float ob = __shfl_xor(best, m, 64);
        const int oi = __shfl_xor(bi, m, 64);
        if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    __shared__ float sb[16];
    __shared__ int si[16];
    if ((threadIdx.x & 63) == 0) { sb[threadIdx.x >> 6] = best; si[threadIdx.x >> 6] = bi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w)
            if (sb[w] > best || (sb[w] == best && si[w] < bi)) { best = sb[w]; bi = si[w]; }
        // no logit compared greater than the start value (a row of NaN or -inf): id 0, never an id outside the
        // vocabulary, which the next step would use as an embedding row
        am[j] = (unsigned)bi < (unsigned)vocab ? bi : 0;
    }
}

// ------------------------------------------------------------------------------------------ sampling
// Temperature sampling per selected row (Sec. 4.2, Experimental Setting: responses are sampled at a temperature):
// token = smallest v with  sum_{v' <= v} e_v'  >  u * sum_v' e_v',  e_v = exp((logit_v - max) * inv_temp),
// u being the draw for (row, token number): supplied by the caller, or generated from a counter (below).  The CDF runs in vocabulary order, so thread t owns
// the contiguous chunk [t*c, (t+1)*c): it sums its chunk in index order, a workgroup scan of the 1024
// chunk sums finds the first chunk whose running total exceeds the target, and that chunk's owner walks
// it again in the same order (same additions, same roundings) to the token.  V-1 when rounding leaves no
// chunk above the target.  1024 threads per row; the row's logits (just written by the LM head) are read
// three times from L2.
// Counter-based draw in [0,1): Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC 2011) on the counter
// (token number, row id, 0, 0) under the 64-bit key; the top 24 bits of the first output word, scaled by 2^-24.
__device__ inline float philox_draw(uint32_t k0, uint32_t k1, uint32_t id, uint32_t t)
{
    uint32_t c0 = t, c1 = id, c2 = 0u, c3 = 0u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return (float)(c0 >> 8) * (1.0f / 16777216.0f);
}

__global__ __launch_bounds__(1024) void k_sample(const float* __restrict__ logits, int vocab,
                                                 const int32_t* __restrict__ d_count, MbState st,
                                                 const float* __restrict__ draws, const int32_t* __restrict__ ids,
                                                 uint32_t key0, uint32_t key1, float inv_temp)
{
    const int j = blockIdx.x;
    if (j >= *d_count) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = st.live_row[j];
    const int t = *st.d_step;
    const float u = draws ? draws[(size_t)row * st.max_new + t] : philox_draw(key0, key1, (uint32_t)ids[row], (uint32_t)t);
    const float* lg = logits + (size_t)j * vocab;
    const int c = (((vocab + 1023) >> 10) + 3) & ~3;   // floats per thread, a multiple of 4 (vocab % 16 == 0)
    const int lo = tid * c;
    const int hi = lo + c < vocab ? lo + c : vocab;    // lo >= vocab: empty chunk

    __shared__ float s_red[16];
    __shared__ float s_tot[17];
    __shared__ int s_owner[16];

    float m = -3.4e38f;
    for (int v = lo; v < hi; v += 4) {
        const float4 q = *(const float4*)(lg + v);
        m = fmaxf(fmaxf(m, fmaxf(q.x, q.y)), fmaxf(q.z, q.w));
    }
    m = wave_max(m);
    if (lane == 0) s_red[wave] = m;
    __syncthreads();
    m = s_red[0];
#pragma unroll
    for (int w = 1; w < 16; ++w) m = fmaxf(m, s_red[w]);

    float csum = 0.f;
    for (int v = lo; v < hi; v += 4) {
        const float4 q = *(const float4*)(lg + v);
        csum += expf((q.x - m) * inv_temp);
        csum += expf((q.y - m) * inv_temp);
        csum += expf((q.z - m) * inv_temp);
        csum += expf((q.w - m) * inv_temp);
    }
    // inclusive scan of the chunk sums: within the wave, then over the 16 wave totals
    float incl = csum;
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
        const float o = __shfl_up(incl, k, 64);
        if (lane >= k) incl += o;
    }
    if (lane == 63) s_tot[wave + 1] = incl;
    __syncthreads();
    if (tid == 0) {
        float a = 0.f;
        s_tot[0] = 0.f;
        for (int w = 1; w <= 16; ++w) { a += s_tot[w]; s_tot[w] = a; }
    }
    __syncthreads();
    const float base = s_tot[wave];
    const float target = u * s_tot[16];
    const float before = base + (incl - csum);   // running total ahead of this chunk
    const float upto = base + incl;
    const unsigned long long hit = __ballot(upto > target);
    if (lane == 0) s_owner[wave] = hit ? (wave << 6) + __ffsll((long long)hit) - 1 : 0x7fffffff;
    __syncthreads();
    int owner = 0x7fffffff;
#pragma unroll
    for (int w = 0; w < 16; ++w) owner = s_owner[w] < owner ? s_owner[w] : owner;
    if (owner == 0x7fffffff) {
        if (tid == 0) st.am[j] = vocab - 1;
        return;
    }
    if (tid != owner) return;
    const float want = target - before;
    float acc = 0.f;
    int pick = hi - 1;
    for (int v = lo; v < hi; ++v) {
        acc += expf((lg[v] - m) * inv_temp);
        if (acc > want) { pick = v; break; }
    }
    st.am[j] = pick;
}

// ------------------------------------------------------------------------------------------ bookkeeping
// After a forward: slot j's chosen token is the row's token number s (s = tokens generated so far).  Emit it
// if the row still owes tokens, then build the next forward: every surviving slot feeds its token back at
// position prompt_len + s.  With `compact` a row leaves the live batch once it has emitted its last token;
// without it the row stays and keeps running on its own output (its later tokens are never emitted).
// A row that emits `eos_id` (never matched when it is -1) has emitted its last token: its limit drops to
// s + 1, which is also where the host reads the row's length afterwards.  *st.d_active counts the rows that
// still owe tokens, for a host that does not know the lengths and polls.
__global__ __launch_bounds__(1024) void k_step_update(MbState st, int compact, int eos_id)
{
    __shared__ int wave_cnt[16];
    __shared__ int wave_act[16];
    __shared__ int wave_off[17];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = *st.d_nlive;
    const int s = *st.d_step;
    int row = -1, tok = 0, keep = 0, owes = 0;
    if (tid < n) {
        row = st.live_row[tid];
        tok = st.am[tid];
        int lim = st.row_limit[row];
        if (s < lim) {
            st.out_tok[(size_t)row * st.max_new + s] = tok;
            if (tok == eos_id && s + 1 < lim) {
                lim = s + 1;
                st.row_limit[row] = lim;
            }
        }
        owes = s + 1 < lim;
        keep = st.row_stay ? s + 1 < st.row_stay[row] : compact ? owes : 1;
    }
    const unsigned long long bal = __ballot(keep);
    const unsigned long long act = __ballot(owes);
    const int before = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) { wave_cnt[wave] = __popcll(bal); wave_act[wave] = __popcll(act); }
    __syncthreads();
    if (tid == 0) {
        int a = 0, b = 0;
        for (int w = 0; w < 16; ++w) { wave_off[w] = a; a += wave_cnt[w]; b += wave_act[w]; }
        wave_off[16] = a;
        *st.d_active = b;
    }
    __syncthreads();
    if (keep) {
        const int jn = wave_off[wave] + before;
        st.tr_tok[jn] = tok;
        st.tr_row[jn] = row;
        st.tr_pos[jn] = st.row_plen[row] + s;
        st.live_row[jn] = row;
    }
    if (tid == 0) {
        *st.d_n = wave_off[16];
        *st.d_nlive = wave_off[16];
        *st.d_step = s + 1;
    }
}

// ------------------------------------------------------------------------------------------ read probe
// Measurement aid: a plain read stream over a packed weight matrix, one wave per 64 KiB chunk, 8 non-temporal
// 16-byte loads per lane in flight, nothing computed.  The rate it reaches at a projection's size is what the
// projection kernels are compared with (no ceiling: small matrices make few such waves).
__global__ __launch_bounds__(256) void k_read_stream(const u32x4* __restrict__ p, int n_chunks, uint32_t* __restrict__ sink)
{
    const int lane = threadIdx.x & 63;
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= n_chunks) return;
    const u32x4* q = p + (size_t)w * 4096 + lane;   // 64 KiB = 4096 vectors of 16 bytes
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (int i = 0; i < 4096; i += 512) {
        u32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(q + i + u * 64);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc ^= v[u];
    }
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u) sink[0] = 1u;   // keeps the loads alive; bf16 weights never hit it in practice
}

// ------------------------------------------------------------------------------------------ launchers
static inline int grid_for(size_t n, int block)
{
    const size_t g = (n + block - 1) / block;
    return (int)(g > (1u << 20) ? (1u << 20) : (g < 1 ? 1 : g));
}

void launch_pack_weight(const void* src, int src_f32, f16_t* dst, int n_src, int k, int kp, int blk_stride,
                        int blk_off, int head_strips, hipStream_t s)
{
    const size_t total = (size_t)n_src * (k / 8);
    hipLaunchKernelGGL(k_pack_weight, dim3(grid_for(total, 256)), dim3(256), 0, s, src, src_f32, dst, n_src, k, kp,
                       blk_stride, blk_off, head_strips);
}

void launch_narrow_weight(const f16_t* src, void* dst, int N, int Kp, int32_t* unfit, hipStream_t s)
{
    const size_t n_groups = (size_t)(N / 16) * (Kp / 128);
    hipLaunchKernelGGL(k_narrow_weight, dim3(grid_for(n_groups * 64, 256)), dim3(256), 0, s, (const u32x4*)src, (u32x4*)dst,
                       n_groups, Kp / 128, unfit);
}

void launch_cast_rows(const void* src, int src_f32, bf16_t* dst, size_t count, hipStream_t s)
{
    hipLaunchKernelGGL(k_cast_rows, dim3(grid_for(count, 256)), dim3(256), 0, s, src, src_f32, dst, count);
}

void launch_fill_i32(int32_t* p, int32_t v, size_t n, hipStream_t s)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
}

void launch_embed(const MbState& st, const bf16_t* embed, float* x, int d, int n_max, hipStream_t s)
{
    hipLaunchKernelGGL(k_embed, dim3(n_max), dim3(256), 0, s, st, embed, x, d);
}

void launch_rmsnorm(const MbState& st, float* x, const float* part, int ksplit, size_t part_stride,
                    const bf16_t* w, float eps, const int32_t* sel, const int32_t* d_nsel, f16_t* h_packed, int d,
                    int n_max, hipStream_t s)
{
    // Few rows: 1024 threads per row, the whole row in one round trip.  Many rows (prompt forwards): 256 threads per
    // row, so that eight rows share a compute unit and the launch is bound by bytes rather than by workgroup
    // start-up (measured at the 7B width: a prompt forward of 640 token-rows takes 13.8 ms, against 15.8 with 1024
    // threads per row, whose norm launches took 47 us each there; up to 256 rows the wide form is the faster one:
    // 24 rows 3.29 against 3.37 ms per decode step, 256 rows equal).
    if (round_up(n_max, 16) >= kNormNarrowFrom)   // by whole strips, like the projections
        hipLaunchKernelGGL((k_rmsnorm<256, 8>), dim3(round_up(n_max, 128)), dim3(256), 0, s, d_nsel ? d_nsel : st.d_n, x, part,
                           part ? ksplit : 0, part_stride, w, eps, sel, h_packed, d, n_max);
    else
        hipLaunchKernelGGL((k_rmsnorm<1024, 2>), dim3(n_max), dim3(1024), 0, s, d_nsel ? d_nsel : st.d_n, x, part,
                           part ? ksplit : 0, part_stride, w, eps, sel, h_packed, d, n_max);
}

// k-blocks per slice; whole groups of 4 where the 12-bit weights are read.  (The halves keep the even shares, and one wave
// per unit up to 96 rows, that suit them: the two forms add up the same products in different orders.)
static inline int slice_kb(const GemmArgs& a)
{
    const int kbs = (a.Kp / 32 + a.ksplit - 1) / a.ksplit;
    return a.narrow ? (kbs + 3) & ~3 : kbs;
}

template <int MT, int NB, int KD, int EPI, int WN = 0>
static void launch_skinny_inst(const GemmArgs& a, hipStream_t s)
{
    const int groups = (a.N / 16 + NB - 1) / NB;
    hipLaunchKernelGGL((k_gemm_skinny<MT, NB, KD, EPI, WN>), dim3(groups * a.ksplit), dim3(256), 0, s, a, groups, slice_kb(a));
}

template <int MT, int EPI>
static void launch_skinny_mt(const GemmArgs& a, hipStream_t s)
{
    if (a.narrow) {   // gemm_plan: for one row strip, 4 k-blocks per load; more strips are several such micro-batches
        if (a.nb == 2) return launch_skinny_inst<MT, 2, 4, EPI, 1>(a, s);
        return launch_skinny_inst<MT, 4, 4, EPI, 1>(a, s);
    }
    if (a.nb == 2) {
        if (a.kd == 2) launch_skinny_inst<MT, 2, 2, EPI>(a, s);
        else launch_skinny_inst<MT, 2, 4, EPI>(a, s);
    } else {
        if (a.kd == 2 || MT > 2) launch_skinny_inst<MT, 4, 2, EPI>(a, s);
        else launch_skinny_inst<MT, 4, 4, EPI>(a, s);
    }
}

template <int P, int MT, int EPI, int KH>
static void launch_sweep_mt(const GemmArgs& a, int units, hipStream_t s)
{
    // strips per wave (sweep_nbw): a gate/up pair with the SwiGLU epilogue, otherwise one
    constexpr int NBW = EPI == EPI_SWIGLU ? 2 : 1;
    const dim3 grid(a.sweep_gn * a.ksplit), block(64 * P);
    if constexpr (MT <= kNarrowMaxRows / 16)
        if (a.narrow) {
            hipLaunchKernelGGL((k_gemm_sweep<P, MT, NBW, EPI, KH, 1>), grid, block, 0, s, a, units, a.sweep_gn, slice_kb(a));
            return;
        }
    hipLaunchKernelGGL((k_gemm_sweep<P, MT, NBW, EPI, KH, 0>), grid, block, 0, s, a, units, a.sweep_gn, slice_kb(a));
}

template <int P, int EPI, int KH>
static void launch_sweep_p(const GemmArgs& a, int units, hipStream_t s)
{
    switch ((a.m_rows + 15) / 16) {
        case 1: launch_sweep_mt<P, 1, EPI, KH>(a, units, s); break;
        case 2: launch_sweep_mt<P, 2, EPI, KH>(a, units, s); break;
        case 3: launch_sweep_mt<P, 3, EPI, KH>(a, units, s); break;
        case 4: launch_sweep_mt<P, 4, EPI, KH>(a, units, s); break;
        case 5: launch_sweep_mt<P, 5, EPI, KH>(a, units, s); break;
        case 6: launch_sweep_mt<P, 6, EPI, KH>(a, units, s); break;
        case 7: launch_sweep_mt<P, 7, EPI, KH>(a, units, s); break;
        case 8: launch_sweep_mt<P, 8, EPI, KH>(a, units, s); break;
        case 9: launch_sweep_mt<P, 9, EPI, KH>(a, units, s); break;
        case 10: launch_sweep_mt<P, 10, EPI, KH>(a, units, s); break;
        case 11: launch_sweep_mt<P, 11, EPI, KH>(a, units, s); break;
        default: launch_sweep_mt<P, 12, EPI, KH>(a, units, s); break;
    }
}

template <int MS, int NS, int WM, int WN, int ST, int EPI>
static void launch_block(const GemmArgs& a, const QkvOut& qo, hipStream_t s)
{
    const int n_ntiles = (a.N / 16 + NS - 1) / NS, n_mtiles = ((a.m_rows + 15) / 16 + MS - 1) / MS;
    hipLaunchKernelGGL((k_gemm_block<MS, NS, WM, WN, ST, EPI>), dim3(n_ntiles * n_mtiles * a.ksplit), dim3(64 * WM * WN), 0, s,
                       a, qo, (a.Kp / 32 + a.ksplit - 1) / a.ksplit, n_ntiles, n_mtiles);
}

// Waves, strips per wave and stages of each tile of block_tiles.
template <int EPI>
static void launch_block_epi(const GemmArgs& a, const QkvOut& qo, hipStream_t s)
{
    switch (a.block) {
        case 0: return launch_block<16, 16, 2, 4, 4, EPI>(a, qo, s);   // 8 waves of 8 x 4 strips, 128 KiB of LDS: one per unit
        case 1: return launch_block<16, 12, 4, 2, 4, EPI>(a, qo, s);   // 8 waves of 4 x 6, 112 KiB
        case 2: return launch_block<8, 16, 2, 2, 3, EPI>(a, qo, s);    // 4 waves of 4 x 8, 72 KiB: two per unit
        case 3: return launch_block<8, 12, 2, 2, 4, EPI>(a, qo, s);    // 4 waves of 4 x 6, 80 KiB
        case 4: return launch_block<8, 8, 2, 2, 4, EPI>(a, qo, s);     // 4 waves of 4 x 4, 64 KiB
        case 5: return launch_block<8, 4, 2, 2, 6, EPI>(a, qo, s);     // 4 waves of 4 x 2, 72 KiB
        case 6: return launch_block<6, 8, 2, 2, 4, EPI>(a, qo, s);     // 4 waves of 3 x 4, 56 KiB
        case 7: return launch_block<10, 8, 2, 2, 4, EPI>(a, qo, s);    // 4 waves of 5 x 4, 72 KiB
        case 8: return launch_block<12, 8, 4, 1, 4, EPI>(a, qo, s);    // 4 waves of 3 x 8, 80 KiB
        case 9: return launch_block<16, 8, 4, 2, 5, EPI>(a, qo, s);    // 8 waves of 4 x 4, 120 KiB: one per unit
        case 10: return launch_block<10, 12, 2, 2, 3, EPI>(a, qo, s);  // 4 waves of 5 x 6, 66 KiB
        case 11: return launch_block<12, 12, 2, 2, 3, EPI>(a, qo, s);  // 4 waves of 6 x 6, 72 KiB
        case 12: return launch_block<14, 16, 2, 4, 4, EPI>(a, qo, s);  // 8 waves of 7 x 4, 120 KiB
        case 13: return launch_block<20, 12, 4, 2, 4, EPI>(a, qo, s);  // 8 waves of 5 x 6, 128 KiB
        default: return launch_block<24, 12, 4, 2, 4, EPI>(a, qo, s);  // 8 waves of 6 x 6, 144 KiB
    }
}

template <int EPI>
static void launch_gemm_epi(const GemmArgs& a, hipStream_t s)
{
    if (a.block < 0 && a.m_rows <= kSweepMaxRows && a.sweep_p > 0 && a.sweep_gn > 0 && a.zero_blk) {
        const int nbw = sweep_nbw(EPI, a.m_rows);
        const int units = (a.N / 16 + nbw - 1) / nbw;
        const int per = (units + a.sweep_gn - 1) / a.sweep_gn;   // most units any workgroup owns
        if (a.sweep_p == 4 && per <= 4) {
            // where the plan asks for it (above 96 rows; with 12-bit weights everywhere): 8 waves, two per unit (see SweepSlot)
            if ((a.narrow ? a.narrow : a.sweep_kh) == 2) return launch_sweep_p<8, EPI, 2>(a, units, s);
            return launch_sweep_p<4, EPI, 1>(a, units, s);
        }
        if (per <= 8) return launch_sweep_p<8, EPI, 1>(a, units, s);
        // a plan this kernel cannot run falls through to the other kernels
    }
    if (a.block < 0 && a.m_rows <= 64) {
        const int mt = (a.m_rows + 15) / 16;
        switch (mt) {
            case 1: launch_skinny_mt<1, EPI>(a, s); break;
            case 2: launch_skinny_mt<2, EPI>(a, s); break;
            case 3: launch_skinny_mt<3, EPI>(a, s); break;
            default: launch_skinny_mt<4, EPI>(a, s); break;
        }
        return;
    }
    launch_block_epi<EPI>(a, QkvOut{}, s);
}

void launch_gemm(const GemmArgs& a, int epilogue, hipStream_t s, const QkvOut* qkv)
{
    switch (epilogue) {
        case EPI_SWIGLU: return launch_gemm_epi<EPI_SWIGLU>(a, s);
        case EPI_QKV: return launch_block_epi<EPI_QKV>(a, *qkv, s);
        case EPI_RESIDUAL: return launch_block_epi<EPI_RESIDUAL>(a, QkvOut{}, s);
        default: return launch_gemm_epi<EPI_PARTIAL>(a, s);
    }
}

template <int R>
static void launch_few_r(const FewArgs& a, int epilogue, hipStream_t s)
{
    const dim3 grid((a.units + a.plan.units_wg - 1) / a.plan.units_wg), block(64 * kFewWaves);
    const size_t lds = few_lds_bytes(R, a.Kp, epilogue);
    if (epilogue == EPI_SWIGLU) hipLaunchKernelGGL((k_gemm_few<R, 2, EPI_SWIGLU, true>), grid, block, lds, s, a);
    else if (epilogue == EPI_RESIDUAL && a.Kp <= 4096) hipLaunchKernelGGL((k_gemm_few<R, 1, EPI_RESIDUAL, false, 1>), grid, block, lds, s, a);
    else if (epilogue == EPI_RESIDUAL && a.Kp <= 12288) hipLaunchKernelGGL((k_gemm_few<R, 1, EPI_RESIDUAL, false, 3>), grid, block, lds, s, a);
    else if (epilogue == EPI_RESIDUAL) hipLaunchKernelGGL((k_gemm_few<R, 1, EPI_RESIDUAL, false, 4>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((k_gemm_few<R, 1, EPI_PARTIAL, true>), grid, block, lds, s, a);
}

void launch_gemm_few(const FewArgs& a, int n_rows, int epilogue, hipStream_t s)
{
    if (n_rows == 1) launch_few_r<1>(a, epilogue, s);
    else if (n_rows == 2) launch_few_r<2>(a, epilogue, s);
    else if (n_rows == 3) launch_few_r<3>(a, epilogue, s);
    else launch_few_r<4>(a, epilogue, s);
}

void launch_rope_append(const MbState& st, const float* qkv_part, int ksplit, size_t part_stride, float* qrot,
                        kv_t* kcache, kv_t* vcache, const float* rope_cos, const float* rope_sin, int d, int H,
                        int hd, int n_max, hipStream_t s)
{
    hipLaunchKernelGGL(k_rope_append, dim3(n_max, (d / 2 + 255) / 256), dim3(256), 0, s, st, qkv_part, ksplit, part_stride, qrot, kcache,
                       vcache, rope_cos, rope_sin, d, H, hd);
}

template <int HD, int NW, int PW = NW, bool SPLIT = false>
static void launch_attention_decode_inst(const MbState& st, const float* qkv_part, int ksplit, size_t part_stride,
                                         kv_t* kcache, kv_t* vcache, const float* rope_cos, const float* rope_sin,
                                         f16_t* out_packed, int d, int H, int n_max, float* shares, int S, hipStream_t s)
{
    hipLaunchKernelGGL((k_attention_decode<HD, NW, PW, SPLIT>), dim3(n_max, H, S), dim3(64 * PW), 0, s, st, qkv_part, ksplit, part_stride,
                       kcache, vcache, rope_cos, rope_sin, out_packed, d, shares);
    if (SPLIT) hipLaunchKernelGGL((k_attention_join<HD>), dim3(n_max, H), dim3(64), 0, s, st, shares, S, out_packed, d);
}

void launch_attention_decode(const MbState& st, const float* qkv_part, int ksplit, size_t part_stride,
                             kv_t* kcache, kv_t* vcache, const float* rope_cos, const float* rope_sin,
                             f16_t* out_packed, int d, int H, int hd, int n_max, int plan_rows, int mb_rows, int max_ctx,
                             float* scratch, hipStream_t s)
{
    const AttentionPlan p = attention_plan(n_max, plan_rows, mb_rows, H, hd, max_ctx);
#define SS_ATTN_ARGS st, qkv_part, ksplit, part_stride, kcache, vcache, rope_cos, rope_sin, out_packed, d, H, n_max, scratch, p.split, s
    if (hd == 128) {
        if (p.split > 1) launch_attention_decode_inst<128, 8, 8, true>(SS_ATTN_ARGS);
        else if (p.slices == 16) launch_attention_decode_inst<128, 16>(SS_ATTN_ARGS);
        else if (p.slices == 8 && p.waves == 2) launch_attention_decode_inst<128, 8, 2>(SS_ATTN_ARGS);
        else if (p.slices == 8 && p.waves == 4) launch_attention_decode_inst<128, 8, 4>(SS_ATTN_ARGS);
        else if (p.slices == 8) launch_attention_decode_inst<128, 8>(SS_ATTN_ARGS);
        else if (p.waves == 2) launch_attention_decode_inst<128, 4, 2>(SS_ATTN_ARGS);
        else launch_attention_decode_inst<128, 4>(SS_ATTN_ARGS);
    } else {
        if (p.split > 1) launch_attention_decode_inst<64, 8, 8, true>(SS_ATTN_ARGS);
        else if (p.slices == 16) launch_attention_decode_inst<64, 16>(SS_ATTN_ARGS);
        else if (p.slices == 8 && p.waves == 2) launch_attention_decode_inst<64, 8, 2>(SS_ATTN_ARGS);
        else if (p.slices == 8 && p.waves == 4) launch_attention_decode_inst<64, 8, 4>(SS_ATTN_ARGS);
        else if (p.slices == 8) launch_attention_decode_inst<64, 8>(SS_ATTN_ARGS);
        else if (p.waves == 2) launch_attention_decode_inst<64, 4, 2>(SS_ATTN_ARGS);
        else launch_attention_decode_inst<64, 4>(SS_ATTN_ARGS);
    }
#undef SS_ATTN_ARGS
}

void launch_attention_prompt(const MbState& st, const float* qrot, const kv_t* kcache, const kv_t* vcache,
                             f16_t* out_packed, int d, int H, int hd, int B, int max_len, hipStream_t s)
{
    // two query tiles per wave from kAttnTallFrom positions on, see k_attention_prompt
    const int per = max_len >= kAttnTallFrom ? 128 : 64;
    const dim3 grid(H, B, (max_len + per - 1) / per);
#define SS_ATTN_ARGS grid, dim3(256), 0, s, st, qrot, kcache, vcache, out_packed, d
    if (hd == 128) {
        if (per == 128) hipLaunchKernelGGL((k_attention_prompt<128, 2, 2>), SS_ATTN_ARGS);
        else hipLaunchKernelGGL((k_attention_prompt<128, 1, 1>), SS_ATTN_ARGS);
    } else {
        if (per == 128) hipLaunchKernelGGL((k_attention_prompt<64, 2, 2>), SS_ATTN_ARGS);
        else hipLaunchKernelGGL((k_attention_prompt<64, 1, 1>), SS_ATTN_ARGS);
    }
#undef SS_ATTN_ARGS
}

void launch_row_step(const MbState& st, const RowStepArgs& a, int hd, int n_max, hipStream_t s)
{
    const size_t lds = row_step_lds_bytes(a.d, a.Fp, hd);
    if (hd == 128) hipLaunchKernelGGL((k_row_step<128>), dim3(n_max), dim3(kRowThreads), lds, s, st, a);
    else hipLaunchKernelGGL((k_row_step<64>), dim3(n_max), dim3(kRowThreads), lds, s, st, a);
}

void launch_argmax(const float* logits, int vocab, const int32_t* d_nsel, int32_t* am, int n_max, hipStream_t s)
{
    hipLaunchKernelGGL(k_argmax, dim3(n_max), dim3(1024), 0, s, logits, vocab, d_nsel, am);
}

void launch_read_stream(const f16_t* p, size_t bytes, uint32_t* sink, hipStream_t s)
{
    const int n_chunks = (int)(bytes >> 16);
    if (n_chunks < 1) return;
    hipLaunchKernelGGL(k_read_stream, dim3((n_chunks + 3) / 4), dim3(256), 0, s, (const u32x4*)p, n_chunks, sink);
}

void launch_sample(const float* logits, int vocab, const int32_t* d_nsel, const MbState& st, const float* draws,
                   const int32_t* ids, uint64_t seed, float inv_temp, int n_max, hipStream_t s)
{
    hipLaunchKernelGGL(k_sample, dim3(n_max), dim3(1024), 0, s, logits, vocab, d_nsel, st, draws, ids,
                       (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32), inv_temp);
}

void launch_step_update(const MbState& st, int compact, int eos_id, hipStream_t s)
{
    hipLaunchKernelGGL(k_step_update, dim3(1), dim3(1024), 0, s, st, compact, eos_id);
}

}  // namespace ss
