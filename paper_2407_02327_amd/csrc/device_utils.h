// Device helpers shared by the gfx950 kernels: wave reductions, 16-byte vector access,
// the Philox4x32-10 block function and the scalar fixed-point quantizer.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "kernels.h"

namespace qsync {

constexpr int kWaveSize = 64;

__device__ __forceinline__ float wave_reduce_max(float v)
{
#pragma unroll
    for(int off = kWaveSize / 2; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWaveSize));
    return v;
}

template <typename F> __device__ __forceinline__ F wave_reduce_sum(F v)
{
#pragma unroll
    for(int off = kWaveSize / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWaveSize);
    return v;
}

// Block-wide maximum for blocks of up to 1024 threads; the result is valid in thread 0.
__device__ __forceinline__ float block_reduce_max(float v, float* lds /* >= 16 floats */)
{
    v = wave_reduce_max(v);
    const int lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
    if(lane == 0) lds[wave] = v;
    __syncthreads();
    if(threadIdx.x == 0)
    {
        const int nw = (blockDim.x + kWaveSize - 1) / kWaveSize;
        for(int i = 1; i < nw; ++i) v = fmaxf(v, lds[i]);
    }
    return v;
}

// Block-wide sum in a fixed order (wave shuffles, then the wave sums in order); valid in thread 0.
template <typename F> __device__ __forceinline__ F block_reduce_sum(F v, F* lds /* >= 16 */)
{
    v = wave_reduce_sum(v);
    const int lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
    if(lane == 0) lds[wave] = v;
    __syncthreads();
    if(threadIdx.x == 0)
    {
        const int nw = (blockDim.x + kWaveSize - 1) / kWaveSize;
        for(int i = 1; i < nw; ++i) v += lds[i];
    }
    return v;
}

// One column of S partials [S][cols]: thread q < 16 of the column folds every sixteenth partial, then the sixteen are folded in
// order (fixed assignment, fixed order).  The first 256 threads of the workgroup take part; the result is valid for q == 0.
template <bool MAX> __device__ __forceinline__ float fold_column(const float* __restrict__ partial, int S, int64_t cols, int64_t c, int q, float* lds)
{
    float acc = 0.0f;
    if(c < cols && threadIdx.x < 256)
    {
        // (the addresses advance: a 64-bit product for each load took as long as the loads; gradient statistics of 2184x65 4.7 us a
        // fold, 4.1)
        const float*  at   = partial + static_cast<int64_t>(q) * cols + c;
        const float*  last = partial + static_cast<int64_t>(S - 1) * cols + c;
        const int64_t step = 16 * cols;
        for(int s0 = q; s0 < S; s0 += 128, at += 8 * step)      // eight loads in flight, past the end the last one again; the fold keeps its order
        {
            float o[8];
#pragma unroll
            for(int u = 0; u < 8; ++u) o[u] = *(s0 + 16 * u < S ? at + u * step : last);
#pragma unroll
            for(int u = 0; u < 8; ++u)
            {
                const float v = s0 + 16 * u < S ? o[u] : 0.0f;
                acc = MAX ? fmaxf(acc, v) : acc + v;
            }
        }
    }
    if(threadIdx.x < 256) lds[threadIdx.x] = acc;
    __syncthreads();
    float t = 0.0f;
    if(q == 0)
        for(int i = 0; i < 16; ++i) t = MAX ? fmaxf(t, lds[i * 16 + threadIdx.x % 16]) : t + lds[i * 16 + threadIdx.x % 16];
    return t;
}
__device__ __forceinline__ void fold_columns(const ColumnFoldArgs& f, uint32_t block, float* lds /* 256 floats */)
{
    const int     q = threadIdx.x / 16;
    const int64_t c = static_cast<int64_t>(block) * 16 + threadIdx.x % 16;
    const float   t = fold_column<false>(f.partial, f.S, f.cols, c, q, lds);
    if(q == 0 && c < f.cols) f.out[c] = t;
}

// Element access that widens to fp32 (binary16 -> fp32 is exact).
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(__half v) { return __half2float(v); }

// 16 bytes of T as fp32 values.
template <typename T> struct Vec16;
template <> struct Vec16<float>
{
    static constexpr int N = 4;
    __device__ static __forceinline__ void decode(const uint4& r, float (&out)[4])
    {
        out[0] = __uint_as_float(r.x); out[1] = __uint_as_float(r.y);
        out[2] = __uint_as_float(r.z); out[3] = __uint_as_float(r.w);
    }
    __device__ static __forceinline__ void load(const float* p, float (&out)[4])
    {
        decode(*reinterpret_cast<const uint4*>(p), out);
    }
};
template <> struct Vec16<__half>
{
    static constexpr int N = 8;
    __device__ static __forceinline__ void load(const __half* p, float (&out)[8])
    {
        decode(*reinterpret_cast<const uint4*>(p), out);
    }
    __device__ static __forceinline__ void decode(const uint4& raw, float (&out)[8])
    {
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for(int i = 0; i < 4; ++i)
        {
            out[2 * i]     = __half2float(__ushort_as_half(static_cast<unsigned short>(w[i] & 0xFFFFu)));
            out[2 * i + 1] = __half2float(__ushort_as_half(static_cast<unsigned short>(w[i] >> 16)));
        }
    }
};

// Philox4x32 with ten rounds (Salmon et al., SC'11).  One round maps
// (c0,c1,c2,c3) -> (hi(M1*c2)^c1^k0, lo(M1*c2), hi(M0*c0)^c3^k1, lo(M0*c0)); the key
// advances by the Weyl constants.  The key is wave-uniform here, so its schedule runs on
// the scalar unit.  A round's two three-input exclusive ors are one instruction each: left to the compiler, six of seven
// become two.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t k_uniform)
{
    uint32_t r;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "s"(k_uniform));
    return r;
}
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for(int r = 0; r < 10; ++r)
    {
        const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c.x;
        const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c.z;
        uint4 n;
        n.x = xor3(static_cast<uint32_t>(p1 >> 32), c.y, k0);
        n.y = static_cast<uint32_t>(p1);
        n.z = xor3(static_cast<uint32_t>(p0 >> 32), c.w, k1);
        n.w = static_cast<uint32_t>(p0);
        c = n;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// The Philox block of the 8-element group `group` of a tensor: counter = offset + group as a
// 128-bit integer (offset and group are 64-bit, so only a carry reaches word 2).
__device__ __forceinline__ uint4 philox_group(uint64_t seed, uint64_t offset, uint64_t group)
{
    const uint64_t lo = offset + group;
    uint4 c;
    c.x = static_cast<uint32_t>(lo);
    c.y = static_cast<uint32_t>(lo >> 32);
    c.z = lo < group ? 1u : 0u;
    c.w = 0u;
    return philox4x32_10(c, static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32));
}

// 16-bit draw number `slot` (0..7) of a Philox block: word slot/2, low half first.
__device__ __forceinline__ uint32_t philox_draw16(const uint4& blk, int slot)
{
    const uint32_t w = (slot >> 1) == 0 ? blk.x : (slot >> 1) == 1 ? blk.y : (slot >> 1) == 2 ? blk.z : blk.w;
    return (slot & 1) ? (w >> 16) : (w & 0xFFFFu);
}

// Fixed-point code of one value: clamp(round(x * inv), -qmax, qmax).  RND is a qsync::Round.
// The product is a single fp32 multiply.  Stochastic rounding: the value rounds up iff
// u16 < floor(residual * 2^16) with residual = x*inv - floor(x*inv).  It is evaluated in 16.16 fixed point:
// t = floor(x*inv * 2^16) is exact (a power-of-two scaling), floor(x*inv) = t >> 16 and floor(residual * 2^16) =
// t & 0xFFFF, so "floor + (u16 < low half)" is the carry of t + (65535 - u16) into bit 16.  Clamping t to
// +-qmax * 2^16 first is the clamp of the code (a clamped t has a zero low half) and keeps the sum inside 32 bits.
__device__ __forceinline__ int floor_to_int(float v)      // saturates; NaN -> 0
{
    int t;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(t) : "v"(v));
    return t;
}
__device__ __forceinline__ int clamped_fixed_point(float v16, int qmax)      // v16 = x * inv * 2^16
{
    int       t   = floor_to_int(v16);
    const int lim = qmax << 16;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(t) : "v"(t), "v"(-lim), "v"(lim));
    return t;
}
template <int RND>
__device__ __forceinline__ int quantize_code(float x, float inv, int qmax, uint32_t u16)
{
    const float v = __fmul_rn(x, inv);
    int         c;
    if(RND == 0) c = static_cast<int>(rintf(v));
    else if(RND == 2) c = floor_to_int(v);
    else return (clamped_fixed_point(__fmul_rn(v, 65536.0f), qmax) + static_cast<int>(65535u - u16)) >> 16;
    return min(max(c, -qmax), qmax);
}

// The products clamped_fixed_point takes, x * inv * 2^16, of eight values.  Of binary16 values in one multiplication by 2^16 inv: 2^16
// only moves the exponent, unless x * inv is subnormal or 2^16 inv overflows, which no binary16 tensor can meet with the
// inverse of its own maximum (|x| >= 2^-24, 2^-16 < inv < 2^31); an inverse scale beyond 2^-100 .. 2^100, which only a
// caller can make up, keeps the two multiplications.
template <typename T> __device__ __forceinline__ void stochastic_products(const float (&v)[8], float inv, float (&p)[8])
{
    if(sizeof(T) == 2 && fabsf(inv) >= 0x1p-100f && fabsf(inv) <= 0x1p100f)
    {
        const float f = __fmul_rn(inv, 65536.0f);
#pragma unroll
        for(int j = 0; j < 8; ++j) p[j] = __fmul_rn(v[j], f);
    }
    else
    {
#pragma unroll
        for(int j = 0; j < 8; ++j) p[j] = __fmul_rn(__fmul_rn(v[j], inv), 65536.0f);
    }
}
// t + (word's low or high half)
template <int HALF> __device__ __forceinline__ uint32_t add_half(int t, uint32_t word)
{
    uint32_t r;
    if constexpr(HALF == 0)
        asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(r) : "v"(t), "v"(word));
    else
        asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(r) : "v"(t), "v"(word));
    return r;
}
// Codes of eight values, packed; `blk` is their Philox block (stochastic rounding).  The stochastic form is bound by the vector
// unit, so its steps are spelled out: 65535 - u of two draws is one complement of their word, added half by half, and the
// codes are byte 2 of the sums.  With the multiplications above and xor3, 585 -> 425 vector instructions for 32 binary16
// values, 76 of them the quarter-rate ones of Philox; maximum, codes and dequantized values of a 16384 x 4096 gradient
// 118.6 -> 113.4 us, 5 of the quantizer's 39.
template <typename T, int RND>
__device__ __forceinline__ void quantize_group(const float (&v)[8], float inv, int qmax, const uint4& blk, uint32_t (&w)[2])
{
    if constexpr(RND == 1)
    {
        float p[8];
        stochastic_products<T>(v, inv, p);
        const uint32_t draws[4] = {~blk.x, ~blk.y, ~blk.z, ~blk.w};
#pragma unroll
        for(int k = 0; k < 2; ++k)
        {
            const uint32_t s0 = add_half<0>(clamped_fixed_point(p[4 * k], qmax), draws[2 * k]);
            const uint32_t s1 = add_half<1>(clamped_fixed_point(p[4 * k + 1], qmax), draws[2 * k]);
            const uint32_t s2 = add_half<0>(clamped_fixed_point(p[4 * k + 2], qmax), draws[2 * k + 1]);
            const uint32_t s3 = add_half<1>(clamped_fixed_point(p[4 * k + 3], qmax), draws[2 * k + 1]);
            w[k] = __builtin_amdgcn_perm(s1, s0, 0x0C0C0602u) | __builtin_amdgcn_perm(s3, s2, 0x06020C0Cu);
        }
        return;
    }
    w[0] = w[1] = 0u;
#pragma unroll
    for(int j = 0; j < 8; ++j) w[j / 4] |= (static_cast<uint32_t>(quantize_code<RND>(v[j], inv, qmax, 0u)) & 0xFFu) << (8 * (j % 4));
}

}  // namespace qsync
