// FP32 GEMM for operands whose rows are not 16-byte multiples, or that do not start on 16 bytes:
// C[M,N] = epilogue( sum_k A[m,k] B[n,k] ).
//
// Such rows cannot go to LDS in 16-byte pieces, so they pass through registers, four bytes a lane (a wavefront reads two rows of
// 128 bytes) and one K tile ahead; the 32x32x2 matrix instruction takes 64 clocks, under which the four-byte loads, their
// addresses and the LDS writes all fit.  Bound by the matrix instructions, as the 16-byte form is; small products by the K tiles one
// behind the other (1024 clocks of instructions each on the 64 tile), which the K splits of the plan shorten.
// Fused multiply-adds
// on the vector units, 64x64 and no splits -> here, us: 128x175x73 15.4 -> 7.1, 500x300x201 32 -> 11, 1000x1000x1001 193 -> 41,
// 200x300x8001 1662 -> 27, 4097x175x1023 174 -> 46, 2049x2047x255 67 -> 51; the 16-byte form takes 0.75 of these times.
#include "gemm_device.h"

namespace qsync {

namespace {

constexpr int kStepK = kRowBytes / 4;      // floats a K tile
constexpr int kPitch = kStepK + 4;         // floats an LDS row: 16-byte reads of sixteen rows meet all banks

template <int T> constexpr int f32_lds_bytes() { return 2 * 2 * T * kPitch * 4 + (2 * T + 4) * 4; }

template <int T, bool SPLIT>
__global__ __launch_bounds__(256) void gemm_f32_any_kernel(const GemmKernelArgs p, int64_t K, int splits)
{
    constexpr int F = T / 64, R = T / 8;      // fragments of a wavefront each way; rows of an operand a lane loads
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    float* const stages = reinterpret_cast<float*>(lds);                       // [stage][A, B][row][kPitch]
    float* const colp   = stages + 2 * 2 * T * kPitch;
    const int    tid = threadIdx.x, lane = tid % kWaveSize, wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
    const int    row = lane % 32, half = lane / 32, wm = wave / 2, wn = wave % 2;
    int          split, tm, tn;
    item_of_block(static_cast<int>(blockIdx.x), p.tiles_m, p.tiles_n, SPLIT ? splits : 1, p.group_m, split, tm, tn);
    const int64_t m0 = static_cast<int64_t>(tm) * T, n0 = static_cast<int64_t>(tn) * T;
    const int64_t first = static_cast<int64_t>(split) * p.ktiles_per_split * kStepK;
    const int64_t end   = SPLIT && first + static_cast<int64_t>(p.ktiles_per_split) * kStepK < K ? first + static_cast<int64_t>(p.ktiles_per_split) * kStepK : K;
    const int     tiles = end > first ? static_cast<int>((end - first + kStepK - 1) / kStepK) : 0;
    const float   alpha = *(p.s0 ? p.s0 : &g_one) * *(p.s1 ? p.s1 : &g_one);
    const uint32_t seen = p.amax_bits ? __hip_atomic_load(p.amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    if constexpr(!SPLIT)
        for(int c = tid; c < T; c += 256)
        {
            const int64_t n = n0 + c < p.N ? n0 + c : p.N - 1;
            colp[c]     = p.col_scale ? p.col_scale[n] : 1.0f;
            colp[T + c] = p.col_bias ? p.col_bias[n] : 0.0f;
        }

    // rows past the last one load that row again (their outputs are never stored); K indices past the end give zeros
    const float*  A = reinterpret_cast<const float*>(p.A) + m0 * K;
    const float*  B = reinterpret_cast<const float*>(p.B) + n0 * K;
    const int     last_a = static_cast<int>(p.M - m0 < T ? p.M - m0 : T) - 1, last_b = static_cast<int>(p.N - n0 < T ? p.N - n0 : T) - 1;
    const int     lk = tid % kStepK, lr = tid / kStepK;
    float         a[R], b[R];
    auto load = [&](int t) {
        const int64_t k  = first + static_cast<int64_t>(t) * kStepK + lk;
        const int64_t at = k < end ? k : 0;
#pragma unroll
        for(int i = 0; i < R; ++i)
        {
            const int     ra = lr + 8 * i < last_a ? lr + 8 * i : last_a, rb = lr + 8 * i < last_b ? lr + 8 * i : last_b;
            a[i] = A[ra * K + at];
            b[i] = B[rb * K + at];
        }
    };
    auto put = [&](int t) {      // (the values are first looked at here: the loads are in flight under a K tile's instructions)
        const bool in  = first + static_cast<int64_t>(t) * kStepK + lk < end;
        float*     dst = stages + t % 2 * (2 * T * kPitch) + lr * kPitch + lk;
#pragma unroll
        for(int i = 0; i < R; ++i)
        {
            dst[8 * i * kPitch]              = in ? a[i] : 0.0f;
            dst[T * kPitch + 8 * i * kPitch] = in ? b[i] : 0.0f;
        }
    };
    v16f32 acc[F][F];
#pragma unroll
    for(int i = 0; i < F; ++i)
#pragma unroll
        for(int j = 0; j < F; ++j)
#pragma unroll
            for(int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    if(tiles > 0)
    {
        load(0);
        put(0);
    }
    __syncthreads();
    for(int t = 0; t < tiles; ++t)
    {
        if(t + 1 < tiles) load(t + 1);
        const float* sa = stages + (t % 2) * (2 * T * kPitch) + (wm * (T / 2) + row) * kPitch;
        const float* sb = stages + (t % 2) * (2 * T * kPitch) + T * kPitch + (wn * (T / 2) + row) * kPitch;
#pragma unroll
        for(int c = 0; c < kStepK; c += 4)
        {   // K ascending: an instruction takes K index c + e of the lower half's lanes, then c + e + 1 of the upper's
            float fa[F][2], fb[F][2];
#pragma unroll
            for(int i = 0; i < F; ++i)
            {
                const float4 va = *reinterpret_cast<const float4*>(sa + i * 32 * kPitch + c), vb = *reinterpret_cast<const float4*>(sb + i * 32 * kPitch + c);
                fa[i][0] = half ? va.y : va.x; fa[i][1] = half ? va.w : va.z;
                fb[i][0] = half ? vb.y : vb.x; fb[i][1] = half ? vb.w : vb.z;
            }
#pragma unroll
            for(int e = 0; e < 2; ++e)
#pragma unroll
                for(int i = 0; i < F; ++i)
#pragma unroll
                    for(int j = 0; j < F; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j][e], fa[i][e], acc[i][j], 0, 0, 0);
        }
        if(t + 1 < tiles) put(t + 1);      // (read last before the barrier that ended the turn before this one)
        __syncthreads();
    }
    store_tile<F32Rows32, T, T, 2, 2, T * kPitch * 4, SPLIT>(p, acc, lds, colp, m0, n0, split, alpha, 0.0f, seen);
}

template <int T> hipError_t launch_any(const GemmKernelArgs& a, int64_t K, int splits, hipStream_t st)
{
    const dim3 grid(static_cast<unsigned>(a.tiles_m) * static_cast<unsigned>(a.tiles_n) * static_cast<unsigned>(splits));
    constexpr int kLds = f32_lds_bytes<T>();
    static bool   attr_set[16] = {};      // per instantiation and device; benign if set twice
    int           dev = 0;
    const bool    known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 16;
    if(!known || !attr_set[dev])
    {
        const void* const kernels[] = {reinterpret_cast<const void*>(&gemm_f32_any_kernel<T, false>), reinterpret_cast<const void*>(&gemm_f32_any_kernel<T, true>)};
        for(const void* k : kernels)
        {
            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
            if(e != hipSuccess) return e;
        }
        if(known) attr_set[dev] = true;
    }
    if(splits > 1) gemm_f32_any_kernel<T, true><<<grid, dim3(256), kLds, st>>>(a, K, splits);
    else           gemm_f32_any_kernel<T, false><<<grid, dim3(256), kLds, st>>>(a, K, 1);
    return hipGetLastError();
}

}  // namespace

// The plan's tile (256: on 128) and K splits; the partial products of more than one are left to the caller.
hipError_t launch_gemm_f32(const GemmProblem& p, const GemmPlan& plan, void* workspace, hipStream_t stream)
{
    const int     T = plan.tile == 2 ? 64 : 128, splits = plan.splits < 1 ? 1 : plan.splits;
    const int64_t ktiles = (p.K + kStepK - 1) / kStepK, per = (ktiles + splits - 1) / splits;
    GemmKernelArgs a{};
    a.A = static_cast<const uint8_t*>(p.A);
    a.B = static_cast<const uint8_t*>(p.B);
    a.M = p.M; a.N = p.N;
    a.C = p.C; a.c_is_f16 = p.c_dtype == kF16;
    a.s0 = p.s0; a.s1 = p.s1; a.col_scale = p.col_scale; a.col_bias = p.col_bias;
    a.partial   = workspace;
    a.amax_bits = splits > 1 ? nullptr : p.out_amax_bits;
    a.ktiles_per_split = static_cast<int>(per < 1 ? 1 : per);
    a.tiles_m = static_cast<int>((p.M + T - 1) / T);
    a.tiles_n = static_cast<int>((p.N + T - 1) / T);
    a.group_m = kGroupM;
    return T == 64 ? launch_any<64>(a, p.K, splits, stream) : launch_any<128>(a, p.K, splits, stream);
}

}  // namespace qsync
