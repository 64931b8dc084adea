// C[M,N] = epilogue( sum_k A[m,k] B[n,k] ), int8 and binary16, where 64 rows and 16 or 32 columns a workgroup are few enough
// workgroups for one on each unit: a handful of tokens, small operators.
//
// On the tiles of 64 columns and more such a product is a few dozen workgroups (or one K split each of them) that walk K one LDS
// stage and barrier after the other, 0.26 us per 128 bytes.  Here a workgroup's eight wavefronts take K in turns of 64 bytes,
// each through stages of its own with two or three turns in flight and no barrier, into the 16x16 matrix instructions; the
// eight sums meet in LDS once at the end.
#include "gemm_device.h"

namespace qsync {

namespace {

constexpr int kRowsWaves = 8;

// MF, NF: fragments of 16 rows, of 16 columns.  The B fragment is the instruction's first operand, so a lane holds four consecutive columns
// (4 (lane / 16) ..) of output row lane % 16.
constexpr int64_t kRowsGroups = 256;                                        // one for each unit
// The dimension of more groups runs fastest and is padded to a multiple of the eight XCDs where that stays within one group for
// each unit: the workgroups that read one piece of the longer operand then share an L2.  4096x128 by 3072, int8: 11.5 -> 7.5 us.
template <int NF> __host__ __device__ constexpr bool rows_first(int64_t M, int64_t N) { return M > N * (4 / NF); }
constexpr int rows_stages(int loads) { return loads > 4 ? 3 : 4; }             // turns in LDS: 144 KB of them at most
template <typename TR, int MF, int NF>
__global__ __launch_bounds__(64 * kRowsWaves) void gemm_rows_kernel(const GemmKernelArgs p)
{
    typedef typename TR::accv_t vec;
    constexpr int kLoads = MF + NF, kStages = rows_stages(kLoads), kTurn = kLoads * 1024;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int     lane = threadIdx.x % kWaveSize, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWaveSize));
    const bool    tall = rows_first<NF>(p.M, p.N);
    const int64_t n0 = static_cast<int64_t>(tall ? blockIdx.y : blockIdx.x) * (16 * NF), m0 = static_cast<int64_t>(tall ? blockIdx.x : blockIdx.y) * 64;
    if(m0 >= p.M || n0 >= p.N) return;                                      // (padded to a multiple of the XCDs)
    uint8_t* const mine = lds + wave * (kStages * kTurn);

    // loads: four lanes read 64 consecutive bytes of a row (lanes on sixteen rows, as the operands want them, took four times as
    // long); the 16-byte chunks land XOR-swizzled so that sixteen rows of one chunk meet all banks
    const int      lrow = lane / 4, lchunk = ((lane % 4) ^ ((lane >> 4) & 3)) * 16;
    const uint8_t* src[kLoads];
#pragma unroll
    for(int f = 0; f < MF; ++f) src[f] = p.A + (m0 + f * 16 + lrow < p.M ? m0 + f * 16 + lrow : p.M - 1) * p.Kb;
#pragma unroll
    for(int j = 0; j < NF; ++j) src[MF + j] = p.B + (n0 + j * 16 + lrow < p.N ? n0 + j * 16 + lrow : p.N - 1) * p.Kb;
    // (rows and columns past the end: any valid one, never stored)
    const int all = static_cast<int>((p.Kb + 63) / 64), turns = all > wave ? (all - wave + kRowsWaves - 1) / kRowsWaves : 0;
    auto issue = [&](int t) {
        const int64_t k   = (static_cast<int64_t>(t) * kRowsWaves + wave) * 64 + lchunk;
        const bool    in  = k < p.Kb;                                        // (16-byte pieces: Kb is a multiple of 16)
        uint8_t*      dst = mine + t % kStages * kTurn;
        static_for<kLoads>([&](auto f) {
            constexpr int i = decltype(f)::value, IMM = i % 4 * 1024;
            const uint8_t* at = in ? src[i] + k : reinterpret_cast<const uint8_t*>(&g_zero_chunk);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(at - IMM),
                                             (__attribute__((address_space(3))) void*)(dst + i / 4 * 4096), 16, IMM, 0);
        });
    };
    vec acc[MF * NF];
#pragma unroll
    for(int f = 0; f < MF * NF; ++f) acc[f] = vec{0, 0, 0, 0};
    const int      row = lane % 16, quad = lane / 16;
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t*)mine));
    const uint32_t frag = static_cast<uint32_t>(row * 64 + ((quad ^ ((row >> 2) & 3)) * 16));
#pragma unroll
    for(int t = 0; t < kStages - 1; ++t)
        if(t < turns) issue(t);
    for(int t = 0; t < turns; ++t)
    {   // (every wavefront by itself: its loads, its slice of LDS)
        if(t + kStages - 1 < turns) issue(t + kStages - 1);
        wait_tiles<kLoads, kStages - 1>(turns - 1 - t);
        v4i32          op[kLoads];
        const uint32_t at = lds0 + static_cast<uint32_t>(t % kStages * kTurn) + frag;
        static_for<kLoads>([&](auto f) { frag_read<decltype(f)::value * 1024>(op[decltype(f)::value], at); });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for(int f = 0; f < MF; ++f)
#pragma unroll
            for(int j = 0; j < NF; ++j) acc[j * MF + f] = TR::mfma(op[MF + j], op[f], acc[j * MF + f]);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();                                                        // (the sums take the place of the stages)
#pragma unroll
    for(int f = 0; f < MF * NF; ++f) *reinterpret_cast<vec*>(lds + ((wave * MF * NF + f) * 64 + lane) * 16) = acc[f];
    __syncthreads();
    if(wave >= MF * NF) return;
    vec sum = *reinterpret_cast<const vec*>(lds + (wave * 64 + lane) * 16);
#pragma unroll
    for(int w = 1; w < kRowsWaves; ++w) sum += *reinterpret_cast<const vec*>(lds + ((w * MF * NF + wave) * 64 + lane) * 16);

    const int64_t m = m0 + wave % MF * 16 + row, n = n0 + wave / MF * 16 + quad * 4;
    if(m >= p.M || n >= p.N) return;
    const float alpha = *(p.s0 ? p.s0 : &g_one) * *(p.s1 ? p.s1 : &g_one);
    float       fs[4], bs[4];
#pragma unroll
    for(int e = 0; e < 4; ++e)
    {
        const int64_t c = n + e < p.N ? n + e : p.N - 1;
        fs[e] = p.col_scale ? alpha * p.col_scale[c] : alpha;
        bs[e] = p.col_bias ? p.col_bias[c] : 0.0f;
    }
    const int64_t at = m * p.N + n;
    const int     os = p.c_is_f16 ? 2 : 4;
    uint8_t* const dst = static_cast<uint8_t*>(p.C) + at * os;
    const bool    vector = p.N % 4 == 0 && (reinterpret_cast<uintptr_t>(p.C) & (4 * os - 1)) == 0;
    float v[4];
#pragma unroll
    for(int e = 0; e < 4; ++e) v[e] = static_cast<float>(sum[e]);
    if(p.c_is_f16)
    {
        const uint2 h = make_uint2(fma_out_half2(v[0], fs[0], bs[0], v[1], fs[1], bs[1]), fma_out_half2(v[2], fs[2], bs[2], v[3], fs[3], bs[3]));
        if(vector) *reinterpret_cast<uint2*>(dst) = h;
        else
            for(int e = 0; e < 4 && n + e < p.N; ++e)
                reinterpret_cast<uint16_t*>(dst)[e] = static_cast<uint16_t>((e < 2 ? h.x : h.y) >> (16 * (e % 2)));
    }
    else
    {
        const float4 y = make_float4(fmaf(v[0], fs[0], bs[0]), fmaf(v[1], fs[1], bs[1]), fmaf(v[2], fs[2], bs[2]), fmaf(v[3], fs[3], bs[3]));
        const float  o[4] = {y.x, y.y, y.z, y.w};
        if(vector) *reinterpret_cast<float4*>(dst) = y;
        else
            for(int e = 0; e < 4 && n + e < p.N; ++e) reinterpret_cast<float*>(dst)[e] = o[e];
    }
}

template <typename TR, int MF, int NF> hipError_t launch_fragments(const GemmKernelArgs& a, hipStream_t st)
{
    static_assert(MF * NF <= kRowsWaves, "a wavefront per fragment in the epilogue");
    constexpr int kLds = kRowsWaves * rows_stages(MF + NF) * (MF + NF) * 1024;
    static bool   attr_set[16] = {};      // per instantiation and device; benign if set twice
    int           dev = 0;
    const bool    known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 16;
    if(!known || !attr_set[dev])
    {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_rows_kernel<TR, MF, NF>), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if(e != hipSuccess) return e;
        if(known) attr_set[dev] = true;
    }
    const int64_t m = (a.M + 63) / 64, n = (a.N + 16 * NF - 1) / (16 * NF), few = rows_first<NF>(a.M, a.N) ? n : m;
    int64_t       many = rows_first<NF>(a.M, a.N) ? m : n;
    if((many + 7) / 8 * 8 * few <= kRowsGroups) many = (many + 7) / 8 * 8;
    gemm_rows_kernel<TR, MF, NF><<<dim3(static_cast<unsigned>(many), static_cast<unsigned>(few)), dim3(64 * kRowsWaves), kLds, st>>>(a);
    return hipGetLastError();
}
template <typename TR> hipError_t launch_rows(const GemmKernelArgs& a, int columns, hipStream_t st)
{
    if(columns == 2) return launch_fragments<TR, 4, 2>(a, st);
    switch(a.M > 64 ? 4 : (a.M + 15) / 16)
    {
    case 1: return launch_fragments<TR, 1, 1>(a, st);
    case 2: return launch_fragments<TR, 2, 1>(a, st);
    case 3: return launch_fragments<TR, 3, 1>(a, st);
    default: return launch_fragments<TR, 4, 1>(a, st);
    }
}
// Fragments of columns a workgroup, 0: other tiles are faster.  A second workgroup on a unit waits for the first (its stages fill
// the LDS; at most 16 rows two fit), which loses at once: 64x16384x64 3.8 us on the tiles, 9.0 here.  Beyond 6 KB of contraction
// (8 KB up to 32 rows) K splits over workgroups win.  The better of the 128 and 64 tiles -> here, operands warm, binary16 outputs, us:
//   int8, 16 columns:  1x4096x1024 5.0 -> 3.3, 64x4096x4096 10.7 -> 8.5, 128x1024x2048 7.2 -> 4.7, 256x1024x4096 10.7 -> 6.9,
//                      512x512x4096 10.7 -> 7.1, 4096x64x3072 9.3 -> 6.0; 100x768x6144 9.7 -> 7.1 and 4096x64x64 3.6 -> 3.4 gain
//                      least, 100x768x8192 9.3 -> 8.7 and 65x1000x8192 9.0 -> 11.8 lie beyond
//   int8, 32 columns:  512x1024x2048 7.6 -> 5.7, 200x2000x4096 12.8 -> 7.9, 4096x128x3072 9.6 -> 7.2, 64x8192x6144 16.3 -> 13.9;
//                      512x1024x128 3.5 -> 3.9 is the loss at the short end (one K tile of the 64 tile: from 256 bytes on)
//   binary16, the same bytes: within 2 % of the int8 times.
// A product whose maximum, codes or accumulators are wanted too stays on the tiles, whose epilogue has them: with the maximum
// 64x128x128 int8 3.7 us (here, without it, 3.3), 45x4096x1024 5.6 (3.9), 512x1024x2048 7.9 (5.7); binary16 1.2 to 2.1 times.
int rows_columns(const GemmProblem& p)
{
    const int64_t bytes = p.K * (p.prec / 8), rows = (p.M + 63) / 64;
    if(bytes > (p.M <= 32 ? 8192 : 6144)) return 0;
    if(rows * ((p.N + 15) / 16) <= (p.M <= 16 ? 2 * kRowsGroups : kRowsGroups)) return 1;
    return bytes > 256 && rows * ((p.N + 31) / 32) <= kRowsGroups ? 2 : 0;
}

}  // namespace

bool gemm_rows_takes(const GemmProblem& p)
{
    if((p.prec != 8 && p.prec != 16) || p.tn || p.conv_H > 0 || p.b_remap_C > 0 || p.acc_dump || p.out_amax_bits || p.out_codes) return false;
    return rows_columns(p) != 0;
}

hipError_t launch_gemm_rows(const GemmProblem& p, bool* taken, hipStream_t st)
{
    *taken = gemm_rows_takes(p);
    if(!*taken) return hipSuccess;
    const int columns = rows_columns(p);
    GemmKernelArgs a{};
    a.A = static_cast<const uint8_t*>(p.A);
    a.B = static_cast<const uint8_t*>(p.B);
    a.M = p.M; a.N = p.N; a.Kb = p.K * (p.prec / 8);
    a.C = p.C; a.c_is_f16 = p.c_dtype == kF16;
    a.s0 = p.s0; a.s1 = p.s1; a.col_scale = p.col_scale; a.col_bias = p.col_bias;
    return p.prec == 8 ? launch_rows<I8Traits>(a, columns, st) : launch_rows<F16Traits>(a, columns, st);
}

}  // namespace qsync
