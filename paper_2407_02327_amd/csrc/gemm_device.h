// What the matrix-instruction kernels share: operand types, kernel arguments, the walk over the tiles, direct loads to LDS, fragment
// reads with hand-placed waits, and the epilogue.
#pragma once
#include "device_utils.h"
#include "kernels.h"

#include <type_traits>
#include <utility>

namespace qsync {

namespace {

typedef int      v4i32 __attribute__((ext_vector_type(4)));
typedef int      v16i32 __attribute__((ext_vector_type(16)));
typedef float    v16f32 __attribute__((ext_vector_type(16)));
typedef float    v4f32 __attribute__((ext_vector_type(4)));
typedef _Float16 v8f16 __attribute__((ext_vector_type(8)));
typedef unsigned v4u32 __attribute__((ext_vector_type(4)));

constexpr int kRowBytes   = 128;  // K bytes per tile row and per LDS row
constexpr int kChunks     = 8;    // 16-byte chunks per LDS row
constexpr int kNumXcd     = 8;
constexpr int kNumCu      = 256;  // compute units of the target: one persistent workgroup each
constexpr int kGroupM     = 8;    // tile rows walked together (default; GemmKernelArgs::group_m)

// A fragment is kRows operand rows of 16 bytes a lane, 64 / kRows lanes side by side along K.  The products run on the instructions of
// 16 rows and columns: with operand values that vary, the chip lowers its clock for either shape, but less for these (nothing but
// matrix instructions, N(0,1) values, 32x32 -> 16x16: int8 3.5 -> 4.2 POP/s, binary16 1.67 -> 1.95 PFLOP/s; the same 4.9 and
// 2.45 on zeros), although they read twice the operand registers per operation.
struct I8Traits
{
    typedef int32_t acc_t;
    typedef v4i32   accv_t;
    static constexpr int kElemBytes = 1, kRows = 16;
    __device__ static __forceinline__ accv_t mfma(const v4i32& a, const v4i32& b, const accv_t& c)
    {
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
    }
};
struct F16Traits
{
    typedef float  acc_t;
    typedef v4f32  accv_t;
    static constexpr int kElemBytes = 2, kRows = 16;
    __device__ static __forceinline__ accv_t mfma(const v4i32& a, const v4i32& b, const accv_t& c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8f16, a), __builtin_bit_cast(v8f16, b), c, 0, 0, 0);
    }
};
// 32 rows and columns
struct I8Rows32
{
    typedef int32_t acc_t;
    typedef v16i32  accv_t;
    static constexpr int kElemBytes = 1, kRows = 32;
    __device__ static __forceinline__ accv_t mfma(const v4i32& a, const v4i32& b, const accv_t& c)
    {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
    }
};
struct F16Rows32
{
    typedef float  acc_t;
    typedef v16f32 accv_t;
    static constexpr int kElemBytes = 2, kRows = 32;
    __device__ static __forceinline__ accv_t mfma(const v4i32& a, const v4i32& b, const accv_t& c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8f16, a), __builtin_bit_cast(v8f16, b), c, 0, 0,
                                                      0);
    }
};

struct GemmKernelArgs
{
    const uint8_t* A;
    const uint8_t* B;
    int64_t        M, N;
    int64_t        Kb;           // bytes per operand row (K * element size), multiple of 16
    void*          C;
    int            c_is_f16;
    const float*   s0;
    const float*   s1;
    const float*   col_scale;
    const float*   col_bias;
    int32_t*       acc_dump;
    void*          partial;      // split-K: [splits][M][N] raw accumulators
    int            ktiles_per_split;
    int            tiles_m, tiles_n;
    int            group_m;      // tile rows that the tile walk keeps together (see item_of_block)
    int            conv_H, conv_W, conv_Cb;   // implicit 3x3 patch matrix: image height, width, bytes per pixel
    // B rows remapped (weight gradient of a 3x3 convolution): logical row (tap, c) = tap*remap_C + c is physical
    // row (tap%3)*remap_C + c of B, read with its K axis displaced by (tap/3 - 1)*remap_shift bytes
    int            remap_C, remap_shift;
    // optional: running maximum of |C| as stored (bit pattern of a non-negative fp32), raised with one atomic
    // maximum per workgroup
    unsigned int*  amax_bits;
    // optional: fixed-point codes of C as stored, clamp(round(C * code_inv[0]), -code_qmax, code_qmax), [M][N] int8
    int8_t*        codes;
    const float*   code_inv;
    int            code_qmax;
};

// A 64-bit value that is the same in every lane, as a pair of scalar registers.
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint64_t u = static_cast<uint64_t>(v);
    // (the builtin returns a signed int: widen each half through uint32_t, never by sign extension)
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(u))));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(u >> 32))));
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | static_cast<uint64_t>(lo));
}

// The lane's index, formed anew where it is asked for: behind a K loop that needs every register, what hangs on it does not have to
// be kept through the loop.
__device__ __forceinline__ int lane_again()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// Work item (K split, tile) of a workgroup.  Workgroups are dealt round-robin to the eight XCDs
// in launch order, each with its own L2, so XCD x takes the x-th contiguous eighth of the item
// list (split-major, tiles in grouped row-major order inside a split): the workgroups that share
// an L2 then read neighbouring operand panels, and with split K also the same K range.
__device__ __forceinline__ void item_of_block(int lin, int tiles_m, int tiles_n, int splits, int group_m, int& split,
                                              int& tm, int& tn)
{
    const int tiles = tiles_m * tiles_n, total = tiles * splits;
    const int per = total / kNumXcd, rem = total % kNumXcd;
    const int xcd = lin % kNumXcd, loc = lin / kNumXcd;
    const int item  = xcd * per + (xcd < rem ? xcd : rem) + loc;
    split           = item / tiles;
    const int L     = item - split * tiles;
    const int width = group_m * tiles_n;
    const int group = L / width, first = group * group_m;
    const int gsz   = (tiles_m - first) < group_m ? (tiles_m - first) : group_m;
    const int in    = L - group * width;
    // the divisions run on the vector unit; hand the (uniform) results back as scalars
    split = __builtin_amdgcn_readfirstlane(split);
    tm    = __builtin_amdgcn_readfirstlane(first + in % gsz);
    tn    = __builtin_amdgcn_readfirstlane(in / gsz);
}

// Output value a*s + b of the fused epilogues.  fp32: the fused multiply-add.  binary16: the same sum rounded ONCE
// to binary16, by the mixed-precision fused multiply-add (fp32 sources, binary16 result) -- written as an
// instruction so that every epilogue (per tile, persistent, reduction of K splits) produces the same bits from the same
// sum; left to the compiler, fmaf + conversion becomes that instruction in some places and a fp32 result converted afterwards
// (two roundings, different at binary16 ties) in others.
template <typename T> __device__ __forceinline__ T fma_out(float a, float s, float b);
template <> __device__ __forceinline__ float fma_out<float>(float a, float s, float b) { return fmaf(a, s, b); }
template <> __device__ __forceinline__ __half fma_out<__half>(float a, float s, float b)
{
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(s), "v"(b));
    return __ushort_as_half(static_cast<unsigned short>(r & 0xFFFFu));
}
// two of them packed in one word (first value in the low half)
__device__ __forceinline__ uint32_t fma_out_half2(float a0, float s0, float b0, float a1, float s1, float b1)
{
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3\n\tv_fma_mixhi_f16 %0, %4, %5, %6"
        : "=&v"(r) : "v"(a0), "v"(s0), "v"(b0), "v"(a1), "v"(s1), "v"(b1));
    return r;
}

// One direct global->LDS load of 16 bytes per lane.  D selects the wavefront's D-th 1 KB slot
// relative to the shared LDS base `lds_mid` (which points DPW/2 KB into the wavefront's slice).
// The hardware adds the instruction's immediate offset to the LDS address and to the global
// address alike.  The global address is formed as uniform base + 32-bit lane offset (scalar base
// addressing), so the K loop spends no vector instructions on addresses: `sbase` is the
// operand panel's address at this K tile minus kDmaBias, and `voff` already contains
// + kDmaBias - IMM.
constexpr int kDmaBias = 4096;
// A wavefront's DPW loads are issued in groups of at most 8 that share one LDS base (the immediate reaches
// +-4 KB); a wavefront with 16 loads per K tile changes the base once in between.
template <int DPW> constexpr int dma_group() { return DPW > 8 ? 8 : DPW; }
template <int D, int DPW> constexpr int dma_imm() { return (D % dma_group<DPW>() - dma_group<DPW>() / 2) * 1024; }   // -4096 .. 3072
template <int D, int DPW> constexpr int dma_lds_shift() { return (D / dma_group<DPW>()) * dma_group<DPW>() * 1024; }
template <int D, int DPW>
__device__ __forceinline__ void dma_issue(const uint8_t* sbase, uint32_t voff, uint8_t* lds_mid)
{
    constexpr int IMM = dma_imm<D, DPW>();
    static_assert(IMM >= -4096 && IMM <= 4095, "immediate offset out of range");
    asm volatile("" : "+v"(voff));      // keep the widening of the lane offset next to the load (scalar-base form)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(sbase + voff),
                                     (__attribute__((address_space(3))) void*)(lds_mid + dma_lds_shift<D, DPW>()), 16, IMM, 0);
}

// The same for one 4-byte column parameter per lane.
__device__ __forceinline__ void column_param_issue(const float* src, uint8_t* lds_dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)lds_dst, 4, 0, 0);
}

template <int DPW, int... Ds>
__device__ __forceinline__ void dma_sequence(std::integer_sequence<int, Ds...>, const uint8_t* sbase,
                                             const uint32_t (&voff)[DPW], uint8_t* lds_mid)
{
    (dma_issue<Ds, DPW>(sbase, voff[Ds], lds_mid), ...);
}

// Last, partial K tile: a chunk past the end of K is fetched from the row's first chunk instead
// (and overwritten with zeros once landed).
template <int DPW, int... Ds>
__device__ __forceinline__ void dma_sequence_tail(std::integer_sequence<int, Ds...>, const uint8_t* sbase,
                                                  const uint32_t (&voff)[DPW], const int (&gchunk)[2], int64_t kb,
                                                  int64_t Kb, uint8_t* lds_mid)
{
    (dma_issue<Ds, DPW>(sbase, voff[Ds] - ((kb + gchunk[Ds & 1] >= Kb) ? gchunk[Ds & 1] : 0), lds_mid), ...);
}

__device__ uint4 g_zero_chunk;     // never written: static storage starts at zero

__device__ const float g_one = 1.0f;     // stands in for an absent scale

template <int DPW, int... Ds>
__device__ __forceinline__ void fill_dma_imms(int (&imm)[DPW], std::integer_sequence<int, Ds...>)
{
    ((imm[Ds] = dma_imm<Ds, DPW>()), ...);
}

__device__ __forceinline__ int swizzle(int row, int chunk) { return (chunk ^ ((row >> 1) & 7)) << 4; }

// Maximum magnitude of the 16 output bytes in `v`, folded into `run`: binary16 magnitudes order like their bit
// patterns without the sign (two per dword), fp32 magnitudes likewise (one per dword).
typedef unsigned short gus2_t __attribute__((ext_vector_type(2)));
template <int OS> __device__ __forceinline__ uint32_t fold_abs_bits(uint32_t run, const v4u32& v)
{
#pragma unroll
    for(int k = 0; k < 4; ++k)
    {
        if(OS == 2)
            run = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(gus2_t, run),
                                                                         __builtin_bit_cast(gus2_t, v[k] & 0x7FFF7FFFu)));
        else
        {
            const uint32_t u = v[k] & 0x7FFFFFFFu;
            run = run > u ? run : u;
        }
    }
    return run;
}
// the folded maximum as the bit pattern of an fp32
template <int OS> __device__ __forceinline__ uint32_t abs_bits_as_f32(uint32_t run)
{
    if(OS == 4) return run;
    const uint32_t h = (run & 0xFFFFu) > (run >> 16) ? (run & 0xFFFFu) : (run >> 16);
    return __float_as_uint(__half2float(__ushort_as_half(static_cast<unsigned short>(h))));
}

// One 16-byte LDS read per fragment, as explicit instructions (the waits are placed by hand in the K loop); OFF is the
// instruction's immediate byte offset (16 bits).
template <int OFF>
__device__ __forceinline__ void frag_read(v4i32& dst, uint32_t addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "immediate offset");
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}
// at most N of this wavefront's LDS operations still in flight (other counters untouched).  The counter holds 15, so a wait for more
// than 14 is one for 14, which also tells a full counter from one that is not.
template <int N> __device__ __forceinline__ void wait_lds()
{
    __builtin_amdgcn_s_waitcnt(0xC07F | ((N < 14 ? N : 14) << 8));
}
typedef unsigned v2u32 __attribute__((ext_vector_type(2)));
// compile-time loop: f(std::integral_constant<int, 0>), ..., f(std::integral_constant<int, N - 1>)
template <typename F, int... Is> __device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}
// Transposing 8-byte reads, sixteen lanes at a time.  ESZ 1: the lanes read 8 rows x 16 bytes (lane s: half s%2 of
// row s/2) and lane j receives the eight bytes of column j.  ESZ 2: they read 4 rows x 32 bytes (lane s: quarter
// s%4 of row s/4) and lane j receives the four 16-bit elements of column j.
template <int ESZ, int OFF> __device__ __forceinline__ void frag_read_tr(v2u32& dst, uint32_t addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "immediate offset");
    if constexpr(ESZ == 1)
        asm volatile("ds_read_b64_tr_b8 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
    else
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}
// XOR term (in 16-byte chunks) of stage row `row` of a TN operand region whose rows are RB bytes long: the rows that one pass of a
// transposing read touches (32 lanes: 8 rows and the 8 rows 16 further down x 16 bytes for ESZ 1; 4 rows and the 4 rows 8
// further down x 32 bytes for ESZ 2) land in different bank groups.  Unchanged by the row steps between the reads of one lane
// (8 and multiples of 64 rows, resp. 4 and multiples of 32).
template <int ESZ, int RB> __device__ __forceinline__ int tn_swizzle(int row)
{
    constexpr int CPR = RB / 16;                                    // chunks per row
    if constexpr(ESZ == 1)
    {
        constexpr int L = CPR == 16 ? 0 : CPR == 8 ? 1 : 2;         // rows that share 256 bytes, as a power of two
        static_assert(CPR == 16 || CPR == 8 || CPR == 4, "rows of 64 to 256 bytes");
        return ((row & 7) >> L) | (((row >> 4) & 1) << (3 - L));
    }
    else
    {
        constexpr int L = CPR >= 16 ? 0 : 1;
        static_assert(CPR == 32 || CPR == 16 || CPR == 8, "rows of 128 to 512 bytes");
        return 2 * (((row & 3) >> L) | (((row >> 3) & 1) << (2 - L)));
    }
}
// Workgroup barrier behind a wait for this wavefront's LDS operations only (the compiler's __syncthreads would also
// wait for every vector-memory operation in flight, i.e. drain the queue of direct loads).
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// at most N of this wavefront's vector-memory operations still in flight
template <int N> __device__ __forceinline__ void wait_direct_loads()
{
    static_assert(N >= 0 && N <= 63, "the vector-memory counter holds 63");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// the direct loads of at most min(n, N) K tiles (DPW instructions each) still in flight
template <int DPW, int N> __device__ __forceinline__ void wait_tiles(int n)
{
    if constexpr(N == 0) wait_direct_loads<0>();
    else if(n >= N)      wait_direct_loads<N * DPW>();
    else                 wait_tiles<DPW, N - 1>(n);
}
__device__ __forceinline__ void lds_write_b32(uint32_t addr, uint32_t v) { asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory"); }

// Epilogue: a workgroup's accumulators to memory.  The B fragment is the matrix instruction's first operand, so a lane holds
// C^T fragments: lane -> output row m = lane%R of the fragment (R = 16 or 32 rows); register v -> output column n = 8*(v/4) +
// 4*(lane/R) + v%4, i.e. four consecutive columns per register quad (one quad for 16 rows).  `lds`: STG_BYTES per wavefront that nobody reads any more behind the
// first barrier here; `colp`: column scales and biases [2][BN], maximum slots behind them.
template <typename TR, int BM, int BN, int WGM, int WGN, int STG_BYTES, bool SPLIT>
__device__ __forceinline__ void store_tile(const GemmKernelArgs& p, typename TR::accv_t (&acc)[BM / WGM / TR::kRows][BN / WGN / TR::kRows], uint8_t* lds,
                                           float* colp, int64_t m0, int64_t n0, int split, float alpha, float code_inv, uint32_t amax_seen)
{
    typedef typename TR::accv_t accv_t;
    typedef typename TR::acc_t  acc_t;
    constexpr int R = TR::kRows, WTM = BM / WGM, WTN = BN / WGN, FM = WTM / R, FN = WTN / R, QUADS = R == 32 ? 4 : 1;
    // (the kernels of 32 rows have registers for the lane's index: formed anew, binary16 convolution 296->24 over 10x17x10 14.2 -> 14.6 us)
    const int lane = R == 32 ? static_cast<int>(threadIdx.x) % kWaveSize : lane_again(), wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWaveSize);
    const int wm = wave / WGN, wn = wave % WGN, frag_row = lane % R, cquad = lane / R;
    const int64_t wrow0 = m0 + wm * WTM, wcol0 = n0 + wn * WTN;
    // Staged stores: pass the wavefront's sub-tile through its private slice of LDS (the K
    // pipeline is drained, so the stages are free) and leave with 16-byte stores whose lanes run
    // along the rows of the destination: every store instruction writes whole 128-byte (or
    // longer) row segments.  RAW writes the accumulators themselves (split-K partials); otherwise
    // they are dequantized in registers first.
    uint8_t*      stg       = lds + wave * STG_BYTES;
    uint32_t out_run = 0u;     // running maximum of |C| of this lane (packed like the output type)
    // one atomic maximum per workgroup at most: lanes -> wavefront (shuffles) -> workgroup (LDS slots behind the
    // column parameters).  Atomics on one word retire about 10 ns apart, so a workgroup skips its own when the
    // word, as read in front of the stores (`amax_seen`: possibly stale, never too large), already covers it.
    auto publish_amax = [&](uint32_t bits_f32) {
#pragma unroll
        for(int off = 32; off >= 1; off >>= 1)
        {
            const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(bits_f32), off));
            bits_f32 = bits_f32 > o ? bits_f32 : o;
        }
        uint32_t* slots = reinterpret_cast<uint32_t*>(colp + 2 * BN);
        if(lane == 0) slots[wave] = bits_f32;
        __syncthreads();
        if(wave == 0 && lane == 0)
        {
            uint32_t m = slots[0];
#pragma unroll
            for(int w = 1; w < WGM * WGN; ++w) m = m > slots[w] ? m : slots[w];
            if(m > amax_seen) atomicMax(p.amax_bits, m);
        }
    };
    // The code of this epilogue runs once per tile, so its length counts as much as its operations: instructions that
    // are not in the instruction cache are fetched while every wavefront waits.  Converting is unrolled (accumulator
    // registers cannot be indexed) but lean: 8 vector operations and one LDS write per four outputs, the column
    // parameters of a fragment column read once for all its rows.  Everything optional (odd N or alignment, maximum,
    // codes, accumulator dump) sits in the short store loop behind it and works on the staged values, instead of in
    // unrolled copies per option, which made 15 000 instructions per kernel.  Measured, unrolled copies -> this form:
    // 16384x4096x1024 int8 on the 256 tile 86.7 -> 82.6 us, 4096x3072x768 18.3 -> 17.2, 512^3 on the 128 tile
    // 7.3 -> 6.5, an odd N (2056x1001x1040, element stores) 40.7 -> 29.5 us.
    auto staged_store = [&](auto out_tag, auto raw_tag, uint8_t* dst_base) {
        typedef decltype(out_tag) out_t;
        constexpr bool RAW   = decltype(raw_tag)::value;
        constexpr int  OS    = sizeof(out_t);
        constexpr int  PITCH = WTN * OS + 16;                    // padded row pitch in the staging slice
        constexpr int  FITS  = STG_BYTES / (R * PITCH);
        constexpr int  FPP   = FITS >= FM ? FM : FITS >= 4 && FM % 4 == 0 ? 4 : FITS >= 2 && FM % 2 == 0 ? 2 : 1;      // row fragments per pass
        static_assert(R * PITCH <= STG_BYTES && FM % FPP == 0, "staging slice too small");
        constexpr int EPV = 16 / OS;                             // elements per 16-byte vector
        constexpr int LPR = WTN / EPV;                           // lanes per output row in the store phase
        constexpr int RPI = 64 / LPR;                            // rows per store instruction
        static_assert(64 % LPR == 0 && (FPP * R) % RPI == 0, "store instructions cover whole rows");
        const bool    vec = (p.N * OS) % 16 == 0 && (reinterpret_cast<uintptr_t>(dst_base) & 15) == 0;
        const int     seg = lane % LPR, lr0 = lane / LPR;
        const int64_t col = wcol0 + seg * EPV;
        __syncthreads();                                  // all wavefronts are done reading the stages
#pragma unroll
        for(int pass = 0; pass < FM / FPP; ++pass)
        {
#pragma unroll
            for(int j = 0; j < FN; ++j)
            {
                float4 fs[QUADS], bs[QUADS];                      // scale and bias of the lane's columns (alpha * column scale, as one product)
                if constexpr(!RAW)
#pragma unroll
                    for(int vq = 0; vq < QUADS; ++vq)
                    {
                        const int c = wn * WTN + j * R + 8 * vq + 4 * cquad;          // column inside the tile
                        const float4 cs = *reinterpret_cast<const float4*>(colp + c);
                        const float4 cb = *reinterpret_cast<const float4*>(colp + BN + c);
                        fs[vq] = p.col_scale ? make_float4(alpha * cs.x, alpha * cs.y, alpha * cs.z, alpha * cs.w)
                                             : make_float4(alpha, alpha, alpha, alpha);
                        bs[vq] = p.col_bias ? cb : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    }
#pragma unroll
                for(int ii = 0; ii < FPP; ++ii)
#pragma unroll
                    for(int vq = 0; vq < QUADS; ++vq)
                    {
                        const accv_t& a   = acc[pass * FPP + ii][j];
                        uint8_t*      dst = stg + (ii * R + frag_row) * PITCH + (j * R + 8 * vq + 4 * cquad) * OS;
                        if constexpr(RAW)
                        {
                            const out_t o[4] = {a[vq * 4], a[vq * 4 + 1], a[vq * 4 + 2], a[vq * 4 + 3]};
                            *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(o);
                        }
                        else
                        {
                            const float a0 = static_cast<float>(a[vq * 4]), a1 = static_cast<float>(a[vq * 4 + 1]);
                            const float a2 = static_cast<float>(a[vq * 4 + 2]), a3 = static_cast<float>(a[vq * 4 + 3]);
                            const float4 f = fs[vq], b = bs[vq];
                            if constexpr(OS == 2)
                                *reinterpret_cast<uint2*>(dst) = make_uint2(fma_out_half2(a0, f.x, b.x, a1, f.y, b.y),
                                                                            fma_out_half2(a2, f.z, b.z, a3, f.w, b.w));
                            else
                                *reinterpret_cast<float4*>(dst) = make_float4(fmaf(a0, f.x, b.x), fmaf(a1, f.y, b.y),
                                                                              fmaf(a2, f.z, b.z), fmaf(a3, f.w, b.w));
                        }
                    }
            }
            // Lanes read what other lanes of the wavefront have just written: the hardware keeps a
            // wavefront's LDS operations in order, and the wavefront-scope fence tells the compiler
            // that these loads may not be satisfied from values a lane has seen before.
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            const int64_t row0 = wrow0 + pass * FPP * R + lr0;
            if constexpr(!RAW)
                if(vec && p.codes && (reinterpret_cast<uintptr_t>(p.codes) & (EPV - 1)) == 0)
                {   // C and its codes as vectors (with the quantizer's arithmetic: one fp32 multiply, ties to even, clamp)
#pragma unroll 2
                    for(int r = 0; r < FPP * R; r += RPI)
                    {
                        const v4u32 val = *reinterpret_cast<const v4u32*>(stg + (r + lr0) * PITCH + seg * 16);
                        uint32_t    cw[EPV / 4];
#pragma unroll
                        for(int g = 0; g < EPV / 4; ++g) cw[g] = 0u;
#pragma unroll
                        for(int e = 0; e < EPV; ++e)
                        {
                            const uint32_t word   = OS == 2 ? (e % 2 ? val[e / 2] >> 16 : val[e / 2] & 0xFFFFu) : val[e % 4];
                            const float    stored = OS == 2 ? __half2float(__ushort_as_half(static_cast<unsigned short>(word))) : __uint_as_float(word);
                            cw[e / 4] |= (static_cast<uint32_t>(quantize_code<kNearest>(stored, code_inv, p.code_qmax, 0u)) & 0xFFu) << (8 * (e % 4));
                        }
                        const int64_t at = (row0 + r) * p.N + col;
                        if(row0 + r < p.M && col < p.N)
                        {
                            out_run = fold_abs_bits<OS>(out_run, val);
                            __builtin_nontemporal_store(val, reinterpret_cast<v4u32*>(dst_base + at * OS));
                            // (read next by the consumer's GEMM: ordinary store)
                            if constexpr(EPV == 8) *reinterpret_cast<uint2*>(p.codes + at) = make_uint2(cw[0], cw[EPV / 4 - 1]);
                            else                   *reinterpret_cast<uint32_t*>(p.codes + at) = cw[0];
                        }
                    }
                    continue;
                }
            if(vec && (RAW || !p.codes))
            {
                uint8_t* dst = dst_base + (row0 * p.N + col) * OS;
                const int64_t step = RPI * p.N * OS;
#pragma unroll
                for(int r = 0; r < FPP * R; r += RPI, dst += step)
                {
                    const v4u32 val = *reinterpret_cast<const v4u32*>(stg + (r + lr0) * PITCH + seg * 16);
                    if(row0 + r < p.M && col < p.N)
                    {
                        if constexpr(!RAW)
                            if(p.amax_bits) out_run = fold_abs_bits<OS>(out_run, val);
                        if constexpr(RAW)
                            *reinterpret_cast<v4u32*>(dst) = val;      // read back soon by the reduction: ordinary store
                        else                 // streaming store: C is not read again here, keep the operand panels in L2
                            __builtin_nontemporal_store(val, reinterpret_cast<v4u32*>(dst));
                    }
                }
                continue;
            }
#pragma unroll 1
            for(int r = 0; r < FPP * R; r += RPI)
            {
                const v4u32   val = *reinterpret_cast<const v4u32*>(stg + (r + lr0) * PITCH + seg * 16);
                const int64_t row = row0 + r, left = row < p.M ? p.N - col : 0;      // valid elements from here on (may be <= 0)
                const int64_t at  = row * p.N + col;
#pragma unroll
                for(int e = 0; e < EPV; ++e)
                {
                    const uint32_t word = OS == 2 ? (e % 2 ? val[e / 2] >> 16 : val[e / 2] & 0xFFFFu) : val[e % 4];
                    if(e >= left) continue;
                    if constexpr(OS == 2)
                        reinterpret_cast<uint16_t*>(dst_base)[at + e] = static_cast<uint16_t>(word);
                    else
                        reinterpret_cast<uint32_t*>(dst_base)[at + e] = word;
                    if constexpr(!RAW)
                    {   // maximum and codes: of the values as stored, with the quantizer's arithmetic (one fp32 multiply,
                        // ties to even, clamp)
                        const uint32_t mag = word & (OS == 2 ? 0x7FFFu : 0x7FFFFFFFu);
                        out_run = out_run > mag ? out_run : mag;
                        if(p.codes)
                        {
                            const float stored = OS == 2 ? __half2float(__ushort_as_half(static_cast<unsigned short>(word))) : __uint_as_float(word);
                            p.codes[at + e] = static_cast<int8_t>(quantize_code<kNearest>(stored, code_inv, p.code_qmax, 0u));
                        }
                    }
                }
            }
        }
    };

    if(SPLIT)
    {
        staged_store(acc_t{}, std::true_type{},
                     reinterpret_cast<uint8_t*>(static_cast<acc_t*>(p.partial) + static_cast<int64_t>(split) * p.M * p.N));
        return;
    }
    if constexpr(std::is_same<acc_t, int32_t>::value)
        if(p.acc_dump) staged_store(acc_t{}, std::true_type{}, reinterpret_cast<uint8_t*>(p.acc_dump));
    if(p.c_is_f16)
    {
        staged_store(__half{}, std::false_type{}, static_cast<uint8_t*>(p.C));
        if(p.amax_bits) publish_amax(abs_bits_as_f32<2>(out_run));
    }
    else
    {
        staged_store(float{}, std::false_type{}, static_cast<uint8_t*>(p.C));
        if(p.amax_bits) publish_amax(abs_bits_as_f32<4>(out_run));
    }
}

}  // namespace

}  // namespace qsync
