// FP32 GEMM:  C[M,N] = epilogue( sum_k A[m,k] B[n,k] ), fp32 operands of any row length, on the bf16 matrix instructions.
//
// An fp32 value is the exact sum of three bf16 values: the nearest one, the nearest one to what remains, and the rest.  The second is at
// most 2^-8 of the value, the third 2^-17.  Of the nine products of two such sums the six largest are added up in fp32, smallest first;
// what is left out is up to 2^-24 of a product (2^-26.8 in the mean square over random mantissas), and of one sign where all products of a
// sum are alike.  (With a first part that is cut off instead it was up to 2^-22, at the same time.)  Six bf16 instructions of 16x16x32 take
// 96 clocks where the eight fp32 ones of 16x16x4 take 256, and
// fewer roundings fall on the sum: an instruction adds 32 products to it, not four.  It cuts off what it shifts out, though, so that a sum
// comes out -1 to 1/2 ulp off, -1/4 on average (measured), where the fp32 instructions round to nearest.  Error against 64 bits in
// the 2-norm, fp32 instructions -> this, values N(0,1): K 24 0.89e-7 -> 0.36e-7, 33 1.04e-7 -> 0.65e-7, 64 1.44e-7 -> 0.92e-7, 256 2.9e-7 ->
// 2.3e-7, 1024 5.7e-7 -> 4.8e-7, 4096 1.14e-6 -> 1.00e-6, without the sums in parts of the smaller tiles, which halve it (2.4e-7 at 1024
// and 2048); products all positive 0.71e-7 -> 0.26e-7 at 24, 2.4e-7 -> 1.6e-7 at 256, all equal 1.66e-7 -> 0.30e-7 and 1.9e-6 -> 0.6e-6.
// Over 120 drawn products 1.5 times smaller on average, at most 1.05 times larger (832x2696x2096, once on the small tile in splits,
// now on the large).  What grows is the error of a sum that rounds little on the fp32 instructions: of up to 16 products (one: 2.5e-8 -> 3.6e-8), which
// therefore stay on those (kF32ShortK), and of longer ones of one product other than zero (at most 1/2 -> 1.4 ulp).
//
// Bound by the matrix instructions, power and the splitting's share of the issue slots: a K tile of 32 takes the 256x128 tile 1.75 us where
// its instructions take 1.28 at 2.4 GHz (1.60 without the splitting, 1.68 without its LDS writes).  Operands go through registers, split
// once a workgroup: each wavefront splitting its own fragments would repeat that two to four times.  fp32 instructions (16-byte rows
// direct to LDS; others through registers) -> this, us: 8192x4096x1024 490 -> 306, 8192x1024x4096 479 -> 286, 4096x1024x8192 490 -> 300,
// 2048^3 132 -> 87, 1000x1000x1001 36 -> 23, 1024^3 23.2 -> 23.4, 512^3 12.1 -> 10.5; over 142 shapes of 64..8192 by 64..4096 by 17..4096
// 1.12 times faster on average; slower are some small ones of up to 100 and rows of fours (by 0.2 us, 503x73x36 5.1 -> 5.5) and large
// outputs of few products for which the plan takes a larger tile than is best (3708x3160x29 23.7 -> 25.3).  40 operator steps 1.12 times
// faster (0.97 to 1.49).
// A remainder behind whole K tiles is loaded like those, as the row's last 32 floats; behind them and float by float, its loads were waited for
// (263x343x80 6.8 -> 6.0 us, 7167x311x43 12.9 -> 10.1; alone, in fours: 3289x72x31 5.4 -> 4.8).
#include "gemm_device.h"

namespace qsync {

namespace {

struct F32Split
{
    typedef float acc_t;
    typedef v4f32 accv_t;
    static constexpr int kElemBytes = 4, kRows = 16;
};
typedef __bf16 v8bf16 __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf16 __attribute__((ext_vector_type(2)));
typedef float  v2f32 __attribute__((ext_vector_type(2)));
typedef float  v4f32_any __attribute__((ext_vector_type(4), aligned(4)));     // 16 bytes of a row that starts on any float

constexpr int kStepK    = kRowBytes / 4;     // floats a K tile: one matrix instruction deep
// LDS bytes of one part of 16 rows, in the order of the instruction's operand: row r, K indices 8 q to 8 q + 7 at 16 bytes times
// (r ^ 2 q) + 16 q.  Reads and writes are free of bank conflicts (with r ^ 4 q half of the LDS cycles were conflicts, 8192x1024x4096 303 -> 300 us).
constexpr int kPlane    = 1024;
constexpr int kFragment = 3 * kPlane;

template <int BM, int BN> constexpr int f32_lds_bytes() { return 2 * (BM + BN) / 16 * kFragment + 2 * BN * 4 + 128; }

// Two values as three pairs of bf16 parts.  `rest` collects the bits behind the third part's: none, down to 2^-110.  A part of anything
// smaller may have bits below 2^-133, the smallest bf16 number, and loses those.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t mask, uint32_t& hi, uint32_t& mid, uint32_t& lo, uint32_t& rest)
{
    hi             = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f32){x0, x1}, v2bf16));
    const float r0 = x0 - __uint_as_float(hi << 16), r1 = x1 - __uint_as_float(hi & mask);
    mid            = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f32){r0, r1}, v2bf16));
    const float    s0 = r0 - __uint_as_float(mid << 16), s1 = r1 - __uint_as_float(mid & mask);
    const uint32_t u0 = __float_as_uint(s0), u1 = __float_as_uint(s1);
    lo   = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
    asm volatile("v_or3_b32 %0, %0, %1, %2" : "+v"(rest) : "v"(u0), "v"(u1));      // (here: gathered up later, both would stay in registers)
}

template <int BM, int BN, int WGM, int WGN, int D, bool SPLIT>
__global__ __launch_bounds__(64 * WGM * WGN, 2) void gemm_f32_kernel(const GemmKernelArgs p, int64_t K, int splits)
{
    constexpr int kThreads = 64 * WGM * WGN, FM = BM / WGM / 16, FN = BN / WGN / 16;
    constexpr int kStage = (BM + BN) / 16 * kFragment;
    // sums of so many K tiles are added up apart where there are registers for both (fewer roundings fall on a long sum)
    constexpr bool kFold = D > 1;
    constexpr int  kFoldSteps = 8;
    constexpr int U = (BM + BN) * 4 / kThreads, kUnitRows = kThreads / 4;      // pieces of eight floats that a thread brings to a stage
    static_assert((BM + BN) * 4 % kThreads == 0 && BM % kUnitRows == 0 && BN % kUnitRows == 0, "a thread's piece is of A or of B in every thread");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    float* const    colp  = reinterpret_cast<float*>(lds + 2 * kStage);        // [2][BN], eight slots of the maximum, eight flags
    uint32_t* const flags = reinterpret_cast<uint32_t*>(colp + 2 * BN) + 16;
    const int       tid = threadIdx.x, lane = tid % kWaveSize, wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
    const int       wm = wave / WGN, wn = wave % WGN, q = lane / 16, fr = lane % 16;
    int             which, tm, tn;
    item_of_block(static_cast<int>(blockIdx.x), p.tiles_m, p.tiles_n, SPLIT ? splits : 1, p.group_m, which, tm, tn);
    const int64_t  m0 = static_cast<int64_t>(tm) * BM, n0 = static_cast<int64_t>(tn) * BN;
    const int64_t  first = static_cast<int64_t>(which) * p.ktiles_per_split * kStepK;
    const int64_t  end   = SPLIT && first + static_cast<int64_t>(p.ktiles_per_split) * kStepK < K ? first + static_cast<int64_t>(p.ktiles_per_split) * kStepK : K;
    const int      tiles = end > first ? static_cast<int>((end - first + kStepK - 1) / kStepK) : 0;
    const float    alpha = *(p.s0 ? p.s0 : &g_one) * *(p.s1 ? p.s1 : &g_one);
    const float    code_inv = *(!SPLIT && p.codes ? p.code_inv : &g_one);
    static_assert(BN <= kThreads, "a column's parameters to a thread");
    float scale = 1.0f, bias = 0.0f;      // of column n0 + tid
    if constexpr(!SPLIT)
    {
        const int64_t n = n0 + tid < p.N ? n0 + tid : p.N - 1;
        if(p.col_scale) scale = p.col_scale[n];
        if(p.col_bias) bias = p.col_bias[n];
    }

    // rows past the last one load that row again (their outputs are never stored); K indices past the end give zeros
    const float* const A = reinterpret_cast<const float*>(p.A);
    const float* const B = reinterpret_cast<const float*>(p.B);
    const float *      row[U], *src[U];
    uint32_t           put_at[U];
#pragma unroll
    for(int i = 0; i < U; ++i)
    {
        const int     line = tid / 4 + i * kUnitRows, g = tid % 4;
        const bool    is_a = i * kUnitRows < BM;
        const int64_t at = is_a ? m0 + line : n0 + line - BM, last = (is_a ? p.M : p.N) - 1;
        row[i]    = (is_a ? A : B) + (at < last ? at : last) * K;
        src[i]    = row[i] + first + 8 * g;
        put_at[i] = static_cast<uint32_t>(line / 16 * kFragment + ((line % 16 ^ 2 * g) + 16 * g) * 16);
    }
    // whole K tiles, D of them on their way in registers; behind them the partial one that ends the row, as the row's last 32 floats
    // (those that the tile before has already are taken as zeros); behind the last one it is loaded again (and not looked at)
    const int whole = tiles > 0 ? static_cast<int>((end - first) / kStepK) : 0, tail = tiles > whole ? static_cast<int>((end - first) % kStepK) : 0;
    float     raw[D][U][8];
    uint32_t  rest[U], mask = 0xFFFF0000u;      // (the rest of a row's values: a piece stays in its row)
#pragma unroll
    for(int i = 0; i < U; ++i) rest[i] = 0u;
    asm volatile("" : "+s"(mask));      // (a scalar register: the instructions that use it are half as long)
    auto load = [&](auto set, int i, int t) {
        const v4f32_any lo = *reinterpret_cast<const v4f32_any*>(src[i]), hi = *reinterpret_cast<const v4f32_any*>(src[i] + 4);
#pragma unroll
        for(int e = 0; e < 4; ++e) { raw[decltype(set)::value][i][e] = lo[e]; raw[decltype(set)::value][i][4 + e] = hi[e]; }
        src[i] += t + 1 < whole ? kStepK : (t + 1 == whole ? tail : 0);
    };
    auto take_tail = [&]() __attribute__((always_inline)) {      // (into the first set)
        static_assert(D <= 2);
        const int  had = kStepK - tail - 8 * (tid % 4);
        const bool odd = whole % D != 0;
#pragma unroll
        for(int i = 0; i < U; ++i)
#pragma unroll
            for(int e = 0; e < 8; ++e)
            {
                const float even = raw[0][i][e], other = raw[D - 1][i][e];
                raw[0][i][e] = e < had ? 0.0f : (odd ? other : even);
            }
    };
    // A partial tile that is all there is (of more than kF32ShortK floats): in fours, the last of which ends with the row.
    auto load_tail = [&]() __attribute__((always_inline)) {
        const int k0 = static_cast<int>(first) + 8 * (tid % 4), ends = static_cast<int>(end), last = static_cast<int>(K) - 4;
#pragma unroll
        for(int i = 0; i < U; ++i)
#pragma unroll
            for(int h = 0; h < 8; h += 4)
            {
                const int from = k0 + h < last ? k0 + h : last, by = k0 + h - from;      // (by four and more: nothing left)
                v4f32     v    = *reinterpret_cast<const v4f32_any*>(row[i] + from);
                v = by & 1 ? v4f32{v[1], v[2], v[3], 0.0f} : v;
                v = by & 2 ? v4f32{v[2], v[3], 0.0f, 0.0f} : v;
#pragma unroll
                for(int e = 0; e < 4; ++e) raw[0][i][h + e] = k0 + h + e < ends ? v[e] : 0.0f;
            }
    };
    v4u32 part[3];
    auto split = [&](auto set, int i, int e) {
        uint32_t hi, mid, lo;
        split2(raw[decltype(set)::value][i][2 * e], raw[decltype(set)::value][i][2 * e + 1], mask, hi, mid, lo, rest[i]);
        part[0][e] = hi; part[1][e] = mid; part[2][e] = lo;
    };
    auto put = [&](int i, int t) {
        uint8_t* dst = lds + (t & 1) * kStage + put_at[i];
#pragma unroll
        for(int s = 0; s < 3; ++s) *reinterpret_cast<v4u32*>(dst + s * kPlane) = part[s];
    };
    v4f32 acc[FM][FN];
#pragma unroll
    for(int i = 0; i < FM; ++i)
#pragma unroll
        for(int j = 0; j < FN; ++j) acc[i][j] = v4f32{0.0f, 0.0f, 0.0f, 0.0f};
    v4f32 total[kFold ? FM : 1][kFold ? FN : 1];
    if constexpr(kFold)
#pragma unroll
        for(int i = 0; i < FM; ++i)
#pragma unroll
            for(int j = 0; j < FN; ++j) total[i][j] = v4f32{0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t read_at = static_cast<uint32_t>(((fr ^ 2 * q) + 16 * q) * 16);
    // The products of a row of fragments, smallest parts first; a column part's registers are free again for the next K tile behind
    // the last row's 1st, 3rd and 6th.
    constexpr int kA[6] = {0, 1, 0, 2, 1, 0}, kB[6] = {2, 1, 1, 0, 0, 0};
    constexpr int kSlots = 6 * FM, kMeet = kSlots - 6, kPer = (kMeet - 2) / U;
    v8bf16        b[FN][3], a[2][3];
    auto read_b = [&](auto s, const uint8_t* stage) {
#pragma unroll
        for(int j = 0; j < FN; ++j) b[j][decltype(s)::value] = *reinterpret_cast<const v8bf16*>(stage + read_at + (BM / 16 + wn * FN + j) * kFragment + decltype(s)::value * kPlane);
    };
    auto read_a = [&](auto i, auto s, const uint8_t* stage) {
        a[decltype(i)::value % 2][decltype(s)::value] = *reinterpret_cast<const v8bf16*>(stage + read_at + (wm * FM + decltype(i)::value) * kFragment + decltype(s)::value * kPlane);
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    // One K tile's products.  Between those of all rows but the last: the next tile's parts into the other stage, the loads of a later one,
    // of a piece as soon as its registers are free, and the next row's fragments.  Then the workgroup meets, and between the last
    // row's products the next tile's first fragments are read.
    enum { kAll, kNoLoads, kLast };
    auto step = [&](auto mode, auto set, int t) __attribute__((always_inline)) {
        constexpr int        MODE = decltype(mode)::value;
        const uint8_t* const cur = lds + (t & 1) * kStage;
        const uint8_t* const nxt = lds + (~t & 1) * kStage;
        read_b(c0, cur);
        static_for<kSlots>([&](auto slot) {
            constexpr int sl = decltype(slot)::value, i = sl / 6, s = sl % 6, u = sl / kPer, at = sl % kPer;
            if constexpr(sl == kMeet && MODE != kLast) wg_barrier();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for(int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][kB[s]], a[i % 2][kA[s]], acc[i][j], 0, 0, 0);
            if constexpr(i + 1 < FM && s < 3) read_a(std::integral_constant<int, i + 1>{}, std::integral_constant<int, s>{}, cur);
            if constexpr(u < U && MODE != kLast)
            {
                static_for<4>([&](auto e) {
                    if constexpr(decltype(e)::value * kPer / 4 == at) split(set, u, decltype(e)::value);
                });
                if constexpr(at == kPer - 1)
                {
                    put(u, t + 1);
                    if constexpr(MODE == kAll) load(set, u, t + 1 + D);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr(MODE != kLast)
            {
                if constexpr(sl == kMeet) { read_a(c0, c0, nxt); read_b(c2, nxt); }
                if constexpr(sl == kMeet + 1) read_a(c0, c1, nxt);
                if constexpr(sl == kMeet + 2) { read_b(c1, nxt); read_a(c0, c2, nxt); }
            }
        });
    };
    auto put_first = [&]() __attribute__((always_inline)) {
#pragma unroll
        for(int i = 0; i < U; ++i)
        {
#pragma unroll
            for(int e = 0; e < 4; ++e) split(c0, i, e);
            put(i, 0);
            if(whole > 0) load(c0, i, D);
            __builtin_amdgcn_sched_barrier(0);
        }
        wg_barrier();
        read_a(c0, c0, lds);
        read_b(c2, lds);
        read_a(c0, c1, lds);
        read_b(c1, lds);
        read_a(c0, c2, lds);
    };
    constexpr std::integral_constant<int, kAll>     all{};
    constexpr std::integral_constant<int, kNoLoads> no_loads{};
    constexpr std::integral_constant<int, kLast>    last_one{};
    // ---- on the fp32 instructions, operands straight from memory: a lane's four K indices of sixteen, of both operands in the same order
    struct Piece { v4f32 a[FM], b[FN]; };
    const float *ra[FM], *rb[FN];
    uint32_t     redo = 0u;      // bit i: the wavefront's sums of rows 16 i and on
    auto point = [&]() {
#pragma unroll
        for(int i = 0; i < FM; ++i)
        {
            const int64_t at = m0 + wm * (BM / WGM) + 16 * i + fr;
            ra[i] = A + (at < p.M ? at : p.M - 1) * K + 4 * q;
        }
#pragma unroll
        for(int j = 0; j < FN; ++j)
        {
            const int64_t at = n0 + wn * (BN / WGN) + 16 * j + fr;
            rb[j] = B + (at < p.N ? at : p.N - 1) * K + 4 * q;
        }
    };
    auto fetch = [&](auto every, Piece& v, int64_t k) {      // (K indices behind the end give zeros)
        const int left = static_cast<int>(end - k) - 4 * q;
#pragma unroll
        for(int i = 0; i < FM; ++i) v.a[i] = v4f32{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for(int j = 0; j < FN; ++j) v.b[j] = v4f32{0.0f, 0.0f, 0.0f, 0.0f};
        if(left >= 4)
        {
#pragma unroll
            for(int i = 0; i < FM; ++i)
                if(decltype(every)::value || redo >> i & 1u) v.a[i] = *reinterpret_cast<const v4f32_any*>(ra[i] + k);
#pragma unroll
            for(int j = 0; j < FN; ++j) v.b[j] = *reinterpret_cast<const v4f32_any*>(rb[j] + k);
        }
        else
#pragma unroll
            for(int e = 0; e < 3; ++e)
                if(e < left)
                {
#pragma unroll
                    for(int i = 0; i < FM; ++i) v.a[i][e] = ra[i][k + e];
#pragma unroll
                    for(int j = 0; j < FN; ++j) v.b[j][e] = rb[j][k + e];
                }
    };
    auto products = [&](auto every, const Piece& v) {
#pragma unroll
        for(int i = 0; i < FM; ++i)
            if(decltype(every)::value || redo >> i & 1u)
#pragma unroll
                for(int e = 0; e < 4; ++e)
#pragma unroll
                    for(int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v.b[j][e], v.a[i][e], acc[i][j], 0, 0, 0);
    };
    auto put_columns = [&]() {
        if constexpr(!SPLIT)
            if(tid < BN)
            {
                colp[tid]      = scale;
                colp[BN + tid] = bias;
            }
    };
    if(!SPLIT && K <= kF32ShortK)
    {
        constexpr std::true_type every{};
        point();
        if(K > 0)
        {
            Piece v;
            fetch(every, v, 0);
            products(every, v);
        }
        put_columns();
        __syncthreads();
    }
    else
    {
        if(whole > 0)
        {
            static_for<D>([&](auto c) {
#pragma unroll
                for(int i = 0; i < U; ++i) load(c, i, decltype(c)::value);
                __builtin_amdgcn_sched_barrier(0);
            });
            put_first();
            // (straight-line, no way from one of the D steps to another's place: the compiler then knows which load each of its waits is for)
            int t = 0, since = 0;
            for(; t + D < whole; t += D)
            {
                static_for<D>([&](auto c) { step(all, std::integral_constant<int, (decltype(c)::value + 1) % D>{}, t + decltype(c)::value); });
                if constexpr(kFold)
                    if((since += D) >= kFoldSteps)
                    {
                        since = 0;
#pragma unroll
                        for(int i = 0; i < FM; ++i)
#pragma unroll
                            for(int j = 0; j < FN; ++j)
                            {
                                total[i][j] += acc[i][j];
                                acc[i][j] = v4f32{0.0f, 0.0f, 0.0f, 0.0f};
                            }
                    }
            }
            static_for<D - 1>([&](auto c) {
                if(t + 1 < whole)
                {
                    step(all, std::integral_constant<int, (decltype(c)::value + 1) % D>{}, t);
                    ++t;
                }
            });
            if(whole < tiles)
            {
                take_tail();
                step(no_loads, c0, t);
                ++t;
            }
            step(last_one, c0, t);
            if constexpr(kFold)
#pragma unroll
                for(int i = 0; i < FM; ++i)
#pragma unroll
                    for(int j = 0; j < FN; ++j) acc[i][j] += total[i][j];
        }
        else if(tiles > 0)
        {
            load_tail();
            put_first();
            step(last_one, c0, 0);
        }
        put_columns();

        // Sums that the bf16 parts do not give as the fp32 instructions would are formed again by those, sixteen rows at a time: sums that
        // are not finite (an infinite value is a NaN in its lower parts, so it shows in every sum that it is part of), denormal ones, and
        // those that the lost bits of a value below 2^-110 may have moved by more than 2^-26: n products with up to the other row's
        // largest value, each off by less than 2^-133 of it.  So such values here and there cost a pass over the other operand, for the
        // largest values of its rows; rows of nothing else, a second turn of sixteen, without LDS; operands of nothing else, all of them.  All
        // of a workgroup's sums again because of one value (before) -> this, us, 8192x4096x1024 (353; on fp32 instructions alone 488): one
        // value in 256 rows 955 -> 381, 5 % of all values 958 -> 382, one row in 256 946 -> 538, an infinity 676 -> 437, all values 941 -> 936;
        // 2048^3 (85; 131) 280 -> 96, 280 -> 95, 281 -> 168, 285 -> 160, 281 -> 272.
        bool odd = false, lost[2] = {false, false};
        auto no_number = [](float v) { return __builtin_amdgcn_classf(v, 0x297); };      // (NaN, infinite or denormal)
#pragma unroll
        for(int i = 0; i < U; ++i) lost[i * kUnitRows < BM ? 0 : 1] |= (rest[i] & 0xFFFFu) != 0u;
#pragma unroll
        for(int i = 0; i < FM; ++i)
#pragma unroll
            for(int j = 0; j < FN; ++j)
#pragma unroll
                for(int e = 0; e < 4; ++e) odd |= no_number(acc[i][j][e]);
        // bit 0: a sum to look at; 1, 2: lost bits in A, in B
        const uint32_t mine = (__any(odd) ? 1u : 0u) | (__any(lost[0]) ? 2u : 0u) | (__any(lost[1]) ? 4u : 0u);
        if(lane == 0) flags[wave] = mine;
        __syncthreads();
        uint32_t looks = 0u;
#pragma unroll
        for(int w = 0; w < WGM * WGN; ++w) looks |= flags[w];
        looks = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(looks)));
        if(looks)
        {
            float* const largest = reinterpret_cast<float*>(lds);      // of a row of A, then of B; with the sign bit where bits of the row are lost
            if(looks & 6u)
            {
#pragma unroll
                for(int i = 0; i < U; ++i)
                {
                    float m = 0.0f;
                    if(looks & (i * kUnitRows < BM ? 4u : 2u))
                    {
#pragma unroll 8
                        for(int64_t k = first; k + kStepK <= end; k += kStepK)
                        {
                            const float* const at = row[i] + k + 8 * (tid % 4);
                            const v4f32_any    u = *reinterpret_cast<const v4f32_any*>(at), v = *reinterpret_cast<const v4f32_any*>(at + 4);
#pragma unroll
                            for(int e = 0; e < 4; ++e) m = fmaxf(m, fmaxf(fabsf(u[e]), fabsf(v[e])));
                        }
                        for(int64_t k = end - (end - first) % kStepK + tid % 4; k < end; k += 4) m = fmaxf(m, fabsf(row[i][k]));
                    }
                    uint32_t r = rest[i] & 0xFFFFu;
#pragma unroll
                    for(int off = 1; off <= 2; off *= 2)
                    {
                        m = fmaxf(m, __shfl_xor(m, off));
                        r |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(r), off));
                    }
                    if(tid % 4 == 0) largest[tid / 4 + i * kUnitRows] = r ? -m : m;
                }
                __syncthreads();
            }
            const float n = static_cast<float>(end - first) * 0x1p-107f;
            float       lb[FN][4];
#pragma unroll
            for(int j = 0; j < FN; ++j)
#pragma unroll
                for(int e = 0; e < 4; ++e) lb[j][e] = looks & 6u ? largest[BM + wn * (BN / WGN) + 16 * j + 4 * q + e] : 0.0f;
#pragma unroll
            for(int i = 0; i < FM; ++i)
            {
                const float la  = looks & 6u ? largest[wm * (BM / WGM) + 16 * i + fr] : 0.0f;
                bool        bad = false;
#pragma unroll
                for(int j = 0; j < FN; ++j)
#pragma unroll
                    for(int e = 0; e < 4; ++e)
                    {
                        const float off = (__builtin_signbitf(la) ? fabsf(lb[j][e]) : 0.0f) + (__builtin_signbitf(lb[j][e]) ? fabsf(la) : 0.0f);
                        bad |= no_number(acc[i][j][e]) || !(fabsf(acc[i][j][e]) >= off * n);
                    }
                if(__any(bad)) redo |= 1u << i;
            }
            redo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(redo)));
            if(looks & 6u) __syncthreads();      // (the epilogue stages its rows where the largest values are)
            if(redo)
            {
                constexpr std::false_type some{};
                constexpr int             kPieces = FM + FN > 4 ? 2 : 3;      // (two sets of them in registers)
                point();
#pragma unroll
                for(int i = 0; i < FM; ++i)
                    if(redo >> i & 1u)
#pragma unroll
                        for(int j = 0; j < FN; ++j) acc[i][j] = v4f32{0.0f, 0.0f, 0.0f, 0.0f};
                Piece now[kPieces], next[kPieces];
#pragma unroll
                for(int s = 0; s < kPieces; ++s)
                    if(first + 16 * s < end) fetch(some, now[s], first + 16 * s);
#pragma unroll 1
                for(int64_t k = first;; k += 16 * kPieces)
                {
#pragma unroll
                    for(int s = 0; s < kPieces; ++s)
                        if(k + 16 * (kPieces + s) < end) fetch(some, next[s], k + 16 * (kPieces + s));
#pragma unroll
                    for(int s = 0; s < kPieces; ++s)
                        if(k + 16 * s < end) products(some, now[s]);
                    if(k + 16 * kPieces >= end) break;
#pragma unroll
                    for(int s = 0; s < kPieces; ++s) now[s] = next[s];
                }
            }
        }
    }
    const uint32_t seen = (!SPLIT && p.amax_bits && wave == 0) ? __hip_atomic_load(p.amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    store_tile<F32Split, BM, BN, WGM, WGN, 2 * kStage / (WGM * WGN) / 16 * 16, SPLIT>(p, acc, lds, colp, m0, n0, which, alpha, code_inv, seen);
}

template <int BM, int BN, int WGM, int WGN, int D> hipError_t launch_tile_f32(const GemmKernelArgs& a, int64_t K, int splits, hipStream_t st)
{
    const dim3 grid(static_cast<unsigned>(a.tiles_m) * static_cast<unsigned>(a.tiles_n) * static_cast<unsigned>(splits)), block(64 * WGM * WGN);
    constexpr int kLds = f32_lds_bytes<BM, BN>();
    static bool   attr_set[16] = {};      // per instantiation and device; benign if set twice
    int           dev = 0;
    const bool    known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 16;
    if(!known || !attr_set[dev])
    {
        const void* const kernels[] = {reinterpret_cast<const void*>(&gemm_f32_kernel<BM, BN, WGM, WGN, D, false>), reinterpret_cast<const void*>(&gemm_f32_kernel<BM, BN, WGM, WGN, D, true>)};
        for(const void* k : kernels)
        {
            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
            if(e != hipSuccess) return e;
        }
        if(known) attr_set[dev] = true;
    }
    if(splits > 1) gemm_f32_kernel<BM, BN, WGM, WGN, D, true><<<grid, block, kLds, st>>>(a, K, splits);
    else           gemm_f32_kernel<BM, BN, WGM, WGN, D, false><<<grid, block, kLds, st>>>(a, K, 1);
    return hipGetLastError();
}

}  // namespace

// The plan's tile and K splits; the partial products of more than one are left to the caller.
hipError_t launch_gemm_f32(const GemmProblem& p, const GemmPlan& plan, void* workspace, hipStream_t stream)
{
    const TileShape ts = gemm_tile_shape(32, plan.tile);
    const int       splits = plan.splits < 1 ? 1 : plan.splits;
    const int64_t   ktiles = (p.K + kStepK - 1) / kStepK, per = (ktiles + splits - 1) / splits;
    GemmKernelArgs  a{};
    a.A = static_cast<const uint8_t*>(p.A);
    a.B = static_cast<const uint8_t*>(p.B);
    a.M = p.M; a.N = p.N;
    a.C = p.C; a.c_is_f16 = p.c_dtype == kF16;
    a.s0 = p.s0; a.s1 = p.s1; a.col_scale = p.col_scale; a.col_bias = p.col_bias;
    a.partial   = workspace;
    a.amax_bits = splits > 1 ? nullptr : p.out_amax_bits;      // with K splits the reduction pass takes the maximum and writes the codes
    a.codes     = splits > 1 ? nullptr : static_cast<int8_t*>(p.out_codes);
    a.code_inv  = p.out_code_inv;
    a.code_qmax = p.out_code_qmax;
    a.ktiles_per_split = static_cast<int>(per < 1 ? 1 : per);
    a.tiles_m = static_cast<int>((p.M + ts.bm - 1) / ts.bm);
    a.tiles_n = static_cast<int>((p.N + ts.bn - 1) / ts.bn);
    a.group_m = kGroupM;
    switch(plan.tile)
    {
    case 0: return launch_tile_f32<256, 128, 4, 2, 1>(a, p.K, splits, stream);
    case 1: return launch_tile_f32<128, 128, 2, 4, 2>(a, p.K, splits, stream);
    default: return launch_tile_f32<64, 64, 2, 2, 2>(a, p.K, splits, stream);
    }
}

}  // namespace qsync
