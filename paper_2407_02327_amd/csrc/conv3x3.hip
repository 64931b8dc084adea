// 3x3 / stride 1 / pad 1 convolution over an NHWC tensor on the matrix cores, forward and data gradient, with the input tile kept
// in LDS: C[m, n] = epilogue( sum over taps (kh, kw) and channels c of x[pixel m shifted by the tap, c] * w[n, kh, kw, c] ).
//
// As an implicit GEMM (gemm_nt_kernel) every input byte is fetched nine times, once per tap, with the gather's address
// arithmetic each time, and the loop waits for that feed, not for the matrix cores.  Here a workgroup owns BM consecutive
// output pixels x BN channels and fetches the BM + 2 W + 2 input pixels its taps reach ONCE per chunk of KC channel bytes;
// a tap is a displacement of the pixel index in LDS, and a neighbour outside the image is an address of zeros, chosen per
// lane by a bit mask.  Steps of one kernel row (three taps) stream the weights through two LDS stages: the loads
// for the next step are in flight behind the barrier, the input of the next chunk behind them.
//   * LDS rows are KC bytes (32 for narrow pixels, 128 for long contractions, else 64); 16-byte chunks are XOR-swizzled with
//     the pixel index so that any sixteen consecutive pixels, whatever the tap, meet all banks once;
//   * a step's fragments are requested together, as many sets as the LDS counter holds, and waited for one by one;
//   * two weight stages: with three, fewer workgroups share a unit (64x56x56 64->64 binary16 41.7 us, with two 28.1).
// What bounds it now: on full grids LDS reads and the stores, on sparse ones the chain barrier - LDS read - matrix
// instruction of each step (0.7 us for 384 bytes of K).
#include "gemm_device.h"

namespace qsync {

namespace {

constexpr int kZeroBytes = 1024;        // LDS offset 0: zeros that lanes of absent neighbours read (KC bytes of them)
constexpr int kMaxLds    = 163840;

struct ConvGeometry
{
    int chunks;          // of KC channel bytes
    int na;              // direct loads of a wavefront per input chunk
    int b_base;          // LDS offset of the weight stages (behind one input buffer, or two)
    int colp;            // LDS offset of the column parameters
};

template <int OFF> __device__ __forceinline__ void lds_frag(v4i32& d, uint32_t addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "immediate offset");
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF) : "memory");
}
template <int IMM> __device__ __forceinline__ void load_to_lds(const uint8_t* src, uint8_t* dst)
{   // (the immediate moves both addresses)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src - IMM),
                                     (__attribute__((address_space(3))) void*)dst, 16, IMM, 0);
}
// at most N + min(n, MAX) vector-memory operations of this wavefront still in flight
template <int N, int MAX> __device__ __forceinline__ void wait_loads_beside(int n)
{
    if constexpr(MAX == 0) wait_direct_loads<N>();
    else if(n >= MAX)      wait_direct_loads<N + MAX>();
    else                   wait_loads_beside<N, MAX - 1>(n);
}

// WGK 2: two sets of WGM x WGN wavefronts, each on its half of every chunk's channels; the second hands its sums over through LDS.
template <typename TR, int BM, int BN, int WGM, int WGN, int WGK, int KC>
__global__ __launch_bounds__(64 * WGM * WGN * WGK) void conv3x3_kernel(const GemmKernelArgs p, const ConvGeometry g)
{
    typedef typename TR::accv_t accv_t;
    constexpr int kWaves = WGM * WGN * WGK;
    constexpr int WTM = BM / WGM, WTN = BN / WGN, FM = WTM / 32, FN = WTN / 32;
    constexpr int LOG_KC = KC == 128 ? 7 : KC == 64 ? 6 : 5, CPR = KC / 16;          // 16-byte chunks per LDS row
    constexpr int PPI = 1024 / KC;                                  // LDS rows a direct load fills
    constexpr int SWZ = KC == 128 ? 1 : KC == 64 ? 2 : 3;           // swizzle of row i: (i >> SWZ) % CPR
    constexpr int NB  = (3 * BN / PPI + kWaves - 1) / kWaves;       // direct loads of a wavefront per weight stage
    constexpr int B_STAGE = NB * kWaves * 1024;
    static_assert((KC == 128 || KC == 64 || (KC == 32 && WGK == 1)) && NB <= 4 && BN % 32 == 0 && WTM % 32 == 0 && WTN % 32 == 0, "tile");

    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t*)lds));
    const int      tid = threadIdx.x, lane = tid % kWaveSize;
    const int      wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize), wk = wave / (WGM * WGN), wm = wave % (WGM * WGN) / WGN, wn = wave % WGN;
    if(tid < KC / 16) *reinterpret_cast<uint4*>(lds + tid * 16) = make_uint4(0, 0, 0, 0);

    int split, tm, tn;
    item_of_block(static_cast<int>(blockIdx.x), p.tiles_m, p.tiles_n, 1, p.group_m, split, tm, tn);
    const int      m0 = tm * BM, n0 = tn * BN, P = static_cast<int>(p.M), W = p.conv_W, H = p.conv_H;      // (P < 2^31: checked)
    const uint32_t Cb = static_cast<uint32_t>(p.conv_Cb);
    const uint8_t* zero = reinterpret_cast<const uint8_t*>(&g_zero_chunk);

    const float  scale0 = *(p.s0 ? p.s0 : &g_one), scale1 = *(p.s1 ? p.s1 : &g_one);
    float* const colp = reinterpret_cast<float*>(lds + g.colp);
    if(wave * 64 < BN && lane < BN)
    {
        const int64_t col = n0 + tid < p.N ? n0 + tid : p.N - 1;
        if(p.col_scale) column_param_issue(p.col_scale + col, lds + g.colp + wave * 256);
        if(p.col_bias) column_param_issue(p.col_bias + col, lds + g.colp + BN * 4 + wave * 256);
    }

    // input: load q of a chunk fills LDS rows [q PPI, (q + 1) PPI) with pixels m0 - W - 1 + row (clamped: rows outside the
    // tensor are never read through the mask)
    const int      pos = lane % CPR, sub = lane / CPR;
    const uint32_t ch  = static_cast<uint32_t>((pos ^ ((sub >> SWZ) % CPR)) * 16);       // channel bytes of the lane in load 0 ...
    constexpr uint32_t kOdd = PPI % (CPR << SWZ) == 0 ? 0u : 64u;                           // ... and what odd loads (KC 128) flip
    auto issue_input = [&](int chunk, int buf) {
        const uint32_t c0 = static_cast<uint32_t>(chunk * KC);
        uint8_t*       dst = lds + kZeroBytes + (buf * kWaves + wave) * g.na * 1024;
        int            px  = m0 - W - 1 + wave * g.na * PPI + sub;
        for(int j = 0; j < g.na; j += 4, dst += 4096, px += 4 * PPI)
        {
            auto one = [&](auto k) {
                if(j + decltype(k)::value >= g.na) return;
                int            q = px + decltype(k)::value * PPI;
                const uint32_t c = c0 + (ch ^ (((wave * g.na + j + decltype(k)::value) & 1) ? kOdd : 0u));
                q     = q < 0 ? 0 : (q < P ? q : P - 1);
                load_to_lds<decltype(k)::value * 1024>(c < Cb ? p.A + (static_cast<uint32_t>(q) * Cb + c) : zero, dst);
            };
            one(std::integral_constant<int, 0>{});
            one(std::integral_constant<int, 1>{});
            one(std::integral_constant<int, 2>{});
            one(std::integral_constant<int, 3>{});
        }
    };
    // weights: stage rows are (kw, n); a wavefront's NB loads are consecutive
    uint32_t b_off[NB];
    auto     b_ch = [&](int d) { return ch ^ (((wave * NB + d) & 1) ? kOdd : 0u); };
#pragma unroll
    for(int d = 0; d < NB; ++d)
    {
        int row = (wave * NB + d) * PPI + sub;
        row     = row < 3 * BN ? row : 3 * BN - 1;                      // (padding of the stage)
        const int     kw = row / BN;
        const int64_t n  = n0 + row % BN < p.N ? row % BN : p.N - 1 - n0;
        b_off[d]         = static_cast<uint32_t>(n) * 9u * Cb + static_cast<uint32_t>(kw) * Cb + b_ch(d);
    }
    const uint8_t* const wbase = p.B + static_cast<int64_t>(n0) * 9 * Cb;
    auto issue_weights = [&](int chunk, int kh, int slot) {
        const uint8_t* src = wbase + static_cast<uint32_t>(kh) * 3u * Cb + static_cast<uint32_t>(chunk * KC);
        uint8_t*       dst = lds + g.b_base + slot * B_STAGE + wave * NB * 1024;
        static_for<NB>([&](auto d) {
            load_to_lds<decltype(d)::value * 1024>(static_cast<uint32_t>(chunk * KC) + b_ch(decltype(d)::value) < Cb ? src + b_off[decltype(d)::value] : zero, dst);
        });
    };

    // fragment rows of this lane: LDS row of the centre tap, and which of the nine neighbours lie inside the image
    const int frag_row = lane & 31, khalf = lane >> 5;
    int       centre[FM];
    uint32_t  inside[FM];
#pragma unroll
    for(int f = 0; f < FM; ++f)
    {
        const int r = wm * WTM + f * 32 + frag_row;
        centre[f]   = r + W + 1;
        const uint32_t m = static_cast<uint32_t>(m0 + r < P ? m0 + r : P - 1), q = m / static_cast<uint32_t>(W);
        const uint32_t h = q % static_cast<uint32_t>(H), w = m - q * static_cast<uint32_t>(W);
        const uint32_t row = (w > 0 ? 1u : 0u) | 2u | (w + 1 < static_cast<uint32_t>(W) ? 4u : 0u);
        inside[f] = (h > 0 ? row : 0u) | (row << 3) | (h + 1 < static_cast<uint32_t>(H) ? row << 6 : 0u);
    }
    const int      b_row  = wn * WTN + frag_row;
    constexpr int  KS = KC / 32 / WGK;                              // 32-byte K chunks of this wavefront's share of a row
    const int      kq = khalf + 2 * KS * wk;                        // first 16-byte chunk of the lane
    const uint32_t b_lane = static_cast<uint32_t>(g.b_base + b_row * KC + ((kq ^ ((b_row >> SWZ) % CPR)) << 4));

    accv_t acc[FM][FN];
#pragma unroll
    for(int i = 0; i < FM; ++i)
#pragma unroll
        for(int j = 0; j < FN; ++j)
#pragma unroll
            for(int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    const int steps = 3 * g.chunks;
    issue_input(0, 0);
    issue_weights(0, 0, 0);
    // fragment sets of a step, (kw, 32-byte K chunk), as many in flight as the LDS counter (15) and the registers allow
    constexpr int ITEMS = 3 * KS, kFit = 15 / (FM + FN), kSets = ITEMS < kFit ? ITEMS : kFit;
    v4i32 af[kSets][FM], bf[kSets][FN];
    int chunk = 0, kh = 0, slot = 0;
    for(int step = 0; step < steps; ++step)
    {
        // Needed: this step's weights and, for kh == 0, this chunk's input.  Requested behind them, so possibly in flight: for
        // kh == 1 the next chunk's input.
        const bool next_chunk = chunk + 1 < g.chunks;
        wait_loads_beside<0, 24>(kh == 1 && next_chunk ? g.na : 0);
        wg_barrier();
        if(step + 1 < steps) issue_weights(kh == 2 ? chunk + 1 : chunk, kh == 2 ? 0 : kh + 1, slot ^ 1);
        if(kh == 0 && next_chunk) issue_input(chunk + 1, (chunk + 1) & 1);

        const uint32_t a_base = lds0 + static_cast<uint32_t>(kZeroBytes + (chunk & 1) * kWaves * g.na * 1024);
        const uint32_t b_base = lds0 + b_lane + static_cast<uint32_t>(slot * B_STAGE);
        const int      shift  = (kh - 1) * W - 1;
        uint32_t       a_tap[FM];
        auto           read = [&](auto item) {
            constexpr int j = decltype(item)::value, kw = j / KS, ks = j % KS, set = j % kSets;
            if constexpr(ks == 0)
#pragma unroll
                for(int f = 0; f < FM; ++f)
                {
                    const int      i = centre[f] + shift + kw;
                    const uint32_t a = a_base + (static_cast<uint32_t>(i) << LOG_KC) + ((static_cast<uint32_t>(kq) ^ ((static_cast<uint32_t>(i) >> SWZ) % CPR)) << 4);
                    const int      m = static_cast<int>(inside[f] << (31 - kw - 3 * kh)) >> 31;      // all ones where the neighbour exists
                    a_tap[f]         = lds0 + ((a - lds0) & static_cast<uint32_t>(m));
                }
            static_for<FM>([&](auto f) { lds_frag<0>(af[set][decltype(f)::value], a_tap[decltype(f)::value] ^ (ks * 32u)); });
            static_for<FN>([&](auto f) { lds_frag<(kw * BN + decltype(f)::value * 32) * KC>(bf[set][decltype(f)::value], b_base ^ (ks * 32u)); });
        };
        static_for<kSets>(read);
        static_for<ITEMS>([&](auto item) {
            constexpr int j = decltype(item)::value, set = j % kSets;
            constexpr int younger = ITEMS - 1 - j < kSets - 1 ? ITEMS - 1 - j : kSets - 1;       // sets that may still be in flight
            constexpr int kWait = 0xC07F | ((younger * (FM + FN)) << 8);
            __builtin_amdgcn_s_waitcnt(kWait);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for(int i = 0; i < FM; ++i)
#pragma unroll
                for(int n = 0; n < FN; ++n) acc[i][n] = TR::mfma(bf[set][n], af[set][i], acc[i][n]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr(j + kSets < ITEMS) read(std::integral_constant<int, j + kSets>{});
        });
        slot ^= 1;
        if(++kh == 3) { kh = 0; ++chunk; }
    }
    if constexpr(WGK == 2)
    {
        uint8_t* mine = lds + (wave % (WGM * WGN)) * (FM * FN * 4096) + lane * 16;
        __syncthreads();                                            // all wavefronts are done reading
        if(wk == 1)
#pragma unroll
            for(int i = 0; i < FM * FN; ++i)
#pragma unroll
                for(int q = 0; q < 4; ++q)
                {
                    const typename TR::acc_t o[4] = {acc[i / FN][i % FN][4 * q], acc[i / FN][i % FN][4 * q + 1], acc[i / FN][i % FN][4 * q + 2], acc[i / FN][i % FN][4 * q + 3]};
                    *reinterpret_cast<uint4*>(mine + i * 4096 + q * 1024) = *reinterpret_cast<const uint4*>(o);
                }
        __syncthreads();
        if(wk == 1) return;
#pragma unroll
        for(int i = 0; i < FM * FN; ++i)
#pragma unroll
            for(int q = 0; q < 4; ++q)
            {
                typename TR::acc_t o[4];
                *reinterpret_cast<uint4*>(o) = *reinterpret_cast<const uint4*>(mine + i * 4096 + q * 1024);
#pragma unroll
                for(int e = 0; e < 4; ++e) acc[i / FN][i % FN][4 * q + e] += o[e];
            }
    }
    const uint32_t amax_seen = p.amax_bits ? __hip_atomic_load(p.amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    store_tile<TR, BM, BN, WGM, WGN, 32 * (WTN * 4 + 16), false>(p, acc, lds, colp, m0, n0, 0, scale0 * scale1, 0.0f, amax_seen);
}

constexpr int kMaxDevices = 16;

template <typename TR, int BM, int BN, int WGM, int WGN, int WGK, int KC> hipError_t launch_tile(GemmKernelArgs a, bool* taken, hipStream_t st)
{
    constexpr int kWaves = WGM * WGN * WGK, PPI = 1024 / KC, NB = (3 * BN / PPI + kWaves - 1) / kWaves;
    constexpr int kEpilogue = WGM * WGN * 32 * (BN / WGN * 4 + 16), kSums = WGK == 2 ? BM * BN * 4 : 0, kStage = kEpilogue > kSums ? kEpilogue : kSums;
    ConvGeometry  g;
    const int64_t rows = BM + 2 * static_cast<int64_t>(a.conv_W) + 2, na = (rows + PPI * kWaves - 1) / (PPI * kWaves);
    const int64_t chunks = (a.conv_Cb + KC - 1) / KC, b_base = kZeroBytes + (chunks > 1 ? 2 : 1) * na * kWaves * 1024;
    int64_t       colp = b_base + 2 * NB * kWaves * 1024;
    colp               = colp < kStage ? kStage : colp;
    const int64_t lds  = colp + 2 * BN * 4 + 64;
    if(lds > kMaxLds) return hipSuccess;                              // (a wide image: the caller takes the implicit GEMM)
    g.chunks = static_cast<int>(chunks); g.na = static_cast<int>(na); g.b_base = static_cast<int>(b_base); g.colp = static_cast<int>(colp);
    a.tiles_m = static_cast<int>((a.M + BM - 1) / BM);
    a.tiles_n = static_cast<int>((a.N + BN - 1) / BN);
    static bool attr_set[kMaxDevices] = {};      // per instantiation and device; benign if set twice
    int         dev = 0;
    const bool  known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices;
    if(!known || !attr_set[dev])
    {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv3x3_kernel<TR, BM, BN, WGM, WGN, WGK, KC>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
        if(e != hipSuccess) return e;
        if(known) attr_set[dev] = true;
    }
    *taken = true;
    conv3x3_kernel<TR, BM, BN, WGM, WGN, WGK, KC><<<dim3(static_cast<unsigned>(a.tiles_m) * a.tiles_n), dim3(64 * kWaves), lds, st>>>(a, g);
    return hipGetLastError();
}

// Shapes: pixels x channels of a workgroup (x2: two sets of wavefronts).
enum Shape { k256x64, k128x64, k128x64x2, k64x64x2, k256x32, k128x32x2 };
template <typename TR, int KC> hipError_t launch_shape(const GemmKernelArgs& a, int shape, bool* taken, hipStream_t st)
{
    constexpr int K2 = KC == 32 ? 1 : 2;
    if constexpr(KC < 128)
        switch(shape)
        {
        case k256x64: return launch_tile<TR, 256, 64, 4, 1, 1, KC>(a, taken, st);
        case k128x64: return launch_tile<TR, 128, 64, 2, 2, 1, KC>(a, taken, st);
        case k256x32: return launch_tile<TR, 256, 32, 4, 1, 1, KC>(a, taken, st);
        }
    switch(shape)
    {
    case k128x64x2: return launch_tile<TR, 128, 64, 2, 2, K2, KC>(a, taken, st);
    case k64x64x2: return launch_tile<TR, 64, 64, 2, 2, K2, KC>(a, taken, st);
    default: return launch_tile<TR, 128, 32, 4, 1, K2, KC>(a, taken, st);
    }
}

}  // namespace

hipError_t launch_conv3x3(const GemmProblem& p, int force_tile, bool* taken, hipStream_t st)
{
    *taken = false;
    const int esz = p.prec / 8;
    if(p.out_codes || p.M + 2 * static_cast<int64_t>(p.conv_W) + 1024 >= (int64_t(1) << 31)) return hipSuccess;
    GemmKernelArgs a{};
    a.A = static_cast<const uint8_t*>(p.A);
    a.B = static_cast<const uint8_t*>(p.B);
    a.M = p.M; a.N = p.N; a.Kb = p.K * esz;
    a.C = p.C; a.c_is_f16 = p.c_dtype == kF16;
    a.s0 = p.s0; a.s1 = p.s1; a.col_scale = p.col_scale; a.col_bias = p.col_bias;
    a.acc_dump  = p.prec == 8 ? p.acc_dump : nullptr;
    a.group_m   = kGroupM;
    a.conv_H = p.conv_H; a.conv_W = p.conv_W; a.conv_Cb = static_cast<int>(p.conv_C * esz);
    a.amax_bits = p.out_amax_bits;
    const int64_t strips = (a.N + 63) / 64;
    auto tiles = [&](int bm) { return (a.M + bm - 1) / bm * strips; };
    // More workgroups of 128 x 64 than units: the implicit GEMM's larger tiles are faster where they read wide rows of weights
    // for many outputs (per unit of work they fetch less of both operands), and where 64-byte rows would be partly empty.  Over 120
    // shapes of 784 to 200704 pixels and 16 to 512 channels this kernel takes, implicit -> here, 64x56x56 64->64 int8 25.5 -> 18.1
    // us, binary16 34.6 -> 28.1; 53x28x48 32->304 binary16 36.0 -> 28.8; left to the other: 25x13x44 208->256 int8 14.5 (18.1
    // here), 46x18x51 80->64 8.9 (10.8), 52x29x32 16->240 13.4 (15.8).  At fewer workgroups it takes them all: 16x14x14
    // 256->256 int8 10.7 -> 8.4, binary16 17.3 -> 12.9; 64x7x7 512->512 21.2 -> 16.8, 45.8 -> 28.9; 11x45x50 192->16 binary16
    // 16.7 -> 10.5; 2x31x43 80->32 7.9 -> 7.8 is the least.
    if(force_tile < 0 && a.N > 32 && tiles(128) > kNumCu
       && !(a.N <= 64 ? a.conv_Cb <= 64 || a.conv_Cb % 64 == 0 : a.conv_Cb >= 32 && a.conv_Cb <= 64))
        return hipSuccess;
    // Narrow outputs by 32 channels; else the largest tile that gives every unit one (beyond: the largest that two of them share).
    // Long contractions on few workgroups run two sets of wavefronts and 128-byte rows, i.e. half the barriers, at one
    // workgroup per unit (24x14x14 256->256 binary16: 23.1 us by 64-byte rows, 16.6).
    int shape;
    if(a.N <= 32) shape = (force_tile >= 0 ? force_tile == 0 : tiles(256) >= 512) ? k256x32 : k128x32x2;
    else if(force_tile >= 0 ? force_tile == 2 : tiles(64) <= kNumCu) shape = k64x64x2;
    else if(force_tile < 0 && tiles(128) <= kNumCu && a.conv_Cb > 64) shape = k128x64x2;
    else if(force_tile >= 0 ? force_tile == 0 : tiles(256) > kNumCu && a.conv_Cb > 32) shape = k256x64;
    else shape = k128x64;
    const int kc = a.conv_Cb <= 32 ? 32 : a.conv_Cb > 64 && (shape == k64x64x2 || shape == k128x64x2 || shape == k128x32x2) ? 128 : 64;
    auto go = [&](auto tr) {
        typedef decltype(tr) TR;
        return kc == 32 ? launch_shape<TR, 32>(a, shape, taken, st) : kc == 64 ? launch_shape<TR, 64>(a, shape, taken, st) : launch_shape<TR, 128>(a, shape, taken, st);
    };
    return p.prec == 8 ? go(I8Rows32{}) : go(F16Rows32{});
}

}  // namespace qsync
