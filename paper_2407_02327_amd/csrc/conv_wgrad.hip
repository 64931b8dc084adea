// Weight gradient of a 3x3 NHWC convolution:  dW[n, (tap, c)] = sum over pixels p of dY[p, n] X[p + displacement(tap), c], pixels outside the
// image zero; int8 or binary16 operands, raw sums per K split.
//
// As a GEMM with gathering loads every pixel of X comes from L2 once a tap and every pixel of dY once a column tile, and a K tile waits
// for them: 64x56x56 64->64 int8 took 26.6 us for 5 us of matrix instructions.  Here a workgroup has 64 rows of dW and all nine taps of 16
// channels; each of its wavefronts goes through a range of pixels by itself, X in a ring in LDS that every pixel enters once.  A tap is a
// displacement in the ring, a neighbour outside the image an address of zeros.  The operands leave LDS through the transposing reads
// (layouts in gemm_mfma.hip), a lane supplying the address of one pixel.  No barrier until the wavefronts' sums are added up.
//
// Bound by the vector instructions that form the 18 addresses of a chunk (about 200 for 36 matrix instructions, 1 us a chunk alone on a
// SIMD; two wavefronts share one) and by what is there once, 11 us with the splits' sum: launch, first loads, the wavefronts' sums.  Gathering
// GEMM -> this with the splits' sum, us: int8 64x56x56 64->64 34.8 -> 29.1, 50x33x38 272->64 39.6 -> 31.9, binary16 24x14x14 256->256 26.7 -> 24.6,
// 58x45x34 272->16 84.8 -> 50.2, 8x34x39 288->160 41.1 -> 31.4.  Tried: chunks four ahead unrolled (code of
// 24 KB, 31.3 us at the first shape), four wavefronts (30.2; 1 % to 10 % slower beyond 9e8, faster below), one chunk ahead (31.0).
#include "gemm_device.h"

#include <cmath>

namespace qsync {

namespace {

constexpr int kWgradWaves = 8, kWgradTaps = 9, kWgradRows = 64, kWgradChannels = 16;
constexpr int kWgradUnit  = 1024;                            // LDS bytes of 16 channels of a chunk's pixels
constexpr int kWgradA     = 4096;                            // ... of 64 columns of dY
constexpr int kWgradSums  = 4 * kWgradTaps * 1024;           // a wavefront's accumulators
constexpr int kWgradAhead = 2;                               // chunks on their way in registers

struct ConvWgradArgs
{
    const uint8_t* x;
    const uint8_t* dy;
    int            M;             // pixels
    int            N, C, H, W;
    int            edge;          // chunks that hold W + 1 pixels: the ring reaches so far in front of and behind a chunk
    int            ring;          // bytes of a wavefront's ring, a power of two: at least 2 edge + 1 chunks
    int            chunks, per;   // chunks of the tensor, of a wavefront
    int            tiles_m, tiles_n, splits;
    void*          partial;
};

// where the rings start
__host__ __device__ constexpr int wgrad_rings(int ring) { return (1024 + kWgradWaves * kWgradA + ring - 1) / ring * ring; }

constexpr int kWgradRingUnits = 8, kWgradLds = kWgradWaves / 2 * kWgradSums;      // the widest ring; the sums need more LDS than the rings
static_assert(wgrad_rings(kWgradRingUnits * kWgradUnit) + kWgradWaves * kWgradRingUnits * kWgradUnit <= kWgradLds && kWgradLds <= 160 * 1024);

template <typename TR> __global__ __launch_bounds__(64 * kWgradWaves, 2) void conv_wgrad_kernel(const ConvWgradArgs p)
{
    constexpr int ESZ = TR::kElemBytes, CH = 64 / ESZ, PX = kWgradChannels * ESZ, AROW = kWgradRows * ESZ;
    constexpr int G = 16 / ESZ;             // pixels of a lane quarter's read: two of its halves side by side fill the banks
    typedef typename TR::accv_t accv_t;
    typedef typename TR::acc_t  acc_t;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int lane = static_cast<int>(threadIdx.x) % kWaveSize, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWaveSize);
    const int q = lane / 16, s = lane % 16;
    int       split, tm, tn;
    item_of_block(static_cast<int>(blockIdx.x), p.tiles_m, p.tiles_n, p.splits, kGroupM, split, tm, tn);
    const int n0 = tm * kWgradRows, c0 = tn * kWgradChannels;

    // LDS: 128 zero bytes, a piece of dY per wavefront, then the rings, each at a multiple of its size
    const uint32_t zero = 0u, a0 = 1024u + static_cast<uint32_t>(wave * kWgradA), ring0 = static_cast<uint32_t>(wgrad_rings(p.ring) + wave * p.ring);
    const uint32_t mask = static_cast<uint32_t>(p.ring) - 1u;
    if(threadIdx.x < 8) *reinterpret_cast<uint4*>(lds + threadIdx.x * 16) = make_uint4(0, 0, 0, 0);
    __syncthreads();

    const int first = (split * kWgradWaves + wave) * p.per, last = first + p.per < p.chunks ? first + p.per : p.chunks;      // (last <= first: nothing to do)
    auto swz = [](int u) { return u ^ (((u / G) & 1) * (G / 2)); };      // place of a pixel among those of its chunk (and back)

    // ---- on the way in.  Ring unit j: pixels CH (j - edge) and on
    const int      slot = ESZ == 1 ? lane : lane / 2, x_px = swz(slot);
    const int      x_col = c0 * ESZ + (ESZ == 2 && (lane & 1) && c0 + 8 < p.C ? 16 : 0);
    // (a scalar base and a 32-bit lane offset, the same for every chunk but those that reach over an end of the tensor)
    const uint32_t x_ld = static_cast<uint32_t>(p.C * ESZ), x_off = static_cast<uint32_t>(x_px) * x_ld + static_cast<uint32_t>(x_col);
    auto load_x = [&](int j) {
        const int      base = (j - p.edge) * CH;
        const uint8_t* src  = p.x + static_cast<int64_t>(base) * x_ld;
        uint32_t       off  = x_off;
        if(base < 0 || base + CH > p.M)
        {   // outside the tensor: any pixel, never used
            const int px = base + x_px;
            src = p.x;
            off = static_cast<uint32_t>(px < 0 ? 0 : px < p.M ? px : p.M - 1) * x_ld + static_cast<uint32_t>(x_col);
        }
        return *reinterpret_cast<const uint4*>(src + off);
    };
    constexpr int  CPR = AROW / 16, RPI = 64 / CPR;                       // 16-byte pieces of a row of dY, rows of a load
    const int      a_row = lane / CPR, a_chunk = lane % CPR;
    const uint32_t a_ld = static_cast<uint32_t>(p.N * ESZ), a_col = static_cast<uint32_t>(n0 * ESZ + (n0 * ESZ + a_chunk * 16 < p.N * ESZ ? a_chunk * 16 : 0));      // (columns past N: never stored)
    uint32_t       a_off[4];
#pragma unroll
    for(int d = 0; d < 4; ++d) a_off[d] = static_cast<uint32_t>(d * RPI + a_row) * a_ld + a_col;
    auto load_a = [&](int t, int d) {
        const uint8_t* src  = p.dy + static_cast<int64_t>(t) * CH * a_ld;
        uint32_t       off  = a_off[d];
        const int      left = p.M - t * CH, row = d * RPI + a_row;
        if(left < CH) off = static_cast<uint32_t>(row < left ? row : left - 1) * a_ld + a_col;
        return *reinterpret_cast<const uint4*>(src + off);
    };
    auto put_x = [&](int j, const uint4& v) {
        *reinterpret_cast<uint4*>(lds + ring0 + ((static_cast<uint32_t>(j) * kWgradUnit) & mask) + lane * 16) = v;
    };
    auto put_a = [&](int d, const uint4& v) {
        const int row = d * RPI + a_row;
        *reinterpret_cast<uint4*>(lds + a0 + row * AROW + ((a_chunk ^ tn_swizzle<ESZ, AROW>(row)) * 16)) = v;
    };

    // ---- on the way out: the pixel that the lane's two reads of a fragment fetch, as chunk-invariant places in the ring
    const int row0 = ESZ == 1 ? 16 * q + s / 2 : 8 * q + s / 4, piece = ESZ == 1 ? 8 * (s & 1) : 8 * (s & 3);
    uint32_t  place[kWgradTaps][2];
#pragma unroll
    for(int t = 0; t < kWgradTaps; ++t)
#pragma unroll
        for(int r = 0; r < 2; ++r)
            place[t][r] = static_cast<uint32_t>(swz(row0 + r * (G / 2) + (t / 3 - 1) * p.W + t % 3 - 1 + p.edge * CH) * PX + piece);
    const uint32_t a_lane = a0 + static_cast<uint32_t>(row0 * AROW + (((ESZ == 1 ? 0 : (s & 3) / 2) ^ tn_swizzle<ESZ, AROW>(row0)) * 16) + 8 * (s & 1));
    int h[2], w[2], px[2];
#pragma unroll
    for(int r = 0; r < 2; ++r)
    {
        px[r] = first * CH + row0 + r * (G / 2);
        const int line = px[r] / p.W;
        w[r] = px[r] - line * p.W;
        h[r] = line % p.H;
    }
    const int dw = CH % p.W, dh = (CH / p.W) % p.H;

    accv_t acc[4][kWgradTaps];
#pragma unroll
    for(int i = 0; i < 4; ++i)
#pragma unroll
        for(int t = 0; t < kWgradTaps; ++t)
#pragma unroll
            for(int e = 0; e < 4; ++e) acc[i][t][e] = 0;

    auto read = [&](uint32_t a, uint32_t b) {
        typedef int   v2i __attribute__((ext_vector_type(2)));
        typedef short v4s __attribute__((ext_vector_type(4)));
        __attribute__((address_space(3))) uint8_t* const base = (__attribute__((address_space(3))) uint8_t*)lds;
        v2i lo, hi;
        if constexpr(ESZ == 1)
        {
            lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) v2i*)(base + a));
            hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) v2i*)(base + b));
        }
        else
        {
            lo = __builtin_bit_cast(v2i, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(base + a)));
            hi = __builtin_bit_cast(v2i, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(base + b)));
        }
        return v4i32{lo.x, lo.y, hi.x, hi.y};
    };
    constexpr int D = kWgradAhead;
    uint4         xr[D], ar[D][4];
    auto request = [&](auto set, int t) {      // (behind the last chunk that one again, not looked at)
        const int at = t < last ? t : last - 1;
        xr[decltype(set)::value] = load_x(at + 2 * p.edge);
#pragma unroll
        for(int d = 0; d < 4; ++d) ar[decltype(set)::value][d] = load_a(at, d);
    };
    auto step = [&](int t) {
        // A wavefront's LDS operations keep their order, so the previous chunk's reads come before these writes and the fence, which
        // costs nothing, keeps the compiler from looking at other lanes' values early.
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        put_x(t + 2 * p.edge, xr[0]);
#pragma unroll
        for(int d = 0; d < 4; ++d) put_a(d, ar[0][d]);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
        for(int k = 0; k + 1 < D; ++k)
        {
            xr[k] = xr[k + 1];
#pragma unroll
            for(int d = 0; d < 4; ++d) ar[k][d] = ar[k + 1][d];
        }
        request(std::integral_constant<int, D - 1>{}, t + D);
        __builtin_amdgcn_sched_barrier(0);

        int      taps[2];      // bit t: the neighbour under tap t lies inside the image
        uint32_t a_at[2];
#pragma unroll
        for(int r = 0; r < 2; ++r)
        {
            const int line = (w[r] > 0 ? 1 : 0) | 2 | (w[r] + 1 < p.W ? 4 : 0);
            const int all  = (h[r] > 0 ? line : 0) | line << 3 | (h[r] + 1 < p.H ? line << 6 : 0);
            taps[r] = px[r] < p.M ? all : 0;
            a_at[r] = px[r] < p.M ? a_lane + static_cast<uint32_t>(r * (G / 2) * AROW) : zero;
        }
        v4i32 af[4];
#pragma unroll
        for(int i = 0; i < 4; ++i) af[i] = read(a_at[0] ^ static_cast<uint32_t>(i * 16 * ESZ), a_at[1] ^ static_cast<uint32_t>(i * 16 * ESZ));
        const uint32_t moved = static_cast<uint32_t>(t) * kWgradUnit;
        static_for<kWgradTaps>([&](auto tt) {
            constexpr int tap = decltype(tt)::value;
            uint32_t      at[2];
#pragma unroll
            for(int r = 0; r < 2; ++r)      // (the zeros lie at address 0)
                at[r] = (((place[tap][r] + moved) & mask) | ring0) & static_cast<uint32_t>(__builtin_amdgcn_sbfe(taps[r], tap, 1));
            const v4i32 bf = read(at[0], at[1]);
#pragma unroll
            for(int i = 0; i < 4; ++i) acc[i][tap] = TR::mfma(bf, af[i], acc[i][tap]);
        });
#pragma unroll
        for(int r = 0; r < 2; ++r)
        {
            px[r] += CH;
            w[r] += dw;
            const int carry = w[r] >= p.W ? 1 : 0;
            w[r] -= carry ? p.W : 0;
            h[r] += dh + carry;
            h[r] -= h[r] >= p.H ? p.H : 0;
        }
    };
    if(first < last)
    {
        uint4 v[4];
#pragma unroll
        for(int k = 0; k < 4; ++k) v[k] = load_x(first + k);
        static_for<D>([&](auto c) { request(c, first + decltype(c)::value); });
        __builtin_amdgcn_sched_barrier(0);
        for(int j = 0;;)
        {   // (what the ring holds in front of the first chunk, four units on their way at once)
#pragma unroll
            for(int k = 0; k < 4; ++k)
                if(j + k < 2 * p.edge) put_x(first + j + k, v[k]);
            j += 4;
            if(j >= 2 * p.edge) break;
#pragma unroll
            for(int k = 0; k < 4; ++k) v[k] = load_x(first + j + k);
        }
        // (one body, the requests moved up a place: unrolled, the code of a few chunks did not fit what is fetched ahead)
#pragma unroll 1
        for(int t = first; t < last; ++t) step(t);
    }

    // ---- the wavefronts' sums, halves onto halves; the last step and the stores divided between wavefronts 0 and 1 by taps
    typedef acc_t v4a __attribute__((ext_vector_type(4)));
    v4a* const sums = reinterpret_cast<v4a*>(lds);
    auto at = [&](int half, int i, int t) -> v4a& { return sums[half * (kWgradSums / 16) + (i * kWgradTaps + t) * 64 + lane]; };
#pragma unroll
    for(int half = kWgradWaves / 2; half >= 2; half /= 2)
    {
        __syncthreads();                                      // (every ring, or what was here before, has been read)
        if(wave >= half && wave < 2 * half)
#pragma unroll
            for(int i = 0; i < 4; ++i)
#pragma unroll
                for(int t = 0; t < kWgradTaps; ++t) at(wave - half, i, t) = acc[i][t];
        __syncthreads();
        if(wave < half)
#pragma unroll
            for(int i = 0; i < 4; ++i)
#pragma unroll
                for(int t = 0; t < kWgradTaps; ++t) acc[i][t] += at(wave, i, t);
    }
    if(wave < 2)
#pragma unroll
        for(int i = 0; i < 4; ++i)
#pragma unroll
            for(int t = 0; t < kWgradTaps; ++t)
                if((t < 5) == (wave == 1)) at(wave, i, t) = acc[i][t];      // (each lane overwrites what it alone has just read)
    __syncthreads();
    if(wave >= 2) return;
    acc_t* const out = static_cast<acc_t*>(p.partial) + static_cast<int64_t>(split) * p.N * 9 * p.C;
#pragma unroll
    for(int i = 0; i < 4; ++i)
    {
        const int n = n0 + 16 * i + s, c = c0 + 4 * q;
        if(n >= p.N || c >= p.C) continue;
#pragma unroll
        for(int t = 0; t < kWgradTaps; ++t)
            if((t < 5) == (wave == 0)) *reinterpret_cast<v4a*>(out + (static_cast<int64_t>(n) * 9 + t) * p.C + c) = acc[i][t] + at(1 - wave, i, t);
    }
}

template <typename TR> hipError_t launch_wgrad(const ConvWgradArgs& a, hipStream_t st)
{
    static bool attr_set[16] = {};      // per instantiation and device; benign if set twice
    int         dev = 0;
    const bool  known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 16;
    if(!known || !attr_set[dev])
    {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_wgrad_kernel<TR>), hipFuncAttributeMaxDynamicSharedMemorySize, kWgradLds);
        if(e != hipSuccess) return e;
        if(known) attr_set[dev] = true;
    }
    conv_wgrad_kernel<TR><<<dim3(static_cast<unsigned>(a.tiles_m) * static_cast<unsigned>(a.tiles_n) * static_cast<unsigned>(a.splits)), dim3(64 * kWgradWaves), kWgradLds, st>>>(a);
    return hipGetLastError();
}

}  // namespace

int& last_wgrad_ring()
{
    static thread_local int splits = 0;
    return splits;
}

// `p`: a weight gradient as launch_gemm takes it (conv_H > 0, tn), checked; at most max_splits partial products fit in `workspace`.  Returns
// the number of splits left there, 0 (nothing launched) where the image is too wide for the ring or the gathering GEMM, `gemm_us`, is the faster.
int launch_conv3x3_wgrad(const GemmProblem& p, int max_splits, double gemm_us, void* workspace, hipStream_t stream, hipError_t* error)
{
    const int esz = p.prec / 8, ch = 64 / esz;
    ConvWgradArgs a{};
    a.edge = (p.conv_W + 1 + ch - 1) / ch;
    int units = 4;
    while(units < 2 * a.edge + 1) units *= 2;
    if(units > kWgradRingUnits || max_splits < 1) return 0;
    a.x = static_cast<const uint8_t*>(p.B); a.dy = static_cast<const uint8_t*>(p.A);
    a.M = static_cast<int>(p.K); a.N = static_cast<int>(p.M); a.C = static_cast<int>(p.conv_C); a.H = p.conv_H; a.W = p.conv_W;
    a.ring    = units * kWgradUnit;
    a.chunks  = static_cast<int>((p.K + ch - 1) / ch);
    a.tiles_m = (a.N + kWgradRows - 1) / kWgradRows;
    a.tiles_n = (a.C + kWgradChannels - 1) / kWgradChannels;
    const int64_t tiles = static_cast<int64_t>(a.tiles_m) * a.tiles_n;
    if(tiles >= (1 << 20)) return 0;
    int64_t splits = 256 / tiles;                                                // a workgroup for each unit
    if(splits > a.chunks / (4 * kWgradWaves)) splits = a.chunks / (4 * kWgradWaves);      // ... of four chunks a wavefront at least
    if(splits > max_splits) splits = max_splits;
    if(splits < 1) splits = 1;
    a.splits = static_cast<int>(splits);
    a.per    = (a.chunks + a.splits * kWgradWaves - 1) / (a.splits * kWgradWaves);
    // The ring's time against the plan's for the gathering GEMM: a start and an end, a wavefront's chunks one after the other, and the partial
    // products' way to memory and back, as in plan_gemm.  Fitted to 843 whole training steps, in which both operands are in cache behind their
    // conversion.  int8 122 of 576 go to the ring, 717 us faster in sum, four slower, by 2 us at most; binary16 208 of 267, 1191 us faster, 29
    // slower, by 1.8 us at most and with dW closer to 64 bits (24x14x14 256->256 59.0 -> 59.7 us, error 1.7e-7 -> 1.0e-7).  A rule on sizes, pixels
    // x C x N from 6e8 and 2.3e8, left 72 and 28 slower, by up to 8 us, and 206 and 109 us ungained.  Of 300 other steps 101 go to the ring, 613 us
    // faster in sum, eleven slower, by 2.3 us at most.
    const double rounds = std::ceil(static_cast<double>(tiles * splits) / 256.0);
    const double parts  = static_cast<double>(splits + 1) * a.N * 9.0 * a.C * 4.0 / 6.24e6;
    const double us     = p.prec == 16 ? 6.2 + 1.05 * a.per * rounds + 3.0 * parts : 11.0 + 1.0 * a.per * rounds + 2.5 * parts;
    if(us >= gemm_us) return 0;
    a.partial = workspace;
    last_wgrad_ring() = a.splits;
    *error = p.prec == 8 ? launch_wgrad<I8Traits>(a, stream) : launch_wgrad<F16Traits>(a, stream);
    return a.splits;
}

}  // namespace qsync
