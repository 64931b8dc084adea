// HBM-bound kernels of the quantized-operator path for gfx950: absmax + scale (two-stage
// reduction), INT8 quantize with optional transposed copy, precision cast / copy with
// optional transpose, standalone dequantize, and column sums (bias gradient).
//
// All of them stream their input once with 16-byte loads per lane when alignment allows,
// reduce at wavefront level with cross-lane shuffles and at block level through LDS, and
// fall back to scalar element access for shapes or pointers that do not meet the vector
// path's alignment rule.
#include "device_utils.h"
#include "kernels.h"

#include <mutex>

#include <type_traits>

namespace qsync {

namespace {

constexpr int kBlock = 256;

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

__device__ __forceinline__ void write_scale(float amax, float qmax, float* scale, float* inv_scale,
                                            float* amax_opt, int64_t i)
{
    float s = 1.0f, iv = 1.0f;
    if(amax != 0.0f)
    {
        s  = __fdiv_rn(amax, qmax);
        iv = __fdiv_rn(qmax, amax);
    }
    scale[i]     = s;
    inv_scale[i] = iv;
    if(amax_opt) amax_opt[i] = amax;
}

// ------------------------------------------------------------------ parts
// A part is the work of one kernel as a value: its arguments and `run(block, lds)`, for workgroups of kThreads threads and
// kLds bytes of LDS.  It is launched by itself (part_kernel) or beside an independent one (two_parts_kernel: the first `na`
// workgroups are a's).  What bounds the small conversions is the launch: a kernel that does nothing takes 2.1 us in a
// replayed graph and 2.7 us of the host otherwise, and few of them fill the chip, so parts that do not wait for each
// other share one.
template <typename P> __global__ __launch_bounds__(P::kThreads) void part_kernel(const P p)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[P::kLds];
    p.run(blockIdx.x, lds);
}
template <typename A, typename B> __global__ __launch_bounds__(A::kThreads) void two_parts_kernel(const A a, const B b, const uint32_t na)
{
    static_assert(A::kThreads == B::kThreads, "one workgroup size");
    __shared__ __attribute__((aligned(16))) uint8_t lds[A::kLds > B::kLds ? A::kLds : B::kLds];
    if(blockIdx.x < na) a.run(blockIdx.x, lds);
    else                b.run(blockIdx.x - na, lds);
}
template <typename P> void launch_part(const P& p, int64_t blocks, hipStream_t st)
{
    part_kernel<P><<<dim3(static_cast<unsigned>(blocks)), dim3(P::kThreads), 0, st>>>(p);
}
template <typename A, typename B> void launch_parts(const A& a, int64_t blocks_a, const B& b, int64_t blocks_b, hipStream_t st)
{
    two_parts_kernel<A, B><<<dim3(static_cast<unsigned>(blocks_a + blocks_b)), dim3(A::kThreads), 0, st>>>(a, b, static_cast<uint32_t>(blocks_a));
}

// Running maximum of |x| over 16-byte vectors.  binary16 magnitudes order like their bit
// patterns with the sign bit cleared, so for binary16 the maximum runs on packed 16-bit
// integers (two elements per VALU operation) and is widened to fp32 once at the end.
typedef unsigned short us2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_absmax_u16(uint32_t m, uint32_t w)
{
    const us2_t a = __builtin_bit_cast(us2_t, m), b = __builtin_bit_cast(us2_t, w & 0x7FFF7FFFu);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, b));
}
__device__ __forceinline__ float half_bits_to_f32(uint32_t h) { return __half2float(__ushort_as_half(static_cast<unsigned short>(h))); }

template <typename T> struct RunMax;
template <> struct RunMax<float>
{
    float m = 0.0f;
    __device__ __forceinline__ void add(const uint4& r)
    {
        m = fmaxf(fmaxf(m, fmaxf(fabsf(__uint_as_float(r.x)), fabsf(__uint_as_float(r.y)))),
                  fmaxf(fabsf(__uint_as_float(r.z)), fabsf(__uint_as_float(r.w))));
    }
    __device__ __forceinline__ void add_scalar(float v) { m = fmaxf(m, fabsf(v)); }
    __device__ __forceinline__ float get() const { return m; }
};
template <> struct RunMax<__half>
{
    uint32_t pk = 0u;
    float    s  = 0.0f;
    __device__ __forceinline__ void add(const uint4& r)
    {
        pk = pk_absmax_u16(pk_absmax_u16(pk, r.x), r.y);
        pk = pk_absmax_u16(pk_absmax_u16(pk, r.z), r.w);
    }
    __device__ __forceinline__ void add_scalar(__half v) { s = fmaxf(s, fabsf(__half2float(v))); }
    __device__ __forceinline__ float get() const
    {
        return fmaxf(s, fmaxf(half_bits_to_f32(pk & 0xFFFFu), half_bits_to_f32(pk >> 16)));
    }
};

// Running sum of squares in fp32 (the squared norm of the indicator statistics).
template <typename T> struct RunSq
{
    float s = 0.0f;
    __device__ __forceinline__ void add(const uint4& r)
    {
        float v[Vec16<T>::N];
        Vec16<T>::decode(r, v);
#pragma unroll
        for(int e = 0; e < Vec16<T>::N; ++e) s = fmaf(v[e], v[e], s);
    }
    __device__ __forceinline__ void add_scalar(T x) { const float v = to_f32(x); s = fmaf(v, v, s); }
};

// ------------------------------------------------------------------ arrival counter
// The per-tensor maximum finishes inside one launch: every block publishes its partial maximum,
// then takes a ticket from an arrival counter; the block that draws the last ticket folds the
// partials (a maximum: the result does not depend on which block that is) and resets the counter
// to zero for the next launch.  The counter lives at the start of the caller's workspace, which
// must be zero before its first use.  Tickets to one address cost about 10 ns each on this
// part, so these kernels run few, large blocks (at most a few hundred).
// Partials are written and read with device-scope atomic accesses (write-through stores, loads
// that bypass the non-coherent cache levels), so no cache-wide flush is needed: a block waits
// until its own partial store has completed, joins its barrier, and only then draws its ticket;
// the last block reads the partials after its ticket has returned.
__device__ __forceinline__ void st_partial(float* p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_partial(const float* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool last_arrival(unsigned int* ctr, unsigned int expected, bool* flag_lds)
{
    __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt(0): this wavefront's partial stores have completed
    __syncthreads();
    if(threadIdx.x == 0)
    {
        const unsigned int t = atomicAdd(ctr, 1u);
        *flag_lds            = (t == expected - 1u);
    }
    __syncthreads();
    return *flag_lds;
}

// ------------------------------------------------------------------ absmax, per tensor
// Each block folds contiguous pieces of the tensor (BLOCK * 8 sixteen-byte vectors each) into one
// partial maximum; the last block to arrive folds the partials and writes amax, scale and
// inverse scale.  With ctr == nullptr only the partials are written (a second launch folds them).
template <typename T, bool VEC, int BLOCK>
__global__ __launch_bounds__(BLOCK) void absmax_tensor_kernel(const T* __restrict__ x, int64_t rows,
                                                              int64_t cols, int64_t ld, float* partial,
                                                              unsigned int* ctr, float qmax, float* scale,
                                                              float* inv_scale, float* amax_opt, float* partial_sq,
                                                              float* sumsq_opt)
{
    __shared__ float  lds[32];
    __shared__ double lds_d[16];
    __shared__ bool   flag;
    RunMax<T>         rm;
    RunSq<T>          sq;                 // only when sumsq_opt is given
    const bool        want_sq = sumsq_opt != nullptr;
    const int64_t     n = rows * cols;
    if(VEC)
    {   // contiguous tensor, 16-byte aligned base
        constexpr int E    = Vec16<T>::N;
        constexpr int U    = 8;                       // 16-byte loads in flight per lane
        const int64_t nvec = n / E;
        const int64_t step = static_cast<int64_t>(gridDim.x) * BLOCK * U;
        const uint4*  xv   = reinterpret_cast<const uint4*>(x);
        for(int64_t c = static_cast<int64_t>(blockIdx.x) * BLOCK * U + threadIdx.x; c < nvec; c += step)
        {
            uint4 v[U];
#pragma unroll
            for(int u = 0; u < U; ++u)
            {
                const int64_t idx = c + static_cast<int64_t>(u) * BLOCK;
                v[u] = idx < nvec ? xv[idx] : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for(int u = 0; u < U; ++u) rm.add(v[u]);
            if(want_sq)
            {
#pragma unroll
                for(int u = 0; u < U; ++u) sq.add(v[u]);
            }
        }
        if(blockIdx.x == 0)
            for(int64_t j = nvec * E + threadIdx.x; j < n; j += BLOCK)
            {
                rm.add_scalar(x[j]);
                if(want_sq) sq.add_scalar(x[j]);
            }
    }
    else
    {
        const int64_t stride = static_cast<int64_t>(gridDim.x) * BLOCK;
        for(int64_t i = static_cast<int64_t>(blockIdx.x) * BLOCK + threadIdx.x; i < n; i += stride)
        {
            const int64_t r = i / cols, c = i - r * cols;
            rm.add_scalar(x[r * ld + c]);
            if(want_sq) sq.add_scalar(x[r * ld + c]);
        }
    }
    const float m = block_reduce_max(rm.get(), lds);
    if(threadIdx.x == 0) st_partial(partial + blockIdx.x, m);
    if(want_sq)
    {
        const float bs = block_reduce_sum(sq.s, lds + 16);
        if(threadIdx.x == 0) st_partial(partial_sq + blockIdx.x, bs);
    }
    if(!ctr) return;
    if(!last_arrival(ctr, gridDim.x, &flag)) return;
    // (Both partials of a block requested together, the sums of squares added up by all threads in a fixed order: by one thread in block
    // order, behind the maxima, 16384x4096 binary16 40.0 -> 32.6 us with cold inputs between other passes.)
    float  mm = 0.0f;
    double d  = 0.0;
    for(int i = threadIdx.x; i < static_cast<int>(gridDim.x); i += BLOCK)
    {
        const float pm = ld_partial(partial + i), ps = want_sq ? ld_partial(partial_sq + i) : 0.0f;
        mm = fmaxf(mm, pm);
        d += static_cast<double>(ps);
    }
    if(want_sq)
    {
        // (up to 64 workgroups' sums are one wavefront's: without the exchange 7x3 5.03 -> 4.90 us, 45x1023 5.31 -> 5.05)
        d = gridDim.x <= kWaveSize ? wave_reduce_sum(d) : block_reduce_sum(d, lds_d);
        if(threadIdx.x == 0) *sumsq_opt = static_cast<float>(d);
    }
    mm = block_reduce_max(mm, lds);
    if(threadIdx.x == 0)
    {
        write_scale(mm, qmax, scale, inv_scale, amax_opt, 0);
        *ctr = 0u;
    }
}

// One maximum per workgroup of a contiguous, 16-byte aligned tensor of whole vectors, for a pass that folds them.
template <typename T> struct BlockMaxima
{
    static constexpr int kThreads = kBlock, kLds = 64, kVectors = kBlock * 8;      // vectors a workgroup has in flight
    const T* x;
    int64_t  n;
    int64_t  blocks;
    float*   partial;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds) const
    {
        const int64_t nvec = n / Vec16<T>::N;
        const uint4*  xv   = reinterpret_cast<const uint4*>(x);
        RunMax<T>     rm;
        for(int64_t c = static_cast<int64_t>(block) * kVectors + threadIdx.x; c < nvec; c += blocks * kVectors)
        {
            uint4 v[8];
#pragma unroll
            for(int u = 0; u < 8; ++u) v[u] = xv[c + u * kBlock < nvec ? c + u * kBlock : nvec - 1];      // (past the end the last one again)
#pragma unroll
            for(int u = 0; u < 8; ++u) rm.add(v[u]);
        }
        const float m = block_reduce_max(rm.get(), reinterpret_cast<float*>(lds));
        if(threadIdx.x == 0) partial[block] = m;
    }
};

// Scale and inverse scale from a maximum some other kernel has collected (a GEMM epilogue); `consume` clears the
// word for the next collection.
struct ScaleFromAmax
{
    static constexpr int kThreads = kBlock, kLds = 16;
    float* amax;
    float  qmax;
    float* scale;
    float* inv_scale;
    int    consume;
    __device__ __forceinline__ void run(uint32_t, uint8_t*) const
    {
        if(threadIdx.x != 0) return;
        const float m = __hip_atomic_load(amax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        write_scale(m, qmax, scale, inv_scale, nullptr, 0);
        if(consume) *amax = 0.0f;
    }
};

// ------------------------------------------------------------------ absmax, per row
// WPR wavefronts per row (1 when there are many rows, 4 = the whole block when there are few),
// up to four 16-byte loads in flight per lane; no second stage.
template <typename T, bool VEC, int WPR>
__global__ __launch_bounds__(kBlock) void absmax_rows_kernel(const T* __restrict__ x, int64_t rows, int64_t cols,
                                                             int64_t ld, float qmax, float* scale, float* inv_scale,
                                                             float* amax_opt)
{
    constexpr int RPB = kBlock / kWaveSize / WPR;       // rows per block
    constexpr int TPR = WPR * kWaveSize;                // threads per row
    __shared__ float lds[kBlock / kWaveSize];
    const int     lane = threadIdx.x % kWaveSize, t = threadIdx.x % TPR;
    const int64_t r    = static_cast<int64_t>(blockIdx.x) * RPB + threadIdx.x / TPR;
    RunMax<T>     rm;
    if(r < rows)
    {
        const T* row  = x + r * ld;
        int64_t  done = 0;
        if(VEC)
        {
            constexpr int E    = Vec16<T>::N;
            const int64_t nvec = cols / E;
            const uint4*  rv   = reinterpret_cast<const uint4*>(row);
            auto         fold = [&](auto ut) {
                constexpr int U = decltype(ut)::value;
                for(int64_t i = t; i < nvec; i += U * TPR)
                {
                    uint4 v[U];
#pragma unroll
                    for(int u = 0; u < U; ++u) v[u] = rv[i + u * TPR < nvec ? i + u * TPR : nvec - 1];      // (past the end the last one again)
#pragma unroll
                    for(int u = 0; u < U; ++u) rm.add(v[u]);
                }
            };
            // As many loads as a lane has vectors, up to four: all four for any row, fp32 14872x120 5.4 us, one 4.6; 8744x408
            // binary16 4.2, one 3.7; 2288x1320 4.1, two 3.9.
            if(nvec <= TPR)          fold(std::integral_constant<int, 1>{});
            else if(nvec <= 2 * TPR) fold(std::integral_constant<int, 2>{});
            else                     fold(std::integral_constant<int, 4>{});
            done = nvec * E;
        }
        for(int64_t c = done + t; c < cols; c += TPR) rm.add_scalar(row[c]);
    }
    float m = wave_reduce_max(rm.get());
    if(WPR > 1)
    {
        if(lane == 0) lds[threadIdx.x / kWaveSize] = m;
        __syncthreads();
        if(t == 0)
        {
            const int w0 = (threadIdx.x / TPR) * WPR;
            for(int w = 1; w < WPR; ++w) m = fmaxf(m, lds[w0 + w]);
        }
    }
    if(t == 0 && r < rows) write_scale(m, qmax, scale, inv_scale, amax_opt, r);
}

// ------------------------------------------------------------------ per-column reductions
// Shared by the per-column absmax (OP_MAX), the column sums of the bias gradient (OP_SUM) and
// their fusion with the tensor-wide absmax (OP_SUMMAX: one pass yields both).
// Stage 1: block (bx, by) reduces rows by*rpb + tr, + gridDim.y*rpb, ... of a strip of tpr*E
// columns, four rows in flight per lane.  Lanes own adjacent columns (one 16-byte vector each
// when VEC); the block's row lanes are folded through LDS, so partial[by][c] holds one value
// per block row; a second launch folds those, and with OP_SUMMAX one more block of it folds the block maxima: a launch that is
// needed anyway, where an arrival counter in the streaming pass cost 7 us of dependent device-scope round trips
// (4096x3072 binary16 14.9 + 4.0 us with it).
enum { OP_MAX = 0, OP_SUM = 1, OP_SUMMAX = 2 };

struct TensorFinal          // OP_SUMMAX: where the tensor-wide result goes
{
    float         qmax;
    float*        scale;
    float*        inv_scale;
    float*        amax_opt;
    float*        partial_sq;   // per-block sums of squares and their total (indicator statistics), or nullptr
    float*        sumsq_opt;
};

template <typename T, bool VEC, int OP, int BLOCK>
__global__ __launch_bounds__(BLOCK) void colreduce_kernel(const T* __restrict__ x, int64_t rows, int64_t cols,
                                                          int64_t ld, int tpr, float* partial, float* partial_max,
                                                          const TensorFinal fin)
{
    constexpr int E = VEC ? Vec16<T>::N : 1;
    constexpr int U = 4;      // rows in flight per lane (eight: 16384x4096 binary16 28.2 -> 30.3 us, 4096x3072 14.3 -> 15.1)
    __shared__ __attribute__((aligned(16))) float lds[BLOCK * E];
    __shared__ float lds_max[16];
    RunMax<T>        rm;                                    // OP_SUMMAX only
    float            sqv     = 0.0f;                        // OP_SUMMAX with fin.sumsq_opt: sum of squares
    const bool       want_sq = OP == OP_SUMMAX && fin.sumsq_opt != nullptr;
    const int     rpb = BLOCK / tpr;                       // row lanes per block
    const int     tc = threadIdx.x % tpr, tr = threadIdx.x / tpr;
    const int64_t c0  = (static_cast<int64_t>(blockIdx.x) * tpr + tc) * E;
    const int64_t S   = static_cast<int64_t>(gridDim.y) * rpb;
    float    acc[E];
    uint32_t pk[4] = {0u, 0u, 0u, 0u};                      // packed binary16 maxima (VEC, OP_MAX, binary16)
    constexpr bool kPacked = VEC && OP == OP_MAX && sizeof(T) == 2;
#pragma unroll
    for(int e = 0; e < E; ++e) acc[e] = 0.0f;
    if(c0 < cols)
    {
        for(int64_t r = static_cast<int64_t>(blockIdx.y) * rpb + tr; r < rows; r += S * U)
        {
            if(VEC)
            {
                uint4 raw[U];
#pragma unroll
                for(int u = 0; u < U; ++u)
                {
                    const int64_t rr = r + u * S;        // rows past the end contribute zeros (neutral for sum and max; a load of
                    // the last row and a choice behind it instead of the branch: 4096x3072x768 INT8 step 78.8 -> 79.8 us)
                    raw[u] = rr < rows ? *reinterpret_cast<const uint4*>(x + rr * ld + c0) : make_uint4(0, 0, 0, 0);
                }
#pragma unroll
                for(int u = 0; u < U; ++u)
                {
                    if(kPacked)
                    {
                        pk[0] = pk_absmax_u16(pk[0], raw[u].x); pk[1] = pk_absmax_u16(pk[1], raw[u].y);
                        pk[2] = pk_absmax_u16(pk[2], raw[u].z); pk[3] = pk_absmax_u16(pk[3], raw[u].w);
                    }
                    else
                    {
                        float v[Vec16<T>::N];
                        Vec16<T>::decode(raw[u], v);
#pragma unroll
                        for(int e = 0; e < E; ++e) acc[e] = OP == OP_MAX ? fmaxf(acc[e], fabsf(v[e])) : acc[e] + v[e];
                        if(OP == OP_SUMMAX) rm.add(raw[u]);
                        if(want_sq)
                        {
#pragma unroll
                            for(int e = 0; e < E; ++e) sqv = fmaf(v[e], v[e], sqv);
                        }
                    }
                }
            }
            else
            {
#pragma unroll
                for(int u = 0; u < U; ++u)
                {
                    const int64_t rr = r + u * S;
                    if(rr < rows)
                    {
                        const T     xv = x[rr * ld + c0];
                        const float v  = to_f32(xv);
                        acc[0] = OP == OP_MAX ? fmaxf(acc[0], fabsf(v)) : acc[0] + v;
                        if(OP == OP_SUMMAX) rm.add_scalar(xv);
                        if(want_sq) sqv = fmaf(v, v, sqv);
                    }
                }
            }
        }
    }
    if(kPacked)
    {
#pragma unroll
        for(int e = 0; e < E; ++e) acc[e] = half_bits_to_f32((pk[e / 2] >> (16 * (e % 2))) & 0xFFFFu);
    }
    if(OP == OP_SUMMAX)
    {   // every thread of the block takes part (threads beyond the last column carry 0)
        const float bm = block_reduce_max(rm.get(), lds_max);
        if(threadIdx.x == 0) partial_max[blockIdx.y * gridDim.x + blockIdx.x] = bm;
        if(want_sq)
        {
            __syncthreads();
            const float bs = block_reduce_sum(sqv, lds_max);
            if(threadIdx.x == 0) fin.partial_sq[blockIdx.y * gridDim.x + blockIdx.x] = bs;
        }
    }
    // fold the block's row lanes in order 0, 1, ... through LDS, a column per thread (consecutive threads, consecutive
    // banks; one row lane folding eight columns each met eight-way conflicts with fifteen of sixteen wavefronts idle)
#pragma unroll
    for(int e = 0; e < E; e += (E % 4 == 0 ? 4 : 1))
    {
        if constexpr(E % 4 == 0)
            *reinterpret_cast<float4*>(lds + (tr * tpr + tc) * E + e) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
        else
            lds[(tr * tpr + tc) * E + e] = acc[e];
    }
    __syncthreads();
    const int strip = tpr * E;
    for(int t = threadIdx.x; t < strip; t += BLOCK)
    {
        const int64_t c = static_cast<int64_t>(blockIdx.x) * strip + t;
        if(c >= cols) break;
        float v = lds[t];
        for(int q = 1; q < rpb; ++q)
        {
            const float o = lds[q * strip + t];
            v = OP == OP_MAX ? fmaxf(v, o) : v + o;
        }
        partial[static_cast<int64_t>(blockIdx.y) * cols + c] = v;
    }
}

// Second launch of the two-launch form: 16 columns per block; sixteen threads per column fold a
// sixteenth of the partials each (fixed assignment, fixed order), then the sixteen are folded in order.
// OP_SUMMAX: the last block folds the `nmax` block maxima (and sums of squares) of the tensor instead.
template <int OP>
__global__ __launch_bounds__(kBlock) void colreduce_finalize_kernel(const float* __restrict__ partial, int S,
                                                                    int64_t cols, float qmax, float* out,
                                                                    float* inv_scale, float* amax_opt,
                                                                    const float* __restrict__ partial_max, int nmax,
                                                                    const TensorFinal fin)
{
    __shared__ float lds[kBlock];
    if constexpr(OP == OP_SUMMAX)
        if(blockIdx.x == gridDim.x - 1)
        {
            __shared__ double lds_d[16];
            float             mm = 0.0f;
            double            d  = 0.0;
            for(int i = threadIdx.x; i < nmax; i += kBlock)
            {
                mm = fmaxf(mm, partial_max[i]);
                if(fin.sumsq_opt) d += static_cast<double>(fin.partial_sq[i]);
            }
            mm = block_reduce_max(mm, lds);
            if(threadIdx.x == 0) write_scale(mm, fin.qmax, fin.scale, fin.inv_scale, fin.amax_opt, 0);
            if(fin.sumsq_opt)
            {
                d = block_reduce_sum(d, lds_d);
                if(threadIdx.x == 0) *fin.sumsq_opt = static_cast<float>(d);
            }
            return;
        }
    const int     tc = threadIdx.x % 16, q = threadIdx.x / 16;
    const int64_t c  = static_cast<int64_t>(blockIdx.x) * 16 + tc;
    const float   t  = fold_column<OP == OP_MAX>(partial, S, cols, c, q, lds);
    if(q == 0 && c < cols)
    {
        if(OP == OP_MAX)
            write_scale(t, qmax, out, inv_scale, amax_opt, c);
        else
            out[c] = t;
    }
}

// The fold of the column sums beside the pass that needs the block maxima.
template <int THREADS> struct ColumnFold
{
    static constexpr int kThreads = THREADS, kLds = kBlock * 4;
    ColumnFoldArgs f;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds) const { fold_columns(f, block, reinterpret_cast<float*>(lds)); }
};

// Column sums of a small tensor in one go: 16 columns per workgroup, THREADS / 16 row lanes, folded in order.  At most
// kColumnSumRows rows: of 512 threads that is two batches of eight loads in flight per lane.
constexpr int64_t kColumnSumRows = 512;
template <typename T, int THREADS> struct ColumnSum
{
    static constexpr int kThreads = THREADS, kLds = THREADS * 4;
    const T* x;
    int64_t  rows, cols;
    float*   out;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds) const
    {
        constexpr int LANES = THREADS / 16;
        float*        part = reinterpret_cast<float*>(lds);
        const int     tc = threadIdx.x % 16, q = threadIdx.x / 16;
        const int64_t c   = static_cast<int64_t>(block) * 16 + tc;
        float         acc = 0.0f;
        if(c < cols)
#pragma unroll 8
            for(int64_t r = q; r < rows; r += LANES) acc += to_f32(x[r * cols + c]);
        part[threadIdx.x] = acc;
        __syncthreads();
        if(q != 0 || c >= cols) return;
        float t = 0.0f;
        for(int i = 0; i < LANES; ++i) t += part[i * 16 + tc];
        out[c] = t;
    }
};

// ------------------------------------------------------------------ INT8 quantize, tiled through LDS
// A workgroup owns a tile of TR rows x 128 columns, a thread four rows x eight columns of it (one Philox block per
// row, four 16-byte loads in flight for binary16, eight for fp32).  The codes of a row leave as 8-byte stores, 128
// contiguous bytes per tile row; the transposed copy goes through LDS as dwords of four rows (a 4x4 byte transpose in
// registers) and leaves as 16-byte stores, TR contiguous bytes per column.  16-byte chunks of a column are
// XOR-swizzled with (column / 8) % 8: writes are two-way, reads conflict free.
// What bounds it is memory latency at small sizes: against one 16 x 32-byte patch per lane with strided 8 or 16-byte
// transposed stores this keeps four times the wavefronts in flight and writes whole lines.
constexpr int kTileCols = 128;

// Maximum over the whole workgroup, handed to every thread.
template <int THREADS> __device__ __forceinline__ float block_max_all(float v, float* lds /* THREADS / 64 floats */)
{
    v = wave_reduce_max(v);
    if(threadIdx.x % kWaveSize == 0) lds[threadIdx.x / kWaveSize] = v;
    __syncthreads();
    float m = lds[0];
#pragma unroll
    for(int w = 1; w < THREADS / kWaveSize; ++w) m = fmaxf(m, lds[w]);
    return m;
}

// Where a per-tensor quantizer takes its scale from.  kInv: the inverse scale in memory.  kPartials: block maxima of
// an earlier launch, folded by every workgroup (a few loads per thread, hidden behind the tile's own loads), which saves the
// maximum pass its arrival counter -- 5 us of dependent device-scope round trips -- and this pass a launch between them.  kWhole: the workgroup finds the maximum of the whole tensor by itself.
enum ScaleFrom { kInv = 0, kPartials = 1, kWhole = 2 };
constexpr int     kFoldMax    = 256;
constexpr int64_t kWholeBytes = 128 << 10;      // largest tensor of kWhole
struct TensorScale
{
    const float* inv;            // kInv
    const float* partial;        // kPartials: n block maxima
    int          n;
    float*       scale;          // kPartials, kWhole: written by workgroup 0
    float*       inv_out;
    float*       amax_opt;
};

// The inverse scale of the tensor in every thread (contains barriers; lds: THREADS / 64 floats).
template <typename T, int SRC, int THREADS>
__device__ __forceinline__ float tensor_inverse_scale(const TensorScale& ts, const T* __restrict__ x, int64_t n, int qmax,
                                                      uint32_t block, float* lds)
{
    if constexpr(SRC == kInv) return ts.inv[0];
    float m = 0.0f;
    if constexpr(SRC == kPartials)
    {
#pragma unroll 4
        for(int i = threadIdx.x; i < ts.n; i += THREADS) m = fmaxf(m, ts.partial[i]);
    }
    else
    {   // (contiguous, 16-byte aligned, whole vectors)  all of it in flight at once
        constexpr int kQuarter = static_cast<int>(kWholeBytes / 64 / THREADS);
        const int64_t nvec  = n / Vec16<T>::N;
        const uint4*  xv    = reinterpret_cast<const uint4*>(x);
        RunMax<T>     rm;
        auto fold = [&](auto ut) {
            constexpr int U = decltype(ut)::value;
            for(int64_t c = threadIdx.x; c < nvec; c += static_cast<int64_t>(THREADS) * U)
            {
                uint4 v[U];
#pragma unroll
                for(int u = 0; u < U; ++u) v[u] = xv[c + u * THREADS < nvec ? c + u * THREADS : nvec - 1];      // (past the end the last one again)
#pragma unroll
                for(int u = 0; u < U; ++u) rm.add(v[u]);
            }
        };
        // As many quarters of the requests as hold the tensor: all four, most on the last vector again, 64x128 fp32 with its
        // column sums 4.7 us, one 3.8; evaluating 45 rows of 4096x1024 (90 KB: three) 9.8 -> 9.2.
        if(nvec <= kQuarter * THREADS)          fold(std::integral_constant<int, kQuarter>{});
        else if(nvec <= 2 * kQuarter * THREADS) fold(std::integral_constant<int, 2 * kQuarter>{});
        else if(nvec <= 3 * kQuarter * THREADS) fold(std::integral_constant<int, 3 * kQuarter>{});
        else                                    fold(std::integral_constant<int, 4 * kQuarter>{});
        m = rm.get();
    }
    m = block_max_all<THREADS>(m, lds);
    if(block == 0 && threadIdx.x == 0) write_scale(m, static_cast<float>(qmax), ts.scale, ts.inv_out, ts.amax_opt, 0);
    return m != 0.0f ? __fdiv_rn(static_cast<float>(qmax), m) : 1.0f;
}

// One thread's share of a tile: rows r0 .. r0 + 3, columns c0 .. c0 + 7 of at least one row and eight columns.  Absent ones raise no
// maximum and their codes are not stored.  Weights (REPEAT) repeat the last row and columns: with each load under a condition, i.e. in
// a branch of its own, converting 192x72 weights took 7.7 us in place of 7.1, 2 % more over 64..4096 by 64..4096.  Elsewhere the
// conditions are the faster: fp32 2096x80 with its transposed copy 3.28 us without them, 3.15 with; maximum and codes of 16x808, where the
// search for the maximum needs the registers, 4.4 and 3.7; both int8 operands of a 32->32 convolution over 16 pixels 9.3 and 8.6.
template <typename T, bool REPEAT> struct TileShare
{
    static constexpr int VG = 8 / Vec16<T>::N;       // 16-byte loads per row
    uint4 raw[4][VG];
    __device__ __forceinline__ void load(const T* __restrict__ x, int64_t r0, int64_t c0, int64_t rows, int64_t cols, int64_t ld)
    {
        const int64_t c = !REPEAT || c0 < cols ? c0 : cols - 8;
#pragma unroll
        for(int i = 0; i < 4; ++i)
        {
            const bool absent = r0 + i >= rows;
            const T*   row    = x + (REPEAT && absent ? rows - 1 : r0 + i) * ld + c;
#pragma unroll
            for(int l = 0; l < VG; ++l)
                raw[i][l] = REPEAT || (!absent && c0 < cols) ? *reinterpret_cast<const uint4*>(row + l * Vec16<T>::N) : make_uint4(0, 0, 0, 0);
        }
    }
    __device__ __forceinline__ void decode(int i, float (&v)[8]) const
    {
#pragma unroll
        for(int l = 0; l < VG; ++l)
        {
            float t[Vec16<T>::N];
            Vec16<T>::decode(raw[i][l], t);
#pragma unroll
            for(int e = 0; e < Vec16<T>::N; ++e) v[l * Vec16<T>::N + e] = t[e];
        }
    }
};

// 4 x 8 codes (two dwords per row) -> eight dwords, one per column, row 0 in the low byte
__device__ __forceinline__ void transpose_codes_4x8(const uint32_t (&code)[4][2], uint32_t (&t)[8])
{
#pragma unroll
    for(int w = 0; w < 2; ++w)
    {   // v_perm_b32: selector bytes 0-3 take from the second operand, 4-7 from the first
        const uint32_t lo01 = __builtin_amdgcn_perm(code[1][w], code[0][w], 0x05010400u);
        const uint32_t hi01 = __builtin_amdgcn_perm(code[1][w], code[0][w], 0x07030602u);
        const uint32_t lo23 = __builtin_amdgcn_perm(code[3][w], code[2][w], 0x05010400u);
        const uint32_t hi23 = __builtin_amdgcn_perm(code[3][w], code[2][w], 0x07030602u);
        t[4 * w + 0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        t[4 * w + 1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        t[4 * w + 2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        t[4 * w + 3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
    }
}

// Transposed codes of a tile through LDS: `trow(c)` is the row of qT that column c lands in.
template <int TR, typename F>
__device__ __forceinline__ void store_transposed_tile(const uint32_t (&t)[8], uint8_t* lds_t, int64_t tile_r, int64_t tile_c,
                                                      int64_t rows, int64_t cols, int8_t* __restrict__ qT, F&& trow)
{
    constexpr int THREADS = TR * 4, CH = TR / 16;            // 16-byte chunks per column
    const int cg = threadIdx.x % 16, quad = threadIdx.x / 16;
#pragma unroll
    for(int j = 0; j < 8; ++j)
        *reinterpret_cast<uint32_t*>(lds_t + (8 * cg + j) * TR + (((quad / 4) ^ (cg % CH)) * 16) + (quad % 4) * 4) = t[j];
    __syncthreads();
    if(rows <= TR && rows % 16 != 0 && (reinterpret_cast<uintptr_t>(qT) & 3) == 0 && trow(tile_c) == tile_c)
    {   // the tile holds whole columns of odd length, i.e. one contiguous piece of qT: dwords across column ends
        const uint32_t len = static_cast<uint32_t>(cols - tile_c < kTileCols ? cols - tile_c : kTileCols) * static_cast<uint32_t>(rows);
        const uint32_t h   = static_cast<uint32_t>(rows);
        int8_t*        dst = qT + tile_c * rows;
        for(uint32_t w = threadIdx.x; 4 * w < len; w += THREADS)
        {
            uint32_t col = 4 * w / h, r = 4 * w - col * h, v = 0u;
#pragma unroll
            for(int b = 0; b < 4; ++b)
            {
                if(4 * w + b < len)
                    v |= static_cast<uint32_t>(lds_t[col * TR + (((r / 16) ^ ((col / 8) % CH)) * 16) + r % 16]) << (8 * b);
                if(++r == h) { r = 0u; ++col; }
            }
            if(4 * w + 4 <= len)
                *reinterpret_cast<uint32_t*>(dst + 4 * w) = v;
            else
                for(uint32_t b = 0; 4 * w + b < len; ++b) dst[4 * w + b] = static_cast<int8_t>((v >> (8 * b)) & 0xFFu);
        }
        return;
    }
    const bool dwords = rows % 4 == 0 && (reinterpret_cast<uintptr_t>(qT) & 3) == 0;      // (300x2048: 6.3 us by bytes, 4.9)
#pragma unroll
    for(int k = threadIdx.x; k < kTileCols * CH; k += THREADS)
    {
        const int     col = k / CH, ch = k % CH;
        const uint4   v   = *reinterpret_cast<const uint4*>(lds_t + col * TR + ((ch ^ ((col / 8) % CH)) * 16));
        const int64_t r   = tile_r + 16 * ch, c = tile_c + col;
        if(c >= cols || r >= rows) continue;
        int8_t* dst = qT + trow(c) * rows + r;
        if(rows % 16 == 0)
            *reinterpret_cast<uint4*>(dst) = v;
        else
        {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            if(dwords)
#pragma unroll
                for(int b = 0; b < 4; ++b)
                {
                    if(r + 4 * b < rows) reinterpret_cast<uint32_t*>(dst)[b] = w[b];
                }
            else
#pragma unroll
                for(int b = 0; b < 16; ++b)
                    if(r + b < rows) dst[b] = static_cast<int8_t>((w[b / 4] >> (8 * (b % 4))) & 0xFFu);
        }
    }
}

// Per-tensor scale.  Needs cols % 8 == 0, 16-byte aligned rows of x, 8-byte aligned q; qT 16-byte aligned when
// rows % 16 == 0 (any alignment and byte stores otherwise).
template <typename T, int RND, int TR, int SRC> struct QuantizeTile
{
    static constexpr int kThreads = TR * 4, kLds = TR * kTileCols + kThreads / kWaveSize * 4;
    const T*    x;
    int64_t     rows, cols, ld;
    int         qmax;
    uint64_t    seed, offset;
    TensorScale ts;
    int8_t*     q;
    int8_t*     qT;
    int         tiles_x;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds) const
    {
        const int     by = static_cast<int>(block) / tiles_x, bx = static_cast<int>(block) - by * tiles_x;
        const int64_t tile_r = static_cast<int64_t>(by) * TR, tile_c = static_cast<int64_t>(bx) * kTileCols;
        const int64_t r0 = tile_r + (threadIdx.x / 16) * 4, c0 = tile_c + (threadIdx.x % 16) * 8;
        TileShare<T, false> s;
        s.load(x, r0, c0, rows, cols, ld);
        const float   inv = tensor_inverse_scale<T, SRC, kThreads>(ts, x, rows * cols, qmax, block, reinterpret_cast<float*>(lds + TR * kTileCols));
        uint32_t      code[4][2];
#pragma unroll
        for(int i = 0; i < 4; ++i)
        {
            float v[8];
            s.decode(i, v);
            uint4 blk = {0u, 0u, 0u, 0u};
            if(RND == kStochastic) blk = philox_group(seed, offset, static_cast<uint64_t>((r0 + i) * cols + c0) >> 3);
            quantize_group<T, RND>(v, inv, qmax, blk, code[i]);
            if(q && r0 + i < rows && c0 < cols) *reinterpret_cast<uint2*>(q + (r0 + i) * cols + c0) = make_uint2(code[i][0], code[i][1]);
        }
        if(!qT) return;
        uint32_t t[8];
        transpose_codes_4x8(code, t);
        store_transposed_tile<TR>(t, lds, tile_r, tile_c, rows, cols, qT, [](int64_t c) { return c; });
    }
};

// ------------------------------------------------------------------ weights: two quantizations in two launches
// The forward wants codes with one scale per row, dX transposed codes with one scale per column.  The first launch
// leaves, per 64 x 128 tile, the maxima of its rows (row_part[bx][row]) and -- per group of row tiles, at most
// kWeightGroups of them -- of its columns (col_part[by][col]).  The second folds what its own tile needs of both
// (a few loads per thread, behind the tile's own loads), so no launch stands between them to fold anything, and
// converts; the first tile column and tile row write the scales out.  Maxima are order free: the results are those of
// the separate passes.
constexpr int kWeightTileRows = 64, kWeightGroups = 64;

template <typename T> struct WeightMaxima
{
    static constexpr int kThreads = 256, kLds = 4 * kTileCols * 4;
    const T* x;
    int64_t  rows, cols;
    int      tiles_x, groups;
    float*   row_part;
    float*   col_part;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds_bytes) const
    {
        constexpr int TR = kWeightTileRows;
        float (*lds)[kTileCols] = reinterpret_cast<float (*)[kTileCols]>(lds_bytes);
        const int     by = static_cast<int>(block) / tiles_x, bx = static_cast<int>(block) - by * tiles_x;
        const int     cg = threadIdx.x % 16, quad = threadIdx.x / 16;
        const int64_t c0 = static_cast<int64_t>(bx) * kTileCols + cg * 8;
        float         cm[8];
#pragma unroll
        for(int j = 0; j < 8; ++j) cm[j] = 0.0f;
        for(int64_t tile_r = static_cast<int64_t>(by) * TR; tile_r < rows; tile_r += static_cast<int64_t>(groups) * TR)
        {
            const int64_t r0 = tile_r + quad * 4;
            TileShare<T, true> s;
            s.load(x, r0, c0, rows, cols, cols);
#pragma unroll
            for(int i = 0; i < 4; ++i)
            {
                float v[8], rm = 0.0f;
                s.decode(i, v);
#pragma unroll
                for(int j = 0; j < 8; ++j)
                {
                    const float a = fabsf(v[j]);
                    cm[j] = fmaxf(cm[j], a);
                    rm    = fmaxf(rm, a);
                }
#pragma unroll
                for(int off = 8; off > 0; off >>= 1) rm = fmaxf(rm, __shfl_xor(rm, off, kWaveSize));     // the 16 lanes of a row
                if(cg == 0 && r0 + i < rows) row_part[bx * rows + r0 + i] = rm;
            }
        }
#pragma unroll
        for(int j = 0; j < 8; ++j)
        {   // the four row quads of the wavefront, then the four wavefronts
            cm[j] = fmaxf(cm[j], __shfl_xor(cm[j], 16, kWaveSize));
            cm[j] = fmaxf(cm[j], __shfl_xor(cm[j], 32, kWaveSize));
        }
        if(quad % 4 == 0)
#pragma unroll
            for(int j = 0; j < 8; ++j) lds[quad / 4][cg * 8 + j] = cm[j];
        __syncthreads();
        const int64_t c = static_cast<int64_t>(bx) * kTileCols + threadIdx.x;
        if(threadIdx.x < kTileCols && c < cols)
            col_part[by * cols + c] = fmaxf(fmaxf(lds[0][threadIdx.x], lds[1][threadIdx.x]), fmaxf(lds[2][threadIdx.x], lds[3][threadIdx.x]));
    }
};

struct WeightOut
{
    float*  row_scale; float* row_inv; float* row_amax_opt;
    float*  col_scale; float* col_inv;
    int8_t* wq;
    int8_t* wqT;
};
// conv_C > 0 (3x3 convolution weights [N, 9 * C]): the column scale belongs to the input channel c = column % C, i.e. it
// covers the nine columns (tap, c), and column (tap, c) lands in row c * 9 + (8 - tap) of the transposed copy, the
// mirrored, channel-exchanged weights.
template <typename T> struct WeightQuantize
{
    static constexpr int TR = kWeightTileRows, kThreads = 256, kLds = TR * kTileCols + (3 * kTileCols + 5 * TR) * 4;
    const T*     x;
    int64_t      rows, cols;
    int          qmax, tiles_x, groups;
    const float* row_part;       // may be o.row_scale
    const float* col_part;
    WeightOut    o;
    int          conv_C;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds_t) const
    {
        float (*lds_c)[kTileCols] = reinterpret_cast<float (*)[kTileCols]>(lds_t + TR * kTileCols);
        float (*lds_r)[TR]        = reinterpret_cast<float (*)[TR]>(lds_c + 2);
        float *inv_c = reinterpret_cast<float*>(lds_r + 4), *inv_r = inv_c + kTileCols;
        const int     by = static_cast<int>(block) / tiles_x, bx = static_cast<int>(block) - by * tiles_x;
        const int64_t tile_r = static_cast<int64_t>(by) * TR, tile_c = static_cast<int64_t>(bx) * kTileCols;
        const int     cg = threadIdx.x % 16, quad = threadIdx.x / 16;
        const int64_t r0 = tile_r + quad * 4, c0 = tile_c + cg * 8;
        TileShare<T, true> s;
        s.load(x, r0, c0, rows, cols, cols);
        {   // columns: two threads each; rows: four threads each
            // (half and part are whole wavefronts': which partials a lane folds is decided, and multiplied out, on the scalar unit; by the
            // lanes, with a 64-bit product for each load, 4096x2376 26.9 us for both launches, so 26.3, before the joint requests 25.7)
            static_assert(kTileCols % kWaveSize == 0 && TR % kWaveSize == 0, "wavefronts of one half, of one part");
            const int     cc = threadIdx.x % kTileCols, half = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kTileCols);
            const int64_t c  = tile_c + cc;
            const int     rr = threadIdx.x % TR, part = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / TR);
            const int64_t r  = tile_r + rr;
            const int64_t step = conv_C > 0 ? conv_C : cols;              // conv: [groups][9][C] read as groups * 9 rows of C
            const int     n    = conv_C > 0 ? groups * 9 : groups;
            const int64_t ca   = c < cols ? c : cols - 1, ra = r < rows ? r : rows - 1;      // (absent ones: any, not used)
            const int64_t cs   = conv_C > 0 ? static_cast<int64_t>(static_cast<uint32_t>(ca) % static_cast<uint32_t>(conv_C)) : ca;
            // Rows and the first batch of columns are requested together, in front of the first wait, past the end the last one
            // again (a maximum does not mind): in loops of four and eight with remainders they were up to four more memory
            // latencies in a row.  Whole INT8 steps, us: 384x1920x736 39.8 -> 38.1, 1120x624x512 35.0 -> 33.9.  (Requested under
            // conditions of their own, i.e. a branch a load, they were slower than the loops: convolution 48->416 60.5 -> 64.4.)
            float pr[4], pc[8], mr = 0.0f, mc = 0.0f;
#pragma unroll
            for(int i = 0; i < 4; ++i) pr[i] = (row_part + (part + 4 * i < tiles_x ? part + 4 * i : tiles_x - 1) * rows)[ra];
            for(int g = half; g < n; g += 16)
            {
#pragma unroll
                for(int i = 0; i < 8; ++i) pc[i] = (col_part + (g + 2 * i < n ? g + 2 * i : n - 1) * step)[cs];
#pragma unroll
                for(int i = 0; i < 8; ++i) mc = fmaxf(mc, pc[i]);
            }
#pragma unroll
            for(int i = 0; i < 4; ++i) mr = fmaxf(mr, pr[i]);
#pragma unroll 4
            for(int b = part + 16; b < tiles_x; b += 4) mr = fmaxf(mr, (row_part + b * rows)[ra]);
            lds_c[half][cc]  = mc;
            lds_r[part][rr] = mr;
        }
        __syncthreads();
        const float fq = static_cast<float>(qmax);
        if(threadIdx.x < kTileCols)
        {
            const int     t = threadIdx.x;
            const float   m = fmaxf(lds_c[0][t], lds_c[1][t]);
            const int64_t c = tile_c + t;
            inv_c[t] = m != 0.0f ? __fdiv_rn(fq, m) : 1.0f;
            if(by == 0 && c < (conv_C > 0 ? conv_C : cols)) write_scale(m, fq, o.col_scale, o.col_inv, nullptr, c);
        }
        else if(threadIdx.x < kTileCols + TR)
        {
            const int     t = threadIdx.x - kTileCols;
            const float   m = fmaxf(fmaxf(lds_r[0][t], lds_r[1][t]), fmaxf(lds_r[2][t], lds_r[3][t]));
            inv_r[t] = m != 0.0f ? __fdiv_rn(fq, m) : 1.0f;
            if(bx == 0 && tile_r + t < rows) write_scale(m, fq, o.row_scale, o.row_inv, o.row_amax_opt, tile_r + t);
        }
        __syncthreads();
        float fc[8];
#pragma unroll
        for(int j = 0; j < 8; ++j) fc[j] = inv_c[cg * 8 + j];
        uint32_t codeT[4][2];
#pragma unroll
        for(int i = 0; i < 4; ++i)
        {
            float v[8];
            s.decode(i, v);
            const float fr = inv_r[quad * 4 + i];
            uint32_t    code[2] = {0u, 0u};
            codeT[i][0] = codeT[i][1] = 0u;
#pragma unroll
            for(int j = 0; j < 8; ++j)
            {
                code[j / 4]     |= (static_cast<uint32_t>(quantize_code<kNearest>(v[j], fr, qmax, 0u)) & 0xFFu) << (8 * (j % 4));
                codeT[i][j / 4] |= (static_cast<uint32_t>(quantize_code<kNearest>(v[j], fc[j], qmax, 0u)) & 0xFFu) << (8 * (j % 4));
            }
            if(r0 + i < rows && c0 < cols) *reinterpret_cast<uint2*>(o.wq + (r0 + i) * cols + c0) = make_uint2(code[0], code[1]);
        }
        uint32_t t[8];
        transpose_codes_4x8(codeT, t);
        store_transposed_tile<TR>(t, lds_t, tile_r, tile_c, rows, cols, o.wqT, [&](int64_t c) {
            if(conv_C == 0) return c;
            const uint32_t tap = static_cast<uint32_t>(c) / static_cast<uint32_t>(conv_C);
            return (c - static_cast<int64_t>(tap) * conv_C) * 9 + (8 - tap);
        });
    }
};

// ------------------------------------------------------------------ INT8 quantize, vector path of per-row and per-column scales
// Each lane owns a patch of 16 (or 8) rows x 32 input bytes (16 binary16 or 8 fp32 columns) and
// requests the eight 16-byte loads of four rows together before it converts them.  A wavefront is up
// to 8 patches wide (fewer for narrow matrices, so that no lane idles) and the rest of its lanes
// stack patches downwards, so every load instruction covers whole 256-byte row segments; the int8
// codes of a patch row leave as one 16-byte (8-byte for fp32 input) store, and -- after a byte
// transpose held entirely in registers -- each column of the patch leaves as one 16-byte (8-byte)
// store to the transposed copy, lanes side by side.  No LDS, no barrier.
// Needs cols % 8 == 0 (Philox groups of 8 never straddle a row), rows % 16 == 0 when the
// transposed copy is written, and 16-byte aligned rows.

__device__ __forceinline__ uint32_t byte_of(uint32_t w, int b) { return (w >> (8 * b)) & 0xFFu; }

template <typename T, int RND, bool PERCOL, int PR>
__global__ __launch_bounds__(kBlock, 3) void quantize_patch_kernel(const T* __restrict__ x, int64_t rows, int64_t cols,
                                                                int64_t ld, int qmax, uint64_t seed,
                                                                uint64_t offset, const float* __restrict__ inv_scale,
                                                                int8_t* __restrict__ q, int8_t* __restrict__ qT,
                                                                int64_t grid_x, int lpr_log2)
{
    // A lane converts a patch of PR rows x PCOLS columns; the 2^lpr_log2 lanes of a wavefront that share
    // rows cover a contiguous row segment, the other lane bits stack patches downwards.  Narrow matrices
    // use fewer lanes per row (no idle lanes), small ones shorter patches (more wavefronts in flight).
    constexpr int E     = Vec16<T>::N;            // elements per 16-byte load (8 or 4)
    constexpr int PCOLS = 2 * E;                  // patch width: 16 (binary16) or 8 (fp32) columns
    constexpr int NH    = PCOLS / 8;              // 8-column halves per patch row (one Philox block each)
    constexpr int CW    = PCOLS / 4;              // code dwords per patch row
    const int     wtile_r = (kWaveSize >> lpr_log2) * PR, wtile_c = PCOLS << lpr_log2;
    const int     lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
    const int64_t by   = blockIdx.x / grid_x, bx = blockIdx.x - by * grid_x;
    const int64_t r0   = (by * (kBlock / kWaveSize) + wave) * wtile_r + (lane >> lpr_log2) * PR;
    const int64_t c0   = bx * wtile_c + (lane & ((1 << lpr_log2) - 1)) * PCOLS;
    if(r0 >= rows || c0 >= cols) return;
    const bool second_ok = NH == 1 || c0 + 8 < cols;      // binary16: the patch's second 8 columns exist

    float fcol[PCOLS];
    if(PERCOL)
#pragma unroll
        for(int j = 0; j < PCOLS; ++j) fcol[j] = (j < 8 || second_ok) ? inv_scale[c0 + j] : 1.0f;

    uint32_t code[PR][CW];   // row i, columns 4w..4w+3 in dword w
    constexpr int RB = 4;                // rows per batch
#pragma unroll
    for(int batch = 0; batch < PR / RB; ++batch)
    {   // four rows at a time: their 8 loads are requested together, then converted
        uint4 raw[RB][2];
#pragma unroll
        for(int ii = 0; ii < RB; ++ii)
        {
            const int64_t r = r0 + batch * RB + ii;
#pragma unroll
            for(int l = 0; l < 2; ++l)
            {
                const bool ok = r < rows && (l == 0 || second_ok);
                raw[ii][l] = ok ? *reinterpret_cast<const uint4*>(x + r * ld + c0 + l * E) : make_uint4(0, 0, 0, 0);
            }
        }
#pragma unroll
        for(int ii = 0; ii < RB; ++ii)
        {
            const int     i    = batch * RB + ii;
            const int64_t r    = r0 + i;
            const float   frow = (!PERCOL && r < rows) ? inv_scale[r] : 1.0f;
            float         v[PCOLS];
            float         t0[E], t1[E];
            Vec16<T>::decode(raw[ii][0], t0);
            Vec16<T>::decode(raw[ii][1], t1);
#pragma unroll
            for(int e = 0; e < E; ++e)
            {
                v[e]     = t0[e];
                v[E + e] = t1[e];
            }
#pragma unroll
            for(int w = 0; w < CW; ++w) code[i][w] = 0u;
#pragma unroll
            for(int h = 0; h < NH; ++h)
            {
                uint4 blk = {0u, 0u, 0u, 0u};
                if(RND == kStochastic)
                    blk = philox_group(seed, offset, static_cast<uint64_t>(r * cols + c0 + 8 * h) >> 3);
#pragma unroll
                for(int j = 0; j < 8; ++j)
                {
                    const int   col = 8 * h + j;
                    const float f   = PERCOL ? fcol[col] : frow;
                    const int   c   = quantize_code<RND>(v[col], f, qmax, philox_draw16(blk, j));
                    code[i][col / 4] |= (static_cast<uint32_t>(c) & 0xFFu) << (8 * (col % 4));
                }
            }
        }
        // Pin the batch's codes here: otherwise the compiler sinks all conversions behind the last
        // batch's loads and keeps every raw vector of the patch alive (register budget).
#pragma unroll
        for(int ii = 0; ii < RB; ++ii)
#pragma unroll
            for(int w = 0; w < CW; ++w) asm volatile("" : "+v"(code[batch * RB + ii][w]));
    }

    if(q)
    {
#pragma unroll
        for(int i = 0; i < PR; ++i)
        {
            const int64_t r = r0 + i;
            if(r >= rows) continue;
            int8_t* dst = q + r * cols + c0;
            if(NH == 1)
                *reinterpret_cast<uint2*>(dst) = make_uint2(code[i][0], code[i][1]);
            else if(cols % 16 == 0)
                *reinterpret_cast<uint4*>(dst) = make_uint4(code[i][0], code[i][1], code[i][CW - 2], code[i][CW - 1]);
            else
            {
                *reinterpret_cast<uint2*>(dst) = make_uint2(code[i][0], code[i][1]);
                if(second_ok) *reinterpret_cast<uint2*>(dst + 8) = make_uint2(code[i][CW - 2], code[i][CW - 1]);
            }
        }
    }
    if(qT)
    {   // rows % 16 == 0 here, so every row of the patch exists
#pragma unroll
        for(int col = 0; col < PCOLS; ++col)
        {
            if(col >= 8 && !second_ok) continue;
            uint32_t t[PR / 4];
#pragma unroll
            for(int g = 0; g < PR / 4; ++g)
            {
                t[g] = byte_of(code[4 * g + 0][col / 4], col % 4) | (byte_of(code[4 * g + 1][col / 4], col % 4) << 8)
                     | (byte_of(code[4 * g + 2][col / 4], col % 4) << 16)
                     | (byte_of(code[4 * g + 3][col / 4], col % 4) << 24);
            }
            int8_t* dst = qT + (c0 + col) * rows + r0;
            if constexpr(PR == 16)
                *reinterpret_cast<uint4*>(dst) = make_uint4(t[0], t[1], t[2], t[3]);
            else
                *reinterpret_cast<uint2*>(dst) = make_uint2(t[0], t[1]);
        }
    }
}

// ------------------------------------------------------------------ INT8 quantize, row-major codes only
// Contiguous tensor, one scale, no transposed copy: nothing ties a lane to a patch, so the lanes of a wavefront take
// adjacent groups of 8 elements (one Philox block each; a load instruction of a wavefront covers 1 KB of consecutive
// memory for binary16 input) with U groups in flight per lane, and the 8 codes of a group leave as one 8-byte store.
template <typename T, int RND, int SRC> struct QuantizeStream
{
    static constexpr int kThreads = kBlock, kLds = kBlock / kWaveSize * 4;
    const T*    x;
    int64_t     ngroups;
    int         qmax;
    uint64_t    seed, offset;
    TensorScale ts;
    int8_t*     q;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds) const
    {
        constexpr int E  = Vec16<T>::N;       // elements per 16-byte load (8 or 4)
        constexpr int VG = 8 / E;             // loads per group
        constexpr int U  = 4;
        const uint4*  xv = reinterpret_cast<const uint4*>(x);
        const int64_t g0 = static_cast<int64_t>(block) * (kBlock * U) + threadIdx.x;
        uint4         raw[U][VG];
#pragma unroll
        for(int u = 0; u < U; ++u)
        {
            const int64_t g = g0 + u * kBlock < ngroups ? g0 + u * kBlock : ngroups - 1;      // (past the end the last one again, not stored)
#pragma unroll
            for(int l = 0; l < VG; ++l) raw[u][l] = xv[g * VG + l];
        }
        const float f = tensor_inverse_scale<T, SRC, kBlock>(ts, x, ngroups * 8, qmax, block, reinterpret_cast<float*>(lds));
#pragma unroll
        for(int u = 0; u < U; ++u)
        {
            const int64_t g = g0 + u * kBlock;
            if(g >= ngroups) continue;
            float v[8];
#pragma unroll
            for(int l = 0; l < VG; ++l)
            {
                float t[E];
                Vec16<T>::decode(raw[u][l], t);
#pragma unroll
                for(int e = 0; e < E; ++e) v[l * E + e] = t[e];
            }
            uint4 blk = {0u, 0u, 0u, 0u};
            if(RND == kStochastic) blk = philox_group(seed, offset, static_cast<uint64_t>(g));
            uint32_t w[2];
            quantize_group<T, RND>(v, f, qmax, blk, w);
            *reinterpret_cast<uint2*>(q + g * 8) = make_uint2(w[0], w[1]);
        }
    }
};

// The code of element i by itself
template <typename T> __device__ __forceinline__ int8_t code_of(float v, float f, int qmax, int rnd, uint64_t seed, uint64_t offset, int64_t i)
{
    if(rnd == kStochastic)
    {
        const uint4 blk = philox_group(seed, offset, static_cast<uint64_t>(i) >> 3);
        return static_cast<int8_t>(quantize_code<kStochastic>(v, f, qmax, philox_draw16(blk, static_cast<int>(i & 7))));
    }
    return static_cast<int8_t>(rnd == kFloor ? quantize_code<kFloor>(v, f, qmax, 0u) : quantize_code<kNearest>(v, f, qmax, 0u));
}

// QuantizeStream of any number of elements: those behind the last whole group one to a thread.  A group is 8 consecutive elements of the
// contiguous tensor, whatever its rows are: odd row lengths used to go an element per thread (8524x2955 binary16, stochastic,
// with its maximum and dequantization 108 -> 48 us)
template <typename T, int RND> struct QuantizeStreamAny : QuantizeStream<T, RND, kInv>
{
    int tail;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds) const
    {
        QuantizeStream<T, RND, kInv>::run(block, lds);
        const int64_t i = this->ngroups * 8 + threadIdx.x;
        if(block == 0 && static_cast<int>(threadIdx.x) < tail)
            this->q[i] = code_of<T>(to_f32(this->x[i]), *this->ts.inv, this->qmax, RND, this->seed, this->offset, i);
    }
};

// Any shape, any alignment: one element per thread.
template <typename T>
__global__ __launch_bounds__(kBlock) void quantize_generic_kernel(const T* __restrict__ x, int64_t rows, int64_t cols,
                                                                  int64_t ld, int qmax, int gran, int rnd,
                                                                  uint64_t seed, uint64_t offset,
                                                                  const float* __restrict__ inv_scale,
                                                                  int8_t* __restrict__ q, int8_t* __restrict__ qT)
{
    const int64_t n      = rows * cols;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for(int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride)
    {
        const int64_t r = i / cols, c = i - r * cols;
        const float   f = inv_scale[gran == kPerTensor ? 0 : (gran == kPerRow ? r : c)];
        const float   v = to_f32(x[r * ld + c]);
        const int8_t  code = code_of<T>(v, f, qmax, rnd, seed, offset, i);
        if(q) q[i] = code;
        if(qT) qT[c * rows + r] = code;
    }
}

// ------------------------------------------------------------------ 3x3 im2col on int8 codes
// Patches of a 3x3, stride-1, pad-1 convolution built from the already quantized NHWC activation:
// A[m, (kh*3+kw)*C + c] = xq[n, h+kh-1, w+kw-1, c] (0 outside the image), m = (n*H + h)*W + w.
// The codes of the patch matrix equal the codes of the quantized fp16 patch matrix (per-tensor
// scale, zeros map to zero), but the activation is read and quantized once instead of nine times.
// Same lane geometry as the quantizer: a lane owns 16 output pixels x 16 K bytes (one tap, 16
// channels; needs C % 16 == 0), a wavefront 128 pixels x 128 K bytes; row-major rows leave as
// 16-byte stores, the transposed copy after a byte transpose in registers (needs M % 16 == 0).
__global__ __launch_bounds__(kBlock) void im2col3x3_i8_kernel(const int8_t* __restrict__ xq, int64_t nimg, int H, int W,
                                                              int C, int8_t* __restrict__ a, int8_t* __restrict__ aT,
                                                              int64_t grid_x)
{
    const int64_t M  = nimg * H * W;
    const int     K  = 9 * C, nchunk = K / 16;
    const int     lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
    const int64_t by = blockIdx.x / grid_x, bx = blockIdx.x - by * grid_x;
    const int64_t m0 = (by * (kBlock / kWaveSize) + wave) * 128 + (lane / 8) * 16;
    const int     ch = static_cast<int>(bx) * 8 + (lane % 8);             // 16-byte chunk of the K axis
    if(m0 >= M || ch >= nchunk) return;
    const int k0  = ch * 16;
    const int tap = k0 / C, c0 = k0 - tap * C;
    const int dh  = tap / 3 - 1, dw = tap % 3 - 1;
    uint32_t  code[16][4];
#pragma unroll
    for(int i = 0; i < 16; ++i)
    {
        const int64_t m = m0 + i;
        uint4         v = make_uint4(0, 0, 0, 0);
        if(m < M)
        {
            const int64_t hw = m % (static_cast<int64_t>(H) * W), n = m / (static_cast<int64_t>(H) * W);
            const int     h = static_cast<int>(hw / W) + dh, w = static_cast<int>(hw % W) + dw;
            if(h >= 0 && h < H && w >= 0 && w < W)
                v = *reinterpret_cast<const uint4*>(xq + ((n * H + h) * W + w) * C + c0);
        }
        code[i][0] = v.x; code[i][1] = v.y; code[i][2] = v.z; code[i][3] = v.w;
    }
    if(a)
    {
#pragma unroll
        for(int i = 0; i < 16; ++i)
            if(m0 + i < M)
                *reinterpret_cast<uint4*>(a + (m0 + i) * K + k0) = make_uint4(code[i][0], code[i][1], code[i][2], code[i][3]);
    }
    if(aT)
    {   // M % 16 == 0 here, so the 16 pixels all exist
#pragma unroll
        for(int col = 0; col < 16; ++col)
        {
            uint32_t t[4];
#pragma unroll
            for(int g = 0; g < 4; ++g)
                t[g] = byte_of(code[4 * g + 0][col / 4], col % 4) | (byte_of(code[4 * g + 1][col / 4], col % 4) << 8)
                     | (byte_of(code[4 * g + 2][col / 4], col % 4) << 16)
                     | (byte_of(code[4 * g + 3][col / 4], col % 4) << 24);
            *reinterpret_cast<uint4*>(aT + (static_cast<int64_t>(k0) + col) * M + m0) = make_uint4(t[0], t[1], t[2], t[3]);
        }
    }
}

// ------------------------------------------------------------------ padded, transposed pixel layout
// Operands of the convolution's weight gradient, which contracts over the pixels.  The codes [M, Ch] of an
// NHWC tensor are transposed to [Ch, Mp] over a padded pixel axis: every image is preceded by a zero row,
// rows are Wp >= W + 1 pixels long (a multiple of 16, the excess zero), one more zero row closes the axis:
//   p = (img * (H + 1) + 1 + h) * Wp + w.
// On this axis a window offset (dh, dw) is the plain displacement dh * Wp + dw and every out-of-image
// neighbour is a stored zero.  NS = 3 writes the three copies displaced by dw = -1, 0, +1
// (out[s][ch][q] = padded[ch][q + s - 1]), so that the GEMM reads 16-byte aligned rows for every tap;
// NS = 1 writes the undisplaced copy (the gradient operand).  A lane gathers 18 (16) pixels x 16 channels
// and leaves with one 16-byte store per channel and copy; pads are written, nothing is assumed zero.
// ES = element size in bytes (1: int8 codes, 2: binary16); `in`/`out` are byte pointers, Ch counts elements.
template <int NS, int ES>
__global__ __launch_bounds__(kBlock) void conv_padded_transpose_kernel(const int8_t* __restrict__ in, int64_t nimg, int H,
                                                                       int W, int Ch, int Wp, int64_t Mp,
                                                                       int8_t* __restrict__ out, int cw_log2,
                                                                       int margin_bytes)
{
    constexpr int NP  = NS == 3 ? 18 : 16;
    constexpr int CPC = 16 / ES;                  // channels per 16-byte chunk
    // margin_bytes > 0: `out` sits between two margins of that many bytes which the GEMM's displaced rows reach
    // into (multiplied by zeros of the other operand); they are cleared here so that no stale NaN pattern can
    // meet a binary16 zero
    if(margin_bytes > 0 && blockIdx.x == 0)
        for(int t = threadIdx.x * 16; t < margin_bytes; t += kBlock * 16)
        {
            *reinterpret_cast<uint4*>(out - margin_bytes + t) = make_uint4(0, 0, 0, 0);
            *reinterpret_cast<uint4*>(out + static_cast<int64_t>(NS) * Ch * Mp * ES + t) = make_uint4(0, 0, 0, 0);
        }
    const int64_t lin  = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const int     ncc  = Ch / CPC, cw = 1 << cw_log2;
    const int64_t nq   = Mp / 16, rest = lin >> cw_log2;
    const int64_t qb   = rest % nq, ccg = rest / nq;
    const int     cc   = static_cast<int>(ccg) * cw + static_cast<int>(lin & (cw - 1));
    if(cc >= ncc) return;
    const int64_t q0 = qb * 16;
    const int     c0 = cc * CPC;
    // first gathered pixel: q0 - 1 (NS = 3) or q0; position -1 is written as the last column of a row "-1"
    int64_t p0 = q0 - (NS == 3 ? 1 : 0);
    int     col, hrow;
    int64_t img;
    if(p0 < 0) { col = Wp - 1; hrow = H; img = -1; }
    else
    {
        const int64_t r = p0 / Wp;
        col  = static_cast<int>(p0 - r * Wp);
        img  = r / (H + 1);
        hrow = static_cast<int>(r - img * (H + 1));
    }
    uint32_t code[NP][4];
#pragma unroll
    for(int i = 0; i < NP; ++i)
    {
        uint4 v = make_uint4(0, 0, 0, 0);
        if(col < W && hrow >= 1 && img >= 0 && img < nimg)
            v = *reinterpret_cast<const uint4*>(in + (((img * H + (hrow - 1)) * W + col) * Ch + c0) * ES);
        code[i][0] = v.x; code[i][1] = v.y; code[i][2] = v.z; code[i][3] = v.w;
        if(++col == Wp)
        {
            col = 0;
            if(++hrow == H + 1) { hrow = 0; ++img; }
        }
    }
#pragma unroll
    for(int s = 0; s < NS; ++s)
#pragma unroll
        for(int ch = 0; ch < CPC; ++ch)
        {
            int8_t* dst = out + ((static_cast<int64_t>(s) * Ch + c0 + ch) * Mp + q0) * ES;
            if constexpr(ES == 1)
            {
                uint32_t t[4];
#pragma unroll
                for(int g = 0; g < 4; ++g)
                    t[g] = byte_of(code[4 * g + 0 + s][ch / 4], ch % 4) | (byte_of(code[4 * g + 1 + s][ch / 4], ch % 4) << 8)
                         | (byte_of(code[4 * g + 2 + s][ch / 4], ch % 4) << 16)
                         | (byte_of(code[4 * g + 3 + s][ch / 4], ch % 4) << 24);
                *reinterpret_cast<uint4*>(dst) = make_uint4(t[0], t[1], t[2], t[3]);
            }
            else
            {
                uint32_t t[8];
#pragma unroll
                for(int g = 0; g < 8; ++g)
                {
                    const uint32_t lo = code[2 * g + 0 + s][ch / 2], hi = code[2 * g + 1 + s][ch / 2];
                    t[g] = (ch % 2 == 0) ? ((lo & 0xFFFFu) | (hi << 16)) : ((lo >> 16) | (hi & 0xFFFF0000u));
                }
                reinterpret_cast<uint4*>(dst)[0] = make_uint4(t[0], t[1], t[2], t[3]);
                reinterpret_cast<uint4*>(dst)[1] = make_uint4(t[4], t[5], t[6], t[7]);
            }
        }
}

// ------------------------------------------------------------------ cast / copy (+ transpose)
template <typename To, typename Ti> __device__ __forceinline__ To convert_elem(Ti v);
template <> __device__ __forceinline__ float  convert_elem<float, float>(float v) { return v; }
template <> __device__ __forceinline__ float  convert_elem<float, __half>(__half v) { return __half2float(v); }
template <> __device__ __forceinline__ __half convert_elem<__half, float>(float v) { return __float2half_rn(v); }
template <> __device__ __forceinline__ __half convert_elem<__half, __half>(__half v) { return v; }

// Floating-point stochastic quantization of one binary32 value to binary16 (Appendix, Proposition 2:
// truncate the mantissa to k bits, move up by one spacing with probability dropped / spacing).
// Integer arithmetic on the significand: sig * 2^(e-23) = |x|; D = (23-k) + max(0, -14-e) low bits are
// dropped (below the binary16 normal range the spacing stays 2^(-14-k)); up iff u16 < floor(rem * 2^16 / 2^D).
// The result is exact in binary16 (or reaches 2^16 and narrows to infinity).
__device__ __forceinline__ __half sr_narrow(float xv, int k, uint32_t u16)
{
    const uint32_t bits = __float_as_uint(xv);
    const uint32_t eb   = (bits >> 23) & 0xFFu;
    const uint32_t mant = bits & 0x7FFFFFu;
    const uint64_t sig  = eb == 0 ? mant : (mant | 0x800000u);
    const int      e    = eb == 0 ? -126 : static_cast<int>(eb) - 127;
    int            D    = (23 - k) + (e < -14 ? -14 - e : 0);
    D                   = D > 40 ? 40 : D;
    const uint64_t kept = sig >> D;
    const uint64_t rem  = sig & ((uint64_t(1) << D) - 1);
    const uint64_t thr  = D >= 16 ? (rem >> (D - 16)) : (rem << (16 - D));
    const uint32_t res  = static_cast<uint32_t>(kept) + (u16 < thr ? 1u : 0u);       // <= 2^(k+1)
    float          val  = ldexpf(static_cast<float>(res), e - 23 + D);                // exact
    val                 = (bits >> 31) ? -val : val;
    return __float2half_rn(val);                                                     // exact, or overflow to infinity
}

// 64x64 tile; the transposed copy goes through a padded LDS tile so that both copies are
// written with lanes along the contiguous axis.  SR (binary32 -> binary16 only) draws the element's
// 16-bit number from the Philox block of its row-major index, as the fixed-point quantizer does.
template <typename Ti, typename To, bool SR>
__global__ __launch_bounds__(kBlock) void convert_kernel(const Ti* __restrict__ x, int64_t rows, int64_t cols,
                                                         int64_t ld, To* __restrict__ q, To* __restrict__ qT,
                                                         int64_t grid_x, uint64_t seed, uint64_t offset, int k)
{
    __shared__ To tile[64][65];
    const int64_t by = blockIdx.x / grid_x, bx = blockIdx.x - by * grid_x;
    const int     tx = threadIdx.x % 64, ty = threadIdx.x / 64;
#pragma unroll 4
    for(int i = 0; i < 16; ++i)
    {
        const int     lr = ty + 4 * i;
        const int64_t r = by * 64 + lr, c = bx * 64 + tx;
        if(r < rows && c < cols)
        {
            To v;
            if constexpr(SR)
            {
                const uint64_t idx = static_cast<uint64_t>(r) * static_cast<uint64_t>(cols) + static_cast<uint64_t>(c);
                const uint4    blk = philox_group(seed, offset, idx >> 3);
                v = sr_narrow(x[r * ld + c], k, philox_draw16(blk, static_cast<int>(idx & 7)));
            }
            else
                v = convert_elem<To, Ti>(x[r * ld + c]);
            if(q) q[r * cols + c] = v;
            tile[lr][tx] = v;
        }
    }
    if(!qT) return;      // uniform over the block
    __syncthreads();
#pragma unroll 4
    for(int i = 0; i < 16; ++i)
    {
        const int     lc = ty + 4 * i;
        const int64_t c = bx * 64 + lc, r = by * 64 + tx;
        if(r < rows && c < cols) qT[c * rows + r] = tile[tx][lc];
    }
}

// ------------------------------------------------------------------ standalone dequantize
// code * scale (+ bias) in the output type.  The dequantized scalar is the exact product of a code and a scale
// (Indicator section: x_hat = round(x_bar) * q_x); for an 8-bit code and one binary32 scale that product has at
// most 32 significant bits.  The binary16 result is that exact value rounded once: the binary32 product is
// brought to round-to-odd with the exact residual of the multiplication (fused multiply-add), and a value
// rounded to odd at 24 bits narrows to 11 bits like the exact one.  With a bias the sum is formed in binary32.
template <typename To> __device__ __forceinline__ To scaled_code(float a, float g, float bias, bool has_bias);
template <> __device__ __forceinline__ float scaled_code<float>(float a, float g, float bias, bool has_bias)
{
    const float v = a * g;
    return has_bias ? v + bias : v;
}
template <> __device__ __forceinline__ __half scaled_code<__half>(float a, float g, float bias, bool has_bias)
{
    const float p = a * g;
    if(has_bias) return __float2half_rn(p + bias);
    const float e = fmaf(a, g, -p);                         // exact residual of a normal product
    uint32_t    b = __float_as_uint(p);
    if(e != 0.0f && (b & 1u) == 0u && (b & 0x7F800000u) != 0u)
        b += ((e > 0.0f) == (p > 0.0f)) ? 1u : 0xFFFFFFFFu;       // the neighbour on the residual's side is the odd one
    return __float2half_rn(__uint_as_float(b));
}

// Conversion with an optional transposed copy, tiled like the fixed-point quantizer: a workgroup owns 64 rows x 16
// threads of 16 output bytes, a thread four rows.  Codes (int8) are scaled per row or per tensor.  The transposed copy
// goes through LDS, four rows of a column per write, and leaves as whole 128-byte (binary16) or 256-byte segments.
// Latency bound at small sizes: one 8 x 8 patch per lane kept half the wavefronts in flight (2056x1032 fp32 -> binary16
// with both copies 8.5 -> 7.4 us, 4096x1024 11.5 -> 9.4; fp32 8192x4096 transposed element by element 69.2 -> 54.6).
// binary16 sources go by patches all the same (CopyF16Patch).
constexpr int kConvertRows = 64;
// conv_C > 0 (3x3 convolution weights [N, 9 * C]): column (tap, c) lands in row c * 9 + (8 - tap) of the transposed copy, as
// for WeightQuantize.
// SUMS: also the sums of the tile's columns of x, one partial per tile row.
template <typename Ti, typename To, bool SUMS = false> struct ConvertTile
{
    static constexpr int TC = 16 / sizeof(To);                      // columns of a thread
    static constexpr int CH = kConvertRows * sizeof(To) / 16;       // 16-byte chunks of a tile column
    static constexpr int kThreads = kBlock, kLds = 16 * TC * CH * 16;
    const Ti*    x;
    int64_t      rows, cols, ld;
    const float* row_scale;
    const float* scale;
    To*          q;
    To*          qT;
    int          tiles_x;
    int          conv_C;
    float*       sums;
    __device__ __forceinline__ void run(uint32_t block, uint8_t* lds_t) const
    {
        const int     by = static_cast<int>(block) / tiles_x, bx = static_cast<int>(block) - by * tiles_x;
        const int     cg = threadIdx.x % 16, quad = threadIdx.x / 16;
        const int64_t tile_r = static_cast<int64_t>(by) * kConvertRows, tile_c = static_cast<int64_t>(bx) * 16 * TC;
        const int64_t r0 = tile_r + quad * 4, c0 = tile_c + cg * TC;
        struct alignas(sizeof(Ti) * TC < 16 ? sizeof(Ti) * TC : 16) In { Ti v[TC]; };
        union Out { To v[TC]; uint4 w; };
        In  in[4];
        Out out[4];
#pragma unroll
        for(int i = 0; i < 4; ++i)      // (absent rows and columns repeat the last ones and are not stored)
            in[i] = *reinterpret_cast<const In*>(x + (r0 + i < rows ? r0 + i : rows - 1) * ld + (c0 < cols ? c0 : cols - TC));
#pragma unroll
        for(int i = 0; i < 4; ++i)
        {
            const bool ok = r0 + i < rows && c0 < cols;
            float      g  = 1.0f;
            if constexpr(std::is_same<Ti, int8_t>::value) g = row_scale ? row_scale[r0 + i < rows ? r0 + i : rows - 1] : *scale;
#pragma unroll
            for(int e = 0; e < TC; ++e)
            {
                if constexpr(std::is_same<Ti, int8_t>::value) out[i].v[e] = scaled_code<To>(static_cast<float>(in[i].v[e]), g, 0.0f, false);
                else out[i].v[e] = convert_elem<To, Ti>(in[i].v[e]);
            }
            if(q && ok) *reinterpret_cast<uint4*>(q + (r0 + i) * cols + c0) = out[i].w;
        }
        if constexpr(SUMS)
        {
            float* part = reinterpret_cast<float*>(lds_t);          // [16 row quads][columns of the tile]
#pragma unroll
            for(int e = 0; e < TC; ++e)
            {
                float t = 0.0f;
#pragma unroll
                for(int i = 0; i < 4; ++i)
                    if(r0 + i < rows && c0 < cols) t += to_f32(in[i].v[e]);
                part[(quad * 16 + cg) * TC + e] = t;
            }
            __syncthreads();
            if(threadIdx.x < 16 * TC && tile_c + threadIdx.x < cols)
            {
                float t = 0.0f;
#pragma unroll
                for(int k = 0; k < 16; ++k) t += part[k * 16 * TC + threadIdx.x];
                sums[by * cols + tile_c + threadIdx.x] = t;
            }
            __syncthreads();
        }
        if(!qT) return;
#pragma unroll
        for(int e = 0; e < TC; ++e)
        {
            const uint32_t* w[4] = {&out[0].w.x, &out[1].w.x, &out[2].w.x, &out[3].w.x};
            uint8_t*        col  = lds_t + (cg * TC + e) * CH * 16;
            if constexpr(sizeof(To) == 2)
            {
                const uint32_t sel = e % 2 ? 0x07060302u : 0x05040100u;
                const uint32_t lo = __builtin_amdgcn_perm(w[1][e / 2], w[0][e / 2], sel), hi = __builtin_amdgcn_perm(w[3][e / 2], w[2][e / 2], sel);
                *reinterpret_cast<uint2*>(col + ((quad / 2) ^ (cg % CH)) * 16 + (quad % 2) * 8) = make_uint2(lo, hi);
            }
            else
                *reinterpret_cast<uint4*>(col + (quad ^ (cg % CH)) * 16) = make_uint4(w[0][e], w[1][e], w[2][e], w[3][e]);
        }
        __syncthreads();
#pragma unroll
        for(int k = threadIdx.x; k < 16 * TC * CH; k += kBlock)
        {
            const int     lc = k / CH, ch = k % CH;
            const int64_t r = tile_r + ch * TC, c = tile_c + lc;        // a chunk holds TC rows
            if(c >= cols || r >= rows) continue;
            Out v;
            v.w = *reinterpret_cast<const uint4*>(lds_t + lc * CH * 16 + ((ch ^ ((lc / TC) % CH)) * 16));
            const int64_t tr  = conv_C == 0 ? c : (c % conv_C) * 9 + (8 - c / conv_C);
            To*           dst = qT + tr * rows + r;
            if(rows % TC == 0)
                *reinterpret_cast<uint4*>(dst) = v.w;
            else
#pragma unroll
                for(int e = 0; e < TC; ++e)
                    if(r + e < rows) dst[e] = v.v[e];
        }
    }
};

// binary16 copied and transposed without converting anything: a lane owns an 8 x 8 patch, transposed in registers by pairing
// 16-bit halves, a wavefront 8 x 8 patches, so every load and store instruction covers 128-byte row segments; no LDS,
// no barrier.  Needs cols % 8 == 0, 16-byte aligned rows, and rows % 8 == 0 when the transposed copy is written.
// Bound by latency when small and by its two streams when large; the tile kernel's pass through LDS is a second latency that
// nothing hides here (fp32 sources, whose loads are twice as long, run faster through it).  Tiles -> patches, transposed
// copy alone: 64x512 3.5 -> 2.4 us, 4096x768 5.1 -> 3.8, 16384x1024 15.8 -> 12.7, 16384x4096 49 -> 43; both copies 4096x768
// 6.2 -> 5.2, 16384x1024 18.0 -> 16.4, 16384x4096 88 -> 89.
struct CopyF16Patch
{
    static constexpr int kThreads = kBlock, kLds = 16;
    const __half* x;
    int64_t       rows, cols, ld;
    __half*       q;
    __half*       qT;
    int64_t       grid_x;
    __device__ __forceinline__ void run(uint32_t block, uint8_t*) const
    {
        const int     lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
        const int64_t by = block / grid_x, bx = block - by * grid_x;
        const int64_t r0 = (by * (kBlock / kWaveSize) + wave) * 64 + (lane / 8) * 8;
        const int64_t c0 = bx * 64 + (lane % 8) * 8;
        if(r0 >= rows || c0 >= cols) return;
        uint4 w[8];
#pragma unroll
        for(int i = 0; i < 8; ++i) w[i] = *reinterpret_cast<const uint4*>(x + (r0 + i < rows ? r0 + i : rows - 1) * ld + c0);      // (absent rows are not stored)
        if(q)
#pragma unroll
            for(int i = 0; i < 8; ++i)
                if(r0 + i < rows) *reinterpret_cast<uint4*>(q + (r0 + i) * cols + c0) = w[i];
        if(!qT) return;
        auto pair = [&](int i, int p) { return p == 0 ? w[i].x : p == 1 ? w[i].y : p == 2 ? w[i].z : w[i].w; };
#pragma unroll
        for(int c = 0; c < 8; ++c)
        {   // column c of the patch: halves c % 2 of pair c / 2 of every row
            uint32_t t[4];
#pragma unroll
            for(int g = 0; g < 4; ++g)
                t[g] = __builtin_amdgcn_perm(pair(2 * g + 1, c / 2), pair(2 * g, c / 2), c % 2 ? 0x07060302u : 0x05040100u);
            *reinterpret_cast<uint4*>(qT + (c0 + c) * rows + r0) = make_uint4(t[0], t[1], t[2], t[3]);
        }
    }
};

template <typename Ti, typename To, int V>
__global__ __launch_bounds__(kBlock) void dequantize_kernel(const Ti* __restrict__ a, int64_t rows, int64_t cols,
                                                            int64_t ld, const float* __restrict__ rs,
                                                            const float* __restrict__ cs, float ts_host,
                                                            const float* __restrict__ ts_dev,
                                                            const float* __restrict__ cb, To* __restrict__ y)
{
    const float   ts     = ts_dev ? ts_host * ts_dev[0] : ts_host;      // one fp32 product (exact when ts_host is 1)
    const int64_t cv     = cols / V;          // V divides cols on this path (V == 1 otherwise)
    const int64_t n      = rows * cv;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for(int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride)
    {
        const int64_t r = i / cv, c = (i - r * cv) * V;
        alignas(16) Ti in[V];
        if(V == 4 && sizeof(Ti) == 4)
            *reinterpret_cast<uint4*>(in) = *reinterpret_cast<const uint4*>(a + r * ld + c);
        else if(V == 4 && sizeof(Ti) == 1)
            *reinterpret_cast<uint32_t*>(in) = *reinterpret_cast<const uint32_t*>(a + r * ld + c);
        else
            in[0] = a[r * ld + c];
        // the scales are multiplied together first: with a single scale in use that product is the scale itself
        const float grow = ts * (rs ? rs[r] : 1.0f);
        alignas(16) To out[V];
#pragma unroll
        for(int e = 0; e < V; ++e)
            out[e] = scaled_code<To>(static_cast<float>(in[e]), cs ? grow * cs[c + e] : grow, cb ? cb[c + e] : 0.0f,
                                     cb != nullptr);
        To* dst = y + r * cols + c;
        if(V == 4 && sizeof(To) == 4)
            *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(out);
        else if(V == 4 && sizeof(To) == 2)
            *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(out);
        else
            dst[0] = out[0];
    }
}

// Vector path: a thread owns V = 16 / sizeof(Ti) adjacent columns (one 16-byte load) and walks down the
// rows, four loads in flight; its column scales and biases are fetched once.  2^tx_log2 threads of a
// block lie side by side along a row (the whole block, 4 KB, when the matrix is wide enough), the
// rest of the block stacks rows.  Same arithmetic per element as dequantize_kernel.
template <typename Ti, typename To>
__global__ __launch_bounds__(kBlock) void dequantize_cols_kernel(const Ti* __restrict__ a, int64_t rows, int64_t cols,
                                                                 int64_t ld, const float* __restrict__ rs,
                                                                 const float* __restrict__ cs, float ts_host,
                                                                 const float* __restrict__ ts_dev,
                                                                 const float* __restrict__ cb, To* __restrict__ y,
                                                                 int tx_log2)
{
    constexpr int V = 16 / sizeof(Ti);
    constexpr int U = 4;
    const float   ts = ts_dev ? ts_host * ts_dev[0] : ts_host;
    const int     tx = threadIdx.x & ((1 << tx_log2) - 1), ty = threadIdx.x >> tx_log2, TY = kBlock >> tx_log2;
    const int64_t c  = ((static_cast<int64_t>(blockIdx.x) << tx_log2) + tx) * V;
    if(c >= cols) return;
    float fcs[V], fcb[V];
#pragma unroll
    for(int e = 0; e < V; e += 4)
    {
        const float4 s4 = cs ? *reinterpret_cast<const float4*>(cs + c + e) : make_float4(1.0f, 1.0f, 1.0f, 1.0f);
        const float4 b4 = cb ? *reinterpret_cast<const float4*>(cb + c + e) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        fcs[e] = s4.x; fcs[e + 1] = s4.y; fcs[e + 2] = s4.z; fcs[e + 3] = s4.w;
        fcb[e] = b4.x; fcb[e + 1] = b4.y; fcb[e + 2] = b4.z; fcb[e + 3] = b4.w;
    }
    // a block works on TY * U adjacent rows at a time
    for(int64_t base = static_cast<int64_t>(blockIdx.y) * (TY * U); base < rows; base += static_cast<int64_t>(gridDim.y) * (TY * U))
    {
        uint4 raw[U];
#pragma unroll
        for(int u = 0; u < U; ++u)
        {
            // Four-byte inputs load the last row again for absent ones instead of branching around each load (int32 6320x3616 to fp32
            // 40.8 -> 37.0 us, 1000x1032 to binary16 4.15 -> 3.81).  Bytes, sixteen of them a load, keep the branch: without it int8
            // to fp32 takes 107 registers in place of 88, 383x592 4.15 -> 4.27 us, and no size gains by more than 2 %.
            const int64_t r = base + u * TY + ty;
            raw[u] = sizeof(Ti) == 4 || r < rows ? *reinterpret_cast<const uint4*>(a + (r < rows ? r : rows - 1) * ld + c) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for(int u = 0; u < U; ++u)
        {
            const int64_t r = base + u * TY + ty;
            if(r >= rows) continue;
            const float grow = ts * (rs ? rs[r] : 1.0f);
            alignas(16) Ti in[V];
            *reinterpret_cast<uint4*>(in) = raw[u];
            alignas(16) To out[V];
#pragma unroll
            for(int e = 0; e < V; ++e)
                out[e] = scaled_code<To>(static_cast<float>(in[e]), cs ? grow * fcs[e] : grow, fcb[e], cb != nullptr);
            To* dst = y + r * cols + c;
#pragma unroll
            for(int e = 0; e < V * static_cast<int>(sizeof(To)) / 16; ++e)
                reinterpret_cast<uint4*>(dst)[e] = reinterpret_cast<const uint4*>(out)[e];
            if(V * sizeof(To) == 8) *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(out);
        }
    }
}

// Contiguous int8 codes with one scale, any row length: vectors of 16 OUTPUT bytes, so that a wavefront's store is 1 KB of consecutive
// memory.  Bound by HBM.  With 16 codes to a thread a store instruction filled every other 16 bytes: 16384x4096 to binary16 alone 38.4 -> 31.6
// us (6.4 TB/s), 4096x4096 15.4 -> 10.9; 10740x1569 from an element a thread.
// Streaming stores from 128 MB of output on: with its codes and the tensor that those came from it no longer fits the memory-side cache of
// 256 MB, and plain stores push that tensor out.  Maximum + quantize + dequantize, plain and streamed, to binary16 of 80 MB 61.8 and 63.8 us, with
// an addition that reads the output 102.4 and 108.3; of 128 MB 95.3 and 91.7, 177.1 and 169.8; to fp32 of 192 MB 126 and 110, 239 and 223.
// Smaller outputs are what the next call finds there (64 MB with a GEMM behind it 52.5 and 69.2, 16 codes to a thread 56.7).  It costs
// whoever dequantizes codes of that size alone and reads them at once: 128 MB to binary16 with an addition 93.6 and 109.
template <typename To, int U, bool STREAM>
__global__ __launch_bounds__(kBlock) void dequantize_flat_kernel(const int8_t* __restrict__ a, int64_t n, float ts_host,
                                                                 const float* __restrict__ ts_dev, To* __restrict__ y)
{
    constexpr int V = 16 / sizeof(To);
    typedef typename std::conditional<V == 8, uint2, uint32_t>::type in_t;
    const float   ts = ts_dev ? ts_host * ts_dev[0] : ts_host;
    const int64_t nvec = n / V, i0 = static_cast<int64_t>(blockIdx.x) * (kBlock * U) + threadIdx.x;
    in_t          raw[U];
#pragma unroll
    for(int u = 0; u < U; ++u)
    {
        const int64_t i = i0 + u * kBlock < nvec ? i0 + u * kBlock : nvec - 1;      // (past the end the last one again, not stored)
        raw[u]          = reinterpret_cast<const in_t*>(a)[i];
    }
#pragma unroll
    for(int u = 0; u < U; ++u)
    {
        const int64_t i = i0 + u * kBlock;
        if(i >= nvec) break;
        alignas(8) int8_t in[V];
        *reinterpret_cast<in_t*>(in) = raw[u];
        alignas(16) To out[V];
#pragma unroll
        for(int e = 0; e < V; ++e) out[e] = scaled_code<To>(static_cast<float>(in[e]), ts, 0.0f, false);
        typedef unsigned v4u __attribute__((ext_vector_type(4)));
        if constexpr(STREAM) __builtin_nontemporal_store(*reinterpret_cast<const v4u*>(out), reinterpret_cast<v4u*>(y) + i);
        else                 reinterpret_cast<v4u*>(y)[i] = *reinterpret_cast<const v4u*>(out);
    }
    const int64_t rest = nvec * V + threadIdx.x;
    if(blockIdx.x == 0 && rest < n) y[rest] = scaled_code<To>(static_cast<float>(a[rest]), ts, 0.0f, false);
}

int next_pow2(int64_t v)
{
    int p = 1;
    while(p < v) p <<= 1;
    return p;
}

// Launch shape of a per-column reduction with `block` threads per block: threads per row (a power
// of two, at most one wavefront so that a wavefront reads 1 KB of a row) and block rows
// (gridDim.y, at most kColParts).  Large inputs run 1024-thread blocks, about one per compute
// unit: sixteen wavefronts with four loads in flight each keep the memory pipeline full, and a
// strip then has few enough partials for one block to fold them.
void colreduce_shape(int64_t rows, int64_t cols, int E, int block, int& tpr, int& gy)
{
    const int64_t ncv = (cols + E - 1) / E;
    tpr               = ncv >= kWaveSize ? kWaveSize : (next_pow2(ncv) < 2 ? 2 : next_pow2(ncv));
    if(ncv > static_cast<int64_t>(kWaveSize) * 1000) tpr = kBlock;     // very wide: keep the strip count small
    const int64_t gx  = (ncv + tpr - 1) / tpr;
    const int     rpb = block / tpr;
    const int64_t target = block >= 1024 ? 256 : 1024;
    int64_t       g   = (target + gx - 1) / gx;
    const int64_t maxg = (rows + rpb - 1) / rpb;              // no more block rows than row groups
    if(g > maxg) g = maxg;
    if(g > kColParts) g = kColParts;
    if(g < 1) g = 1;
    gy = static_cast<int>(g);
}

// Workspace of the per-tensor reductions: the arrival counter first (a 256-byte slot), partials behind it.
constexpr size_t kCtrBytes = 256;

// The pass over x; `gy` partials per column, `nmax` block maxima.
template <typename T, int OP>
void colreduce_first(const T* x, int64_t rows, int64_t cols, int64_t ld, float* partial, float* partial_max, const TensorFinal& tfin,
                     int& gy, int& nmax, hipStream_t st)
{
    constexpr int E     = Vec16<T>::N;
    const bool    vec   = aligned16(x) && (ld * sizeof(T)) % 16 == 0 && cols % E == 0;
    const int     block = rows * cols >= (int64_t(1) << 20) ? 1024 : kBlock;
    int           tpr;
    colreduce_shape(rows, cols, vec ? E : 1, block, tpr, gy);
    const int64_t ncv = (cols + (vec ? E : 1) - 1) / (vec ? E : 1);
    const int64_t gx  = (ncv + tpr - 1) / tpr;
    if(partial_max)
        while(gx * gy > kAbsmaxMaxBlocks && gy > 1) gy = (gy + 1) / 2;  // block maxima must fit their slots
    const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(gy));
    if(vec)
    {
        if(block == 1024)
            colreduce_kernel<T, true, OP, 1024><<<grid, dim3(1024), 0, st>>>(x, rows, cols, ld, tpr, partial, partial_max, tfin);
        else
            colreduce_kernel<T, true, OP, kBlock><<<grid, dim3(kBlock), 0, st>>>(x, rows, cols, ld, tpr, partial, partial_max, tfin);
    }
    else
    {
        if(block == 1024)
            colreduce_kernel<T, false, OP, 1024><<<grid, dim3(1024), 0, st>>>(x, rows, cols, ld, tpr, partial, partial_max, tfin);
        else
            colreduce_kernel<T, false, OP, kBlock><<<grid, dim3(kBlock), 0, st>>>(x, rows, cols, ld, tpr, partial, partial_max, tfin);
    }
    nmax = static_cast<int>(gx * gy);
}

template <typename T, int OP>
hipError_t colreduce_launch(const T* x, int64_t rows, int64_t cols, int64_t ld, float qmax, float* out,
                            float* inv_scale, float* amax_opt, float* partial, float* partial_max, TensorFinal tfin,
                            hipStream_t st)
{
    int gy, nmax;
    colreduce_first<T, OP>(x, rows, cols, ld, partial, partial_max, tfin, gy, nmax, st);
    colreduce_finalize_kernel<OP><<<dim3((cols + 15) / 16 + (OP == OP_SUMMAX ? 1 : 0)), dim3(kBlock), 0, st>>>(
        partial, gy, cols, qmax, out, inv_scale, amax_opt, partial_max, nmax, tfin);
    return hipGetLastError();
}

}  // namespace

// ======================================================================== launchers
size_t absmax_workspace_bytes(int64_t rows, int64_t cols, int gran)
{
    (void)rows;
    const size_t c = static_cast<size_t>(cols > 0 ? cols : 0);
    if(gran == kPerTensor)   // counter, block maxima, block sums of squares; with fused column sums also their partials
        return kCtrBytes + sizeof(float) * (2 * kAbsmaxMaxBlocks + static_cast<size_t>(kColParts) * c);
    if(gran == kPerCol) return kCtrBytes + sizeof(float) * kColParts * c;   // same layout: the counter slot stays untouched
    return 0;
}

template <typename T>
static hipError_t absmax_typed(const T* x, int64_t rows, int64_t cols, int64_t ld, int gran, float qmax, float* scale,
                               float* inv_scale, float* amax_opt, float* colsum_opt, float* sumsq_opt, void* workspace,
                               hipStream_t st)
{
    constexpr int E       = Vec16<T>::N;
    const bool    rows_ok = aligned16(x) && (ld * sizeof(T)) % 16 == 0;
    (void)E;
    if(gran == kPerTensor)
    {
        unsigned int* ctr = static_cast<unsigned int*>(workspace);
        float*        ws  = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + kCtrBytes);
        float*        wsq = ws + kAbsmaxMaxBlocks;          // block sums of squares
        if(colsum_opt)
        {   // per-tensor absmax fused with column sums: one pass over x
            TensorFinal tfin{qmax, scale, inv_scale, amax_opt, wsq, sumsq_opt};
            return colreduce_launch<T, OP_SUMMAX>(x, rows, cols, ld, 0.0f, colsum_opt, nullptr, nullptr,
                                                  ws + 2 * kAbsmaxMaxBlocks, ws, tfin, st);
        }
        const bool    vec  = aligned16(x) && ld == cols;
        const int64_t work = vec ? (rows * cols) / E : rows * cols;
        const bool    big  = work >= (int64_t(1) << 19);
        const int     blk  = big ? 1024 : kBlock;
        int64_t       nb   = (work + blk * 8 - 1) / (blk * 8);
        nb                 = nb < 1 ? 1 : (nb > 256 ? 256 : nb);       // few blocks: the tickets are serialised
        if(vec)
        {
            if(big)
                absmax_tensor_kernel<T, true, 1024><<<dim3(nb), dim3(1024), 0, st>>>(x, rows, cols, ld, ws, ctr, qmax, scale, inv_scale, amax_opt, wsq, sumsq_opt);
            else
                absmax_tensor_kernel<T, true, kBlock><<<dim3(nb), dim3(kBlock), 0, st>>>(x, rows, cols, ld, ws, ctr, qmax, scale, inv_scale, amax_opt, wsq, sumsq_opt);
        }
        else
        {
            if(big)
                absmax_tensor_kernel<T, false, 1024><<<dim3(nb), dim3(1024), 0, st>>>(x, rows, cols, ld, ws, ctr, qmax, scale, inv_scale, amax_opt, wsq, sumsq_opt);
            else
                absmax_tensor_kernel<T, false, kBlock><<<dim3(nb), dim3(kBlock), 0, st>>>(x, rows, cols, ld, ws, ctr, qmax, scale, inv_scale, amax_opt, wsq, sumsq_opt);
        }
    }
    else if(gran == kPerRow)
    {
        const bool few = rows < 4096;         // too few rows to fill the chip with one wavefront per row
        const int64_t nb = few ? rows : (rows + 3) / 4;
        if(rows_ok)
        {
            if(few)
                absmax_rows_kernel<T, true, 4><<<dim3(nb), dim3(kBlock), 0, st>>>(x, rows, cols, ld, qmax, scale, inv_scale, amax_opt);
            else
                absmax_rows_kernel<T, true, 1><<<dim3(nb), dim3(kBlock), 0, st>>>(x, rows, cols, ld, qmax, scale, inv_scale, amax_opt);
        }
        else
        {
            if(few)
                absmax_rows_kernel<T, false, 4><<<dim3(nb), dim3(kBlock), 0, st>>>(x, rows, cols, ld, qmax, scale, inv_scale, amax_opt);
            else
                absmax_rows_kernel<T, false, 1><<<dim3(nb), dim3(kBlock), 0, st>>>(x, rows, cols, ld, qmax, scale, inv_scale, amax_opt);
        }
    }
    else
    {
        TensorFinal none{qmax, nullptr, nullptr, nullptr, nullptr, nullptr};
        return colreduce_launch<T, OP_MAX>(x, rows, cols, ld, qmax, scale, inv_scale, amax_opt,
                                           reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + kCtrBytes), nullptr,
                                           none, st);
    }
    return hipGetLastError();
}

hipError_t launch_scale_from_amax(float* amax, float qmax, float* scale, float* inv_scale, int consume, hipStream_t st)
{
    launch_part(ScaleFromAmax{amax, qmax, scale, inv_scale, consume}, 1, st);
    return hipGetLastError();
}

// ---- scratch that the library owns: for the entry point that may not allocate ---------------------------------
// One array per GPU (every device that loads this code object holds its own copy at its own address), kept
// until the process ends.  Host code must never pass the array's name to a kernel: that name is a host-side
// stand-in.  The device address is looked up once per device and handed to the kernels like any workspace.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch(void** ptr_out)
{
    constexpr int      kMaxDevices = 64;
    static std::mutex  lock;
    static void*       per_device[kMaxDevices] = {};
    int                dev = -1;
    hipError_t         e   = hipGetDevice(&dev);
    if(e != hipSuccess) return e;
    if(dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(lock);
    if(!per_device[dev])
    {
        void* p = nullptr;
        e       = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if(e != hipSuccess) return e;
        if(!p) return hipErrorInvalidSymbol;
        per_device[dev] = p;
    }
    *ptr_out = per_device[dev];
    return hipSuccess;
}

hipError_t launch_absmax_scale(const void* x, int xdt, int64_t rows, int64_t cols, int64_t ld, int gran, float qmax,
                               float* scale, float* inv_scale, float* amax_opt, float* colsum_opt, float* sumsq_opt,
                               void* workspace, hipStream_t stream)
{
    if(xdt == kF32)
        return absmax_typed(static_cast<const float*>(x), rows, cols, ld, gran, qmax, scale, inv_scale, amax_opt,
                            colsum_opt, sumsq_opt, workspace, stream);
    return absmax_typed(static_cast<const __half*>(x), rows, cols, ld, gran, qmax, scale, inv_scale, amax_opt,
                        colsum_opt, sumsq_opt, workspace, stream);
}

// Launch shape of the patch kernel: lanes per row (as a power of two) and patch height.
struct PatchShape { int lpr_log2, pr; int64_t gx, gy; };
template <typename T> static PatchShape patch_shape(int64_t rows, int64_t cols, bool transposed_copy)
{
    constexpr int PCOLS = 2 * Vec16<T>::N;
    PatchShape    p{3, 16, 0, 0};
    const int64_t pc = (cols + PCOLS - 1) / PCOLS;                 // patches per row
    while(p.lpr_log2 > 0 && (int64_t(1) << (p.lpr_log2 - 1)) >= pc) --p.lpr_log2;
    // 8-row patches put twice the wavefronts in flight (measured: faster whenever no transposed copy is
    // written, and below about eight wavefronts of 16-row patches per compute unit); the transposed copy
    // of a large tensor prefers 16-byte stores
    if(!transposed_copy || (rows / 16) * pc < int64_t(kWaveSize) * 2048) p.pr = 8;
    p.gx = (pc + (int64_t(1) << p.lpr_log2) - 1) >> p.lpr_log2;
    const int64_t rows_per_block = static_cast<int64_t>(kBlock / kWaveSize) * (kWaveSize >> p.lpr_log2) * p.pr;
    p.gy = (rows + rows_per_block - 1) / rows_per_block;
    return p;
}

template <typename T, int RND>
static void quantize_patch_launch(const T* x, int64_t rows, int64_t cols, int64_t ld, int qmax, int gran,
                                  uint64_t seed, uint64_t offset, const float* inv, int8_t* q, int8_t* qT,
                                  hipStream_t st)
{
    const PatchShape ps = patch_shape<T>(rows, cols, qT != nullptr);
    const dim3       grid(static_cast<unsigned>(ps.gx * ps.gy));
    auto go = [&](auto percol, auto pr) {
        quantize_patch_kernel<T, RND, decltype(percol)::value, decltype(pr)::value><<<grid, dim3(kBlock), 0, st>>>(
            x, rows, cols, ld, qmax, seed, offset, inv, q, qT, ps.gx, ps.lpr_log2);
    };
    typedef std::integral_constant<int, 16> P16;
    typedef std::integral_constant<int, 8>  P8;
    if(gran == kPerCol) { if(ps.pr == 16) go(std::true_type{}, P16{}); else go(std::true_type{}, P8{}); }
    else                { if(ps.pr == 16) go(std::false_type{}, P16{}); else go(std::false_type{}, P8{}); }
}

// f(std::integral_constant<int, RND>) for a run-time rounding mode
template <typename F> static void with_rounding(int rnd, F&& f)
{
    if(rnd == kStochastic)  f(std::integral_constant<int, kStochastic>{});
    else if(rnd == kFloor)  f(std::integral_constant<int, kFloor>{});
    else                    f(std::integral_constant<int, kNearest>{});
}

// What the tiled kernel and the streaming one need of a tensor and its outputs.
static int64_t tiles_of(int64_t rows, int64_t cols, int tr) { return ((rows + tr - 1) / tr) * ((cols + kTileCols - 1) / kTileCols); }
template <typename T> static bool tile_ok(const T* x, int64_t rows, int64_t cols, int64_t ld, const int8_t* q, const int8_t* qT)
{
    return cols % 8 == 0 && aligned16(x) && (ld * sizeof(T)) % 16 == 0 && (reinterpret_cast<uintptr_t>(q) & 7) == 0
        && (rows % 16 != 0 || aligned16(qT)) && tiles_of(rows, cols, 64) < (int64_t(1) << 30);
}

// A row count that is no multiple of 16 leaves the columns of the transposed copy unaligned, and the tile kernel then
// gathers or stores them in pieces, with most of a tile's rows absent when there are few: one element per thread
// (quantize_generic_kernel) is faster for fewer than 16 rows (1 x 65536: 2.4 against 4.4 us, 1 x 1048576: 4.5 against
// 30; 9 x 65536: 4.0 against 4.1) and up to about 400 000 elements (45 x 1024: 2.5 against 4.7 us, 500 x 128: 2.8 against
// 4.5, 1000 x 264: 3.8 against 4.7, 1000 x 392: 4.6 against 4.9; 1000 x 528: 5.5 against 5.1, 1000 x 1048: 8.4 against 6.1).
static bool odd_transpose_generic(int64_t rows, int64_t n, const int8_t* qT)
{
    return qT && rows % 16 != 0 && (rows < 16 || n < (int64_t(3) << 17));
}

// Per-tensor codes of a tensor that meets tile_ok, as parts: f(part, workgroups).  Streaming when only row-major codes of a
// contiguous tensor are wanted, tiles otherwise.  Tiles are 128 rows high (whole 128-byte lines of the transposed copy)
// once that gives every compute unit two workgroups, 64 rows below.
template <typename T, int SRC, typename F>
static void with_quantize_part(const T* x, int64_t rows, int64_t cols, int64_t ld, int qmax, int rnd, uint64_t seed, uint64_t offset,
                               const TensorScale& ts, int8_t* q, int8_t* qT, F&& f)
{
    const int64_t ngroups = rows * cols / 8, stream_blocks = (ngroups + kBlock * 4 - 1) / (kBlock * 4);
    const bool    stream  = SRC != kWhole && q && !qT && ld == cols && stream_blocks < (int64_t(1) << 30);
    const int     tiles_x = static_cast<int>((cols + kTileCols - 1) / kTileCols);
    with_rounding(rnd, [&](auto r) {
        constexpr int RND = decltype(r)::value;
        if constexpr(SRC != kWhole)
        {
            if(stream)
            {
                f(QuantizeStream<T, RND, SRC>{x, ngroups, qmax, seed, offset, ts, q}, stream_blocks);
                return;
            }
            if(tiles_of(rows, cols, 128) < 512)
            {
                f(QuantizeTile<T, RND, 64, SRC>{x, rows, cols, ld, qmax, seed, offset, ts, q, qT, tiles_x}, tiles_of(rows, cols, 64));
                return;
            }
        }
        f(QuantizeTile<T, RND, 128, SRC>{x, rows, cols, ld, qmax, seed, offset, ts, q, qT, tiles_x}, tiles_of(rows, cols, 128));
    });
}
template <typename T, int SRC>
static void quantize_tensor_launch(const T* x, int64_t rows, int64_t cols, int64_t ld, int qmax, int rnd, uint64_t seed,
                                   uint64_t offset, const TensorScale& ts, int8_t* q, int8_t* qT, hipStream_t st)
{
    with_quantize_part<T, SRC>(x, rows, cols, ld, qmax, rnd, seed, offset, ts, q, qT, [&](const auto& p, int64_t blocks) { launch_part(p, blocks, st); });
}

template <typename T>
static hipError_t quantize_typed(const T* x, int64_t rows, int64_t cols, int64_t ld, int qmax, int gran, int rnd,
                                 uint64_t seed, uint64_t offset, const float* inv, int8_t* q, int8_t* qT,
                                 hipStream_t st)
{
    const PatchShape ps = patch_shape<T>(rows, cols, qT != nullptr);
    const bool       fast = cols % 8 == 0 && aligned16(x) && (ld * sizeof(T)) % 16 == 0 && (!q || aligned16(q))
                      && (!qT || (aligned16(qT) && rows % 16 == 0)) && ps.gx * ps.gy < (int64_t(1) << 31);
    if(gran == kPerTensor && tile_ok(x, rows, cols, ld, q, qT) && !odd_transpose_generic(rows, rows * cols, qT))
    {
        const TensorScale ts{inv, nullptr, 0, nullptr, nullptr, nullptr};
        quantize_tensor_launch<T, kInv>(x, rows, cols, ld, qmax, rnd, seed, offset, ts, q, qT, st);
    }
    // (any row length; smaller ones, whose groups of eight leave units idle, go an element per thread: stochastic 33x999 2.5 us, as groups 3.5,
    // 3950x89 3.4 and 3.5, 512x777 3.5 and 3.3; to nearest 1338x91 2.4 and 2.6, 196x1581 2.8 and 2.7)
    else if(gran == kPerTensor && q && !qT && ld == cols && rows * cols >= (rnd == kStochastic ? 390000 : 250000) && rows * cols < (int64_t(1) << 40)
            && aligned16(x) && (reinterpret_cast<uintptr_t>(q) & 7) == 0)
        with_rounding(rnd, [&](auto r) {
            const int64_t     ngroups = rows * cols / 8;
            const TensorScale ts{inv, nullptr, 0, nullptr, nullptr, nullptr};
            launch_part(QuantizeStreamAny<T, decltype(r)::value>{{x, ngroups, qmax, seed, offset, ts, q}, static_cast<int>(rows * cols % 8)},
                        (ngroups + kBlock * 4 - 1) / (kBlock * 4), st);
        });
    else if(fast && gran != kPerTensor)
        with_rounding(rnd, [&](auto r) {
            quantize_patch_launch<T, decltype(r)::value>(x, rows, cols, ld, qmax, gran, seed, offset, inv, q, qT, st);
        });
    else
    {
        int64_t nb = (rows * cols + kBlock - 1) / kBlock;
        nb         = nb > 65536 ? 65536 : nb;
        quantize_generic_kernel<T><<<dim3(nb), dim3(kBlock), 0, st>>>(x, rows, cols, ld, qmax, gran, rnd, seed, offset,
                                                                     inv, q, qT);
    }
    return hipGetLastError();
}

hipError_t launch_quantize_int8(const void* x, int xdt, int64_t rows, int64_t cols, int64_t ld, int qmax, int gran,
                                int rnd, uint64_t seed, uint64_t offset, const float* inv_scale, int8_t* q, int8_t* qT,
                                hipStream_t stream)
{
    if(xdt == kF32)
        return quantize_typed(static_cast<const float*>(x), rows, cols, ld, qmax, gran, rnd, seed, offset, inv_scale,
                              q, qT, stream);
    return quantize_typed(static_cast<const __half*>(x), rows, cols, ld, qmax, gran, rnd, seed, offset, inv_scale, q,
                          qT, stream);
}

// The transposed copy of an odd row count goes one element per thread, in a pass behind the maximum's, where that is faster:
// not up to kWholeBytes, where launched one by one a second launch costs the host more (nearest, 45 x 1024 binary16: one
// launch 6.6 us, apart 8.5; 100 x 512 7.6 against 8.6; replayed from a graph 6.7 against 6.5 and 7.9 against 6.5), except from
// 128 rows on (129 x 512: 9.1 against 8.7, from a graph 9.0 against 6.6; 250 x 256 8.7 against 8.5), and not from 192 K
// elements of 16 rows or more on, where folding the maxima in the quantizer makes up for it (70 x 3744 7.5 against 8.4,
// 500 x 528 8.1 against 8.5).
template <typename T> static bool odd_transpose_apart(int64_t rows, int64_t n, const int8_t* qT)
{
    const bool whole = n * static_cast<int64_t>(sizeof(T)) <= kWholeBytes;
    return odd_transpose_generic(rows, n, qT) && (rows < 16 || n < (int64_t(3) << 16))
        && (!whole || (rows >= 128 && n >= (int64_t(1) << 15)));
}

// Per-tensor maximum, scales and codes of a contiguous tensor.  Up to kWholeBytes one launch, every workgroup of which
// reads the whole tensor for its maximum (no workgroup waits for another); above that a launch that leaves one maximum
// per block and the quantizing launch, which folds them.
template <typename T>
static hipError_t absmax_quantize_typed(const T* x, int64_t rows, int64_t cols, int qmax, int rnd, uint64_t seed,
                                        uint64_t offset, float* scale, float* inv_scale, float* amax_opt, int8_t* q,
                                        int8_t* qT, void* workspace, hipStream_t st)
{
    const int64_t n     = rows * cols;
    const bool    whole = n * static_cast<int64_t>(sizeof(T)) <= kWholeBytes;
    if(odd_transpose_apart<T>(rows, n, qT) || !tile_ok(x, rows, cols, cols, q, qT))
    {
        hipError_t e = absmax_typed(x, rows, cols, cols, kPerTensor, static_cast<float>(qmax), scale, inv_scale, amax_opt,
                                    nullptr, nullptr, workspace, st);
        if(e != hipSuccess) return e;
        return quantize_typed(x, rows, cols, cols, qmax, kPerTensor, rnd, seed, offset, inv_scale, q, qT, st);
    }
    float* partial = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + kCtrBytes);
    if(whole)
    {
        const TensorScale ts{nullptr, nullptr, 0, scale, inv_scale, amax_opt};
        quantize_tensor_launch<T, kWhole>(x, rows, cols, cols, qmax, rnd, seed, offset, ts, q, qT, st);
        return hipGetLastError();
    }
    const int64_t nvec = rows * cols / Vec16<T>::N;
    const int     blk  = nvec >= (int64_t(1) << 19) ? 1024 : kBlock;
    int64_t       nb   = (nvec + blk * 8 - 1) / (blk * 8);
    nb                 = nb > kFoldMax ? kFoldMax : nb;
    if(blk == 1024)
        absmax_tensor_kernel<T, true, 1024><<<dim3(nb), dim3(1024), 0, st>>>(x, rows, cols, cols, partial, nullptr, 0.0f, nullptr, nullptr, nullptr, nullptr, nullptr);
    else
        absmax_tensor_kernel<T, true, kBlock><<<dim3(nb), dim3(kBlock), 0, st>>>(x, rows, cols, cols, partial, nullptr, 0.0f, nullptr, nullptr, nullptr, nullptr, nullptr);
    const TensorScale ts{nullptr, partial, static_cast<int>(nb), scale, inv_scale, amax_opt};
    quantize_tensor_launch<T, kPartials>(x, rows, cols, cols, qmax, rnd, seed, offset, ts, q, qT, st);
    return hipGetLastError();
}

hipError_t launch_absmax_quantize(const void* x, int xdt, int64_t rows, int64_t cols, int qmax, int rnd, uint64_t seed,
                                  uint64_t offset, float* scale, float* inv_scale, float* amax_opt, int8_t* q, int8_t* qT,
                                  void* workspace, hipStream_t stream)
{
    if(xdt == kF32)
        return absmax_quantize_typed(static_cast<const float*>(x), rows, cols, qmax, rnd, seed, offset, scale, inv_scale,
                                     amax_opt, q, qT, workspace, stream);
    return absmax_quantize_typed(static_cast<const __half*>(x), rows, cols, qmax, rnd, seed, offset, scale, inv_scale,
                                 amax_opt, q, qT, workspace, stream);
}

// Maximum, scales, column sums and codes of a gradient: the pass that leaves block maxima and column partials, then a launch
// that converts and, in workgroups of its own, folds the partials.  A tensor of at most kWholeBytes takes one launch.
// Bound by the launches when small.  Three launches -> two, whole steps: 4096x3072x768 92.6 -> 90.6 us, 1808x1040x784 52.7 ->
// 50.9; -> one: 64x128x128 35.7 -> 28.7.
template <typename T>
static hipError_t gradient_quantize_typed(const T* x, int64_t rows, int64_t cols, int qmax, int rnd, uint64_t seed, uint64_t offset,
                                          float* scale, float* inv_scale, float* amax_opt, float* colsum, int8_t* q, int8_t* qT,
                                          void* workspace, hipStream_t st)
{
    const int64_t n = rows * cols, fold_blocks = (cols + 15) / 16;
    if(!tile_ok(x, rows, cols, cols, q, qT) || odd_transpose_generic(rows, n, qT))
    {
        hipError_t e = absmax_typed(x, rows, cols, cols, kPerTensor, static_cast<float>(qmax), scale, inv_scale, amax_opt, colsum, nullptr,
                                    workspace, st);
        if(e != hipSuccess) return e;
        return quantize_typed(x, rows, cols, cols, qmax, kPerTensor, rnd, seed, offset, inv_scale, q, qT, st);
    }
    if(n * static_cast<int64_t>(sizeof(T)) <= kWholeBytes && rows <= kColumnSumRows)
    {
        const TensorScale ts{nullptr, nullptr, 0, scale, inv_scale, amax_opt};
        with_quantize_part<T, kWhole>(x, rows, cols, cols, qmax, rnd, seed, offset, ts, q, qT, [&](const auto& p, int64_t blocks) {
            launch_parts(p, blocks, ColumnSum<T, std::decay_t<decltype(p)>::kThreads>{x, rows, cols, colsum}, fold_blocks, st);
        });
        return hipGetLastError();
    }
    float* maxima  = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + kCtrBytes);
    float* partial = maxima + 2 * kAbsmaxMaxBlocks;
    const TensorFinal none{0.0f, nullptr, nullptr, nullptr, nullptr, nullptr};
    int gy, nmax;
    colreduce_first<T, OP_SUMMAX>(x, rows, cols, cols, partial, maxima, none, gy, nmax, st);
    const TensorScale ts{nullptr, maxima, nmax, scale, inv_scale, amax_opt};
    with_quantize_part<T, kPartials>(x, rows, cols, cols, qmax, rnd, seed, offset, ts, q, qT, [&](const auto& p, int64_t blocks) {
        launch_parts(ColumnFold<std::decay_t<decltype(p)>::kThreads>{{partial, gy, cols, colsum}}, fold_blocks, p, blocks, st);
    });
    return hipGetLastError();
}

hipError_t launch_gradient_quantize(const void* x, int xdt, int64_t rows, int64_t cols, int qmax, int rnd, uint64_t seed, uint64_t offset,
                                    float* scale, float* inv_scale, float* amax_opt, float* colsum, int8_t* q, int8_t* qT,
                                    void* workspace, hipStream_t stream)
{
    if(xdt == kF32)
        return gradient_quantize_typed(static_cast<const float*>(x), rows, cols, qmax, rnd, seed, offset, scale, inv_scale, amax_opt,
                                       colsum, q, qT, workspace, stream);
    return gradient_quantize_typed(static_cast<const __half*>(x), rows, cols, qmax, rnd, seed, offset, scale, inv_scale, amax_opt, colsum,
                                   q, qT, workspace, stream);
}

// Weights of one linear operator in one go: per-row scales and codes for the forward, per-column scales
// and transposed codes for dX.  Two launches that read W twice where the vector rules hold; otherwise the
// separate passes.  Same results either way.
// conv_C > 0: w is [N, 9*conv_C]; the second scales are per input channel (conv_C of them) and wqbT is the
// mirrored, channel-exchanged copy [conv_C, 9*N]; only the two launches serve this case.
template <typename T>
static bool weights_in_two_passes(const T* w, int64_t N, int64_t K, const int8_t* wq, const int8_t* wqbT, const void* workspace)
{
    return aligned16(w) && K % 8 == 0 && N % 16 == 0 && N <= 16 * kColParts && aligned16(wq) && aligned16(wqbT) && aligned16(workspace);
}
template <typename T> struct WeightParts { WeightMaxima<T> maxima; int64_t maxima_blocks; WeightQuantize<T> quantize; int64_t quantize_blocks; };
template <typename T>
static WeightParts<T> weight_parts(const T* w, int64_t N, int64_t K, float qmax, float* sw, float* iw, float* aw_opt, int8_t* wq,
                                   float* swb, float* iwb, int8_t* wqbT, void* workspace, int64_t conv_C)
{
    float*        partial = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + kCtrBytes);
    const int64_t tiles_x = (K + kTileCols - 1) / kTileCols, row_tiles = (N + kWeightTileRows - 1) / kWeightTileRows;
    const int groups = static_cast<int>(row_tiles < kWeightGroups ? row_tiles : kWeightGroups);
    // Row maxima lie behind the 64 K column maxima in a workspace of 512 K floats: ceil(K / 128) N of them fit while K > 128
    // (N <= 8192 here).  Of a single tile column they are final and wait in sw, where the tile that owns the rows replaces
    // them by their scales (they need not fit then: 4096x8 fp32 in separate passes 17.2 us, so 9.5).
    float*    row_part = tiles_x == 1 ? sw : partial + kWeightGroups * K;
    return WeightParts<T>{WeightMaxima<T>{w, N, K, static_cast<int>(tiles_x), groups, row_part, partial}, tiles_x * groups,
                          WeightQuantize<T>{w, N, K, static_cast<int>(qmax), static_cast<int>(tiles_x), groups, row_part, partial,
                                            WeightOut{sw, iw, aw_opt, swb, iwb, wq, wqbT}, static_cast<int>(conv_C)}, tiles_x * row_tiles};
}

template <typename T>
static hipError_t prepare_weights_typed(const T* w, int64_t N, int64_t K, float qmax, float* sw, float* iw,
                                        float* aw_opt, int8_t* wq, float* swb, float* iwb, int8_t* wqbT,
                                        void* workspace, hipStream_t st, int64_t conv_C = 0)
{
    if(weights_in_two_passes(w, N, K, wq, wqbT, workspace))
    {
        const WeightParts<T> p = weight_parts(w, N, K, qmax, sw, iw, aw_opt, wq, swb, iwb, wqbT, workspace, conv_C);
        launch_part(p.maxima, p.maxima_blocks, st);
        launch_part(p.quantize, p.quantize_blocks, st);
        return hipGetLastError();
    }
    if(conv_C > 0) return hipErrorInvalidValue;      // the caller tests the same conditions before choosing this form
    hipError_t e = absmax_typed(w, N, K, K, kPerRow, qmax, sw, iw, aw_opt, nullptr, nullptr, workspace, st);
    if(e != hipSuccess) return e;
    e = quantize_typed(w, N, K, K, static_cast<int>(qmax), kPerRow, kNearest, 0, 0, iw, wq, nullptr, st);
    if(e != hipSuccess) return e;
    e = absmax_typed(w, N, K, K, kPerCol, qmax, swb, iwb, nullptr, nullptr, nullptr, workspace, st);
    if(e != hipSuccess) return e;
    return quantize_typed(w, N, K, K, static_cast<int>(qmax), kPerCol, kNearest, 0, 0, iwb, nullptr, wqbT, st);
}

hipError_t launch_prepare_weights(const void* w, int wdt, int64_t N, int64_t K, float qmax, float* sw, float* iw,
                                  float* aw_opt, int8_t* wq, float* swb, float* iwb, int8_t* wqbT, void* workspace,
                                  hipStream_t stream)
{
    if(wdt == kF32)
        return prepare_weights_typed(static_cast<const float*>(w), N, K, qmax, sw, iw, aw_opt, wq, swb, iwb, wqbT, workspace, stream);
    return prepare_weights_typed(static_cast<const __half*>(w), N, K, qmax, sw, iw, aw_opt, wq, swb, iwb, wqbT, workspace, stream);
}

// The tiled conversion as a part, f(part, workgroups), where its vector rules hold; false: f was not called.
template <typename Ti, typename To, bool SUMS = false, typename F>
static bool with_convert_tiles(const Ti* x, int64_t rows, int64_t cols, int64_t ld, const float* row_scale, const float* scale, To* q,
                               To* qT, int conv_C, F&& f, float* sums = nullptr)
{
    constexpr int64_t TC = 16 / sizeof(To), in_bytes = TC * sizeof(Ti) < 16 ? TC * sizeof(Ti) : 16;
    const int64_t     bx = (cols + 16 * TC - 1) / (16 * TC), by = (rows + kConvertRows - 1) / kConvertRows;
    if(conv_C > 0 && cols != 9 * conv_C) return false;
    if(cols % TC != 0 || (reinterpret_cast<uintptr_t>(x) & (in_bytes - 1)) != 0 || (ld * sizeof(Ti)) % in_bytes != 0 || !aligned16(q)
       || (rows % TC == 0 && !aligned16(qT)) || bx * by >= (int64_t(1) << 30))
        return false;
    f(ConvertTile<Ti, To, SUMS>{x, rows, cols, ld, row_scale, scale, q, qT, static_cast<int>(bx), conv_C, sums}, bx * by);
    return true;
}
template <typename Ti, typename To>
static bool convert_tiles(const Ti* x, int64_t rows, int64_t cols, int64_t ld, const float* row_scale, const float* scale, To* q,
                          To* qT, hipStream_t st)
{
    return with_convert_tiles(x, rows, cols, ld, row_scale, scale, q, qT, 0, [&](const auto& p, int64_t blocks) { launch_part(p, blocks, st); });
}

// binary16 to binary16 by patches, as a part, where their vector rules hold; false: f was not called.  A row-major copy alone gains from
// them below 2 M elements (1024x1024 3.0 -> 2.7 us) and, while every patch column is whole, below 8 M (4096x768 3.8 -> 3.4,
// 100000x64 5.5 -> 4.8; but 2256x2640 5.6 -> 6.0, and 16384x1024 from memory 13.8 -> 14.7); not with so few rows that most of
// a workgroup's are absent (1x2097152 9.9 -> 12.3).
template <typename F> static bool with_copy_patches(const __half* x, int64_t rows, int64_t cols, int64_t ld, __half* q, __half* qT, F&& f)
{
    const int64_t bx = (cols + 63) / 64, by = (rows + 255) / 256;
    if(cols % 8 != 0 || !aligned16(x) || ld % 8 != 0 || !aligned16(q) || !aligned16(qT) || (qT && rows % 8 != 0)
       || (!qT && (rows < 32 || rows * cols >= (int64_t(1) << (cols % 64 == 0 ? 23 : 21)))) || bx * by >= (int64_t(1) << 30))
        return false;
    f(CopyF16Patch{x, rows, cols, ld, q, qT, bx}, bx * by);
    return true;
}

// The conversion as a part, f(part, workgroups), unless convert_kernel is to do it (false).
template <typename Ti, typename To, bool SUMS = false, typename F>
static bool with_convert_part(const Ti* x, int64_t rows, int64_t cols, int64_t ld, To* q, To* qT, F&& f, float* sums = nullptr)
{
    if constexpr(std::is_same<Ti, __half>::value && std::is_same<To, __half>::value)
        if(with_copy_patches(x, rows, cols, ld, q, qT, f)) return true;
    // columns of a binary16 copy that are no multiple of 16 bytes leave a tile of eight-row chunks element by element; the
    // kernel below, a column per wavefront and store, is faster for large ones of some rows (10002x1032 binary16, transposed
    // alone, 25.3 -> 17.7 us, fp32 28.6 -> 18.5, with both copies 30.7 -> 21.3; but 1569x320 4.7 -> 5.2, 9x262144 7.8 -> 10.2).
    // binary16 with both copies gains in between only (30004x256 19.3 -> 15.3; 7001x304 from memory 9.7 -> 11.4, 10002x1032
    // 28.7 -> 38.6)
    const int64_t n   = rows * cols;
    const bool    odd = std::is_same<To, __half>::value && qT && rows % 8 != 0 && rows >= 32
                     && (std::is_same<Ti, float>::value || !q ? n >= (int64_t(1) << 21) : n >= (int64_t(1) << 22) && n < (int64_t(1) << 23));
    return !odd && with_convert_tiles<Ti, To, SUMS>(x, rows, cols, ld, nullptr, nullptr, q, qT, 0, f, sums);
}

template <typename Ti, typename To>
static hipError_t convert_typed(const void* x, int64_t rows, int64_t cols, int64_t ld, void* q, void* qT,
                                hipStream_t st)
{
    if(with_convert_part(static_cast<const Ti*>(x), rows, cols, ld, static_cast<To*>(q), static_cast<To*>(qT),
                         [&](const auto& p, int64_t blocks) { launch_part(p, blocks, st); }))
        return hipGetLastError();
    const int64_t gx = (cols + 63) / 64, gy = (rows + 63) / 64;
    convert_kernel<Ti, To, false><<<dim3(static_cast<unsigned>(gx * gy)), dim3(kBlock), 0, st>>>(
        static_cast<const Ti*>(x), rows, cols, ld, static_cast<To*>(q), static_cast<To*>(qT), gx, 0, 0, 0);
    return hipGetLastError();
}

// ---- both operands of a forward pass, activation and weights, in shared launches
// What the two conversions do one after the other, stage by stage beside each other: the passes that leave maxima, then the
// passes that fold them and convert.  The weights of an ordinary operator fill a fraction of the chip and each pass over
// them is one memory latency long, so beside the activation they cost next to nothing; a small operator is bound by the
// number of launches.  Whole steps, apart -> beside each other: 64x128x128 28.7 -> 22.9 us, 1808x1040x784 50.9 -> 43.5, INT8
// 4096x3072x768 87.8 -> 80.0, FP16 2056x1000x1032 64.9 -> 61.7, convolution 64x56x56x64 126.4 -> 115.8.  Merged where every part is one of 256 threads: weights fp32 and, for codes, in two passes or small;
// an activation whose transposed copy is large enough for 128-row tiles keeps its own launches.
template <typename T> static bool small_tiles(int64_t rows, int64_t cols, const int8_t* qT, int64_t n)
{
    return tiles_of(rows, cols, 128) < 512 && !odd_transpose_apart<T>(rows, n, qT);
}
template <typename T> static int64_t maxima_blocks(int64_t n)
{
    const int64_t nb = (n / Vec16<T>::N + BlockMaxima<T>::kVectors - 1) / BlockMaxima<T>::kVectors;
    return nb > 1024 ? 1024 : nb;
}

template <typename TX> static bool convert_int8_operands(const OperandConversion& c, hipStream_t st)
{
    const TX*     x = static_cast<const TX*>(c.x);
    const float*  w = static_cast<const float*>(c.w);
    const int64_t nx = c.M * c.C, K = c.taps * c.C, nw = c.N * K;
    int8_t *const xq = static_cast<int8_t*>(c.xq), *const xqT = static_cast<int8_t*>(c.xqT);
    int8_t *const wq = static_cast<int8_t*>(c.wq), *const wqbT = static_cast<int8_t*>(c.wqbT);
    const bool    stream = xq && !xqT;
    if(!tile_ok(x, c.M, c.C, c.C, xq, xqT) || !(stream || small_tiles<TX>(c.M, c.C, xqT, nx))) return false;
    const bool w_rows = c.w_gran == kPerRow;
    if(w_rows ? !weights_in_two_passes(w, c.N, K, wq, wqbT, c.ws_w)
              : c.taps != 1 || !tile_ok(w, c.N, K, K, wq, wqbT) || !small_tiles<float>(c.N, K, wqbT, nw)) return false;
    const bool    x_whole = !c.x_amax && nx * static_cast<int64_t>(sizeof(TX)) <= kWholeBytes;
    const bool    w_whole = !w_rows && nw * 4 <= kWholeBytes;
    const float   qm = static_cast<float>(c.qmax);
    float* const  px = reinterpret_cast<float*>(static_cast<uint8_t*>(c.ws_x) + kCtrBytes);
    float* const  pw = reinterpret_cast<float*>(static_cast<uint8_t*>(c.ws_w) + kCtrBytes);
    const int64_t bx = maxima_blocks<TX>(nx), bw = maxima_blocks<float>(nw);
    const int     tx = static_cast<int>((c.C + kTileCols - 1) / kTileCols), tw = static_cast<int>((K + kTileCols - 1) / kTileCols);
    const TensorScale sx{c.ix, px, static_cast<int>(bx), c.sx, c.ix, c.ax}, sw{nullptr, pw, static_cast<int>(bw), c.sw, c.iw, c.aw};
    const int64_t tiles_x = tiles_of(c.M, c.C, 64), tiles_w = tiles_of(c.N, K, 64);
    const int64_t groups = nx / 8, stream_blocks = (groups + kBlock * 4 - 1) / (kBlock * 4);
    if(stream_blocks + tiles_x + tiles_w >= (int64_t(1) << 31)) return false;
    const WeightParts<float> wp = w_rows ? weight_parts(w, c.N, K, qm, c.sw, c.iw, c.aw, wq, c.swb, c.iwb, wqbT, c.ws_w, c.taps == 9 ? c.C : 0)
                                         : WeightParts<float>{};
    auto x1 = [&](auto&& f) {
        if(c.x_amax)     f(ScaleFromAmax{c.x_amax, qm, c.sx, c.ix, 1}, 1);
        else if(x_whole) f(QuantizeTile<TX, kNearest, 64, kWhole>{x, c.M, c.C, c.C, c.qmax, 0, 0, sx, xq, xqT, tx}, tiles_x);
        else             f(BlockMaxima<TX>{x, nx, bx, px}, bx);
    };
    auto x2 = [&](auto&& f) {
        if(c.x_amax && stream) f(QuantizeStream<TX, kNearest, kInv>{x, groups, c.qmax, 0, 0, sx, xq}, stream_blocks);
        else if(c.x_amax)      f(QuantizeTile<TX, kNearest, 64, kInv>{x, c.M, c.C, c.C, c.qmax, 0, 0, sx, xq, xqT, tx}, tiles_x);
        else if(stream)        f(QuantizeStream<TX, kNearest, kPartials>{x, groups, c.qmax, 0, 0, sx, xq}, stream_blocks);
        else                   f(QuantizeTile<TX, kNearest, 64, kPartials>{x, c.M, c.C, c.C, c.qmax, 0, 0, sx, xq, xqT, tx}, tiles_x);
    };
    auto w1 = [&](auto&& f) {
        if(w_rows)       f(wp.maxima, wp.maxima_blocks);
        else if(w_whole) f(QuantizeTile<float, kNearest, 64, kWhole>{w, c.N, K, K, c.qmax, 0, 0, sw, wq, wqbT, tw}, tiles_w);
        else             f(BlockMaxima<float>{w, nw, bw, pw}, bw);
    };
    auto w2 = [&](auto&& f) {
        if(w_rows) f(wp.quantize, wp.quantize_blocks);
        else       f(QuantizeTile<float, kNearest, 64, kPartials>{w, c.N, K, K, c.qmax, 0, 0, sw, wq, wqbT, tw}, tiles_w);
    };
    // (weights first: theirs are the longer chains of dependent accesses)
    auto together = [&](auto&& a, auto&& b) {
        a([&](const auto& pa, int64_t na) { b([&](const auto& pb, int64_t nb) { launch_parts(pa, na, pb, nb, st); }); });
    };
    auto alone = [&](const auto& p, int64_t blocks) { launch_part(p, blocks, st); };
    if(x_whole && w_whole)
    {   // tiles of 512 threads: half the loads per thread for the maximum, which is what these launches wait for
        // (64x128 and 128x128 fp32 6.2 -> 5.0 us)
        launch_parts(QuantizeTile<float, kNearest, 128, kWhole>{w, c.N, K, K, c.qmax, 0, 0, sw, wq, wqbT, tw}, tiles_of(c.N, K, 128),
                     QuantizeTile<TX, kNearest, 128, kWhole>{x, c.M, c.C, c.C, c.qmax, 0, 0, sx, xq, xqT, tx}, tiles_of(c.M, c.C, 128), st);
        return true;
    }
    together(w1, x1);
    if(!x_whole && !w_whole) together(w2, x2);
    else if(!x_whole)        x2(alone);
    else                     w2(alone);
    return true;
}

// Casts and copies: activation (unless it is used as it is) and weights in one launch.
template <typename TX, typename To> static bool convert_float_operands(const OperandConversion& c, hipStream_t st)
{
    const int64_t K = c.taps * c.C;
    const float*  w = static_cast<const float*>(c.w);
    To *const     wq = static_cast<To*>(c.wq), *const wqbT = static_cast<To*>(c.wqbT);
    bool          done = false;
    auto weights = [&](auto&& f) {
        return c.taps == 9 ? with_convert_tiles(w, c.N, K, K, nullptr, nullptr, wq, wqbT, static_cast<int>(c.C), f)
                           : with_convert_part(w, c.N, K, K, wq, wqbT, f);
    };
    if(!c.xq && !c.xqT)
        return weights([&](const auto& p, int64_t blocks) { launch_part(p, blocks, st); });
    weights([&](const auto& pw, int64_t bw) {
        done = with_convert_part(static_cast<const TX*>(c.x), c.M, c.C, c.C, static_cast<To*>(c.xq), static_cast<To*>(c.xqT),
                                 [&](const auto& px, int64_t bx) { launch_parts(pw, bw, px, bx, st); });
    });
    return done;
}

hipError_t launch_convert_operands(const OperandConversion& c, int tag, int xdt, bool* taken, hipStream_t st)
{
    const bool half = xdt == kF16;
    *taken = tag == 8    ? (half ? convert_int8_operands<__half>(c, st) : convert_int8_operands<float>(c, st))
             : tag == 16 ? (half ? convert_float_operands<__half, __half>(c, st) : convert_float_operands<float, __half>(c, st))
                         : (half ? convert_float_operands<__half, float>(c, st) : convert_float_operands<float, float>(c, st));
    return *taken ? hipGetLastError() : hipSuccess;
}

hipError_t launch_convert(const void* x, int xdt, int64_t rows, int64_t cols, int64_t ld, int outdt, void* q, void* qT,
                          hipStream_t stream)
{
    if(xdt == kF32 && outdt == kF16) return convert_typed<float, __half>(x, rows, cols, ld, q, qT, stream);
    if(xdt == kF32 && outdt == kF32) return convert_typed<float, float>(x, rows, cols, ld, q, qT, stream);
    if(xdt == kF16 && outdt == kF16) return convert_typed<__half, __half>(x, rows, cols, ld, q, qT, stream);
    return convert_typed<__half, float>(x, rows, cols, ld, q, qT, stream);
}

hipError_t launch_convert_sr(const float* x, int64_t rows, int64_t cols, int64_t ld, int mantissa_bits, uint64_t seed,
                             uint64_t offset, void* q, void* qT, hipStream_t stream)
{
    const int64_t gx = (cols + 63) / 64, gy = (rows + 63) / 64;
    convert_kernel<float, __half, true><<<dim3(static_cast<unsigned>(gx * gy)), dim3(kBlock), 0, stream>>>(
        x, rows, cols, ld, static_cast<__half*>(q), static_cast<__half*>(qT), gx, seed, offset, mantissa_bits);
    return hipGetLastError();
}

template <typename Ti, typename To>
static hipError_t dequantize_typed(const void* a, int64_t rows, int64_t cols, int64_t ld, const float* rs,
                                   const float* cs, float ts, const float* tsd, const float* cb, void* y, hipStream_t st)
{
    if constexpr(std::is_same<Ti, int8_t>::value)
    {
        constexpr int V = 16 / sizeof(To);
        const int64_t n = rows * cols;
        if(ld == cols && !rs && !cs && !cb && n >= V && aligned16(y) && reinterpret_cast<uintptr_t>(a) % V == 0)
        {
            auto go = [&](auto u, auto stream) {
                constexpr int U = decltype(u)::value;
                const int64_t nb = (n / V + kBlock * U - 1) / (kBlock * U);
                dequantize_flat_kernel<To, U, decltype(stream)::value><<<dim3(static_cast<unsigned>(nb)), dim3(kBlock), 0, st>>>(
                    static_cast<const int8_t*>(a), n, ts, tsd, static_cast<To*>(y));
            };
            if(n < (int64_t(1) << 20)) go(std::integral_constant<int, 1>{}, std::false_type{});
            else if(n < (int64_t(1) << 24)) go(std::integral_constant<int, 4>{}, std::false_type{});
            else if(n * static_cast<int64_t>(sizeof(To)) < (int64_t(1) << 27)) go(std::integral_constant<int, 2>{}, std::false_type{});
            else go(std::integral_constant<int, 8>{}, std::true_type{});
            return hipGetLastError();
        }
    }
    constexpr int V16 = 16 / sizeof(Ti);
    const bool    wide = cols % V16 == 0 && (ld * sizeof(Ti)) % 16 == 0 && aligned16(a) && aligned16(y)
                      && (!cs || aligned16(cs)) && (!cb || aligned16(cb));
    // (without per-column parameters the flat kernel below streams 32-bit inputs a little faster: measured)
    if(wide && (cs || cb || sizeof(Ti) == 1))
    {
        const int64_t cv = cols / V16;
        int           tx_log2 = 8;                                   // the whole block along the row when possible
        while(tx_log2 > 0 && (int64_t(1) << (tx_log2 - 1)) >= cv) --tx_log2;
        const int64_t gx = (cv + (int64_t(1) << tx_log2) - 1) >> tx_log2;
        const int64_t ty = kBlock >> tx_log2;
        int64_t       gy = (rows + ty * 4 - 1) / (ty * 4);           // four rows in flight per thread
        if(gy > 65535) gy = 65535;
        if(gy < 1) gy = 1;
        if(gx < (int64_t(1) << 31))
        {
            dequantize_cols_kernel<Ti, To><<<dim3(static_cast<unsigned>(gx), static_cast<unsigned>(gy)), dim3(kBlock), 0, st>>>(
                static_cast<const Ti*>(a), rows, cols, ld, rs, cs, ts, tsd, cb, static_cast<To*>(y), tx_log2);
            return hipGetLastError();
        }
    }
    const bool vec = cols % 4 == 0 && ld % 4 == 0 && (reinterpret_cast<uintptr_t>(a) % (4 * sizeof(Ti))) == 0
                  && (reinterpret_cast<uintptr_t>(y) % (4 * sizeof(To))) == 0;
    const int64_t work = vec ? rows * (cols / 4) : rows * cols;
    int64_t       nb   = (work + kBlock - 1) / kBlock;
    nb                 = nb > (1 << 20) ? (1 << 20) : nb;
    if(vec)
        dequantize_kernel<Ti, To, 4><<<dim3(nb), dim3(kBlock), 0, st>>>(static_cast<const Ti*>(a), rows, cols, ld, rs,
                                                                       cs, ts, tsd, cb, static_cast<To*>(y));
    else
        dequantize_kernel<Ti, To, 1><<<dim3(nb), dim3(kBlock), 0, st>>>(static_cast<const Ti*>(a), rows, cols, ld, rs,
                                                                       cs, ts, tsd, cb, static_cast<To*>(y));
    return hipGetLastError();
}

hipError_t launch_dequantize_f16_tiles(const int8_t* a, int64_t rows, int64_t cols, const float* row_scale, const float* scale, void* y,
                                      void* yT, hipStream_t stream)
{
    if(convert_tiles(a, rows, cols, cols, row_scale, scale, static_cast<__half*>(y), static_cast<__half*>(yT), stream)) return hipGetLastError();
    const hipError_t e = launch_dequantize(a, kI8, rows, cols, cols, row_scale, nullptr, 1.0f, row_scale ? nullptr : scale, nullptr, y, kF16, stream);
    return e != hipSuccess || !yT ? e : launch_convert(y, kF16, rows, cols, cols, kF16, nullptr, yT, stream);
}

hipError_t launch_dequantize_f16_both(const int8_t* x, int64_t xr, int64_t xc, const float* x_scale, void* xh, const int8_t* w, int64_t N,
                                      int64_t K, const float* w_row_scale, const float* w_scale, void* wh, void* whT, hipStream_t st)
{
    bool done = false;
    with_convert_tiles(w, N, K, K, w_row_scale, w_scale, static_cast<__half*>(wh), static_cast<__half*>(whT), 0, [&](const auto& pw, int64_t bw) {
        done = with_convert_tiles(x, xr, xc, xc, nullptr, x_scale, static_cast<__half*>(xh), static_cast<__half*>(nullptr), 0,
                                  [&](const auto& px, int64_t bx) { launch_parts(pw, bw, px, bx, st); });
    });
    if(done) return hipGetLastError();
    const hipError_t e = launch_dequantize_f16_tiles(x, xr, xc, nullptr, x_scale, xh, nullptr, st);
    return e != hipSuccess ? e : launch_dequantize_f16_tiles(w, N, K, w_row_scale, w_scale, wh, whT, st);
}

hipError_t launch_dequantize(const void* a, int adt, int64_t rows, int64_t cols, int64_t ld, const float* row_scale,
                             const float* col_scale, float tensor_scale, const float* tensor_scale_dev,
                             const float* col_bias, void* y, int ydt, hipStream_t stream)
{
    if(adt == kI32 && ydt == kF32)
        return dequantize_typed<int32_t, float>(a, rows, cols, ld, row_scale, col_scale, tensor_scale, tensor_scale_dev, col_bias, y, stream);
    if(adt == kI32 && ydt == kF16)
        return dequantize_typed<int32_t, __half>(a, rows, cols, ld, row_scale, col_scale, tensor_scale, tensor_scale_dev, col_bias, y, stream);
    if(adt == kI8 && ydt == kF32)
        return dequantize_typed<int8_t, float>(a, rows, cols, ld, row_scale, col_scale, tensor_scale, tensor_scale_dev, col_bias, y, stream);
    return dequantize_typed<int8_t, __half>(a, rows, cols, ld, row_scale, col_scale, tensor_scale, tensor_scale_dev, col_bias, y, stream);
}

// wflip[c, (8 - tap)*N + n] = w[n, tap*C + c]: a few kilobytes of weights, one element per thread.
template <typename T>
__global__ __launch_bounds__(256) void conv3x3_wflip_kernel(const T* __restrict__ w, int64_t N, int64_t C, T* __restrict__ wflip)
{
    const int64_t total = 9 * N * C;
    for(int64_t o = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; o < total; o += static_cast<int64_t>(gridDim.x) * 256)
    {
        const int64_t c = o / (9 * N), r = o - c * 9 * N, tap = r / N, n = r - tap * N;
        wflip[o] = w[n * 9 * C + (8 - tap) * C + c];
    }
}

hipError_t launch_conv3x3_wflip(const void* w, int elem_bytes, int64_t N, int64_t C, void* wflip, hipStream_t stream)
{
    const int64_t total = 9 * N * C;
    if(total <= 0) return hipSuccess;
    int64_t nb = (total + 255) / 256;
    nb         = nb > 4096 ? 4096 : nb;
    if(elem_bytes == 1)
        conv3x3_wflip_kernel<int8_t><<<dim3(static_cast<unsigned>(nb)), dim3(256), 0, stream>>>(
            static_cast<const int8_t*>(w), N, C, static_cast<int8_t*>(wflip));
    else
        conv3x3_wflip_kernel<uint16_t><<<dim3(static_cast<unsigned>(nb)), dim3(256), 0, stream>>>(
            static_cast<const uint16_t*>(w), N, C, static_cast<uint16_t*>(wflip));
    return hipGetLastError();
}

hipError_t launch_conv3x3_prepare_weights(const void* w, int wdt, int64_t N, int64_t C, float qmax, float* sw, float* iw,
                                          float* swb, float* iwb, int8_t* wq, int8_t* wflip, void* workspace,
                                          hipStream_t st)
{
    const int64_t K = 9 * C;
    const int64_t e2 = wdt == kF32 ? 8 : 16;
    if(K % e2 == 0 && weights_in_two_passes(w, N, K, wq, wflip, workspace))
    {
        if(wdt == kF32)
            return prepare_weights_typed(static_cast<const float*>(w), N, K, qmax, sw, iw, nullptr, wq, swb, iwb, wflip, workspace, st, C);
        return prepare_weights_typed(static_cast<const __half*>(w), N, K, qmax, sw, iw, nullptr, wq, swb, iwb, wflip, workspace, st, C);
    }
    // large weights: the separate passes; the per-c codes go through the workspace (behind the absmax scratch)
    int8_t*    wqb = static_cast<int8_t*>(workspace) + absmax_workspace_bytes(N, K, kPerCol);
    hipError_t e   = launch_absmax_scale(w, wdt, N, K, K, kPerRow, qmax, sw, iw, nullptr, nullptr, nullptr, workspace, st);
    if(e != hipSuccess) return e;
    e = launch_quantize_int8(w, wdt, N, K, K, static_cast<int>(qmax), kPerRow, kNearest, 0, 0, iw, wq, nullptr, st);
    if(e != hipSuccess) return e;
    e = launch_absmax_scale(w, wdt, 9 * N, C, C, kPerCol, qmax, swb, iwb, nullptr, nullptr, nullptr, workspace, st);
    if(e != hipSuccess) return e;
    e = launch_quantize_int8(w, wdt, 9 * N, C, C, static_cast<int>(qmax), kPerCol, kNearest, 0, 0, iwb, wqb, nullptr, st);
    if(e != hipSuccess) return e;
    return launch_conv3x3_wflip(wqb, 1, N, C, wflip, st);
}


hipError_t launch_im2col3x3_i8(const int8_t* xq, int64_t nimg, int H, int W, int C, int8_t* a, int8_t* aT,
                               hipStream_t stream)
{
    const int64_t M  = nimg * H * W;
    const int64_t gx = (9 * C / 16 + 7) / 8, gy = (M + 511) / 512;
    im2col3x3_i8_kernel<<<dim3(static_cast<unsigned>(gx * gy)), dim3(kBlock), 0, stream>>>(xq, nimg, H, W, C, a, aT, gx);
    return hipGetLastError();
}

ConvPaddedAxis conv_padded_axis(int64_t nimg, int H, int W)
{
    ConvPaddedAxis a;
    a.Wp = (W + 1 + 15) / 16 * 16;
    a.Mp = (nimg * (H + 1) + 1) * a.Wp;          // a multiple of 16
    return a;
}

hipError_t launch_conv_padded_transpose(const void* in, int elem_bytes, int64_t nimg, int H, int W, int Ch, int copies,
                                        void* out, int margin_bytes, hipStream_t stream)
{
    const ConvPaddedAxis ax = conv_padded_axis(nimg, H, W);
    const int     ncc = Ch / (16 / elem_bytes);
    int           cw_log2 = 2;                                   // four channel chunks side by side when there are that many
    while(cw_log2 > 0 && (1 << (cw_log2 - 1)) >= ncc) --cw_log2;
    const int64_t groups = (ncc + (1 << cw_log2) - 1) >> cw_log2;
    const int64_t lanes  = (ax.Mp / 16) * groups << cw_log2;
    const int64_t nb     = (lanes + kBlock - 1) / kBlock;
    if(nb >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    const dim3    grid(static_cast<unsigned>(nb)), block(kBlock);
    const int8_t* src = static_cast<const int8_t*>(in);
    int8_t*       dst = static_cast<int8_t*>(out);
    if(elem_bytes == 1)
    {
        if(copies == 3) conv_padded_transpose_kernel<3, 1><<<grid, block, 0, stream>>>(src, nimg, H, W, Ch, ax.Wp, ax.Mp, dst, cw_log2, margin_bytes);
        else            conv_padded_transpose_kernel<1, 1><<<grid, block, 0, stream>>>(src, nimg, H, W, Ch, ax.Wp, ax.Mp, dst, cw_log2, margin_bytes);
    }
    else
    {
        if(copies == 3) conv_padded_transpose_kernel<3, 2><<<grid, block, 0, stream>>>(src, nimg, H, W, Ch, ax.Wp, ax.Mp, dst, cw_log2, margin_bytes);
        else            conv_padded_transpose_kernel<1, 2><<<grid, block, 0, stream>>>(src, nimg, H, W, Ch, ax.Wp, ax.Mp, dst, cw_log2, margin_bytes);
    }
    return hipGetLastError();
}

size_t colsum_workspace_bytes(int64_t rows, int64_t cols)
{
    (void)rows;
    return sizeof(float) * static_cast<size_t>(kColParts) * static_cast<size_t>(cols > 0 ? cols : 0);
}

// ------------------------------------------------------------------ transpose of int8 codes
// out[c, r] = in[r, c].  A lane owns a 16 x 16 byte patch: sixteen 16-byte loads, a byte transpose in registers,
// sixteen 16-byte stores; a wavefront is 8 patches wide (128-byte row segments) and 8 patches high.
__global__ __launch_bounds__(kBlock) void transpose_i8_patch_kernel(const int8_t* __restrict__ in, int64_t rows, int64_t cols,
                                                                   int8_t* __restrict__ out, int64_t grid_x)
{
    const int     lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
    const int64_t by = blockIdx.x / grid_x, bx = blockIdx.x - by * grid_x;
    const int64_t r0 = (by * (kBlock / kWaveSize) + wave) * 128 + (lane / 8) * 16;
    const int64_t c0 = bx * 128 + (lane % 8) * 16;
    if(r0 >= rows || c0 >= cols) return;                   // rows and cols are multiples of 16: patches are whole
    uint4 raw[16];
#pragma unroll
    for(int i = 0; i < 16; ++i) raw[i] = *reinterpret_cast<const uint4*>(in + (r0 + i) * cols + c0);
#pragma unroll
    for(int c = 0; c < 16; ++c)
    {
        uint32_t t[4];
#pragma unroll
        for(int g = 0; g < 4; ++g)
        {
            auto word = [&](int r) -> uint32_t {
                const uint4& v = raw[r];
                return (c / 4) == 0 ? v.x : (c / 4) == 1 ? v.y : (c / 4) == 2 ? v.z : v.w;
            };
            t[g] = byte_of(word(4 * g + 0), c % 4) | (byte_of(word(4 * g + 1), c % 4) << 8)
                 | (byte_of(word(4 * g + 2), c % 4) << 16) | (byte_of(word(4 * g + 3), c % 4) << 24);
        }
        *reinterpret_cast<uint4*>(out + (c0 + c) * rows + r0) = make_uint4(t[0], t[1], t[2], t[3]);
    }
}

__global__ __launch_bounds__(kBlock) void transpose_i8_generic_kernel(const int8_t* __restrict__ in, int64_t rows, int64_t cols,
                                                                     int8_t* __restrict__ out)
{
    const int64_t n = rows * cols, stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for(int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride)
    {
        const int64_t r = i / cols, c = i - r * cols;
        out[c * rows + r] = in[i];
    }
}

hipError_t launch_transpose_i8(const int8_t* in, int64_t rows, int64_t cols, int8_t* out, hipStream_t stream)
{
    if(rows <= 0 || cols <= 0) return hipSuccess;
    const int64_t gx = (cols + 127) / 128, gy = (rows + 128 * (kBlock / kWaveSize) - 1) / (128 * (kBlock / kWaveSize));
    if(rows % 16 == 0 && cols % 16 == 0 && aligned16(in) && aligned16(out) && gx * gy < (int64_t(1) << 31))
        transpose_i8_patch_kernel<<<dim3(static_cast<unsigned>(gx * gy)), dim3(kBlock), 0, stream>>>(in, rows, cols, out, gx);
    else
    {
        int64_t nb = (rows * cols + kBlock - 1) / kBlock;
        nb         = nb > 65536 ? 65536 : nb;
        transpose_i8_generic_kernel<<<dim3(static_cast<unsigned>(nb)), dim3(kBlock), 0, stream>>>(in, rows, cols, out);
    }
    return hipGetLastError();
}

// Clears n floats with a kernel (a memset node recorded into a captured graph is avoided on purpose).
__global__ __launch_bounds__(256) void zero_f32_kernel(float* __restrict__ p, int64_t n)
{
    for(int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * 256)
        p[i] = 0.0f;
}

hipError_t launch_zero_f32(float* p, int64_t n, hipStream_t stream)
{
    if(n <= 0) return hipSuccess;
    int64_t nb = (n + 255) / 256;
    nb         = nb > 1024 ? 1024 : nb;
    zero_f32_kernel<<<dim3(static_cast<unsigned>(nb)), dim3(256), 0, stream>>>(p, n);
    return hipGetLastError();
}

template <typename T>
static void colsum_partials(const T* x, int64_t rows, int64_t cols, float* workspace, int& S, hipStream_t st)
{
    const TensorFinal none{0.0f, nullptr, nullptr, nullptr, nullptr, nullptr};
    int               nmax;
    colreduce_first<T, OP_SUM>(x, rows, cols, cols, workspace, nullptr, none, S, nmax, st);
}
hipError_t launch_colsum_partials(const void* x, int xdt, int64_t rows, int64_t cols, float* out, float* workspace, ColumnFoldArgs* fold,
                                  hipStream_t stream)
{
    int S;
    if(xdt == kF32) colsum_partials(static_cast<const float*>(x), rows, cols, workspace, S, stream);
    else            colsum_partials(static_cast<const __half*>(x), rows, cols, workspace, S, stream);
    *fold = ColumnFoldArgs{workspace, S, cols, out};
    return hipGetLastError();
}

hipError_t launch_column_fold(const ColumnFoldArgs& fold, hipStream_t stream)
{
    launch_part(ColumnFold<kBlock>{fold}, fold.blocks(), stream);
    return hipGetLastError();
}

template <typename To>
static bool convert_sums(const float* x, int64_t rows, int64_t cols, void* q, void* qT, float* workspace, hipStream_t st)
{
    return with_convert_part<float, To, true>(x, rows, cols, cols, static_cast<To*>(q), static_cast<To*>(qT),
                                              [&](const auto& p, int64_t blocks) { launch_part(p, blocks, st); }, workspace);
}
hipError_t launch_convert_sums(const float* x, int64_t rows, int64_t cols, int outdt, void* q, void* qT, float* out, float* workspace,
                               ColumnFoldArgs* fold, bool* taken, hipStream_t stream)
{
    const int64_t S = (rows + kConvertRows - 1) / kConvertRows;
    *taken = S <= kColParts && (outdt == kF16 ? convert_sums<__half>(x, rows, cols, q, qT, workspace, stream)
                                              : convert_sums<float>(x, rows, cols, q, qT, workspace, stream));
    if(!*taken) return hipSuccess;
    *fold = ColumnFoldArgs{workspace, static_cast<int>(S), cols, out};
    return hipGetLastError();
}

}  // namespace qsync
