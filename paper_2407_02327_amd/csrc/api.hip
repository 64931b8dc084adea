// C ABI of libqsync: argument validation (the "front-end security wrapper" the paper's backend
// puts around its tensorized kernels) and dispatch to the gfx950 kernels.  Validation never
// touches the HIP runtime, so every argument error is reported even on a machine with no GPU.
#include "../../include/qsync.h"
#include "../../include/qsync_debug.h"
#include "kernels.h"

#include <limits>

using namespace qsync;

namespace {

thread_local int g_last_hip_error = 0;
thread_local int g_last_pair_tile = -1;      // see qsync_debug_last_gradient_pair
thread_local int g_last_pair_splits = 0;     // see qsync_debug_last_gradient_splits

int hip_status(hipError_t e)
{
    if(e == hipSuccess) return QSYNC_OK;
    g_last_hip_error = static_cast<int>(e);
    (void)hipGetLastError();   // clear the sticky launch error
    return QSYNC_ERR_HIP;
}

bool is_float_dtype(int dt) { return dt == QSYNC_F32 || dt == QSYNC_F16; }
bool is_tag(int t) { return t == QSYNC_INT8 || t == QSYNC_FP16 || t == QSYNC_FP32; }
bool is_gran(int g) { return g == QSYNC_PER_TENSOR || g == QSYNC_PER_ROW || g == QSYNC_PER_COL; }
bool is_round(int r) { return r == QSYNC_ROUND_NEAREST || r == QSYNC_ROUND_STOCHASTIC || r == QSYNC_ROUND_FLOOR; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// rows*cols (and a few multiples of it) must fit comfortably in int64
bool count_ok(int64_t a, int64_t b)
{
    if(a < 0 || b < 0) return false;
    if(a == 0 || b == 0) return true;
    return a <= (std::numeric_limits<int64_t>::max() / 64) / b;
}

// the contraction axis of an MFMA GEMM: rows of at most 16 MiB (32-bit lane offsets inside an operand panel)
bool gemm_row_ok(int tag, int64_t k)
{
    const int64_t esz = tag == QSYNC_INT8 ? 1 : (tag == QSYNC_FP16 ? 2 : 4);
    return k <= kGemmMaxRowBytes / esz;
}

size_t round256(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }

GemmProblem data_gradient(int tag, int64_t M, int64_t N, int64_t K, const void* dyq, const float* sdy, const void* wqbT,
                          const float* swb, int wbgran, void* dx, int dxdt, int32_t* acc_dump)
{
    GemmProblem p{};
    p.prec = tag; p.M = M; p.N = K; p.K = N;
    p.A = dyq; p.B = wqbT; p.C = dx; p.c_dtype = dxdt;
    if(tag == QSYNC_INT8)
    {
        p.s0 = sdy;
        if(wbgran == QSYNC_PER_TENSOR) p.s1 = swb; else p.col_scale = swb;
        p.acc_dump = acc_dump;
    }
    return p;
}

bool overlap(const void* a, int64_t a_bytes, const void* b, int64_t b_bytes)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return a && b && x < y + static_cast<uintptr_t>(b_bytes) && y < x + static_cast<uintptr_t>(a_bytes);
}

// (Beside the last launch and with the cast of dY summing its columns, whole steps: FP16 2056x1000x1032 from fp32 gradients 61.7
// -> 56.1 us, INT8 forward with FP16 backward 4096x768x3072 123.5 -> 121.4 -- with the two dequantizations in one launch --,
// fp32 8192x4096x1024 1611 -> 1580.)
// The gradient GEMMs that are wanted, in one launch where that is estimated faster, and the fold of the column sums: in
// workgroups of the last launch that can take it, unless the sums go where the GEMMs read or write.
int run_gradients(const GemmProblem* dx, const GemmPlan& plan_dx, void* ws_dx, const GemmProblem* dw, const GemmPlan& plan_dw, void* ws_dw,
                  ColumnFoldArgs fold, hipStream_t st)
{
    auto touches = [&](const GemmProblem* p) {
        const int64_t esz = p ? p->prec / 8 : 0, n = fold.cols * 4;
        return p && (overlap(fold.out, n, p->A, p->M * p->K * esz) || overlap(fold.out, n, p->B, p->N * p->K * esz)
                     || overlap(fold.out, n, p->C, p->M * p->N * (p->c_dtype == kF16 ? 2 : 4)) || overlap(fold.out, n, p->acc_dump, p->M * p->N * 4)
                     || overlap(fold.out, n, p->s0, 4) || overlap(fold.out, n, p->s1, 4) || overlap(fold.out, n, p->col_scale, p->N * 4));
    };
    const bool beside = fold.out && !touches(dx) && !touches(dw);
    const GradientPair pair = dx && dw ? gradient_pair(*dx, plan_dx, *dw, plan_dw) : GradientPair{};
    g_last_pair_tile   = pair.splits == 1 ? pair.tile : -1;
    g_last_pair_splits = pair.tile >= 0 ? pair.splits : 0;
    int rc = QSYNC_OK;
    if(pair.tile >= 0)
    {
        rc = hip_status(launch_gradient_pair(*dx, ws_dx, *dw, ws_dw, pair, beside ? fold : ColumnFoldArgs{}, st));
        if(beside) fold = ColumnFoldArgs{};
    }
    else
    {
        if(dx) rc = hip_status(launch_gemm(*dx, plan_dx, ws_dx, st, beside && !dw ? &fold : nullptr));
        if(dw && rc == QSYNC_OK) rc = hip_status(launch_gemm(*dw, plan_dw, ws_dw, st, beside ? &fold : nullptr));
    }
    if(rc == QSYNC_OK && fold.out) rc = hip_status(launch_column_fold(fold, st));
    return rc;
}

}  // namespace

extern "C" {

int qsync_version(void) { return 100; }

int qsync_last_hip_error(void) { return g_last_hip_error; }

const char* qsync_strerror(int status)
{
    switch(status)
    {
    case QSYNC_OK: return "ok";
    case QSYNC_ERR_NULL: return "a required pointer is NULL";
    case QSYNC_ERR_BAD_ENUM: return "an enum argument holds no enumerator";
    case QSYNC_ERR_BAD_SHAPE: return "bad shape: negative dimension, ld < cols, or element count overflow";
    case QSYNC_ERR_UNSUPPORTED: return "unsupported combination of arguments";
    case QSYNC_ERR_ALIGN: return "pointer or dimension violates an alignment rule";
    case QSYNC_ERR_WORKSPACE: return "workspace missing or too small";
    case QSYNC_ERR_HIP: return "a HIP runtime call failed (see qsync_last_hip_error)";
    default: return "unknown status";
    }
}

size_t qsync_absmax_workspace_bytes(int64_t rows, int64_t cols, int gran)
{
    if(rows < 0 || cols < 0 || !is_gran(gran)) return 0;
    return round256(absmax_workspace_bytes(rows, cols, gran));
}

int qsync_absmax_scale(const void* x, int xdt, int64_t rows, int64_t cols, int64_t ld, int gran, int bits,
                       float* scale, float* inv_scale, float* amax_opt, float* colsum_opt, float* sumsq_opt,
                       void* workspace, size_t workspace_bytes, void* stream)
{
    if(!x || !scale || !inv_scale) return QSYNC_ERR_NULL;
    if(!is_float_dtype(xdt) || !is_gran(gran)) return QSYNC_ERR_BAD_ENUM;
    if(!count_ok(rows, cols) || ld < cols || !count_ok(rows, ld)) return QSYNC_ERR_BAD_SHAPE;
    if(bits < 2 || bits > 8) return QSYNC_ERR_UNSUPPORTED;
    if((colsum_opt || sumsq_opt) && gran != QSYNC_PER_TENSOR) return QSYNC_ERR_UNSUPPORTED;
    if(colsum_opt && cols > (int64_t(1) << 19)) return QSYNC_ERR_UNSUPPORTED;   // one block-maximum slot per column strip
    if(rows == 0 || cols == 0) return QSYNC_OK;
    const size_t need = qsync_absmax_workspace_bytes(rows, cols, gran);
    if(need > 0)
    {
        if(!workspace || workspace_bytes < need) return QSYNC_ERR_WORKSPACE;
        if(!aligned16(workspace)) return QSYNC_ERR_ALIGN;
    }
    const float qmax = static_cast<float>((1 << (bits - 1)) - 1);
    return hip_status(launch_absmax_scale(x, xdt, rows, cols, ld, gran, qmax, scale, inv_scale, amax_opt, colsum_opt,
                                          sumsq_opt, workspace, static_cast<hipStream_t>(stream)));
}

int qsync_absmax_scale_static(const void* x, int xdt, int64_t rows, int64_t cols, int64_t ld, int bits, float* scale,
                              float* inv_scale, float* amax_opt, float* colsum_opt, float* sumsq_opt, void* stream)
{
    if(!x || !scale || !inv_scale) return QSYNC_ERR_NULL;
    if(!is_float_dtype(xdt)) return QSYNC_ERR_BAD_ENUM;
    if(!count_ok(rows, cols) || ld < cols || !count_ok(rows, ld)) return QSYNC_ERR_BAD_SHAPE;
    if(bits < 2 || bits > 8) return QSYNC_ERR_UNSUPPORTED;
    // the library's own scratch holds the column-sum partials of at most kStaticMaxCols columns
    if(colsum_opt && cols > kStaticMaxCols) return QSYNC_ERR_WORKSPACE;
    if(rows == 0 || cols == 0) return QSYNC_OK;
    if(absmax_workspace_bytes(rows, colsum_opt ? cols : 0, kPerTensor) > kStaticScratchBytes) return QSYNC_ERR_WORKSPACE;
    void*      ws = nullptr;
    hipError_t e  = static_scratch(&ws);
    if(e != hipSuccess) return hip_status(e);
    hipStream_t st = static_cast<hipStream_t>(stream);
    // the arrival counter must start at zero whatever an earlier call left behind (cleared by a kernel, not by a
    // memset node, so that the call can be captured into a graph)
    e = launch_zero_f32(static_cast<float*>(ws), 64, st);
    if(e != hipSuccess) return hip_status(e);
    const float qmax = static_cast<float>((1 << (bits - 1)) - 1);
    return hip_status(launch_absmax_scale(x, xdt, rows, cols, ld, kPerTensor, qmax, scale, inv_scale, amax_opt, colsum_opt,
                                          sumsq_opt, ws, st));
}

int qsync_quantize(const void* x, int xdt, int64_t rows, int64_t cols, int64_t ld, int tag, int bits, int gran,
                   int rnd, uint64_t philox_seed, uint64_t philox_offset, const float* inv_scale, void* q_opt,
                   void* qT_opt, void* stream)
{
    if(!x || (!q_opt && !qT_opt)) return QSYNC_ERR_NULL;
    if(!is_tag(tag) || !is_float_dtype(xdt)) return QSYNC_ERR_BAD_ENUM;
    if(tag == QSYNC_INT8)
    {
        if(!inv_scale) return QSYNC_ERR_NULL;
        if(!is_gran(gran) || !is_round(rnd)) return QSYNC_ERR_BAD_ENUM;
    }
    if(!count_ok(rows, cols) || ld < cols || !count_ok(rows, ld)) return QSYNC_ERR_BAD_SHAPE;
    if(tag == QSYNC_INT8 && (bits < 2 || bits > 8)) return QSYNC_ERR_UNSUPPORTED;
    const bool fp_sr = tag == QSYNC_FP16 && rnd == QSYNC_ROUND_STOCHASTIC && xdt == QSYNC_F32;
    if(fp_sr && bits != 0 && (bits < 7 || bits > 10)) return QSYNC_ERR_UNSUPPORTED;
    if(rows == 0 || cols == 0) return QSYNC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if(fp_sr)
        return hip_status(launch_convert_sr(static_cast<const float*>(x), rows, cols, ld, bits == 0 ? 9 : bits,
                                            philox_seed, philox_offset, q_opt, qT_opt, st));
    if(tag == QSYNC_INT8)
    {
        const int qmax = (1 << (bits - 1)) - 1;
        return hip_status(launch_quantize_int8(x, xdt, rows, cols, ld, qmax, gran, rnd, philox_seed, philox_offset,
                                               inv_scale, static_cast<int8_t*>(q_opt), static_cast<int8_t*>(qT_opt),
                                               st));
    }
    return hip_status(launch_convert(x, xdt, rows, cols, ld, tag == QSYNC_FP16 ? kF16 : kF32, q_opt, qT_opt, st));
}

size_t qsync_absmax_quantize_workspace_bytes(int64_t rows, int64_t cols)
{
    return qsync_absmax_workspace_bytes(rows, cols, QSYNC_PER_TENSOR);
}

int qsync_absmax_quantize(const void* x, int xdt, int64_t rows, int64_t cols, int bits, int rnd, uint64_t philox_seed,
                          uint64_t philox_offset, float* scale, float* inv_scale, float* amax_opt, void* q_opt,
                          void* qT_opt, void* workspace, size_t workspace_bytes, int poll_limit, void* stream)
{
    if(!x || !scale || !inv_scale || (!q_opt && !qT_opt)) return QSYNC_ERR_NULL;
    if(!is_float_dtype(xdt) || !is_round(rnd)) return QSYNC_ERR_BAD_ENUM;
    if(!count_ok(rows, cols)) return QSYNC_ERR_BAD_SHAPE;
    if(bits < 2 || bits > 8) return QSYNC_ERR_UNSUPPORTED;
    if(rows == 0 || cols == 0) return QSYNC_OK;
    const size_t need = qsync_absmax_quantize_workspace_bytes(rows, cols);
    if(!workspace || workspace_bytes < need) return QSYNC_ERR_WORKSPACE;
    if(!aligned16(workspace)) return QSYNC_ERR_ALIGN;
    const int qmax = (1 << (bits - 1)) - 1;
    (void)poll_limit;       // nothing waits any more
    return hip_status(launch_absmax_quantize(x, xdt, rows, cols, qmax, rnd, philox_seed, philox_offset, scale, inv_scale,
                                             amax_opt, static_cast<int8_t*>(q_opt), static_cast<int8_t*>(qT_opt),
                                             workspace, static_cast<hipStream_t>(stream)));
}

int qsync_gradient_quantize(const void* dy, int dydt, int64_t rows, int64_t cols, int bits, int rnd, uint64_t philox_seed,
                            uint64_t philox_offset, float* scale, float* inv_scale, float* amax_opt, float* colsum, void* q_opt,
                            void* qT_opt, void* workspace, size_t workspace_bytes, void* stream)
{
    if(!dy || !scale || !inv_scale || !colsum || (!q_opt && !qT_opt)) return QSYNC_ERR_NULL;
    if(!is_float_dtype(dydt) || !is_round(rnd)) return QSYNC_ERR_BAD_ENUM;
    if(!count_ok(rows, cols)) return QSYNC_ERR_BAD_SHAPE;
    if(bits < 2 || bits > 8 || cols > (int64_t(1) << 19)) return QSYNC_ERR_UNSUPPORTED;
    if(rows == 0 || cols == 0) return QSYNC_OK;
    if(!workspace || workspace_bytes < qsync_absmax_workspace_bytes(rows, cols, QSYNC_PER_TENSOR)) return QSYNC_ERR_WORKSPACE;
    if(!aligned16(workspace)) return QSYNC_ERR_ALIGN;
    return hip_status(launch_gradient_quantize(dy, dydt, rows, cols, (1 << (bits - 1)) - 1, rnd, philox_seed, philox_offset, scale,
                                               inv_scale, amax_opt, colsum, static_cast<int8_t*>(q_opt), static_cast<int8_t*>(qT_opt),
                                               workspace, static_cast<hipStream_t>(stream)));
}

// fp32 products split their contraction only where the workspace has room for the parts: many of them once asked for none, and a
// caller that brings that still gets the result.
static bool splits_optional(int tag) { return tag == QSYNC_FP32; }
static void unsplit(GemmPlan& plan) { plan.splits = 1; plan.workspace = 0; }

size_t qsync_qlinear_workspace_bytes(int tag, int64_t M, int64_t N, int64_t K)
{
    if(!is_tag(tag) || M < 0 || N < 0 || K < 0) return 0;
    return round256(plan_gemm(tag, M, N, K).workspace);
}

size_t qsync_qlinear_bwd_workspace_bytes(int tag, int64_t M, int64_t N, int64_t K)
{
    if(!is_tag(tag) || M < 0 || N < 0 || K < 0) return 0;
    return round256(plan_gemm(tag, M, K, N).workspace) + round256(plan_gemm(tag, N, K, M).workspace)
         + round256(colsum_workspace_bytes(M, N));
}

static int qlinear_fwd_impl(int tag, int64_t M, int64_t N, int64_t K, const void* xq, const float* sx, const void* wq,
                            const float* sw, int wgran, const float* bias_opt, void* y, int ydt, int32_t* acc_dump_opt,
                            float* y_amax_opt, void* workspace, size_t workspace_bytes, void* stream,
                            void* yq_opt = nullptr, const float* yq_inv = nullptr, int yq_qmax = 127)
{
    if(!xq || !wq || !y) return QSYNC_ERR_NULL;
    if(!is_tag(tag) || !is_float_dtype(ydt)) return QSYNC_ERR_BAD_ENUM;
    if(tag == QSYNC_INT8)
    {
        if(!sx || !sw) return QSYNC_ERR_NULL;
        if(!is_gran(wgran)) return QSYNC_ERR_BAD_ENUM;
    }
    if(!count_ok(M, N) || !count_ok(M, K) || !count_ok(N, K)) return QSYNC_ERR_BAD_SHAPE;
    if(!gemm_row_ok(tag, K)) return QSYNC_ERR_UNSUPPORTED;
    if(tag == QSYNC_INT8 && wgran == QSYNC_PER_COL) return QSYNC_ERR_UNSUPPORTED;
    if(tag != QSYNC_INT8 && acc_dump_opt) return QSYNC_ERR_UNSUPPORTED;
    if(tag != QSYNC_FP32)
    {
        if(K % (tag == QSYNC_INT8 ? 16 : 8) != 0) return QSYNC_ERR_ALIGN;
        if(!aligned16(xq) || !aligned16(wq)) return QSYNC_ERR_ALIGN;
    }
    if(M == 0 || N == 0) return QSYNC_OK;
    GemmPlan plan = plan_gemm(tag, M, N, K);
    if(splits_optional(tag) && !(workspace && aligned16(workspace) && workspace_bytes >= plan.workspace)) unsplit(plan);
    if(plan.workspace > 0)
    {
        if(!workspace || workspace_bytes < plan.workspace) return QSYNC_ERR_WORKSPACE;
        if(!aligned16(workspace)) return QSYNC_ERR_ALIGN;
    }
    GemmProblem p{};
    p.prec = tag; p.M = M; p.N = N; p.K = K;
    p.A = xq; p.B = wq; p.C = y; p.c_dtype = ydt;
    if(tag == QSYNC_INT8)
    {
        p.s0 = sx;
        if(wgran == QSYNC_PER_TENSOR) p.s1 = sw; else p.col_scale = sw;
        p.acc_dump = acc_dump_opt;
    }
    p.col_bias = bias_opt;
    p.out_amax_bits = reinterpret_cast<unsigned int*>(y_amax_opt);
    p.out_codes = yq_opt; p.out_code_inv = yq_inv; p.out_code_qmax = yq_qmax;
    return hip_status(launch_gemm(p, plan, workspace, static_cast<hipStream_t>(stream)));
}

int qsync_qlinear_fwd(int tag, int64_t M, int64_t N, int64_t K, const void* xq, const float* sx, const void* wq,
                      const float* sw, int wgran, const float* bias_opt, void* y, int ydt, int32_t* acc_dump_opt,
                      void* workspace, size_t workspace_bytes, void* stream)
{
    return qlinear_fwd_impl(tag, M, N, K, xq, sx, wq, sw, wgran, bias_opt, y, ydt, acc_dump_opt, nullptr, workspace,
                            workspace_bytes, stream);
}

int qsync_qlinear_fwd_amax(int tag, int64_t M, int64_t N, int64_t K, const void* xq, const float* sx, const void* wq,
                           const float* sw, int wgran, const float* bias_opt, void* y, int ydt, int32_t* acc_dump_opt,
                           float* y_amax, void* workspace, size_t workspace_bytes, void* stream)
{
    if(!y_amax) return QSYNC_ERR_NULL;
    if((reinterpret_cast<uintptr_t>(y_amax) & 3u) != 0) return QSYNC_ERR_ALIGN;
    return qlinear_fwd_impl(tag, M, N, K, xq, sx, wq, sw, wgran, bias_opt, y, ydt, acc_dump_opt, y_amax, workspace,
                            workspace_bytes, stream);
}

int qsync_qlinear_fwd_codes(int tag, int64_t M, int64_t N, int64_t K, const void* xq, const float* sx, const void* wq,
                            const float* sw, int wgran, const float* bias_opt, void* y, int ydt, int bits,
                            const float* next_inv_scale, void* yq, float* y_amax_opt, void* workspace,
                            size_t workspace_bytes, void* stream)
{
    if(!yq || !next_inv_scale) return QSYNC_ERR_NULL;
    if(bits < 2 || bits > 8) return QSYNC_ERR_UNSUPPORTED;
    if(y_amax_opt && (reinterpret_cast<uintptr_t>(y_amax_opt) & 3u) != 0) return QSYNC_ERR_ALIGN;
    // fp32 operands whose rows are not 16-byte multiples are refused, as the header says
    if(tag == QSYNC_FP32 && ((K * 4) % 16 != 0 || !aligned16(xq) || !aligned16(wq))) return QSYNC_ERR_UNSUPPORTED;
    return qlinear_fwd_impl(tag, M, N, K, xq, sx, wq, sw, wgran, bias_opt, y, ydt, nullptr, y_amax_opt, workspace,
                            workspace_bytes, stream, yq, next_inv_scale, (1 << (bits - 1)) - 1);
}

int qsync_transpose_i8(const void* in, int64_t rows, int64_t cols, void* out, void* stream)
{
    if(!in || !out) return QSYNC_ERR_NULL;
    if(!count_ok(rows, cols)) return QSYNC_ERR_BAD_SHAPE;
    if(in == out) return QSYNC_ERR_UNSUPPORTED;
    return hip_status(launch_transpose_i8(static_cast<const int8_t*>(in), rows, cols, static_cast<int8_t*>(out),
                                          static_cast<hipStream_t>(stream)));
}

int qsync_scale_from_amax(float* amax, int bits, float* scale, float* inv_scale, int consume, void* stream)
{
    if(!amax || !scale || !inv_scale) return QSYNC_ERR_NULL;
    if(bits < 2 || bits > 8) return QSYNC_ERR_UNSUPPORTED;
    const float qmax = static_cast<float>((1 << (bits - 1)) - 1);
    return hip_status(launch_scale_from_amax(amax, qmax, scale, inv_scale, consume != 0, static_cast<hipStream_t>(stream)));
}

// sums: partial column sums that lie in the workspace already (their number), or 0
static int qlinear_bwd_impl(int tag, int64_t M, int64_t N, int64_t K, const void* dyq, const void* dyqT, const float* sdy,
                            const void* xqT, const float* sx, const void* wqbT, const float* swb, int wbgran, void* dx_opt,
                            int dxdt, void* dw_opt, int dwdt, float* db_opt, const void* dy_float_opt, int dydt,
                            int32_t* acc_dx_dump_opt, int32_t* acc_dw_dump_opt, void* workspace, size_t workspace_bytes,
                            void* stream, int sums)
{
    if(dx_opt && (!dyq || !wqbT)) return QSYNC_ERR_NULL;
    if(dw_opt && (!dyqT || !xqT)) return QSYNC_ERR_NULL;
    if(db_opt && !dy_float_opt) return QSYNC_ERR_NULL;
    if(!is_tag(tag)) return QSYNC_ERR_BAD_ENUM;
    if(dx_opt && !is_float_dtype(dxdt)) return QSYNC_ERR_BAD_ENUM;
    if(dw_opt && !is_float_dtype(dwdt)) return QSYNC_ERR_BAD_ENUM;
    if(db_opt && !is_float_dtype(dydt)) return QSYNC_ERR_BAD_ENUM;
    if(tag == QSYNC_INT8)
    {
        if((dx_opt || dw_opt) && !sdy) return QSYNC_ERR_NULL;
        if(dx_opt && !swb) return QSYNC_ERR_NULL;
        if(dw_opt && !sx) return QSYNC_ERR_NULL;
        if(dx_opt && !is_gran(wbgran)) return QSYNC_ERR_BAD_ENUM;
    }
    if(!count_ok(M, N) || !count_ok(M, K) || !count_ok(N, K)) return QSYNC_ERR_BAD_SHAPE;
    if((dx_opt && !gemm_row_ok(tag, N)) || (dw_opt && !gemm_row_ok(tag, M))) return QSYNC_ERR_UNSUPPORTED;
    if(tag == QSYNC_INT8 && dx_opt && wbgran == QSYNC_PER_COL) return QSYNC_ERR_UNSUPPORTED;
    if(tag != QSYNC_INT8 && (acc_dx_dump_opt || acc_dw_dump_opt)) return QSYNC_ERR_UNSUPPORTED;
    if(tag != QSYNC_FP32)
    {
        const int64_t mult = tag == QSYNC_INT8 ? 16 : 8;
        if(dx_opt && (N % mult != 0 || !aligned16(dyq) || !aligned16(wqbT))) return QSYNC_ERR_ALIGN;
        if(dw_opt && (M % mult != 0 || !aligned16(dyqT) || !aligned16(xqT))) return QSYNC_ERR_ALIGN;
    }
    GemmPlan plan_dx = plan_gemm(tag, M, K, N);
    GemmPlan plan_dw = plan_gemm(tag, N, K, M);
    const bool full = workspace && aligned16(workspace) && workspace_bytes >= qsync_qlinear_bwd_workspace_bytes(tag, M, N, K);
    if(!full && splits_optional(tag))
    {
        unsplit(plan_dx);
        unsplit(plan_dw);
    }
    const size_t   off_dw  = round256(plan_dx.workspace);
    const size_t   off_db  = off_dw + round256(plan_dw.workspace);
    const size_t   need    = (dx_opt ? plan_dx.workspace : 0) + (dw_opt ? plan_dw.workspace : 0)
                        + ((db_opt && M > 0 && N > 0) ? colsum_workspace_bytes(M, N) : 0);
    if(need > 0)
    {
        if(!workspace || workspace_bytes < off_db + round256(colsum_workspace_bytes(M, N))) return QSYNC_ERR_WORKSPACE;
        if(!aligned16(workspace)) return QSYNC_ERR_ALIGN;
    }
    hipStream_t st  = static_cast<hipStream_t>(stream);
    char*       wsb = static_cast<char*>(workspace);
    GemmProblem pdx = data_gradient(tag, M, N, K, dyq, sdy, wqbT, swb, wbgran, dx_opt, dxdt, acc_dx_dump_opt), pdw{};
    pdw.prec = tag; pdw.M = N; pdw.N = K; pdw.K = M;
    pdw.A = dyqT; pdw.B = xqT; pdw.C = dw_opt; pdw.c_dtype = dwdt;
    if(tag == QSYNC_INT8)
    {
        pdw.s0 = sdy; pdw.s1 = sx;
        pdw.acc_dump = acc_dw_dump_opt;
    }
    const bool want_dx = dx_opt && M > 0 && K > 0, want_dw = dw_opt && N > 0 && K > 0;
    ColumnFoldArgs fold;
    if(db_opt && N > 0 && M > 0)
    {
        float* part = reinterpret_cast<float*>(wsb + off_db);
        if(sums > 0) fold = ColumnFoldArgs{part, sums, N, db_opt};
        else
        {
            const int rc = hip_status(launch_colsum_partials(dy_float_opt, dydt, M, N, db_opt, part, &fold, st));
            if(rc != QSYNC_OK) return rc;
        }
    }
    const int rc = run_gradients(want_dx ? &pdx : nullptr, plan_dx, wsb, want_dw ? &pdw : nullptr, plan_dw, wsb ? wsb + off_dw : nullptr, fold, st);
    // no rows to sum: the bias gradient is zero (the column-sum kernels need their workspace, which an empty batch does not
    // have to bring)
    if(rc == QSYNC_OK && db_opt && N > 0 && M == 0) return hip_status(launch_zero_f32(db_opt, N, st));
    return rc;
}

int qsync_qlinear_bwd(int tag, int64_t M, int64_t N, int64_t K, const void* dyq, const void* dyqT, const float* sdy,
                      const void* xqT, const float* sx, const void* wqbT, const float* swb, int wbgran, void* dx_opt,
                      int dxdt, void* dw_opt, int dwdt, float* db_opt, const void* dy_float_opt, int dydt,
                      int32_t* acc_dx_dump_opt, int32_t* acc_dw_dump_opt, void* workspace, size_t workspace_bytes,
                      void* stream)
{
    return qlinear_bwd_impl(tag, M, N, K, dyq, dyqT, sdy, xqT, sx, wqbT, swb, wbgran, dx_opt, dxdt, dw_opt, dwdt, db_opt, dy_float_opt,
                            dydt, acc_dx_dump_opt, acc_dw_dump_opt, workspace, workspace_bytes, stream, 0);
}

// Row-major backward: data gradient's and weight gradient's partial products, then the column sums, behind both so that they can be
// folded last.  A workspace without room for the column sums there keeps them behind the transposed form's parts, folded first.
static size_t rm_products_bytes(int tag, int64_t M, int64_t N, int64_t K)
{
    return round256(plan_gemm(tag, M, K, N).workspace) + round256(plan_gemm(tag, N, K, M, -1, -1, true, /*tn=*/M > 0).workspace);
}
static size_t rm_sums_offset(int tag, int64_t M, int64_t N, int64_t K)
{
    const size_t nt = round256(plan_gemm(tag, M, K, N).workspace) + round256(plan_gemm(tag, N, K, M).workspace);
    const size_t rm = rm_products_bytes(tag, M, N, K);
    return nt > rm ? nt : rm;
}

size_t qsync_qlinear_bwd_rm_workspace_bytes(int tag, int64_t M, int64_t N, int64_t K)
{
    if((tag != QSYNC_INT8 && tag != QSYNC_FP16) || M < 0 || N < 0 || K < 0) return 0;
    // the data gradient (and bias gradient) go through qsync_qlinear_bwd, which asks for its own full size
    const size_t nt = qsync_qlinear_bwd_workspace_bytes(tag, M, N, K);
    const size_t rm = rm_sums_offset(tag, M, N, K) + round256(colsum_workspace_bytes(M, N));
    return nt > rm ? nt : rm;
}

static int qlinear_bwd_rm_impl(int tag, int64_t M, int64_t N, int64_t K, const void* dyq, const float* sdy, const void* xq, const float* sx,
                               const void* wqbT, const float* swb, int wbgran, void* dx_opt, int dxdt, void* dw_opt, int dwdt,
                               float* db_opt, const void* dy_float_opt, int dydt, int32_t* acc_dx_dump_opt,
                               int32_t* acc_dw_dump_opt, void* workspace, size_t workspace_bytes, void* stream, int sums)
{
    if(!is_tag(tag)) return QSYNC_ERR_BAD_ENUM;
    if(tag != QSYNC_INT8 && tag != QSYNC_FP16) return QSYNC_ERR_UNSUPPORTED;
    const bool i8 = tag == QSYNC_INT8;
    if((dx_opt || dw_opt) && (!dyq || (i8 && !sdy))) return QSYNC_ERR_NULL;
    if(dx_opt && (!wqbT || (i8 && !swb))) return QSYNC_ERR_NULL;
    if(dw_opt && (!xq || (i8 && !sx))) return QSYNC_ERR_NULL;
    if(db_opt && !dy_float_opt) return QSYNC_ERR_NULL;
    if(!i8 && (acc_dx_dump_opt || acc_dw_dump_opt)) return QSYNC_ERR_UNSUPPORTED;
    if(dx_opt && (!is_float_dtype(dxdt) || !is_gran(wbgran))) return QSYNC_ERR_BAD_ENUM;
    if(dw_opt && !is_float_dtype(dwdt)) return QSYNC_ERR_BAD_ENUM;
    if(db_opt && !is_float_dtype(dydt)) return QSYNC_ERR_BAD_ENUM;
    if(!count_ok(M, N) || !count_ok(M, K) || !count_ok(N, K)) return QSYNC_ERR_BAD_SHAPE;
    if(dx_opt && wbgran == QSYNC_PER_COL) return QSYNC_ERR_UNSUPPORTED;
    if((dx_opt && !gemm_row_ok(tag, N)) || (dw_opt && (N >= (int64_t(1) << 24) || K >= (int64_t(1) << 24))))
        return QSYNC_ERR_UNSUPPORTED;
    const int64_t mult = i8 ? 16 : 8;                           // elements per 16-byte chunk
    if(dx_opt && (N % mult != 0 || !aligned16(dyq) || !aligned16(wqbT))) return QSYNC_ERR_ALIGN;
    // the weight gradient reads both operands row-major: whole K tiles of contraction rows, 16-byte column chunks
    if(dw_opt && (M % 128 != 0 || N % mult != 0 || K % mult != 0 || !aligned16(dyq) || !aligned16(xq))) return QSYNC_ERR_ALIGN;
    const GemmPlan plan   = plan_gemm(tag, N, K, M, -1, -1, true, /*tn=*/M > 0), plan_dx = plan_gemm(tag, M, K, N);
    const size_t   off_dw = round256(plan_dx.workspace);
    const bool     want_dw = dw_opt && N > 0 && K > 0;
    GemmProblem p{};
    p.prec = tag; p.M = N; p.N = K; p.K = M;
    p.A = dyq; p.B = xq; p.C = dw_opt; p.c_dtype = dwdt;
    p.s0 = i8 ? sdy : nullptr; p.s1 = i8 ? sx : nullptr; p.acc_dump = acc_dw_dump_opt;
    p.tn = M > 0;      // (empty contraction: the NT form writes the zeros, no operand is read)
    const GemmProblem pdx  = data_gradient(tag, M, N, K, dyq, sdy, wqbT, swb, wbgran, dx_opt, dxdt, acc_dx_dump_opt);
    const bool want_dx = dx_opt && M > 0 && K > 0, want_db = db_opt && M > 0 && N > 0;
    const size_t nt = qsync_qlinear_bwd_workspace_bytes(tag, M, N, K), products = rm_products_bytes(tag, M, N, K);
    const bool   need_nt = (dx_opt && plan_dx.workspace > 0) || want_db, need_rm = want_dw && plan.workspace > 0;
    if((need_nt && (!workspace || workspace_bytes < nt)) || (need_rm && (!workspace || workspace_bytes < (nt > products ? nt : products))))
        return QSYNC_ERR_WORKSPACE;
    if((need_nt || need_rm) && !aligned16(workspace)) return QSYNC_ERR_ALIGN;
    hipStream_t st  = static_cast<hipStream_t>(stream);
    char*       wsb = static_cast<char*>(workspace);
    int         rc  = QSYNC_OK;
    ColumnFoldArgs fold;
    if(want_db)
    {
        const bool   last = workspace_bytes >= rm_sums_offset(tag, M, N, K) + colsum_workspace_bytes(M, N);
        float* const part = reinterpret_cast<float*>(wsb + (last ? rm_sums_offset(tag, M, N, K)
                                                                 : round256(plan_dx.workspace) + round256(plan_gemm(tag, N, K, M).workspace)));
        if(sums > 0) fold = ColumnFoldArgs{part, sums, N, db_opt};
        else rc = hip_status(launch_colsum_partials(dy_float_opt, dydt, M, N, db_opt, part, &fold, st));
        if(rc == QSYNC_OK && !last)
        {
            rc   = hip_status(launch_column_fold(fold, st));
            fold = ColumnFoldArgs{};
        }
        if(rc != QSYNC_OK) return rc;
    }
    rc = run_gradients(want_dx ? &pdx : nullptr, plan_dx, wsb, want_dw ? &p : nullptr, plan, wsb ? wsb + off_dw : nullptr, fold, st);
    if(rc == QSYNC_OK && db_opt && N > 0 && M == 0) return hip_status(launch_zero_f32(db_opt, N, st));
    return rc;
}

int qsync_qlinear_bwd_rm(int tag, int64_t M, int64_t N, int64_t K, const void* dyq, const float* sdy, const void* xq, const float* sx,
                         const void* wqbT, const float* swb, int wbgran, void* dx_opt, int dxdt, void* dw_opt, int dwdt,
                         float* db_opt, const void* dy_float_opt, int dydt, int32_t* acc_dx_dump_opt,
                         int32_t* acc_dw_dump_opt, void* workspace, size_t workspace_bytes, void* stream)
{
    return qlinear_bwd_rm_impl(tag, M, N, K, dyq, sdy, xq, sx, wqbT, swb, wbgran, dx_opt, dxdt, dw_opt, dwdt, db_opt, dy_float_opt, dydt,
                               acc_dx_dump_opt, acc_dw_dump_opt, workspace, workspace_bytes, stream, 0);
}

int qsync_qlinear_backward(int tag, int64_t M, int64_t N, int64_t K, const void* dy, int dydt, void* dyq_opt, void* dyqT_opt, const void* x,
                           int x_rowmajor, const void* wqbT, void* dx_opt, int dxdt, void* dw_opt, int dwdt, float* db_opt,
                           void* workspace, size_t workspace_bytes, void* stream)
{
    if(!is_tag(tag) || !is_float_dtype(dydt) || (x_rowmajor != 0 && x_rowmajor != 1)) return QSYNC_ERR_BAD_ENUM;
    if(tag == QSYNC_INT8) return QSYNC_ERR_UNSUPPORTED;
    if(!dy) return QSYNC_ERR_NULL;
    const void* dyq = dyq_opt ? dyq_opt : dy;
    if(!dyq_opt && (dydt == QSYNC_F16) != (tag == QSYNC_FP16)) return QSYNC_ERR_UNSUPPORTED;      // used as it is: of the operand type
    int sums = 0;
    if(dyq_opt || dyqT_opt)
    {
        const bool   shape = count_ok(M, N) && count_ok(M, K) && count_ok(N, K) && M > 0 && N > 0 && K > 0;
        const size_t need  = !shape ? 0 : x_rowmajor ? qsync_qlinear_bwd_rm_workspace_bytes(tag, M, N, K) : qsync_qlinear_bwd_workspace_bytes(tag, M, N, K);
        bool         taken = false;
        if(shape && db_opt && dydt == QSYNC_F32 && workspace && workspace_bytes >= need && aligned16(workspace)
           && (!x_rowmajor || tag == QSYNC_FP16))
        {   // the cast reads dY once for both
            const size_t off = x_rowmajor ? rm_sums_offset(tag, M, N, K)
                                          : round256(plan_gemm(tag, M, K, N).workspace) + round256(plan_gemm(tag, N, K, M).workspace);
            ColumnFoldArgs fold;
            const int rc = hip_status(launch_convert_sums(static_cast<const float*>(dy), M, N, tag == QSYNC_FP16 ? kF16 : kF32, dyq_opt, dyqT_opt,
                                                          db_opt, reinterpret_cast<float*>(static_cast<char*>(workspace) + off), &fold, &taken,
                                                          static_cast<hipStream_t>(stream)));
            if(rc != QSYNC_OK) return rc;
            sums = taken ? fold.S : 0;
        }
        if(!taken)
        {
            const int rc = qsync_quantize(dy, dydt, M, N, N, tag, 0, QSYNC_PER_TENSOR, QSYNC_ROUND_NEAREST, 0, 0, nullptr, dyq_opt, dyqT_opt, stream);
            if(rc != QSYNC_OK) return rc;
        }
    }
    if(x_rowmajor)
        return qlinear_bwd_rm_impl(tag, M, N, K, dyq, nullptr, x, nullptr, wqbT, nullptr, QSYNC_PER_TENSOR, dx_opt, dxdt, dw_opt, dwdt, db_opt,
                                   dy, dydt, nullptr, nullptr, workspace, workspace_bytes, stream, sums);
    return qlinear_bwd_impl(tag, M, N, K, dyq, dyqT_opt, nullptr, x, nullptr, wqbT, nullptr, QSYNC_PER_TENSOR, dx_opt, dxdt, dw_opt, dwdt,
                            db_opt, dy, dydt, nullptr, nullptr, workspace, workspace_bytes, stream, sums);
}

// Workspace of qsync_qlinear_bwd_fp16_of_int8: binary16 operands of the FP16 backward, then the GEMMs' own scratch;
// every part starts on a 256-byte boundary.
namespace {
struct Fp16BwdLayout { size_t off_xhT, off_wh, off_whT, off_dyh, off_dyhT, off_gemm, total; };
Fp16BwdLayout fp16_bwd_layout(int64_t M, int64_t N, int64_t K, int dydt)
{
    Fp16BwdLayout l;
    size_t at = 0;
    auto take = [&](int64_t elems) { const size_t o = at; at += round256(static_cast<size_t>(elems) * 2); return o; };
    l.off_xhT  = take(K * M);
    l.off_wh   = take(N * K);
    l.off_whT  = take(K * N);
    l.off_dyh  = take(dydt == QSYNC_F16 ? 0 : M * N);          // a binary16 gradient is used in place
    l.off_dyhT = take(N * M);
    l.off_gemm = at;
    const size_t nt = qsync_qlinear_bwd_workspace_bytes(QSYNC_FP16, M, N, K), rm = qsync_qlinear_bwd_rm_workspace_bytes(QSYNC_FP16, M, N, K);
    l.total    = at + (nt > rm ? nt : rm);
    return l;
}
}  // namespace

size_t qsync_qlinear_bwd_fp16_of_int8_workspace_bytes(int64_t M, int64_t N, int64_t K, int dydt)
{
    if(M < 0 || N < 0 || K < 0 || !is_float_dtype(dydt) || !count_ok(M, N) || !count_ok(M, K) || !count_ok(N, K)) return 0;
    return fp16_bwd_layout(M, N, K, dydt).total;
}

int qsync_qlinear_bwd_fp16_of_int8(int64_t M, int64_t N, int64_t K, const void* dy, int dydt, const void* xqT,
                                   int x_rowmajor, const float* sx, const void* wq, const float* sw, int wgran, void* dx_opt, int dxdt,
                                   void* dw_opt, int dwdt, float* db_opt, void* workspace, size_t workspace_bytes,
                                   size_t* operand_offsets_opt, void* stream)
{
    if(!dy || !workspace) return !dy ? QSYNC_ERR_NULL : QSYNC_ERR_WORKSPACE;
    if(dx_opt && (!wq || !sw)) return QSYNC_ERR_NULL;
    if(dw_opt && (!xqT || !sx)) return QSYNC_ERR_NULL;
    if(!is_float_dtype(dydt)) return QSYNC_ERR_BAD_ENUM;
    if(dx_opt && (!is_float_dtype(dxdt) || (wgran != QSYNC_PER_TENSOR && wgran != QSYNC_PER_ROW))) return QSYNC_ERR_BAD_ENUM;
    if(dw_opt && !is_float_dtype(dwdt)) return QSYNC_ERR_BAD_ENUM;
    if(!count_ok(M, N) || !count_ok(M, K) || !count_ok(N, K)) return QSYNC_ERR_BAD_SHAPE;
    if(x_rowmajor != 0 && x_rowmajor != 1) return QSYNC_ERR_BAD_ENUM;
    if((dx_opt && N % 8 != 0) || (dw_opt && M % 8 != 0) || !aligned16(dy)) return QSYNC_ERR_ALIGN;
    if(dw_opt && x_rowmajor && (M % 128 != 0 || N % 8 != 0 || K % 8 != 0)) return QSYNC_ERR_ALIGN;
    const Fp16BwdLayout l = fp16_bwd_layout(M, N, K, dydt);
    if(workspace_bytes < l.total) return QSYNC_ERR_WORKSPACE;
    if((reinterpret_cast<uintptr_t>(workspace) & 255) != 0) return QSYNC_ERR_ALIGN;
    if(operand_offsets_opt)
    {   // where the binary16 operands lie in the workspace (host array of 5: xhT, wh, whT, dyh, dyhT)
        const size_t offs[5] = {l.off_xhT, l.off_wh, l.off_whT, l.off_dyh, l.off_dyhT};
        for(int i = 0; i < 5; ++i) operand_offsets_opt[i] = offs[i];
    }
    if(M == 0 || N == 0 || K == 0)
        return qsync_qlinear_bwd(QSYNC_FP16, M, N, K, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                                 QSYNC_PER_TENSOR, nullptr, dxdt, nullptr, dwdt, db_opt, dy, dydt, nullptr, nullptr,
                                 static_cast<char*>(workspace) + l.off_gemm, workspace_bytes - l.off_gemm, stream);
    hipStream_t st   = static_cast<hipStream_t>(stream);
    char*       base = static_cast<char*>(workspace);
    void *xhT = base + l.off_xhT, *wh = base + l.off_wh, *whT = base + l.off_whT, *dyhT = base + l.off_dyhT;
    const void* dyh = dydt == QSYNC_F16 ? dy : base + l.off_dyh;
    hipError_t e = hipSuccess;
    // x_hat = code * q_x narrowed to binary16, [M,K] or [K,M] like the codes; w_hat with the forward's scales (one per output
    // channel, or one) and its transpose for dX: side by side when both are wanted
    const int64_t xr = x_rowmajor ? M : K, xc = x_rowmajor ? K : M;
    const float *w_rows = wgran == QSYNC_PER_ROW ? sw : nullptr, *w_one = wgran == QSYNC_PER_ROW ? nullptr : sw;
    if(dw_opt && dx_opt)
        e = launch_dequantize_f16_both(static_cast<const int8_t*>(xqT), xr, xc, sx, xhT, static_cast<const int8_t*>(wq), N, K, w_rows, w_one, wh, whT, st);
    else if(dw_opt)
        e = launch_dequantize_f16_tiles(static_cast<const int8_t*>(xqT), xr, xc, nullptr, sx, xhT, nullptr, st);
    else if(dx_opt)
        e = launch_dequantize_f16_tiles(static_cast<const int8_t*>(wq), N, K, w_rows, w_one, wh, whT, st);
    if(e != hipSuccess) return hip_status(e);
    // dY narrowed to binary16 (or used in place) and transposed, then the FP16 gradients
    void* const dyh_out  = dydt == QSYNC_F16 ? nullptr : const_cast<void*>(dyh);
    void* const dyhT_out = (dw_opt && !x_rowmajor) ? dyhT : nullptr;
    return qsync_qlinear_backward(QSYNC_FP16, M, N, K, dy, dydt, dyh_out, dyhT_out, xhT, x_rowmajor, whT, dx_opt, dxdt, dw_opt, dwdt, db_opt,
                                  base + l.off_gemm, workspace_bytes - l.off_gemm, stream);
}

int qsync_prepare_weights(const void* w, int wdt, int64_t N, int64_t K, int bits, float* sw, float* iw, float* aw_opt,
                          void* wq, float* swb, float* iwb, void* wqbT, void* workspace, size_t workspace_bytes,
                          void* stream)
{
    if(!w || !sw || !iw || !wq || !swb || !iwb || !wqbT) return QSYNC_ERR_NULL;
    if(!is_float_dtype(wdt)) return QSYNC_ERR_BAD_ENUM;
    if(!count_ok(N, K)) return QSYNC_ERR_BAD_SHAPE;
    if(bits < 2 || bits > 8) return QSYNC_ERR_UNSUPPORTED;
    if(N == 0 || K == 0) return QSYNC_OK;
    if(!workspace || workspace_bytes < absmax_workspace_bytes(N, K, kPerCol)) return QSYNC_ERR_WORKSPACE;
    if(!aligned16(workspace)) return QSYNC_ERR_ALIGN;
    const float qmax = static_cast<float>((1 << (bits - 1)) - 1);
    return hip_status(launch_prepare_weights(w, wdt == QSYNC_F32 ? kF32 : kF16, N, K, qmax, sw, iw, aw_opt,
                                             static_cast<int8_t*>(wq), swb, iwb, static_cast<int8_t*>(wqbT), workspace,
                                             static_cast<hipStream_t>(stream)));
}

// Workspace of qsync_conv3x3_wgrad over padded copies: [margin][three displaced copies of the activation, C x Mp each]
// [margin][gradient operand, N x Mp][split-K partials]; every part starts on a 256-byte boundary.
namespace {
struct WgradLayout { ConvPaddedAxis ax; size_t margin, off_x, off_dy, off_part, total; GemmPlan plan; };
WgradLayout wgrad_layout(int tag, int64_t nimg, int64_t H, int64_t W, int64_t C, int64_t N)
{
    const size_t esz = tag == QSYNC_INT8 ? 1 : 2;
    WgradLayout  l;
    l.ax       = conv_padded_axis(nimg, static_cast<int>(H), static_cast<int>(W));
    l.margin   = round256(static_cast<size_t>(l.ax.Wp) * esz);
    l.off_x    = l.margin;
    l.off_dy   = l.off_x + round256(static_cast<size_t>(3 * C * l.ax.Mp) * esz) + l.margin;
    l.off_part = l.off_dy + round256(static_cast<size_t>(N * l.ax.Mp) * esz);
    l.plan     = plan_gemm(tag, N, 9 * C, l.ax.Mp);
    l.total    = l.off_part + l.plan.workspace;
    return l;
}
// The gathering form: the weight-gradient GEMM reads the row-major gradient and the NHWC activation themselves (TN
// form, patches formed by its loads).  It needs rows of at most 2^24 elements for its 32-bit lane offsets, so gradients
// with more output channels take the padded copies.  Its other bounds (9 C below 2^24, an activation below 2^31 bytes,
// H and W below 2^16) follow from wgrad_shape_ok, whose three padded copies stay below 2^32 bytes.
bool wgrad_gathers(int64_t N) { return N < (int64_t(1) << 24); }
bool wgrad_shape_ok(int tag, int64_t nimg, int64_t H, int64_t W, int64_t C, int64_t N)
{
    const int64_t esz = tag == QSYNC_INT8 ? 1 : 2;
    if(nimg < 0 || H < 0 || W < 0 || C < 0 || N < 0 || H > 65535 || (W + 16) * esz > 1024 || C > (1 << 20)
       || N > (int64_t(1) << 31))
        return false;
    if(H > 0 && W > 0 && nimg > ((int64_t(1) << 31) - 1) / ((H + 1) * (W + 16))) return false;
    const ConvPaddedAxis ax = conv_padded_axis(nimg, static_cast<int>(H), static_cast<int>(W));
    return 3 * C * ax.Mp * esz < (int64_t(1) << 32) - (1 << 20) && count_ok(N, ax.Mp) && count_ok(N, 9 * C);
}
}  // namespace

size_t qsync_conv3x3_wgrad_workspace_bytes(int tag, int64_t nimg, int64_t H, int64_t W, int64_t C, int64_t N)
{
    if((tag != QSYNC_INT8 && tag != QSYNC_FP16) || nimg <= 0 || H <= 0 || W <= 0 || C <= 0 || N <= 0
       || !wgrad_shape_ok(tag, nimg, H, W, C, N))
        return 0;
    if(!wgrad_gathers(N)) return wgrad_layout(tag, nimg, H, W, C, N).total;
    // split-K partials only (the largest over the tile shapes, so that a pinned tile fits too)
    size_t need = plan_gemm(tag, N, 9 * C, nimg * H * W, -1, -1, true, true).workspace;
    for(int t = 0; t < 3; ++t)
    {
        const size_t w = plan_gemm(tag, N, 9 * C, nimg * H * W, t, 0, true, true).workspace;
        need = w > need ? w : need;
    }
    return round256(need);
}

int qsync_conv3x3_wgrad(int tag, int64_t nimg, int64_t H, int64_t W, int64_t C, int64_t N, const void* xq, const float* sx,
                        const void* dyq, const float* sdy, void* dw, int dwdt, int32_t* acc_dump_opt, void* workspace,
                        size_t workspace_bytes, void* stream)
{
    if(!xq || !dyq || !dw) return QSYNC_ERR_NULL;
    if(!is_tag(tag) || !is_float_dtype(dwdt)) return QSYNC_ERR_BAD_ENUM;
    if(tag == QSYNC_FP32) return QSYNC_ERR_UNSUPPORTED;
    if(tag == QSYNC_INT8 && (!sx || !sdy)) return QSYNC_ERR_NULL;
    if(tag != QSYNC_INT8 && acc_dump_opt) return QSYNC_ERR_UNSUPPORTED;
    if(!wgrad_shape_ok(tag, nimg, H, W, C, N)) return QSYNC_ERR_BAD_SHAPE;
    if(nimg == 0 || H == 0 || W == 0 || C == 0 || N == 0) return QSYNC_OK;
    const int esz = tag == QSYNC_INT8 ? 1 : 2;
    if((C * esz) % 16 != 0 || (N * esz) % 16 != 0 || !aligned16(xq) || !aligned16(dyq)) return QSYNC_ERR_ALIGN;
    hipStream_t st  = static_cast<hipStream_t>(stream);
    last_wgrad_ring() = 0;
    if(wgrad_gathers(N))
    {
        const int64_t  M    = nimg * H * W;
        const GemmPlan plan = plan_gemm(tag, N, 9 * C, M, -1, -1, true, /*tn=*/true);
        if(plan.workspace > 0)
        {
            if(!workspace || workspace_bytes < plan.workspace) return QSYNC_ERR_WORKSPACE;
            if((reinterpret_cast<uintptr_t>(workspace) & 255) != 0) return QSYNC_ERR_ALIGN;
        }
        GemmProblem p{};
        p.prec = tag; p.M = N; p.N = 9 * C; p.K = M;
        p.A = dyq; p.B = xq; p.C = dw; p.c_dtype = dwdt; p.tn = true;
        p.conv_H = static_cast<int>(H); p.conv_W = static_cast<int>(W); p.conv_C = C;
        if(tag == QSYNC_INT8) { p.s0 = sdy; p.s1 = sx; p.acc_dump = acc_dump_opt; }
        return hip_status(launch_gemm(p, plan, workspace, st));
    }
    const WgradLayout l = wgrad_layout(tag, nimg, H, W, C, N);
    if(!workspace || workspace_bytes < l.total) return QSYNC_ERR_WORKSPACE;
    if((reinterpret_cast<uintptr_t>(workspace) & 255) != 0) return QSYNC_ERR_ALIGN;
    uint8_t*    xT  = static_cast<uint8_t*>(workspace) + l.off_x;
    uint8_t*    dyT = static_cast<uint8_t*>(workspace) + l.off_dy;
    hipError_t  e   = launch_conv_padded_transpose(xq, esz, nimg, static_cast<int>(H), static_cast<int>(W), static_cast<int>(C), 3, xT, static_cast<int>(l.margin), st);
    if(e != hipSuccess) return hip_status(e);
    e = launch_conv_padded_transpose(dyq, esz, nimg, static_cast<int>(H), static_cast<int>(W), static_cast<int>(N), 1, dyT, 0, st);
    if(e != hipSuccess) return hip_status(e);
    GemmProblem p{};
    p.prec = tag; p.M = N; p.N = 9 * C; p.K = l.ax.Mp;
    p.A = dyT; p.B = xT; p.C = dw; p.c_dtype = dwdt;
    if(tag == QSYNC_INT8) { p.s0 = sdy; p.s1 = sx; p.acc_dump = acc_dump_opt; }
    p.b_remap_C = C; p.b_remap_shift = static_cast<int64_t>(l.ax.Wp) * esz;
    return hip_status(launch_gemm(p, l.plan, static_cast<uint8_t*>(workspace) + l.off_part, st));
}

size_t qsync_conv3x3_prepare_weights_workspace_bytes(int64_t N, int64_t C)
{
    if(N <= 0 || C <= 0) return 0;
    return absmax_workspace_bytes(N, 9 * C, kPerCol) + static_cast<size_t>(9 * N * C);
}

int qsync_conv3x3_prepare_weights(const void* w, int wdt, int64_t N, int64_t C, int bits, float* sw, float* iw, void* wq,
                                  float* swb, float* iwb, void* wflip, void* workspace, size_t workspace_bytes,
                                  void* stream)
{
    if(!w || !sw || !iw || !wq || !swb || !iwb || !wflip) return QSYNC_ERR_NULL;
    if(!is_float_dtype(wdt)) return QSYNC_ERR_BAD_ENUM;
    if(N < 0 || C < 0 || C > (1 << 20) || !count_ok(N, 9 * C)) return QSYNC_ERR_BAD_SHAPE;
    if(bits < 2 || bits > 8) return QSYNC_ERR_UNSUPPORTED;
    if(N == 0 || C == 0) return QSYNC_OK;
    if(!workspace || workspace_bytes < qsync_conv3x3_prepare_weights_workspace_bytes(N, C)) return QSYNC_ERR_WORKSPACE;
    if(!aligned16(workspace)) return QSYNC_ERR_ALIGN;
    const float qmax = static_cast<float>((1 << (bits - 1)) - 1);
    return hip_status(launch_conv3x3_prepare_weights(w, wdt == QSYNC_F32 ? kF32 : kF16, N, C, qmax, sw, iw, swb, iwb,
                                                     static_cast<int8_t*>(wq), static_cast<int8_t*>(wflip), workspace,
                                                     static_cast<hipStream_t>(stream)));
}

int qsync_probe_mfma(int tag, int random_operands, int iters, void* out, double* ops_out, void* stream)
{
    if(!out) return QSYNC_ERR_NULL;
    if(tag != QSYNC_INT8 && tag != QSYNC_FP16) return QSYNC_ERR_BAD_ENUM;
    if(iters < 1 || iters > (1 << 24)) return QSYNC_ERR_BAD_SHAPE;
    iters = (iters + 3) / 4 * 4;               // the kernel runs whole groups of four iterations
    if(random_operands < 0 || random_operands > 2) return QSYNC_ERR_BAD_ENUM;
    if(ops_out)   // a 16x16x64 int8 instruction is 2*16*16*64 operations, the 16x16x32 binary16 one half of that
        *ops_out = static_cast<double>(kProbeBlocks) * 4.0 * 8.0 * iters * (tag == QSYNC_INT8 ? 32768.0 : 16384.0);
    return hip_status(launch_probe_mfma(tag, random_operands, iters, out, static_cast<hipStream_t>(stream)));
}

void qsync_debug_set_gemm_tile(int tile) { set_gemm_tile_override(tile); }
void qsync_debug_set_gemm_persistent(int mode) { set_gemm_persistent_mode(mode); }
int qsync_debug_last_gradient_pair(void) { return g_last_pair_tile; }
int qsync_debug_last_gradient_splits(void) { return g_last_pair_splits; }
int qsync_debug_last_wgrad_ring(void) { return last_wgrad_ring(); }

static int conv3x3_fwd_impl(int tag, int64_t nimg, int64_t H, int64_t W, int64_t C, int64_t N, const void* xq,
                            const float* sx, const void* wq, const float* sw, int wgran, const float* bias_opt, void* y,
                            int ydt, int32_t* acc_dump_opt, float* y_amax_opt, void* stream)
{
    if(!xq || !wq || !y) return QSYNC_ERR_NULL;
    if(!is_tag(tag) || !is_float_dtype(ydt)) return QSYNC_ERR_BAD_ENUM;
    if(tag == QSYNC_INT8)
    {
        if(!sx || !sw) return QSYNC_ERR_NULL;
        if(!is_gran(wgran)) return QSYNC_ERR_BAD_ENUM;
    }
    if(nimg < 0 || H < 0 || W < 0 || C < 0 || N < 0 || H > 65535 || W > 65535 || C > (1 << 20) || N > (int64_t(1) << 31))
        return QSYNC_ERR_BAD_SHAPE;
    if(tag == QSYNC_FP32) return QSYNC_ERR_UNSUPPORTED;
    if(tag == QSYNC_INT8 && wgran == QSYNC_PER_COL) return QSYNC_ERR_UNSUPPORTED;
    if(tag != QSYNC_INT8 && acc_dump_opt) return QSYNC_ERR_UNSUPPORTED;
    const int64_t esz = tag == QSYNC_INT8 ? 1 : 2;
    if(H > 0 && W > 0 && C > 0 && nimg > ((int64_t(1) << 31) - 1) / (H * W * C * esz)) return QSYNC_ERR_BAD_SHAPE;
    const int64_t M = nimg * H * W;
    if(!count_ok(M, N) || !count_ok(N, 9 * C)) return QSYNC_ERR_BAD_SHAPE;
    if((C * esz) % 16 != 0 || !aligned16(xq) || !aligned16(wq)) return QSYNC_ERR_ALIGN;
    if(M == 0 || N == 0) return QSYNC_OK;
    const GemmPlan plan = plan_gemm(tag, M, N, 9 * C, -1, -1, /*allow_split=*/false);
    GemmProblem p{};
    p.prec = tag; p.M = M; p.N = N; p.K = 9 * C;
    p.A = xq; p.B = wq; p.C = y; p.c_dtype = ydt;
    p.conv_H = static_cast<int>(H); p.conv_W = static_cast<int>(W); p.conv_C = C;
    if(tag == QSYNC_INT8)
    {
        p.s0 = sx;
        if(wgran == QSYNC_PER_TENSOR) p.s1 = sw; else p.col_scale = sw;
        p.acc_dump = acc_dump_opt;
    }
    p.col_bias = bias_opt;
    p.out_amax_bits = reinterpret_cast<unsigned int*>(y_amax_opt);
    return hip_status(launch_gemm(p, plan, nullptr, static_cast<hipStream_t>(stream)));
}

int qsync_conv3x3_fwd(int tag, int64_t nimg, int64_t H, int64_t W, int64_t C, int64_t N, const void* xq,
                      const float* sx, const void* wq, const float* sw, int wgran, const float* bias_opt, void* y,
                      int ydt, int32_t* acc_dump_opt, void* stream)
{
    return conv3x3_fwd_impl(tag, nimg, H, W, C, N, xq, sx, wq, sw, wgran, bias_opt, y, ydt, acc_dump_opt, nullptr, stream);
}

int qsync_conv3x3_fwd_amax(int tag, int64_t nimg, int64_t H, int64_t W, int64_t C, int64_t N, const void* xq,
                           const float* sx, const void* wq, const float* sw, int wgran, const float* bias_opt, void* y,
                           int ydt, int32_t* acc_dump_opt, float* y_amax, void* stream)
{
    if(!y_amax) return QSYNC_ERR_NULL;
    if((reinterpret_cast<uintptr_t>(y_amax) & 3u) != 0) return QSYNC_ERR_ALIGN;
    return conv3x3_fwd_impl(tag, nimg, H, W, C, N, xq, sx, wq, sw, wgran, bias_opt, y, ydt, acc_dump_opt, y_amax, stream);
}

// The operands of a forward pass one after the other, activation first.
static int convert_operands_apart(int tag, const void* x, int xdt, int64_t M, int64_t C, float* x_amax_opt, const void* w, int wdt,
                                  int64_t N, int taps, int bits, int w_gran, float* sx, float* ix, float* ax_opt, void* xq, void* xqT_opt,
                                  float* sw, float* iw, float* aw_opt, void* wq, float* swb, float* iwb, void* wqbT, void* ws_x,
                                  size_t ws_x_bytes, void* ws_w, size_t ws_w_bytes, void* stream)
{
    const int64_t K  = taps * C;
    int           rc = QSYNC_OK;
    if(tag == QSYNC_INT8 && !x_amax_opt)
        rc = qsync_absmax_quantize(x, xdt, M, C, bits, QSYNC_ROUND_NEAREST, 0, 0, sx, ix, ax_opt, xq, xqT_opt, ws_x, ws_x_bytes, -1, stream);
    else
    {
        if(tag == QSYNC_INT8) rc = qsync_scale_from_amax(x_amax_opt, bits, sx, ix, 1, stream);
        if(rc == QSYNC_OK && (tag == QSYNC_INT8 || xq || xqT_opt))
            rc = qsync_quantize(x, xdt, M, C, C, tag, tag == QSYNC_INT8 ? bits : 0, QSYNC_PER_TENSOR, QSYNC_ROUND_NEAREST, 0, 0,
                                tag == QSYNC_INT8 ? ix : nullptr, xq, xqT_opt, stream);
    }
    if(rc != QSYNC_OK) return rc;
    if(tag == QSYNC_INT8 && w_gran == QSYNC_PER_ROW)
        return taps == 9 ? qsync_conv3x3_prepare_weights(w, wdt, N, C, bits, sw, iw, wq, swb, iwb, wqbT, ws_w, ws_w_bytes, stream)
                         : qsync_prepare_weights(w, wdt, N, K, bits, sw, iw, aw_opt, wq, swb, iwb, wqbT, ws_w, ws_w_bytes, stream);
    void* const wT = taps == 9 ? nullptr : wqbT;
    rc = tag == QSYNC_INT8 ? qsync_absmax_quantize(w, wdt, N, K, bits, QSYNC_ROUND_NEAREST, 0, 0, sw, iw, aw_opt, wq, wT, ws_w, ws_w_bytes, -1, stream)
                           : qsync_quantize(w, wdt, N, K, K, tag, 0, QSYNC_PER_TENSOR, QSYNC_ROUND_NEAREST, 0, 0, nullptr, wq, wT, stream);
    if(rc != QSYNC_OK || taps == 1) return rc;
    return qsync_conv3x3_wflip(wq, tag == QSYNC_INT8 ? QSYNC_I8 : QSYNC_F16, N, C, wqbT, stream);
}

int qsync_convert_operands(int tag, const void* x, int xdt, int64_t M, int64_t C, float* x_amax_opt, const void* w, int wdt, int64_t N,
                           int taps, int bits, int w_gran, float* sx, float* ix, float* ax_opt, void* xq, void* xqT_opt, float* sw,
                           float* iw, float* aw_opt, void* wq, float* swb, float* iwb, void* wqbT, void* ws_x, size_t ws_x_bytes,
                           void* ws_w, size_t ws_w_bytes, void* stream)
{
    if(!is_tag(tag)) return QSYNC_ERR_BAD_ENUM;
    if(tag == QSYNC_INT8 && w_gran != QSYNC_PER_TENSOR && w_gran != QSYNC_PER_ROW) return QSYNC_ERR_BAD_ENUM;
    if((taps != 1 && taps != 9) || (taps == 9 && (tag == QSYNC_FP32 || xqT_opt))) return QSYNC_ERR_UNSUPPORTED;
    // shared launches where each conversion by itself would pass its checks and neither writes what the other reads or writes
    const bool   i8 = tag == QSYNC_INT8, rows = w_gran == QSYNC_PER_ROW;
    bool         ok = x && w && wq && wqbT && is_float_dtype(xdt) && wdt == QSYNC_F32 && M > 0 && C > 0 && N > 0 && C <= (1 << 28)
              && count_ok(M, C) && count_ok(N, taps * C) && (taps == 1 || C <= (1 << 20));
    size_t need_x = 0, need_w = 0;
    if(ok && i8)
    {
        need_x = x_amax_opt ? 0 : qsync_absmax_workspace_bytes(M, C, QSYNC_PER_TENSOR);
        need_w = !rows ? qsync_absmax_workspace_bytes(N, taps * C, QSYNC_PER_TENSOR)
                 : taps == 9 ? qsync_conv3x3_prepare_weights_workspace_bytes(N, C) : absmax_workspace_bytes(N, C, kPerCol);
        ok = bits >= 2 && bits <= 8 && sx && ix && sw && iw && (!rows || (swb && iwb)) && (xq || xqT_opt)
          && (x_amax_opt || (ws_x && ws_x_bytes >= need_x && aligned16(ws_x))) && ws_w && ws_w_bytes >= need_w && aligned16(ws_w);
    }
    if(ok)
    {
        struct Span { const void* p; int64_t n; };
        const int64_t xe = xdt == QSYNC_F16 ? 2 : 4, oe = i8 ? 1 : (tag == QSYNC_FP16 ? 2 : 4), nx = M * C, nw = N * taps * C;
        const int64_t nsw = rows ? N : 1, nsb = rows ? C : 1;
        const Span x_in[] = {{x, nx * xe}, {x_amax_opt, 4}};
        const Span x_out[] = {{xq, nx * oe}, {xqT_opt, nx * oe}, {i8 ? sx : nullptr, 4}, {i8 ? ix : nullptr, 4}, {i8 ? ax_opt : nullptr, 4},
                              {i8 ? ws_x : nullptr, static_cast<int64_t>(need_x)}, {x_amax_opt, 4}};
        const Span w_in[] = {{w, nw * 4}};
        const Span w_out[] = {{wq, nw * oe}, {wqbT, nw * oe}, {i8 ? sw : nullptr, nsw * 4}, {i8 ? iw : nullptr, nsw * 4},
                              {i8 ? aw_opt : nullptr, nsw * 4}, {i8 && rows ? swb : nullptr, nsb * 4}, {i8 && rows ? iwb : nullptr, nsb * 4},
                              {i8 ? ws_w : nullptr, static_cast<int64_t>(need_w)}};
        auto apart = [](const Span& a, const Span& b) {
            const uintptr_t p = reinterpret_cast<uintptr_t>(a.p), q = reinterpret_cast<uintptr_t>(b.p);
            return !a.p || !b.p || p >= q + static_cast<uintptr_t>(b.n) || q >= p + static_cast<uintptr_t>(a.n);
        };
        for(const Span& o : x_out)
        {
            for(const Span& i : w_in) ok = ok && apart(o, i);
            for(const Span& i : w_out) ok = ok && apart(o, i);
        }
        for(const Span& o : w_out)
            for(const Span& i : x_in) ok = ok && apart(o, i);
    }
    if(ok)
    {
        const OperandConversion c{x, M, C, i8 ? x_amax_opt : nullptr, w, N, taps, i8 ? (1 << (bits - 1)) - 1 : 0, w_gran, sx, ix, ax_opt,
                                  xq, xqT_opt, sw, iw, taps == 9 && rows ? nullptr : aw_opt, wq, swb, iwb, wqbT, ws_x, ws_w};
        bool      taken = false;
        const int rc    = hip_status(launch_convert_operands(c, tag, xdt, &taken, static_cast<hipStream_t>(stream)));
        if(taken || rc != QSYNC_OK) return rc;
    }
    return convert_operands_apart(tag, x, xdt, M, C, x_amax_opt, w, wdt, N, taps, bits, w_gran, sx, ix, ax_opt, xq, xqT_opt, sw, iw,
                                  aw_opt, wq, swb, iwb, wqbT, ws_x, ws_x_bytes, ws_w, ws_w_bytes, stream);
}

int qsync_conv3x3_wflip(const void* w, int wdt, int64_t N, int64_t C, void* wflip, void* stream)
{
    if(!w || !wflip) return QSYNC_ERR_NULL;
    if(wdt != QSYNC_I8 && wdt != QSYNC_F16) return QSYNC_ERR_BAD_ENUM;
    if(N < 0 || C < 0 || !count_ok(N, 9 * C)) return QSYNC_ERR_BAD_SHAPE;
    if(w == wflip) return QSYNC_ERR_UNSUPPORTED;
    return hip_status(launch_conv3x3_wflip(w, wdt == QSYNC_I8 ? 1 : 2, N, C, wflip, static_cast<hipStream_t>(stream)));
}

int qsync_im2col3x3_i8(const void* xq, int64_t nimg, int64_t H, int64_t W, int64_t C, void* a_opt, void* aT_opt,
                       void* stream)
{
    if(!xq || (!a_opt && !aT_opt)) return QSYNC_ERR_NULL;
    if(nimg < 0 || H < 0 || W < 0 || C < 0 || H > (1 << 15) || W > (1 << 15) || C > (1 << 15)) return QSYNC_ERR_BAD_SHAPE;
    if(nimg > 0 && H > 0 && W > 0 && nimg > (int64_t(1) << 40) / (H * W)) return QSYNC_ERR_BAD_SHAPE;
    const int64_t M = nimg * H * W;
    if(M == 0 || C == 0) return QSYNC_OK;
    if(C % 16 != 0) return QSYNC_ERR_UNSUPPORTED;
    if(((M + 511) / 512) * ((9 * C / 16 + 7) / 8) >= (int64_t(1) << 31)) return QSYNC_ERR_BAD_SHAPE;
    if(!aligned16(xq) || (a_opt && !aligned16(a_opt)) || (aT_opt && (!aligned16(aT_opt) || M % 16 != 0))) return QSYNC_ERR_ALIGN;
    return hip_status(launch_im2col3x3_i8(static_cast<const int8_t*>(xq), nimg, static_cast<int>(H), static_cast<int>(W),
                                          static_cast<int>(C), static_cast<int8_t*>(a_opt), static_cast<int8_t*>(aT_opt),
                                          static_cast<hipStream_t>(stream)));
}

int qsync_dequantize(const void* a, int adt, int64_t rows, int64_t cols, int64_t ld, const float* row_scale_opt,
                     const float* col_scale_opt, float tensor_scale, const float* tensor_scale_dev_opt,
                     const float* col_bias_opt, void* y, int ydt, void* stream)
{
    if(!a || !y) return QSYNC_ERR_NULL;
    if((adt != QSYNC_I32 && adt != QSYNC_I8) || !is_float_dtype(ydt)) return QSYNC_ERR_BAD_ENUM;
    if(!count_ok(rows, cols) || ld < cols || !count_ok(rows, ld)) return QSYNC_ERR_BAD_SHAPE;
    if(rows == 0 || cols == 0) return QSYNC_OK;
    return hip_status(launch_dequantize(a, adt == QSYNC_I32 ? kI32 : kI8, rows, cols, ld, row_scale_opt, col_scale_opt,
                                        tensor_scale, tensor_scale_dev_opt, col_bias_opt, y, ydt,
                                        static_cast<hipStream_t>(stream)));
}

}  // extern "C"
