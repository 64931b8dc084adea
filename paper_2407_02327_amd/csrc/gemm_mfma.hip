// LDS-tiled MFMA GEMM for gfx950 (CDNA4):  C[M,N] = epilogue( sum_k A[m,k] * B[n,k] ).
//
// Both operands are K-contiguous ("NT"), which is exactly the operand shape of the gfx950
// 16x16 matrix instructions: every lane feeds 16 contiguous K-bytes of one row of A and of
// one row of B (v_mfma_i32_16x16x64_i8: 16 int8; v_mfma_f32_16x16x32_f16: 8 binary16).  The
// INT8 and FP16 kernels therefore move identical bytes and share one tiling:
//
//   * block tile BM x BN, K step of 128 bytes per row; WGM x WGN wavefronts, each owning a
//     (BM/WGM) x (BN/WGN) sub-tile as 16x16 accumulator fragments.  The large tile is
//     256x256 with 8 wavefronts (2 per SIMD, 128 accumulator registers each), so that one
//     wavefront's LDS reads and barrier waits hide behind the other's matrix instructions;
//   * global -> LDS with direct 16-byte loads (global_load_lds_dwordx4), bypassing the VGPRs;
//     LDS rows are 128 bytes.  The LDS of gfx950 serves a 16-byte read in groups of 16 lanes,
//     one 256-byte bank row per group, so the chunk position is XOR-swizzled with (row/2)%8
//     (applied on the global-address side of the direct load): the 16 lanes that read one
//     chunk index of 16 consecutive rows then touch 16 different 16-byte bank groups;
//   * two LDS stages: the next K step streams in while the current one feeds the matrix cores; a fragment of the next
//     64-byte K chunk is requested behind the last matrix instruction that reads its registers; one barrier per K step.
//     The 128x128 tile, while no compute unit gets a second workgroup, has three stages, or four and wavefronts of their
//     own for the loads (launch_traits);
//   * the dequantizer (scalar scales, per-column scale vector, per-column bias) runs on the
//     accumulator registers (the paper fuses dequantization at the same point: before the
//     accumulators are copied to shared memory); the B fragment is fed as the instruction's
//     first operand so that a lane holds four consecutive output columns per register quad,
//     which are packed, passed through the wavefront's private LDS slice and stored to C as
//     16-byte vectors along the rows;
//   * workgroup ids are remapped so that consecutive tiles stay on one XCD (ids are dealt
//     round-robin to the 8 XCDs, each with its own L2) and walk the tile grid in groups of
//     rows, which keeps the A and B panels of neighbouring tiles in that L2;
//   * split-K (for outputs with too few tiles to fill 256 CUs) writes raw partial
//     accumulators to a workspace; a second kernel adds them in a fixed order and applies
//     the epilogue, so results do not depend on scheduling.
#include "gemm_device.h"

#include <cmath>

namespace qsync {

namespace {

constexpr int kPersistentLdsBytes = 159744;   // two 64 KB stages, hand-over area, column parameters

// Implicit patch matrix of a 3x3 / stride 1 / pad 1 convolution over an NHWC tensor: row m of A is
// output pixel m, its K axis runs (kh, kw, c).  A 16-byte chunk lies inside one tap because the
// pixel size is a multiple of 16 bytes, so the direct load of a lane either reads 16 bytes of the
// neighbouring pixel (same image, inside the border) or, for padding and for chunks past the end
// of K, 16 zero bytes from a constant block.
// Where a lane's two chunk positions (by parity of the load slot) stand on the K axis: the byte offset (less W + 1 pixels,
// modulo 2^32), the tap it lies in and the channel offset in that tap.  Requests go over consecutive K tiles, so the position is carried on instead of
// divided out of the tile index (a division per parity and tile, and border tests per load, made the gather's own
// arithmetic the bound of the K loop: four loads took about 130 vector instructions, now about 55).
struct ConvTap { uint32_t koff[2], tap[2], c0[2]; };

// `mask`: bit t says that tap t of the lane's output pixel lies inside the image; taps from 9 on (chunks past the end
// of K) have no bit.  `delta`: byte distance from the pixel to the chunk's source, modulo 2^32: their sum is the source's
// offset in the tensor, below 2^31 wherever the mask has the bit.  (Without the modulus, on a base W + 1 pixels in front
// of the tensor, the sum reaches 2 W + 1 pixels and left 32 bits for one row of nearly 2^31 bytes.)
template <int D, int DPW>
__device__ __forceinline__ void conv_issue(const uint8_t* a, const uint8_t* zero, uint32_t pix_off, uint32_t mask,
                                           const ConvTap& t, const uint32_t (&delta)[2], uint8_t* lds_mid)
{
    constexpr int IMM = dma_imm<D, DPW>();
    constexpr int par = D & 1;
    const uint8_t* src = ((mask >> t.tap[par]) & 1u) ? a + (pix_off + delta[par]) : zero;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src - IMM),
                                     (__attribute__((address_space(3))) void*)(lds_mid + dma_lds_shift<D, DPW>()), 16, IMM, 0);
}

template <int DPW, int... Ds>
__device__ __forceinline__ void conv_sequence(std::integer_sequence<int, Ds...>, const uint8_t* a, const uint8_t* zero,
                                              const uint32_t (&pix_off)[DPW], const uint32_t (&mask)[DPW],
                                              const ConvTap& t, const uint32_t (&delta)[2], uint8_t* lds_mid)
{
    (conv_issue<Ds, DPW>(a, zero, pix_off[Ds], mask[Ds], t, delta, lds_mid), ...);
}

// TN form with the B operand gathered from an NHWC tensor (weight gradient of the 3x3 convolution): stage row r of
// K tile kt is pixel m = kt * KR + r, and a lane's 16-byte chunk lies in one tap (dh, dw) at channel offset c0, both
// fixed per load slot; what changes from K tile to K tile is the pixel, i.e. (h, w).  `delta` holds the slot's whole
// constant part ((dh W + dw) Cb + c0 + r Cb), modulo 2^32; `code`, low byte: (dh + 1) | (dw + 1) << 2 | valid << 4; `hw` = h << 16 | w of the
// pixel of the NEXT K tile to be requested and is advanced by KR pixels here (dr = KR % W, hq = (KR / W) % H).
template <int D, int DPW>
__device__ __forceinline__ void conv_tn_issue(const uint8_t* x, const uint8_t* zero, uint32_t pix_base, uint32_t delta, int code,
                                              uint32_t& hw, int H, int W, int dr, int hq, uint8_t* lds_mid)
{
    constexpr int IMM = dma_imm<D, DPW>();
    int        h = static_cast<int>(hw >> 16), w = static_cast<int>(hw & 0xffffu);
    const int  hh = h + (code & 3) - 1, ww = w + ((code >> 2) & 3) - 1;
    const bool inb = ((code >> 4) & 1) != 0 && static_cast<unsigned>(hh) < static_cast<unsigned>(H)
                     && static_cast<unsigned>(ww) < static_cast<unsigned>(W);
    const uint8_t* src = inb ? x + (pix_base + delta) : zero;       // (an offset in the tensor, below 2^31, wherever it is read)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src - IMM),
                                     (__attribute__((address_space(3))) void*)(lds_mid + dma_lds_shift<D, DPW>()), 16, IMM, 0);
    w += dr;
    const int carry = w >= W ? 1 : 0;
    w -= carry ? W : 0;
    h += hq + carry;
    h -= h >= H ? H : 0;
    hw = (static_cast<uint32_t>(h) << 16) | static_cast<uint32_t>(w);
}

template <int DPW, int... Ds>
__device__ __forceinline__ void conv_tn_sequence(std::integer_sequence<int, Ds...>, const uint8_t* x, const uint8_t* zero,
                                                 uint32_t pix_base, const uint32_t (&delta)[DPW], const uint32_t (&codes)[(DPW + 3) / 4],
                                                 uint32_t (&hw)[DPW], int H, int W, int dr, int hq, uint8_t* lds_mid)
{
    (conv_tn_issue<Ds, DPW>(x, zero, pix_base, delta[Ds], static_cast<int>(codes[Ds / 4] >> (8 * (Ds % 4))), hw[Ds], H, W, dr, hq, lds_mid), ...);
}

// TN, last K tile with fewer contraction rows than a stage holds: rows from `rows` on are fetched from the tile's first
// row instead (and overwritten with zeros once landed).
template <int DPW, int RPS, int... Ds>
__device__ __forceinline__ void dma_sequence_short(std::integer_sequence<int, Ds...>, const uint8_t* sbase,
                                                   const uint32_t (&voff)[DPW], int row0, int rows, uint32_t row_bytes, uint8_t* lds_mid)
{
    (dma_issue<Ds, DPW>(sbase, voff[Ds] - (row0 + Ds * RPS >= rows ? static_cast<uint32_t>(row0 + Ds * RPS) * row_bytes : 0u), lds_mid), ...);
}

// TN (int8 and binary16): both operands are handed over with the contraction axis as their ROW axis, A [P, M] and
// B [P, N] row-major (C[m,n] = sum_p A[p,m] B[p,n]): the weight gradient dW = dY^T X straight from the row-major
// operands, no transposed copies.  A stage then holds 128 (int8) or 64 (binary16) contraction rows of each operand
// (rows of BM / BN elements), and the fragments come out of LDS through the transposing reads of gfx950
// (ds_read_b64_tr_b8 / _b16): sixteen lanes read 8 rows x 16 bytes (4 rows x 32 bytes) and receive, lane j, the
// eight (four) elements of column j -- consecutive contraction indices of one output row, which is what the
// matrix instruction wants; two reads make a lane's 16 operand bytes.  16-byte chunks are XOR-swizzled per row so
// that the lanes of one access pass touch all banks once.  Everything behind the fragments
// (matrix instructions, epilogue, split K) is shared with the NT form.  Kb is the contraction length P here.
// `lin` is the workgroup's index among the `splits` x tiles workgroups of the problem.
// MIXED: whether the workgroup leaves raw sums (its problem is in K splits) is known at run time only (`raw`).
template <typename TR, int BM, int BN, int WGM, int WGN, int ST, int NL, bool SPLIT, bool CONV, bool TN, bool MIXED = false>
__device__ __forceinline__ void gemm_tile(const GemmKernelArgs& p, int lin, int splits, bool raw = SPLIT)
{
    static_assert(!MIXED || SPLIT, "one body for both");
    constexpr bool WHOLE = !SPLIT || MIXED;      // the epilogue may be this workgroup's
    static_assert(!(SPLIT && CONV && !TN), "the implicit patch matrix of the forward is not combined with split K");
    static_assert(!TN || (TR::kElemBytes <= 2 && BM == BN && BM >= 64), "TN: int8 or binary16 operands, square tiles");
    constexpr bool CONVA  = CONV && !TN;       // NT form: the A operand is the implicit patch matrix (forward, data gradient)
    constexpr bool CONVTN = CONV && TN;        // TN form: the B operand is gathered from the NHWC tensor (weight gradient)
    constexpr int ESZ = TR::kElemBytes;
    typedef typename TR::accv_t accv_t;
    typedef typename TR::acc_t  acc_t;
    constexpr int kThreads = 64 * WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;   // wavefront sub-tile
    constexpr int R = TR::kRows, FM = WTM / R, FN = WTN / R;         // fragments per wavefront
    constexpr int CH = kRowBytes / (16 * (64 / R));                 // K chunks (16 bytes of each of 64 / R lanes) per K tile
    constexpr int STAGE_BYTES = (BM + BN) * kRowBytes;
    constexpr int WC = WGM * WGN, WL = NL > 0 ? NL : WC;            // wavefronts that compute, that load
    constexpr int DPW = (BM + BN) / 8 / WL;                         // direct-load instructions per loading wavefront per K tile
    static_assert(R == 16 && CH == 2 && WTM % R == 0 && WTN % R == 0 && FM >= FN && (FN == 2 || FN == 4), "fragments of a wavefront");
    static_assert((BM + BN) % (8 * WL) == 0 && BM % 16 == 0, "stage rows must split evenly over the wavefronts");

    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

    int split, tm, tn;
    item_of_block(lin, p.tiles_m, p.tiles_n, SPLIT ? splits : 1, p.group_m, split, tm, tn);
    const int64_t m0 = static_cast<int64_t>(tm) * BM, n0 = static_cast<int64_t>(tn) * BN;
    const int     tid = threadIdx.x, lane = tid % kWaveSize;
    const int     wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize);     // wavefront index, held in an SGPR
    const int     wm = wave / WGN, wn = wave % WGN;
    const int     lwave = NL == 0 ? wave : wave >= WC ? wave - WC : 0;          // index among the loading wavefronts

    // K-tile indices are 32-bit so that the loop control stays on the scalar unit
    const int ktiles_all = static_cast<int>((p.Kb + kRowBytes - 1) / kRowBytes);
    const int tail_kt    = (p.Kb % kRowBytes) ? ktiles_all - 1 : -1;     // index of a partial last tile, if any
    int       kt_begin = 0, kt_end = ktiles_all;
    if(SPLIT)
    {
        kt_begin = split * p.ktiles_per_split;
        kt_end   = kt_begin + p.ktiles_per_split < ktiles_all ? kt_begin + p.ktiles_per_split : ktiles_all;
    }

    // Global -> LDS with direct loads (global_load_lds_dwordx4): the data never passes through
    // VGPRs and no LDS store instruction is issued.  One such instruction of a wavefront fills
    // 1 KB of LDS = 8 consecutive stage rows (A rows first, then B rows): lane l lands at row l/8,
    // chunk position l%8, so it fetches the logical chunk (l%8) ^ ((row/2)%8) of that row.
    // Rows beyond M (or N) are clamped to the last row: they only feed accumulators of outputs
    // that are never stored.  Chunks beyond the end of K (last, partial K tile only) are
    // fetched from the row's first chunk of that tile and overwritten with zeros once landed.
    // A wavefront's DPW instructions cover 8*DPW consecutive stage rows, all of A or all of B, so
    // its source is one uniform base pointer plus a 32-bit lane offset per instruction.
    constexpr bool kUniformSide = (BM / 8) % DPW == 0;
    static_assert(kUniformSide, "a wavefront must not straddle the A/B boundary of a stage");
    const bool     is_a      = lwave * DPW < BM / 8;
    // TN: the panel starts at the tile's first column of the operand (its rows are contraction indices)
    const uint8_t* gbase     = TN ? (is_a ? p.A + m0 * ESZ : (CONVTN ? p.B : p.B + n0 * ESZ))
                                  : (is_a ? p.A + m0 * p.Kb : ((!CONV && p.remap_C > 0) ? p.B : p.B + n0 * p.Kb));
    const int64_t  rows_left = is_a ? p.M - m0 : p.N - n0;           // >= 1
    uint32_t       voff[DPW];                                         // lane offset + kDmaBias - immediate
    uint32_t       hw[CONV ? DPW : 1];       // CONVTN: (h << 16) | w of the lane's pixels; CONVA: their taps inside the image
    uint32_t       tnc_code[CONVTN ? (DPW + 3) / 4 : 1] = {};      // CONVTN, B side (see conv_tn_issue), a byte per load; voff holds the deltas there
    int            gchunk[2];                                         // the swizzle term depends on d%2 only
    {
        int imm[DPW];
        fill_dma_imms<DPW>(imm, std::make_integer_sequence<int, DPW>{});
        if constexpr(TN)
        {   // instruction q of the stage fills LDS bytes [1024 q, 1024 q + 1024) of the A region (128 / ESZ rows of
            // BM elements), then of the B region; a lane's 16 bytes are chunk (position ^ swizzle(row)) of its row
            constexpr int RB = BM * ESZ;                                   // bytes per region row
            const int64_t ld    = (is_a ? p.M : p.N) * ESZ;                // operand row length in bytes
            const int64_t width = (is_a ? p.M - m0 : p.N - n0) * ESZ;      // valid bytes of this tile's columns (>= 16)
#pragma unroll
            for(int d = 0; d < DPW; ++d)
            {
                const int q     = lwave * DPW + d - (is_a ? 0 : BM / 8);
                const int o     = q * 1024 + lane * 16;
                const int row   = o / RB, pos = (o % RB) / 16;
                int       chunk = pos ^ tn_swizzle<ESZ, RB>(row);
                if constexpr(CONVTN)
                    if(!is_a)
                    {   // B side: column byte (n0 * ESZ + 16 chunk) of the implicit [pixels, 9 C] matrix = tap, channel offset
                        constexpr int KR = kRowBytes / ESZ;                       // pixels per K tile
                        const uint32_t colb  = static_cast<uint32_t>(n0) * ESZ + static_cast<uint32_t>(chunk) * 16u;      // (9 C < 2^24)
                        const bool     valid = colb < 9u * static_cast<uint32_t>(p.conv_Cb);      // tile columns past 9 C: zeros, never stored
                        const int      tap   = valid ? static_cast<int>(colb / static_cast<uint32_t>(p.conv_Cb)) : 0;
                        const int      c0    = valid ? static_cast<int>(colb) - tap * p.conv_Cb : 0;
                        const int     kh = (tap * 11) >> 5, kw = tap - 3 * kh;          // tap / 3 for tap < 12
                        voff[d]      = static_cast<uint32_t>(((kh - 1) * p.conv_W + (kw - 1)) * p.conv_Cb + c0 + row * p.conv_Cb);
                        tnc_code[d / 4] |= static_cast<uint32_t>(kh | (kw << 2) | (valid ? 16 : 0)) << (8 * (d % 4));
                        const uint32_t m  = static_cast<uint32_t>(kt_begin) * KR + static_cast<uint32_t>(row);
                        const uint32_t qq = m / static_cast<uint32_t>(p.conv_W);
                        hw[d]   = ((qq % static_cast<uint32_t>(p.conv_H)) << 16) | (m - qq * static_cast<uint32_t>(p.conv_W));
                        continue;
                    }
                if(static_cast<int64_t>(chunk) * 16 >= width) chunk = 0;    // columns past the matrix: any valid chunk, never stored
                voff[d] = static_cast<uint32_t>(static_cast<int64_t>(row) * ld + chunk * 16 + kDmaBias - imm[d]);
            }
            gchunk[0] = gchunk[1] = 0;
        }
        else
#pragma unroll
        for(int d = 0; d < DPW; ++d)
        {
            const int srow  = (lwave * DPW + d) * 8 + lane / 8;           // row inside the stage
            const int chunk = (lane % 8) ^ ((srow >> 1) & 7);             // BM % 16 == 0: same term for A and B rows
            int64_t   lrow  = srow - (is_a ? 0 : BM);
            if(lrow >= rows_left) lrow = rows_left - 1;
            voff[d] = static_cast<uint32_t>(lrow * p.Kb + chunk * 16 + kDmaBias - imm[d]);
            if constexpr(CONVA)
                if(is_a)
                {   // A side: voff holds the byte offset of output pixel m in the NHWC tensor instead
                    const uint32_t m = static_cast<uint32_t>(m0 + lrow), q = m / static_cast<uint32_t>(p.conv_W);
                    voff[d] = m * static_cast<uint32_t>(p.conv_Cb);
                    const uint32_t h = q % static_cast<uint32_t>(p.conv_H), w = m - q * static_cast<uint32_t>(p.conv_W);
                    const uint32_t row = (w > 0 ? 1u : 0u) | 2u | (w + 1 < static_cast<uint32_t>(p.conv_W) ? 4u : 0u);
                    hw[d] = (h > 0 ? row : 0u) | (row << 3) | (h + 1 < static_cast<uint32_t>(p.conv_H) ? row << 6 : 0u);
                }
            if(d < 2) gchunk[d] = chunk * 16;
        }
        if constexpr(!CONV && !TN)
            if(p.remap_C > 0 && !is_a)
            {   // offset from p.B itself (the base below is not advanced to this tile's rows); in a block of its own, so
                // that the ordinary kernel's first instructions are not spread over these divisions
#pragma unroll
                for(int d = 0; d < DPW; ++d)
                {
                    const int      lrow = (lwave * DPW + d) * 8 + lane / 8 - BM;
                    const uint32_t row  = static_cast<uint32_t>(n0 + (lrow < rows_left ? lrow : rows_left - 1));
                    const int      tap  = static_cast<int>(row / static_cast<uint32_t>(p.remap_C));
                    const int      c    = static_cast<int>(row) - tap * p.remap_C;
                    const int      kh = (tap * 11) >> 5, kw = tap - 3 * kh;      // tap / 3 for tap < 12
                    voff[d] = static_cast<uint32_t>(static_cast<int64_t>(kw * p.remap_C + c) * p.Kb + (kh - 1) * p.remap_shift
                                                    + gchunk[d & 1] + kDmaBias - imm[d]);
                }
            }
    }
    // the panel base as two scalar registers (the wavefront index is uniform, so is the choice of panel)
    const uint64_t gbits = reinterpret_cast<uint64_t>(gbase) - kDmaBias;
    const uint8_t* sbase0 = reinterpret_cast<const uint8_t*>(uniform64(static_cast<int64_t>(gbits)));
    // All DPW instructions of a wavefront share one LDS base (M0): instruction d reaches its 1 KB
    // slot through the instruction's immediate offset (d - DPW/2) KB.  Rewriting M0 between direct
    // loads would stall the wavefront until the previous load has left the issue queue
    // (measured: +20 % GEMM throughput without it).
    // CONVTN: pixels per K tile, and how far (h, w) of a stage row move from one K tile to the next
    constexpr int tnc_KR = kRowBytes / ESZ;
    const int     tnc_dr = CONVTN ? tnc_KR % p.conv_W : 0, tnc_hq = CONVTN ? (tnc_KR / p.conv_W) % p.conv_H : 0;
    // CONVA: the K axis position of the lane's two chunks, how it moves from one K tile to the next, and the extra distance
    // of a step in kh
    ConvTap        conv_t;
    const uint32_t conv_cb = CONVA ? static_cast<uint32_t>(p.conv_Cb) : 1u;
    const uint32_t conv_q = kRowBytes / conv_cb, conv_r = kRowBytes % conv_cb;
    const uint32_t conv_kh_step = CONVA ? static_cast<uint32_t>((p.conv_W - 3) * p.conv_Cb) : 0u;       // (modulo 2^32 for W < 3)
    if constexpr(CONVA)
#pragma unroll
        for(int par = 0; par < 2; ++par)
        {
            conv_t.koff[par] = static_cast<uint32_t>(gchunk[par]);
            conv_t.tap[par]  = conv_t.koff[par] / conv_cb;
            conv_t.c0[par]   = conv_t.koff[par] % conv_cb;
            conv_t.koff[par] -= (static_cast<uint32_t>(p.conv_W) + 1u) * conv_cb;
        }
    const int64_t tn_ld = TN ? uniform64(is_a ? p.M : p.N) : 0;      // operand row length in elements
    // TN: stage row of the lane in load slot 0, rows from slot to slot, and the contraction rows of a partial last K tile
    constexpr int tn_rps = TN ? 1024 / (BM * ESZ) : 0;
    auto          tn_first_row = [&]() { return ((lwave * DPW - (is_a ? 0 : BM / 8)) * 1024 + lane_again() * 16) / (BM * ESZ); };
    const int     tn_tail_rows = TN ? static_cast<int>(p.Kb % kRowBytes) / ESZ : 0;
    auto dma = [&](int stage, int kt) {
        const int64_t  kb    = static_cast<int64_t>(kt) * kRowBytes;
        uint8_t*       lbase = lds + stage * STAGE_BYTES + lwave * (DPW * 1024) + (dma_group<DPW>() / 2) * 1024;
        if constexpr(CONVTN)
            if(!is_a)
            {   // (requested for consecutive K tiles only, starting at kt_begin: hw is advanced by every call)
                if(kt == tail_kt)      // (the last request) stage rows without a pixel read zeros
                {
                    const int row0 = tn_first_row();
#pragma unroll
                    for(int d = 0; d < DPW; ++d)
                        if(row0 + d * tn_rps >= tn_tail_rows) tnc_code[d / 4] &= ~(0xFFu << (8 * (d % 4)));
                }
                conv_tn_sequence<DPW>(std::make_integer_sequence<int, DPW>{}, p.B, reinterpret_cast<const uint8_t*>(&g_zero_chunk),
                                      static_cast<uint32_t>(kt) * static_cast<uint32_t>(tnc_KR) * static_cast<uint32_t>(p.conv_Cb), voff, tnc_code, hw, p.conv_H, p.conv_W,
                                      tnc_dr, tnc_hq, lbase);
                return;
            }
        if constexpr(CONVA)
            if(is_a)
            {
                // (for consecutive K tiles, starting at 0)  Source of a chunk: pixel + (kh - 1) rows + (kw - 1) pixels + c0
                // = pixel - (W + 1) pixels + K offset + kh (W - 3) pixels, since the K offset = (3 kh + kw) pixels + c0;
                // koff carries the constant part.
                uint32_t delta[2];
#pragma unroll
                for(int par = 0; par < 2; ++par)
                    delta[par] = conv_t.koff[par] + (conv_t.tap[par] >= 3 ? conv_kh_step : 0u) + (conv_t.tap[par] >= 6 ? conv_kh_step : 0u);
                conv_sequence<DPW>(std::make_integer_sequence<int, DPW>{}, p.A, reinterpret_cast<const uint8_t*>(&g_zero_chunk),
                                   voff, hw, conv_t, delta, lbase);
#pragma unroll
                for(int par = 0; par < 2; ++par)
                {
                    conv_t.koff[par] += kRowBytes;
                    conv_t.tap[par]  += conv_q;
                    conv_t.c0[par]   += conv_r;
                    if(conv_t.c0[par] >= static_cast<uint32_t>(p.conv_Cb)) { conv_t.c0[par] -= static_cast<uint32_t>(p.conv_Cb); ++conv_t.tap[par]; }
                }
                return;
            }
        const uint8_t* sb    = TN ? sbase0 + kb * tn_ld : sbase0 + kb;      // TN: 128 operand rows further
        asm volatile("" : "+s"(sb));      // keep base + K offset a scalar pair: the lane offsets stay loop-invariant 32-bit values
        if(TN && kt == tail_kt)
            dma_sequence_short<DPW, tn_rps>(std::make_integer_sequence<int, DPW>{}, sb, voff, tn_first_row(), tn_tail_rows,
                                            static_cast<uint32_t>(tn_ld * ESZ), lbase);
        else if(!TN && kt == tail_kt)
            dma_sequence_tail<DPW>(std::make_integer_sequence<int, DPW>{}, sb, voff, gchunk, kb, p.Kb, lbase);
        else
            dma_sequence<DPW>(std::make_integer_sequence<int, DPW>{}, sb, voff, lbase);
    };
    // Waits for this wavefront's direct loads and for its outstanding fragment reads (the barrier hands the
    // stage they read to the next direct load, and the compiler does not see those reads), zero-fills its
    // out-of-K chunks, then joins the block.
    auto zero_tail = [&](int stage, int kt) {
        if((!CONVTN || is_a) && kt == tail_kt)
        {
            const int64_t kb   = static_cast<int64_t>(kt) * kRowBytes;
            const int     l    = lane_again(), row0 = TN ? ((lwave * DPW - (is_a ? 0 : BM / 8)) * 1024 + l * 16) / (BM * ESZ) : 0;
#pragma unroll
            for(int d = 0; d < DPW; ++d)
                if(TN ? row0 + d * tn_rps >= tn_tail_rows : kb + gchunk[d & 1] >= p.Kb)
                    *reinterpret_cast<uint4*>(lds + stage * STAGE_BYTES + (lwave * DPW + d) * 1024 + l * 16)
                        = make_uint4(0, 0, 0, 0);
        }
    };
    auto land = [&](int stage, int kt) {
        // direct loads retire in order: tile kt has landed when at most the loads of the tiles requested behind it
        // (up to ST - 2 of them; fewer at the end of K) are outstanding
        wait_tiles<DPW, ST - 2>(kt_end - 1 - kt);
        zero_tail(stage, kt);
        wg_barrier();
    };
    float*     colp  = reinterpret_cast<float*>(lds + ST * STAGE_BYTES);       // [2][BN]: scale, bias
    const bool any_k = kt_begin < kt_end;
    // Column parameters and as many K tiles as there are stages; the wait for tile 0 (up to ST - 1 tiles are requested behind it).
    // Nothing in front of the K loop waits for global memory except that wait (a load into a register here would make the
    // compiler drain the queue before its use).
    auto request_first = [&]() {
        if(WHOLE && lwave < BN / 64)
        {
            const int64_t c = n0 + lwave * 64 + lane, col = c < p.N ? c : p.N - 1;       // columns past N: any valid one, never stored
            if(p.col_scale) column_param_issue(p.col_scale + col, lds + ST * STAGE_BYTES + lwave * 256);
            if(p.col_bias) column_param_issue(p.col_bias + col, lds + ST * STAGE_BYTES + BN * 4 + lwave * 256);
        }
#pragma unroll
        for(int t = 0; t < ST; ++t)
            if(kt_begin + t < kt_end) dma(t, kt_begin + t);
    };
    auto await_first = [&]() {
        wait_tiles<DPW, ST - 1>(kt_end - 1 - kt_begin);
        zero_tail(0, kt_begin);
        wg_barrier();
    };
    // Loading wavefronts of their own (NL): they meet the others at every K tile's barrier and do nothing but request, wait and
    // clear.  A direct load occupies the compute unit's vector-memory path for 16 clocks, the 32 of a 128 tile's K tile for
    // 512, and a wavefront whose loads queue there issues nothing else; with two computing wavefronts a SIMD that was twice
    // what their instructions and LDS reads took.
    if constexpr(NL > 0)
        if(wave >= WC)
        {
            request_first();
            if(!any_k)
            {
                wait_direct_loads<0>();              // the column parameters
                return;
            }
            await_first();
            int stage = 0;
            for(int kt = kt_begin; kt + 1 < kt_end; ++kt)
            {
                const int next = stage + 1 < ST ? stage + 1 : 0;
                land(next, kt + 1);
                if(kt + ST < kt_end) dma(stage, kt + ST);
                stage = next;
            }
            return;
        }

    accv_t acc[FM][FN];
#pragma unroll
    for(int i = 0; i < FM; ++i)
#pragma unroll
        for(int j = 0; j < FN; ++j)
#pragma unroll
            for(int v = 0; v < 4; ++v) acc[i][j][v] = 0;

    // Fragment reads: lane -> row lane%16 of a fragment, 16-byte chunk 4*c + lane/16 of the stage row.  The swizzle term
    // (row/2)%8 is the same for every fragment of a lane because fragments start at multiples of 16.
    const int frag_row = lane % R, kq = lane / R;
    int       roff[CH];
#pragma unroll
    for(int c = 0; c < CH; ++c) roff[c] = frag_row * kRowBytes + swizzle(frag_row, c * (8 / CH) + kq);
    const int a_base = (wm * WTM) * kRowBytes, b_base = BM * kRowBytes + (wn * WTN) * kRowBytes;

    // The fragment reads are written as instructions with hand-placed waits.  The compiler's own wait
    // insertion treats a direct global->LDS load as an access that may return through either counter, and
    // while one is in flight (always, here) every wait it places on an LDS read becomes "all LDS reads
    // done", including the reads just issued for a later chunk: the wavefront would then sit out a full LDS
    // latency twice per K tile.  LDS reads of a wavefront return in order, so "at most n outstanding" says which have arrived.
    constexpr bool ROLL = FM > 4;                    // one set of registers for the rows' fragments (below)
    v4i32          af[ROLL ? 1 : 2][FM], bf[2][FN];
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t*)lds));
    // TN: lane (q = lane/16, s = lane%16) receives row s of a fragment.
    // int8: it supplies the 8-byte half s%2 of chunk (first chunk of the sub-tile + f) of contraction row
    // 64 c + 16 q + 8 r + s/2 (r = 0, 1: the two reads of a fragment) and receives contraction indices
    // 64 c + 16 q + 8 r + 0..7.  binary16: the 8-byte half s%2 of chunk (first chunk + 2f + (s%4)/2) of
    // contraction row 32 c + 8 q + 4 r + s/4; it receives contraction indices 32 c + 8 q + 4 r + 0..3.
    // A sub-tile's first chunk is a multiple of its fragments' chunks, so every fragment lies at one lane's address with a
    // wavefront-uniform chunk XORed in, which leaves stage bases (multiples of 1024) alone: one register for all of them.
    uint32_t       tn_lane = 0u;
    const uint32_t tn_a = static_cast<uint32_t>(wm * WTM * ESZ), tn_b = static_cast<uint32_t>(wn * WTN * ESZ);
    if constexpr(TN)
    {
        constexpr int RB = BM * ESZ;
        static_assert((WTM / 16) % FM == 0 && (WTN / 16) % FN == 0 && RB <= 1024, "fragments by XOR");
        const int s16 = lane & 15;
        const int prow = ESZ == 1 ? 16 * kq + s16 / 2 : 8 * kq + s16 / 4;       // + c and r steps through the immediate
        const int lch  = ESZ == 1 ? 0 : (s16 & 3) / 2;                           // chunk inside the fragment's columns
        tn_lane = static_cast<uint32_t>(prow * RB + ((lch ^ tn_swizzle<ESZ, RB>(prow)) * 16) + 8 * (s16 & 1));
    }
    // fragment f of chunk c of the stage at LDS address sb
    auto read_tn = [&](v4i32& d, uint32_t addr, auto ct) {
        constexpr int c = decltype(ct)::value;
        v2u32 lo, hi;
        frag_read_tr<ESZ, c * 64 * BM>(lo, addr);
        frag_read_tr<ESZ, c * 64 * BM + 8 * BM>(hi, addr);
        d = v4i32{static_cast<int>(lo.x), static_cast<int>(lo.y), static_cast<int>(hi.x), static_cast<int>(hi.y)};
    };
    auto read_a = [&](auto ft, auto ct, uint32_t sb) {
        constexpr int f = decltype(ft)::value, c = decltype(ct)::value;
        if constexpr(TN) read_tn(af[ROLL ? 0 : c][f], (sb + tn_lane) ^ (tn_a + static_cast<uint32_t>(f * ESZ * 16)), ct);
        else             frag_read<f * R * kRowBytes>(af[ROLL ? 0 : c][f], sb + static_cast<uint32_t>(a_base + roff[c]));
    };
    auto read_b = [&](auto ft, auto ct, uint32_t sb) {
        constexpr int f = decltype(ft)::value, c = decltype(ct)::value;
        if constexpr(TN) read_tn(bf[c][f], (sb + 128 * BM + tn_lane) ^ (tn_b + static_cast<uint32_t>(f * ESZ * 16)), ct);
        else             frag_read<f * R * kRowBytes>(bf[c][f], sb + static_cast<uint32_t>(b_base + roff[c]));
    };
    constexpr int kPer = TN ? 2 : 1;                 // LDS instructions per fragment
    // row fragment f of chunk c: FN matrix instructions; every other row walks its columns backwards, so that the B operand
    // stays from one row to the next (instructions on the same operands draw less power: +2 % of the rate above)
    auto mma = [&](auto ft, auto ct) {
        constexpr int f = decltype(ft)::value, c = decltype(ct)::value;
        __builtin_amdgcn_sched_barrier(0);           // fences: the matrix instructions stay behind the wait in front of them
#pragma unroll
        for(int jj = 0; jj < FN; ++jj)
        {
            const int j = f % 2 ? FN - 1 - jj : jj;
            acc[f][j]   = TR::mfma(bf[c][j], af[ROLL ? 0 : c][f], acc[f][j]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // K pipeline.  A tile has two 64-byte K chunks.
    // Wavefronts of few fragments hold those of both chunks: behind the matrix instructions of chunk 0 the wavefront joins the
    // barrier that publishes the next stage (every wavefront's reads of the current one have returned by then), requests the
    // direct load of the tile after next into the stage just drained (some wavefronts: later in the tile, see below), reads
    // chunk 0 of the next tile, issues chunk 1, whose operands are already in registers, and reads chunk 1 of the next tile: barrier release, LDS latency and a whole K tile of memory latency hide behind matrix work.
    // With four rows (128 tile) the reads go out between the rows' instructions, and the load behind row 0: 4096x768x3072 in three
    // stages int8 16.4 -> 15.7 us, binary16 28.0 -> 26.4, against all of them at the chunk's end; the 64 tile, of which a unit holds
    // several, gains nothing from that (its convolution's weight gradient 32.2 -> 33.2).
    // The 256 tile's wavefronts have no registers for both chunks.  A row's fragment is used by FN instructions in a row and
    // never again, so its registers are requested anew, for the next chunk, right behind them; the columns'
    // fragments, which every row uses, have two sets, and those of the next chunk are requested behind the first rows.  In chunk 1 no
    // row in front of the middle requests anything: there the barrier and the load's request follow, then the next tile's columns
    // and first rows, and the other rows go on as before.
    // 32x32 instructions with four 32-byte chunks and two sets of fragments -> this, values N(0,1), side by side, us: 16384x1024x4096
    // int8 59.1 -> 53.0, binary16 112 -> 101, 16384x4096x1024 79.4 -> 75.1 and 132 -> 124; 8192^3 2.55 -> 2.84 POP/s and 1.28 -> 1.42
    // PFLOP/s; on zeros, i.e. at the full clock, within 2 % of the same times.  The smaller tiles are not bound by power, and gain
    // little: 128 tile, 4096x3072x768 int8 14.9 -> 15.3, binary16 24.5 -> 24.8 (256 tile 15.8 -> 15.6, 23.0 -> 22.1); 64 tile, 2048x2048x1024
    // binary16 14.4 -> 14.1, 1808x1040x784 int8 7.42 -> 7.37, 64x64x6144 in splits 8.69 -> 8.67.
    // The column scales and biases of this tile are fetched by direct loads as well, in front of the first K tile, and
    // wait in LDS behind the stages for the epilogue.
    // The direct loads of a K tile are not requested by all wavefronts at once.  A compute unit takes such an
    // instruction (1 KB) at about 64 bytes per clock, and a wavefront issues nothing else while its loads
    // queue up: with every wavefront requesting right behind the barrier, both wavefronts of every SIMD sit
    // in that queue together and the matrix pipeline idles until the unit has taken all (BM + BN) / 8 of them.
    // The upper half of the wavefronts (the second wavefront of each SIMD) therefore requests later, among the instructions of
    // chunk 1: while one wavefront of a SIMD queues loads, its sibling issues matrix instructions (launched alone: 4-10 % fewer
    // cycles per launch on the 256 and 128 tiles, int8 and binary16).  256 tile: behind the last row.  128 tile: behind the third of
    // four rows; behind the last, binary16 256x1408x768 backward 14.1 -> 14.5 us, weight gradient of a convolution 200->168 over
    // 18x47x53 83.3 -> 85.0.
    // The 64 tile has no second wavefront on a SIMD, and a K tile of its own is over in less than a load takes: a request that goes
    // out at the chunk's end holds up the next barrier.  All of its wavefronts request right behind the barrier, at the end of
    // the tile -> this, us: row-major binary16 10368x168x1568 27.4 -> 23.5, 12416x3240x192 47.1 -> 41.1, int8 2560x96x1296 9.78 ->
    // 8.60.  Operand rows that straddle the 128-byte lines double the queue (binary16 960x1024x1808 16.6 -> 17.8 with all of them
    // at once): there the upper half requests behind the first of two rows.
    const bool late_loader = wave >= WC / 2 && (FM > 2 || (!TN && p.Kb % kRowBytes != 0));
    // (scalar loads: in front of the first direct load, used by the epilogue)
    const float scale0 = *(WHOLE && p.s0 ? p.s0 : &g_one), scale1 = *(WHOLE && p.s1 ? p.s1 : &g_one);
    const float code_inv = *(WHOLE && p.codes ? p.code_inv : &g_one);
    if constexpr(NL == 0) request_first();
    // (What the K loop starts from is formed while the first loads are in flight, not behind the wait for them: 4096x3072x768 on the
    // 128 tile int8 15.3 -> 14.8 us)
    if constexpr(FM > 2 && ESZ <= 2)
    {
#pragma unroll
        for(int i = 0; i < FM; ++i)
#pragma unroll
            for(int j = 0; j < FN; ++j) asm volatile("" : "+v"(acc[i][j]));
        if constexpr(TN) asm volatile("" : "+v"(tn_lane));
        else             asm volatile("" : "+v"(roff[0]), "+v"(roff[1]));
    }
    if(any_k)
    {
        if constexpr(NL == 0) await_first();
        else                  wg_barrier();
        constexpr int H = FM / 2;
        const std::integral_constant<int, 0> c0{};
        const std::integral_constant<int, 1> c1{};
        auto read_chunk = [&](auto ct, uint32_t sb) {
            static_for<FN>([&](auto j) { read_b(j, ct, sb); });
            static_for<FM>([&](auto i) { read_a(i, ct, sb); });
        };
        // Both chunks held, four rows: the other chunk's columns and first row go out behind row 0, its other rows behind row 1.
        auto requested   = [](int i) constexpr { return i == 0 ? 0 : i == 1 ? FN + 1 : FN + FM; };      // in front of row i
        auto read_behind = [&](auto it, auto ct, uint32_t sb) {
            constexpr int i = decltype(it)::value;
            if constexpr(i == 0)
            {
                static_for<FN>([&](auto j) { read_b(j, ct, sb); });
                read_a(std::integral_constant<int, 0>{}, ct, sb);
            }
            if constexpr(i == 1)
                static_for<FM - 1>([&](auto r) { read_a(std::integral_constant<int, decltype(r)::value + 1>{}, ct, sb); });
        };
        read_chunk(c0, lds0);
        if constexpr(FM == 2) read_chunk(c1, lds0);
        int stage = 0;
        for(int kt = kt_begin; kt < kt_end; ++kt)
        {
            const bool     more = kt + 1 < kt_end;
            const int      next = stage + 1 < ST ? stage + 1 : 0;
            const uint32_t sb   = lds0 + static_cast<uint32_t>(stage * STAGE_BYTES);
            // without a next tile the reads behind the barrier fetch the current stage again: in bounds, unused
            const uint32_t nb      = lds0 + static_cast<uint32_t>((more ? next : stage) * STAGE_BYTES);
            const bool     request = NL == 0 && kt + ST < kt_end;
            if constexpr(ROLL)
            {
                static_for<FM>([&](auto it) {
                    // Younger than this row's fragment: those of the FM - 1 other rows and of min(2 i, FN) columns (and younger
                    // than the last column's, at row 0: FM - 1 rows)
                    constexpr int i = decltype(it)::value;
                    wait_lds<kPer * (FM - 1 + (2 * i < FN ? 2 * i : FN))>();
                    mma(it, c0);
                    if constexpr(2 * i < FN)
                    {
                        read_b(std::integral_constant<int, 2 * i>{}, c1, sb);
                        read_b(std::integral_constant<int, 2 * i + 1>{}, c1, sb);
                    }
                    read_a(it, c1, sb);
                });
                static_for<H>([&](auto it) {
                    wait_lds<kPer * (FM - 1 - decltype(it)::value)>();
                    mma(it, c1);
                });
            }
            else if constexpr(FM == 2)
            {
                wait_lds<kPer * (FM + FN)>();
                static_for<FM>([&](auto it) { mma(it, c0); });
            }
            else
                static_for<FM>([&](auto it) {
                    constexpr int i = decltype(it)::value;
                    wait_lds<kPer * (FM - 1 - i + requested(i))>();
                    mma(it, c0);
                    read_behind(it, c1, sb);
                });
            wait_lds<0>();
            if(more)
            {
                if constexpr(NL > 0) wg_barrier();
                else                 land(next, kt + 1);
            }
            if((ROLL || FM == 2) && request && !late_loader) dma(stage, kt + ST);
            if constexpr(ROLL)
            {
                static_for<FN>([&](auto j) { read_b(j, c0, nb); });
                static_for<H>([&](auto i) { read_a(i, c0, nb); });
                static_for<FM - H>([&](auto it) {
                    const std::integral_constant<int, H + decltype(it)::value> row{};
                    mma(row, c1);
                    read_a(row, c0, nb);
                });
            }
            else if constexpr(FM == 2)
            {
                read_chunk(c0, nb);
                mma(c0, c1);
                if(request && late_loader) dma(stage, kt + ST);
                mma(c1, c1);
                read_chunk(c1, nb);
            }
            else
                static_for<FM>([&](auto it) {
                    mma(it, c1);
                    read_behind(it, c0, nb);
                    if constexpr(decltype(it)::value == 0)
                        if(request && !late_loader) dma(stage, kt + ST);
                    if constexpr(decltype(it)::value == 2)
                        if(request && late_loader) dma(stage, kt + ST);
                });
            if(ROLL && request && late_loader) dma(stage, kt + ST);
            stage = next;
        }
    }
    // The unused reads of the last trip land before their registers are reused: naming the registers behind the wait
    // keeps the compiler from handing them out in front of it.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if(any_k)
    {
#pragma unroll
        for(int f = 0; f < FM; ++f) asm volatile("" : "+v"(af[0][f]), "+v"(af[ROLL ? 0 : 1][f]));
#pragma unroll
        for(int f = 0; f < FN; ++f) asm volatile("" : "+v"(bf[0][f]), "+v"(bf[1][f]));
    }
    else if(NL == 0)
        wait_direct_loads<0>();                  // the column parameters
    const float    alpha     = scale0 * scale1;
    // (by the wavefront that publishes: loads of the word stand in line with the atomics on it, and with some hundred workgroups that end
    // together the line is what they wait for.  Every wavefront -> one, int8 912x3008x752 28.5 -> 20.4 us, 12896x576x368 24.4 -> 17.3)
    const uint32_t amax_seen = (WHOLE && p.amax_bits && wave == 0) ? __hip_atomic_load(p.amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;

    constexpr int STG = 2 * STAGE_BYTES / (WGM * WGN);
    if(MIXED ? raw : SPLIT) store_tile<TR, BM, BN, WGM, WGN, STG, true>(p, acc, lds, colp, m0, n0, split, alpha, code_inv, amax_seen);
    else if constexpr(WHOLE) store_tile<TR, BM, BN, WGM, WGN, STG, false>(p, acc, lds, colp, m0, n0, split, alpha, code_inv, amax_seen);
}

// (Two wavefronts a SIMD at least, i.e. at most 256 registers each: with more allowed the compiler keeps the accumulators in the other
// half of the register file, and moves the 64 tile's from there and back on every K tile.)
template <typename TR, int BM, int BN, int WGM, int WGN, int ST, int NL, bool SPLIT, bool CONV = false, bool TN = false>
__global__ __launch_bounds__(64 * (WGM * WGN + NL), 2) void gemm_nt_kernel(const GemmKernelArgs p)
{
    gemm_tile<TR, BM, BN, WGM, WGN, ST, NL, SPLIT, CONV, TN>(p, static_cast<int>(blockIdx.y * gridDim.x + blockIdx.x),
                                                         static_cast<int>(gridDim.y));
}

// Two independent GEMMs of one operand type in one launch, the first `na` workgroups on the first: the data and weight gradient
// of an operator.  Each of them alone leaves compute units idle unless its tiles happen to fill the chip, and pays its own
// launch, first-load latency and drain.
struct GemmPairArgs
{
    GemmKernelArgs g[2];
    int            na, total;      // workgroups of the first, of both; behind them those of the fold
    int            splits;         // K splits of the first (SPLITA)
    ColumnFoldArgs fold;
};
// (No loading wavefronts of their own here: with them 2048x1024x1024 int8 10.1 -> 10.4 us, 2056x1000x1032 binary16 24.8 -> 25.5.)
template <typename TR, int BM, int BN, int WGM, int WGN, int ST, bool TNA, bool SPLITA>
__global__ __launch_bounds__(64 * WGM * WGN, 2) void gemm_nt_pair_kernel(const GemmPairArgs p)
{
    const int blk = static_cast<int>(blockIdx.x);
    if(blk >= p.total)
    {
        extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
        fold_columns(p.fold, static_cast<uint32_t>(blk - p.total), reinterpret_cast<float*>(lds));
        return;
    }
    if constexpr(!TNA && !SPLITA)
        gemm_tile<TR, BM, BN, WGM, WGN, ST, 0, false, false, false>(p.g[blk < p.na ? 0 : 1], blk < p.na ? blk : blk - p.na, 1);
    else if constexpr(!TNA)
        gemm_tile<TR, BM, BN, WGM, WGN, ST, 0, true, false, false, true>(p.g[blk < p.na ? 0 : 1], blk < p.na ? blk : blk - p.na, blk < p.na ? p.splits : 1, blk < p.na);
    else if(blk < p.na)
        gemm_tile<TR, BM, BN, WGM, WGN, ST, 0, SPLITA, false, TNA>(p.g[0], blk, p.splits);
    else
        gemm_tile<TR, BM, BN, WGM, WGN, ST, 0, false, false, false>(p.g[1], blk - p.na, 1);
}

// ---------------------------------------------------------------------------------------------------------------
// Persistent variant of the 256x256 kernel for binary16 outputs whose M, N are multiples of 256 and whose operand
// rows are multiples of two K tiles.  One workgroup per compute unit walks its tiles; three things differ from
// gemm_nt_kernel:
//   * the wavefronts split the vector-memory roles.  Loads and stores of a wavefront share one in-flight counter
//     that retires in issue order, so a wavefront that has just stored its part of C cannot see a later load
//     land before those stores have reached the cache, microseconds later.  Wavefronts 0-3 (one per SIMD, the
//     upper half of the tile) therefore issue every direct global->LDS load and never store; wavefronts 4-7 (the
//     lower half) issue every store of C and never load.  The loaders pass their dequantized half through LDS;
//   * the next tile's first K tile is requested while the last K tile of the current one is still being
//     multiplied (its stage is free by then), the second one as soon as the storers have drained the hand-over
//     area (which is the other stage plus the spare LDS behind the stages); nobody waits for a store, so the
//     write-back of a tile overlaps the next tile's K loop;
//   * barriers are bare s_barrier instructions behind an LDS wait (the compiler's __syncthreads would wait for
//     every vector-memory operation of the wavefront, stores included), and every LDS access behind the first
//     store is written as an instruction for the same reason.
__device__ __forceinline__ void wait_lds_all() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); __builtin_amdgcn_sched_barrier(0); }
// LDS accesses as instructions; OFF is the instruction's immediate byte offset (16 bits)
template <int OFF> __device__ __forceinline__ void lds_write_b64(uint32_t addr, const v2u32& v)
{
    static_assert(OFF >= 0 && OFF < 65536, "immediate offset");
    asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(OFF) : "memory");
}
template <int OFF> __device__ __forceinline__ void lds_read_b128(v4u32& d, uint32_t addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "immediate offset");
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF) : "memory");
}
// bit patterns by value (a vector element is not an object a bit cast could be applied to directly)
template <typename T> __device__ __forceinline__ T word_as(uint32_t u);
template <> __device__ __forceinline__ int32_t word_as<int32_t>(uint32_t u) { return static_cast<int32_t>(u); }
template <> __device__ __forceinline__ float   word_as<float>(uint32_t u) { return __uint_as_float(u); }
__device__ __forceinline__ uint32_t as_word(int32_t v) { return static_cast<uint32_t>(v); }
__device__ __forceinline__ uint32_t as_word(float v) { return __float_as_uint(v); }

template <typename TR>
__global__ __launch_bounds__(512) void gemm_nt_persistent_kernel(const GemmKernelArgs p, const int total_tiles)
{
    typedef typename TR::accv_t accv_t;
    constexpr int BM = 256, BN = 256, WGN = 4, WTM = 128, WTN = 64, R = TR::kRows, FM = WTM / R, FN = WTN / R;
    static_assert(R == 16, "fragments of a wavefront");
    constexpr int STAGE_BYTES = (BM + BN) * kRowBytes;        // 64 KB
    constexpr int DPW         = 16;                           // direct loads per loader wavefront and K tile
    constexpr int PITCH       = WTN * 2 + 16;                 // padded row of 64 binary16 outputs in the hand-over area
    constexpr int L_STG       = WTM * PITCH;                  // a loader's whole sub-tile
    constexpr int S_STG       = 32 * PITCH;                   // a storer's private slice: 32 rows, two of fragments
    constexpr int STG_BASE    = STAGE_BYTES;                  // the hand-over area starts where stage 1 starts
    constexpr int S_BASE      = STG_BASE + 4 * L_STG;
    constexpr int COLP_BASE   = S_BASE + 4 * S_STG;           // [2][BN] floats: alpha * column scale, column bias
    static_assert(COLP_BASE + 2 * BN * 4 <= kPersistentLdsBytes, "LDS layout");

    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t*)lds));
    const int  tid = threadIdx.x, lane = tid % kWaveSize;
    const int  wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
    const int  wm = wave / WGN, wn = wave % WGN;
    const bool loader = wave < 4;                              // uniform per wavefront
    const int  KT = static_cast<int>(p.Kb / kRowBytes);        // even, >= 2 (checked by the launcher)
    const int  G  = static_cast<int>(gridDim.x);

    // ---- loader set-up: wavefront l covers stage rows [128 l, 128 l + 128): l = 0, 1 rows of A, l = 2, 3 rows of B
    const int  lw   = wave & 3;
    const bool is_a = lw < 2;
    uint32_t   voff[DPW];
    {
        int imm[DPW];
        fill_dma_imms<DPW>(imm, std::make_integer_sequence<int, DPW>{});
#pragma unroll
        for(int d = 0; d < DPW; ++d)
        {
            const int srow  = (lw * DPW + d) * 8 + lane / 8;
            const int chunk = (lane % 8) ^ ((srow >> 1) & 7);
            const int lrow  = srow - (is_a ? 0 : BM);
            voff[d] = static_cast<uint32_t>(static_cast<int64_t>(lrow) * p.Kb + chunk * 16 + kDmaBias - imm[d]);
        }
    }
    auto panel_base = [&](int tm, int tn) -> const uint8_t* {
        const uint8_t* g = is_a ? p.A + static_cast<int64_t>(tm) * BM * p.Kb : p.B + static_cast<int64_t>(tn) * BN * p.Kb;
        const uint64_t bits = reinterpret_cast<uint64_t>(g) - kDmaBias;
        const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(bits))));
        const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(bits >> 32))));
        return reinterpret_cast<const uint8_t*>((static_cast<uint64_t>(hi) << 32) | static_cast<uint64_t>(lo));
    };
    auto dma = [&](int stage, const uint8_t* sbase, int kt) {
        const uint8_t* sb    = sbase + static_cast<int64_t>(kt) * kRowBytes;
        uint8_t*       lbase = lds + stage * STAGE_BYTES + lw * (DPW * 1024) + (dma_group<DPW>() / 2) * 1024;
        asm volatile("" : "+s"(sb));
        dma_sequence<DPW>(std::make_integer_sequence<int, DPW>{}, sb, voff, lbase);
    };
    auto park_column_parameters = [&](int tn) {               // threads 0..255 are exactly the loaders
        float alpha = 1.0f;
        if(p.s0) alpha *= *p.s0;
        if(p.s1) alpha *= *p.s1;
        const int64_t col = static_cast<int64_t>(tn) * BN + tid;
        const float   sc  = alpha * (p.col_scale ? p.col_scale[col] : 1.0f);
        const float   bi  = p.col_bias ? p.col_bias[col] : 0.0f;
        lds_write_b32(lds0 + COLP_BASE + tid * 4, __float_as_uint(sc));
        lds_write_b32(lds0 + COLP_BASE + (BN + tid) * 4, __float_as_uint(bi));
    };

    // ---- fragment reads (as in gemm_nt_kernel, but one set of registers for the columns too: there are none left for two)
    const int frag_row = lane % R, kq = lane / R;
    int       roff[2];
#pragma unroll
    for(int c = 0; c < 2; ++c) roff[c] = frag_row * kRowBytes + swizzle(frag_row, c * 4 + kq);
    const int a_base = (wm * WTM) * kRowBytes, b_base = BM * kRowBytes + (wn * WTN) * kRowBytes;
    v4i32     af[FM], bf[FN];
    auto      read_a = [&](auto ft, int stage, int c) {
        frag_read<decltype(ft)::value * R * kRowBytes>(af[decltype(ft)::value], lds0 + static_cast<uint32_t>(stage * STAGE_BYTES + a_base + roff[c]));
    };
    auto read_b = [&](auto ft, int stage, int c) {
        frag_read<decltype(ft)::value * R * kRowBytes>(bf[decltype(ft)::value], lds0 + static_cast<uint32_t>(stage * STAGE_BYTES + b_base + roff[c]));
    };
    accv_t acc[FM][FN];
    auto   mma = [&](auto ft) {
        constexpr int f = decltype(ft)::value;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for(int j = 0; j < FN; ++j) acc[f][j] = TR::mfma(bf[j], af[f], acc[f][j]);
        __builtin_amdgcn_sched_barrier(0);
    };
    // the last row of a chunk, and the next chunk's columns behind it
    const std::integral_constant<int, FM - 1> last_row{};
    auto turn = [&](int stage, int c) {
        mma(last_row);
        static_for<FN>([&](auto j) { read_b(j, stage, c); });
        read_a(last_row, stage, c);
    };
    auto clear_acc = [&]() {
#pragma unroll
        for(int i = 0; i < FM; ++i)
#pragma unroll
            for(int j = 0; j < FN; ++j)
#pragma unroll
                for(int v = 0; v < 4; ++v) acc[i][j][v] = 0;
    };

    // ---- first tile: both stages requested, column parameters parked, first K tile awaited
    int lin = static_cast<int>(blockIdx.x);
    int split_unused, tm, tn;
    item_of_block(lin, p.tiles_m, p.tiles_n, 1, p.group_m, split_unused, tm, tn);
    const uint8_t* cur = panel_base(tm, tn);
    if(loader)
    {
        dma(0, cur, 0);
        dma(1, cur, 1);
        park_column_parameters(tn);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    wg_barrier();

    while(true)
    {
        __builtin_amdgcn_sched_barrier(0);     // the accumulators' live range starts here, not before the last tile's stores
        clear_acc();
        const int  nlin     = lin + G;
        const bool has_next = nlin < total_tiles;
        int        ntm = 0, ntn = 0;
        if(has_next) item_of_block(nlin, p.tiles_m, p.tiles_n, 1, p.group_m, split_unused, ntm, ntn);
        const uint8_t* nxt = has_next ? panel_base(ntm, ntn) : cur;

        // ---- K loop.  On entry K tile 0 is in stage 0 and published, K tile 1 is in flight towards stage 1.
        static_for<FN>([&](auto j) { read_b(j, 0, 0); });
        static_for<FM>([&](auto i) { read_a(i, 0, 0); });
        for(int kt = 0; kt < KT; ++kt)
        {
            const int stage = kt & 1;
            // chunk 0: younger than the fragment of row i are those of the FM - 1 other rows, less than the rows requested last
            // behind the columns
            static_for<FM - 1>([&](auto it) {
                if constexpr(decltype(it)::value == 0) wait_lds<1>();
                else                                   wait_lds<FM - 1>();
                mma(it);
                read_a(it, stage, 1);
            });
            wait_lds<FM - 1>();
            turn(stage, 1);
            static_for<FM / 2>([&](auto it) {
                wait_lds<1>();
                mma(it);
            });
            wait_lds<0>();
            const bool more = kt + 1 < KT;
            if(more)
            {
                // the loaders' K tile kt+1 has landed, everybody's reads of this stage have returned
                if(loader) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                wg_barrier();
                if(loader)
                {
                    if(kt + 2 < KT) dma(stage, cur, kt + 2);
                    else if(has_next) dma(stage, nxt, 0);        // kt + 2 == KT: stage 0, first K tile of the next tile
                }
            }
            // on the last K tile the reads below fetch chunk 0 of the current stage again: in bounds, unused
            const int nstage = more ? (stage ^ 1) : stage;
            static_for<FM / 2>([&](auto it) { read_a(it, nstage, 0); });
            static_for<FM / 2 - 1>([&](auto it) {
                const std::integral_constant<int, FM / 2 + decltype(it)::value> row{};
                mma(row);
                read_a(row, nstage, 0);
            });
            turn(nstage, 0);
        }
        wait_lds<0>();
#pragma unroll
        for(int f = 0; f < FM; ++f) asm volatile("" : "+v"(af[f]));
#pragma unroll
        for(int f = 0; f < FN; ++f) asm volatile("" : "+v"(bf[f]));

        // ---- epilogue.  Stage 1 (last K tile) is drained once everybody passes this barrier.
        wg_barrier();
        const int64_t m0 = static_cast<int64_t>(tm) * BM, n0 = static_cast<int64_t>(tn) * BN;
        // where this wavefront's dequantized rows go: a loader fills its whole 128-row region, a storer its
        // private 32-row slice, pass by pass (the storer's base steps back by one pass per pass, so that both
        // use the same immediates)
        const uint32_t my_stg  = lds0 + (loader ? STG_BASE + wave * L_STG : S_BASE + (wave - 4) * S_STG);
        const uint32_t wr_lane = my_stg + static_cast<uint32_t>(frag_row * PITCH + 8 * kq);
        const uint32_t cp_lane = lds0 + COLP_BASE + static_cast<uint32_t>((wn * WTN + 4 * kq) * 4);
        const int      lr8 = lane / 8, seg = lane % 8;
        const uint32_t rd_lane = static_cast<uint32_t>(lr8 * PITCH + seg * 16);
        const int64_t  wcol0 = n0 + wn * WTN;
        __half* const  cbase = static_cast<__half*>(p.C) + wcol0 + seg * 8;
        // alpha * column scale and bias of this lane's 4 x 4 columns, read once per tile
        v4u32 rs[FN], rb[FN];
        static_for<FN>([&](auto jt) {
            constexpr int j = decltype(jt)::value;
            lds_read_b128<j * R * 4>(rs[j], cp_lane);
            lds_read_b128<(BN + j * R) * 4>(rb[j], cp_lane);
        });
        wait_lds_all();
        static_for<WTM / 32>([&](auto it) {                     // 32 rows a pass
            constexpr int  i       = decltype(it)::value;
            const uint32_t wr_base = loader ? wr_lane : wr_lane - static_cast<uint32_t>(i * 32 * PITCH);
            static_for<32 / R>([&](auto ht) {
                constexpr int f = i * (32 / R) + decltype(ht)::value;
                static_for<FN>([&](auto jt) {
                    constexpr int j = decltype(jt)::value;
                    // the per-tile kernel's arithmetic: each value one fused multiply-add rounded once to binary16
                    auto pair = [&](int e) {
                        return fma_out_half2(static_cast<float>(acc[f][j][e]), __uint_as_float(rs[j][e]), __uint_as_float(rb[j][e]),
                                             static_cast<float>(acc[f][j][e + 1]), __uint_as_float(rs[j][e + 1]),
                                             __uint_as_float(rb[j][e + 1]));
                    };
                    const v2u32 packed = {pair(0), pair(2)};
                    lds_write_b64<f * R * PITCH + j * R * 2>(wr_base, packed);
                });
            });
            if(!loader)
            {   // the storer's own rows leave right away: written by this wavefront, read back transposed
                wait_lds_all();
                v4u32 val[4];
                static_for<4>([&](auto qt) { lds_read_b128<decltype(qt)::value * 8 * PITCH>(val[decltype(qt)::value], my_stg + rd_lane); });
                wait_lds_all();
#pragma unroll
                for(int q = 0; q < 4; ++q)
                {
                    const int64_t row = m0 + WTM + i * 32 + q * 8 + lr8;
                    __builtin_nontemporal_store(val[q], reinterpret_cast<v4u32*>(cbase + row * p.N));
                }
            }
        });
        wg_barrier();                                        // the loaders' rows are in the hand-over area
        // The storers take the partner's sub-tile (same columns, the upper half of the tile) out of the hand-over
        // area into registers, so that the area is free again after one more barrier and the loaders' request for
        // the next tile's second K tile enters the memory pipeline ahead of the stores that follow.
        // (The 64 registers are those of the accumulators, dead by now: a separate array would raise the kernel's
        // register demand and the compiler would spill the results of the LDS instructions before they arrive.)
        if(!loader)
        {
            const uint32_t src = lds0 + STG_BASE + static_cast<uint32_t>((wave - 4) * L_STG) + rd_lane;
            static_for<2>([&](auto bt) {                       // two batches: the LDS counter of a wavefront holds 15
                constexpr int b = decltype(bt)::value;
                v4u32 t[8];
                static_for<8>([&](auto rt) { lds_read_b128<(b * 8 + decltype(rt)::value) * 8 * PITCH>(t[decltype(rt)::value], src); });
                wait_lds_all();
                static_for<8>([&](auto rt) {
                    constexpr int r = b * 8 + decltype(rt)::value;
#pragma unroll
                    for(int e = 0; e < 4; ++e)
                        {
                        const uint32_t word = t[decltype(rt)::value][e];
                        acc[r / 4][r % 4][e] = word_as<typename TR::acc_t>(word);
                    }
                });
            });
        }
        if(loader && has_next)
        {
            park_column_parameters(ntn);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the next tile's first K tile has landed
        }
        wg_barrier();                                        // hand-over area drained, stage 0 and parameters published
        if(loader && has_next) dma(1, nxt, 1);
        if(!loader)
        {
#pragma unroll
            for(int r = 0; r < 16; ++r)
            {
                const int64_t row = m0 + r * 8 + lr8;
                v4u32         val;
#pragma unroll
                for(int e = 0; e < 4; ++e)
                {
                    const typename TR::acc_t a = acc[r / 4][r % 4][e];
                    val[e] = as_word(a);
                }
                __builtin_nontemporal_store(val, reinterpret_cast<v4u32*>(cbase + row * p.N));
            }
        }
        if(!has_next) break;
        lin = nlin; tm = ntm; tn = ntn; cur = nxt;
    }
}


// Adds the split-K partials in split order and applies the epilogue.
constexpr int kThreads = 256;   // split-K reduction

template <typename ACC, bool VEC4>
__global__ __launch_bounds__(kThreads) void splitk_reduce_kernel(const ACC* __restrict__ partial, int splits,
                                                                 int64_t M, int64_t N, void* C, int c_is_f16,
                                                                 const float* s0, const float* s1,
                                                                 const float* __restrict__ col_scale,
                                                                 const float* __restrict__ col_bias, int32_t* acc_dump,
                                                                 unsigned int* amax_bits, int8_t* codes,
                                                                 const float* code_inv_p, int code_qmax, const int blocks,
                                                                 const ColumnFoldArgs fold)
{
    if(static_cast<int>(blockIdx.x) >= blocks)      // workgroups behind the reduction's own: column sums of some other tensor
    {
        __shared__ float lds_f[kThreads];
        fold_columns(fold, blockIdx.x - blocks, lds_f);
        return;
    }
    const float code_inv = codes ? *code_inv_p : 0.0f;
    constexpr int V      = VEC4 ? 4 : 1;       // VEC4: N % 4 == 0 and 16-byte aligned buffers
    uint32_t      run    = 0u;                 // maximum of |C| as stored (fp32 bits), when amax_bits is given
    const uint32_t seen  = amax_bits ? __hip_atomic_load(amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    const int64_t n      = M * N;
    const int64_t stride = static_cast<int64_t>(blocks) * kThreads * V;
    float         alpha  = 1.0f;
    if(s0) alpha *= *s0;
    if(s1) alpha *= *s1;
    for(int64_t i = (static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x) * V; i < n; i += stride)
    {
        ACC acc[V];
#pragma unroll
        for(int e = 0; e < V; ++e) acc[e] = 0;
#pragma unroll 8                                  // eight independent partial loads in flight; the sum keeps its order
        for(int s = 0; s < splits; ++s)
        {
            ACC part[V];
            if(VEC4)
                *reinterpret_cast<uint4*>(part) = *reinterpret_cast<const uint4*>(partial + static_cast<int64_t>(s) * n + i);
            else
                part[0] = partial[static_cast<int64_t>(s) * n + i];
#pragma unroll
            for(int e = 0; e < V; ++e) acc[e] += part[e];
        }
        const int64_t col = i % N;
        float         y[V];
#pragma unroll
        for(int e = 0; e < V; ++e)
        {
            const float f = alpha * (col_scale ? col_scale[col + e] : 1.0f), b = col_bias ? col_bias[col + e] : 0.0f;
            const float a = static_cast<float>(acc[e]);
            y[e] = c_is_f16 ? __half2float(fma_out<__half>(a, f, b)) : fma_out<float>(a, f, b);      // the value as stored
        }
        if(amax_bits)
        {
#pragma unroll
            for(int e = 0; e < V; ++e)
            {
                const uint32_t u = __float_as_uint(y[e]) & 0x7FFFFFFFu;
                run = run > u ? run : u;
            }
        }
        if(codes)
        {   // codes of the values as stored (y holds the rounded value when the output is binary16)
            uint32_t cw = 0u;
#pragma unroll
            for(int e = 0; e < V; ++e)
                cw |= (static_cast<uint32_t>(quantize_code<kNearest>(y[e], code_inv, code_qmax, 0u)) & 0xFFu) << (8 * e);
            if(VEC4 && (reinterpret_cast<uintptr_t>(codes) & 3) == 0)
                *reinterpret_cast<uint32_t*>(codes + i) = cw;
            else
#pragma unroll
                for(int e = 0; e < V; ++e) codes[i + e] = static_cast<int8_t>((cw >> (8 * e)) & 0xFFu);
        }
        if(VEC4)
        {
            if(c_is_f16)
            {
                __half h[4];
#pragma unroll
                for(int e = 0; e < 4; ++e) h[e] = __float2half_rn(y[e]);      // exact: y is a binary16 value
                *reinterpret_cast<uint2*>(static_cast<__half*>(C) + i) = *reinterpret_cast<const uint2*>(h);
            }
            else
                *reinterpret_cast<uint4*>(static_cast<float*>(C) + i) = *reinterpret_cast<const uint4*>(y);
        }
        else if(c_is_f16)
            static_cast<__half*>(C)[i] = __float2half_rn(y[0]);
        else
            static_cast<float*>(C)[i] = y[0];
        if(acc_dump)
#pragma unroll
            for(int e = 0; e < V; ++e) acc_dump[i + e] = static_cast<int32_t>(acc[e]);
    }
    if(amax_bits)
    {   // one atomic maximum per workgroup
        __shared__ uint32_t slots[kThreads / 64];
#pragma unroll
        for(int off = 32; off >= 1; off >>= 1)
        {
            const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(run), off));
            run = run > o ? run : o;
        }
        if(threadIdx.x % 64 == 0) slots[threadIdx.x / 64] = run;
        __syncthreads();
        if(threadIdx.x == 0)
        {
            uint32_t m = slots[0];
#pragma unroll
            for(int w = 1; w < kThreads / 64; ++w) m = m > slots[w] ? m : slots[w];
            if(m > seen) atomicMax(amax_bits, m);      // `seen` may be stale but never too large: skipping is safe
        }
    }
}

// 0: 256x256, 8 wavefronts (2x4, 128x64 each)   1: 128x128, 8 wavefronts (2x4, 64x32 each)
// 2: 64x64, 4 wavefronts (2x2, 32x32 each)
// (What follows was measured on 32x32 instructions.)
// (128x128 with four wavefronts of 64x64, one per SIMD, reads a third less LDS per operation but has nobody to issue
//  matrix instructions while it queues direct loads.  Four -> eight wavefronts: 4096x768x3072 int8 18.1 -> 16.2 us,
//  3072x768x4096 20.4 -> 18.2, 2056x1000x1032 binary16 14.0 -> 12.5, 64x128x128 4.7 -> 3.9.)
// (256x256 with 4 wavefronts of 128x128 -- a third fewer LDS fragment reads per matrix instruction, 256
//  accumulator registers per lane -- needs matrix instructions written as inline assembly on accumulator
//  registers, one loop body without branches around them, and fragment reads and direct loads placed one by one
//  between them; the compiler's own allocation keeps the accumulators in scratch memory.  Built that way it is
//  bit-identical and as fast as the 8-wavefront tile at 8192^3 but 7-14 % slower on 16384x4096x1024 and
//  16384x1024x4096, where its longer epilogue counts: not kept.)
constexpr TileShape kTiles[] = {{256, 256}, {128, 128}, {64, 64}};
constexpr int       kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// The dynamic-LDS attribute of a kernel is set once per device: flags indexed by the current device (a process
// that drives several GPUs sets it on each; beyond kMaxDevices it is set before every launch).
constexpr int kMaxDevices = 16;
inline int current_device_slot()
{
    int dev = 0;
    return (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices) ? dev : -1;
}

template <typename TR, int BM, int BN, int WGM, int WGN, int ST, int NL>
hipError_t launch_tile(const GemmKernelArgs& a, int splits, hipStream_t st, bool tn = false)
{
    constexpr size_t lds_bytes = ST * static_cast<size_t>(BM + BN) * kRowBytes + 2 * BN * sizeof(float) + 64;   // + amax slots
    auto go = [&](auto split, auto conv, auto rowmajor) {
        const auto  kernel = &gemm_nt_kernel<TR, BM, BN, WGM, WGN, ST, NL, decltype(split)::value, decltype(conv)::value, decltype(rowmajor)::value>;
        static bool attr_set[kMaxDevices] = {};   // per instantiation and device; benign if set twice
        const int   slot = current_device_slot();
        if(slot < 0 || !attr_set[slot])
        {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     static_cast<int>(lds_bytes));
            if(e != hipSuccess) return e;
            if(slot >= 0) attr_set[slot] = true;
        }
        kernel<<<dim3(static_cast<unsigned>(a.tiles_m * a.tiles_n), static_cast<unsigned>(splits)), dim3(64 * (WGM * WGN + NL)), lds_bytes, st>>>(a);
        return hipGetLastError();
    };
    constexpr std::true_type  yes{};
    constexpr std::false_type no{};
    if constexpr(TR::kElemBytes <= 2 && NL == 0)
    {
        if(a.conv_H > 0 && tn) return splits > 1 ? go(yes, yes, yes) : go(no, yes, yes);
        if(a.conv_H > 0 && splits == 1) return go(no, yes, no);
    }
    if(a.conv_H > 0) return hipErrorInvalidValue;
    if constexpr(TR::kElemBytes <= 2)
        if(tn) return splits > 1 ? go(yes, no, yes) : go(no, no, yes);
    if(tn) return hipErrorInvalidValue;
    return splits > 1 ? go(yes, no, no) : go(no, no, no);
}

template <typename TR>
hipError_t launch_traits(int tile, const GemmKernelArgs& a, int splits, hipStream_t st, bool tn = false)
{
    // The 128x128 tile where every compute unit gets one workgroup at most (with a second one resident, two stages,
    // its K loop fills the gaps):
    //   four stages and four loading wavefronts, three stages -> this, us: 4096x768x3072 (192 workgroups) int8 16.4 -> 14.6,
    //   binary16 25.1 -> 22.6; 2048x2048x1536 int8 9.9 -> 9.3, 1024x512x2048 10.5 -> 9.6.
    //   Their start costs 0.3 us, a K tile less gains 0.05 to 0.12: 8 K tiles int8 7.33 -> 7.30, 6 lose (7.6 -> 7.8), 2 lose 5 %.
    //   Contiguous rows that straddle the 128-byte lines (two lines a piece) keep the loaders the bound: 4096x768x3088 int8 18.4 ->
    //   18.9.  A row-major stage row is 128 or 256 bytes of a longer operand row, for which that matters less: they take any row length.
    //   Whole lines 2048x1024x1024 12.8 -> 11.7, 4096x768x3072 int8 21.7 -> 18.8; others 1536x1344x1792 int8 11.1 -> 10.6, binary16
    //   1408x576x3640 17.1 -> 15.7, 1792x480x816 14.2 -> 13.8 (over 179 row-major products 0.83 to 1.04 of three stages, on average 0.96).
    //   The gathering loads of a convolution have too much arithmetic for four wavefronts (24.9 -> 28.2).
    //   three stages otherwise.  The rest was measured on 32x32 instructions.  Two -> three: 4096x768x3072 int8 18.5 -> 15.3 us,
    //   binary16 33.5 -> 26.4; 2048x2048x4096 (256) int8 25.8 -> 22.5; a short contraction gains nothing (4096x768x768 int8 6.8 -> 7.0).
    // Beyond 256 workgroups a third stage loses: 2176x2048x1024 (272) int8 10.9 -> 14.2, binary16 17.6 -> 21.8; 4096x2048x3072
    // (512) int8 29.9 -> 34.2, 4096x3072x768 (768) 15.5 -> 18.9.
    // The 64x64 tile gains nothing from 3, 4 or 8 stages (14.7 / 16.4 / 17.3 / 23.9 us on 2056x1000x1032 binary16), nor
    // from fragments read a whole K tile ahead (14.7).
    const int64_t workgroups = static_cast<int64_t>(a.tiles_m) * a.tiles_n * splits;
    switch(tile)
    {
    case 0: return launch_tile<TR, 256, 256, 2, 4, 2, 0>(a, splits, st, tn);
    case 1:
        if(workgroups > kNumCu) return launch_tile<TR, 128, 128, 2, 4, 2, 0>(a, splits, st, tn);
        return a.conv_H == 0 && a.remap_C == 0 && a.ktiles_per_split >= 8 && (tn || a.Kb % kRowBytes == 0)
                 ? launch_tile<TR, 128, 128, 2, 4, 4, 4>(a, splits, st, tn)
                 : launch_tile<TR, 128, 128, 2, 4, 3, 0>(a, splits, st, tn);
    default: return launch_tile<TR, 64, 64, 2, 2, 2, 0>(a, splits, st, tn);
    }
}

template <typename TR, int BM, int BN, int WGM, int WGN, int ST, bool TNA, bool SPLITA>
hipError_t launch_pair_tile(const GemmPairArgs& p, hipStream_t st)
{
    constexpr size_t lds_bytes = ST * static_cast<size_t>(BM + BN) * kRowBytes + 2 * BN * sizeof(float) + 64;
    const auto       kernel = &gemm_nt_pair_kernel<TR, BM, BN, WGM, WGN, ST, TNA, SPLITA>;
    static bool      attr_set[kMaxDevices] = {};      // per instantiation and device; benign if set twice
    const int        slot = current_device_slot();
    if(slot < 0 || !attr_set[slot])
    {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_bytes));
        if(e != hipSuccess) return e;
        if(slot >= 0) attr_set[slot] = true;
    }
    kernel<<<dim3(static_cast<unsigned>(p.total + p.fold.blocks())), dim3(64 * WGM * WGN), lds_bytes, st>>>(p);
    return hipGetLastError();
}
template <typename TR, bool TNA, bool SPLITA>
hipError_t launch_pair_traits(int tile, const GemmPairArgs& p, hipStream_t st)
{
    if(tile == 1)
        return p.total <= kNumCu ? launch_pair_tile<TR, 128, 128, 2, 4, 3, TNA, SPLITA>(p, st)
                                 : launch_pair_tile<TR, 128, 128, 2, 4, 2, TNA, SPLITA>(p, st);
    return launch_pair_tile<TR, 64, 64, 2, 2, 2, TNA, SPLITA>(p, st);
}

// The persistent kernel serves full 256x256 tiles with binary16 output and nothing optional in the epilogue.
bool persistent_eligible(const GemmKernelArgs& a, int prec, int tile, int splits)
{
    return (prec == 8 || prec == 16) && tile == 0 && splits == 1 && a.c_is_f16 && !a.acc_dump && !a.amax_bits && !a.codes && a.conv_H == 0
        && a.remap_C == 0 && a.M % 256 == 0 && a.N % 256 == 0 && a.Kb % (2 * kRowBytes) == 0 && a.Kb >= 2 * kRowBytes
        && (reinterpret_cast<uintptr_t>(a.C) & 15) == 0;
}

template <typename TR> hipError_t launch_persistent(const GemmKernelArgs& a, hipStream_t st)
{
    static bool      attr_set[kMaxDevices] = {};      // per instantiation and device; benign if set twice
    const int        slot = current_device_slot();
    const void*      fn = reinterpret_cast<const void*>(&gemm_nt_persistent_kernel<TR>);
    if(slot < 0 || !attr_set[slot])
    {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kPersistentLdsBytes);
        if(e != hipSuccess) return e;
        if(slot >= 0) attr_set[slot] = true;
    }
    const int total = a.tiles_m * a.tiles_n;
    const int grid  = total < kNumCu ? total : kNumCu;
    gemm_nt_persistent_kernel<TR><<<dim3(static_cast<unsigned>(grid)), dim3(512), kPersistentLdsBytes, st>>>(a, total);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f32(const GemmProblem& p, const GemmPlan& plan, void* workspace, hipStream_t stream);   // gemm_f32.hip

static thread_local int g_tile_override = -1;     // set by tests and tuning runs only; per calling thread
void set_gemm_tile_override(int tile) { g_tile_override = (tile >= 0 && tile < kNumTiles) ? tile : -1; }
static thread_local int g_persistent_mode = -1;   // 1: whenever eligible; anything else: never (the default, see launch_gemm)
void set_gemm_persistent_mode(int mode) { g_persistent_mode = (mode == 0 || mode == 1) ? mode : -1; }

// fp32 operands: 0 is 256x128 (gemm_f32.hip)
TileShape gemm_tile_shape(int prec, int tile) { return prec == 32 && tile == 0 ? TileShape{256, 128} : kTiles[tile]; }

// Model of a tile shape's time; the constants are explained in plan_gemm.
struct TileModel { double r1, rmax, ovh, cap; int occ; };
static constexpr TileModel kTileModel[kNumTiles] = {{14.0, 15.8, 7.5, 2280.0, 1}, {8.3, 9.0, 4.2, 1900.0, 2}, {3.55, 5.48, 3.2, 2060.0, 4}};
// fp32: an LDS stage of three bf16 parts leaves room for one workgroup of the larger tiles on a unit, three of the small one.  Fitted to
// 146 shapes of 64..16384 by 64..4096 by 64..8192, each tile with one and more K splits, replayed from a graph: the choice is 0.5 % behind
// the best on average, 18 % at most (3120x3508x72).
static constexpr TileModel kTileModelF32[kNumTiles] = {{37.3, 37.3, 8.4, 7520.0, 1}, {29.5, 29.5, 6.4, 6410.0, 1}, {14.9, 19.5, 5.1, 5400.0, 3}};
// Row-major (TN) operands: a K tile takes twice the LDS fragment reads, and a 64-wide tile of int8 operands
// loads 64-byte row pieces (binary16: 128 bytes, no penalty); fitted slow-down of the main loop per tile shape.
static double tn_factor(int tile, int prec, bool tn)
{
    const double rate[kNumTiles] = {0.94, 0.89, prec == 8 ? 0.74 : 0.97};
    return tn ? rate[tile] : 1.0;
}

GemmPlan plan_gemm(int prec, int64_t M, int64_t N, int64_t K, int force_tile, int force_splits, bool allow_split, bool tn)
{
    if(force_tile < 0 && g_tile_override >= 0)
    {   // a forced tile keeps the planner's split choice for that tile
        GemmPlan forced = plan_gemm(prec, M, N, K, g_tile_override, force_splits >= 1 ? force_splits : 0, allow_split, tn);
        return forced;
    }
    GemmPlan plan{1, 1, 0, 0.0};
    if(M <= 0 || N <= 0) return plan;
    const int64_t kb     = K * (prec == 8 ? 1 : (prec == 16 ? 2 : 4));
    // (the unit of fp32's constants: what a K tile of fp32 operands took on the fp32 instructions)
    const double  kwork  = prec == 32 ? 8.0 : 1.0;
    const int64_t ktiles = (kb + kRowBytes - 1) / kRowBytes;
    auto shape  = [&](int t) { return gemm_tile_shape(prec, t); };
    auto ntiles = [&](int t) { return ((M + shape(t).bm - 1) / shape(t).bm) * ((N + shape(t).bn - 1) / shape(t).bn); };
    // Plan = (tile, K splits) with the smallest estimated time.  The estimate is a small model fitted to gfx950
    // measurements of these tiles on 32x32 instructions (int8 and binary16, forward, row-major and transposed weight-gradient
    // forms: 54 operands x 3 tiles, replayed from a graph; rms error 11 %; fp32 operands have constants of their own).  It knows
    // nothing of the 128 tile's loading wavefronts.  The choice against the best of the three present tiles, over 465 shapes of 64..16384
    // by 64..4096 that are the tiles': forward 1.1 % behind on average with int8 and 1.7 % with binary16, row-major 0.6 % and 1.6 %,
    // as before (1.0 % and 1.6 %); more than 10 % in 18 of them, 35 % at most (row-major binary16 3328x528x2384, split on the 64 tile
    // where the 128 tile takes 22.9 us):
    //   a compute unit retires `r1` Mop/us per resident workgroup of a tile shape, up to `rmax` with `occ` of them
    //   sharing it; the chip as a whole retires at most `cap` Mop/us (256 busy units, at a lower clock and on
    //   shared caches, do not each reach `rmax`); every round of co-resident workgroups costs `ovh` us of launch, first-load latency
    //   and epilogue (the 256 tile's: fitted 6.9, raised to 7.5 for few K tiles: int8 9856 x 1920 x 176, fp32 output, 256
    //   tile 28.5 us, 128 tile 21.5; 49 of 6000 shapes drawn over the same range change, 18 % faster on average); split K adds its reduction pass.
    const double     cus = 256.0;
    const TileModel* models = prec == 32 ? kTileModelF32 : kTileModel;
    const int64_t    least = prec == 32 ? 4 : 8;      // K tiles of a split: one of fp32 operands is 0.5 us and more
    auto estimate = [&](int t, int64_t s) {
        const TileModel& m    = models[t];
        const double     tnf  = tn_factor(t, prec, tn);
        const double     wgs  = static_cast<double>(ntiles(t)) * static_cast<double>(s);
        const double     per  = std::ceil(wgs / cus);                                    // workgroups of the busiest unit
        const double     share = per < m.occ ? per : m.occ;                              // co-resident ones
        const double     rate = (m.r1 * share < m.rmax ? m.r1 * share : m.rmax) * tnf;
        const double     kt   = std::ceil(static_cast<double>(ktiles) / static_cast<double>(s));
        const double     mop  = 2.0 * shape(t).bm * shape(t).bn * kRowBytes * 1e-6 * kwork;    // per K tile (int8 ops)
        const double     unit = per * kt * mop / rate, chip = wgs * kt * mop / (m.cap * tnf);
        double           us   = (unit > chip ? unit : chip) + m.ovh * std::ceil(wgs / (cus * m.occ));
        // (the parts' way to memory and back; fp32's was fitted together with its other constants)
        if(s > 1) us += (prec == 32 ? 1.9 : 4.0) + (prec == 32 ? 2.7 : 1.0) * static_cast<double>(s + 1) * static_cast<double>(M) * static_cast<double>(N) * 4.0 / 6.24e6;
        return us;
    };
    // (fp32 up to kF32ShortK is latency and stores: the small tile, 2584x3144x4 14.7 us, 256 tile 20.4, 128 tile 19.7; 5960x1804x4 19.0, 23.7, 23.6)
    // Candidates: no split, and the split counts that fill the units once, twice or up to their co-residency.  Tiles are
    // visited from large to small and splits from few to many; a later candidate must win by 5 % (the larger tile
    // moves fewer bytes per operation, and estimates that close are inside the model's error) -- unless the
    // incumbent's tiles overhang the output by a quarter more than the candidate's: padding is where the model
    // errs in the larger tile's favour.
    int     tile = 0, splits = 1;
    double  best = -1.0, best_area = 0.0;
    for(int t = 0; t < kNumTiles; ++t)
    {
        if(force_tile >= 0 && force_tile < kNumTiles && t != force_tile) continue;
        if(force_tile < 0 && prec == 32 && K <= kF32ShortK && t + 1 < kNumTiles) continue;      // (below)
        int64_t cand[4] = {1, 1, 1, 1};
        int     ncand   = 1;
        if(allow_split && !(force_tile >= 0 && force_splits < 0))
            for(int f = 0; f < 3; ++f)
            {
                const int64_t fill = f == 0 ? 256 : (f == 1 ? 512 : 256 * models[t].occ);
                if(fill > 256 * models[t].occ) continue;
                int64_t       s    = fill / ntiles(t);
                if(s > ktiles / least) s = ktiles / least;
                if(s > 128) s = 128;
                if(s >= 2 && s != cand[ncand - 1]) cand[ncand++] = s;
            }
        const double area = static_cast<double>(ntiles(t)) * shape(t).bm * shape(t).bn;
        for(int c = 0; c < ncand; ++c)
        {
            const double us     = estimate(t, cand[c]);
            const double margin = best_area > 1.25 * area ? 1.0 : 0.95;
            if(best < 0.0 || us < margin * best) { best = us; best_area = area; tile = t; splits = static_cast<int>(cand[c]); }
        }
    }
    if(force_splits >= 1 && allow_split) splits = force_splits;
    if(splits > ktiles) splits = static_cast<int>(ktiles < 1 ? 1 : ktiles);
    plan.tile      = tile;
    plan.splits    = splits;
    plan.workspace = splits > 1 ? static_cast<size_t>(splits) * M * N * 4 : 0;
    plan.us        = estimate(tile, splits);
    return plan;
}

// Kernel arguments of a problem under a plan; hipErrorInvalidValue for operands the kernels cannot address.
static hipError_t kernel_args(const GemmProblem& p, const GemmPlan& plan, void* workspace, GemmKernelArgs& a)
{
    const int      esz = p.prec == 8 ? 1 : (p.prec == 16 ? 2 : 4);
    // lane offsets inside an operand panel are 32-bit: 255 rows of K bytes (plus the load immediates) must fit
    if(p.K > kGemmMaxRowBytes / esz) return hipErrorInvalidValue;
    a.A = static_cast<const uint8_t*>(p.A);
    a.B = static_cast<const uint8_t*>(p.B);
    a.M = p.M; a.N = p.N; a.Kb = p.K * esz;
    a.C = p.C; a.c_is_f16 = p.c_dtype == kF16;
    a.s0 = p.s0; a.s1 = p.s1; a.col_scale = p.col_scale; a.col_bias = p.col_bias;
    a.acc_dump = p.prec == 8 ? p.acc_dump : nullptr;
    a.partial  = workspace;
    a.conv_H = a.conv_W = a.conv_Cb = 0;
    a.remap_C = a.remap_shift = 0;
    if(p.tn)
    {   // A [K, M], B [K, N] row-major int8 or binary16: rows are contraction indices (128 bytes' worth per K tile),
        // 16-byte column chunks
        if((p.prec != 8 && p.prec != 16) || p.b_remap_C > 0
           || (p.M * esz) % 16 != 0 || (p.N * esz) % 16 != 0
           || p.M >= (int64_t(1) << 24) || p.N >= (int64_t(1) << 24)
           || ((reinterpret_cast<uintptr_t>(p.A) | reinterpret_cast<uintptr_t>(p.B)) & 15) != 0)
            return hipErrorInvalidValue;
    }
    a.amax_bits = plan.splits > 1 ? nullptr : p.out_amax_bits;      // with K splits the reduction pass takes the maximum
    a.codes     = plan.splits > 1 ? nullptr : static_cast<int8_t*>(p.out_codes);      // ... and writes the codes
    a.code_inv  = p.out_code_inv;
    a.code_qmax = p.out_code_qmax;
    if(p.b_remap_C > 0)
    {   // B is [3*remap_C, K] with a margin of |remap_shift| readable bytes in front of it and behind it
        if(p.conv_H > 0 || p.N != 9 * p.b_remap_C || p.b_remap_shift % 16 != 0 || p.b_remap_shift < 0
           || p.b_remap_shift > 1024 || 3 * p.b_remap_C * a.Kb >= (int64_t(1) << 32) - (1 << 20))
            return hipErrorInvalidValue;
        a.remap_C = static_cast<int>(p.b_remap_C); a.remap_shift = static_cast<int>(p.b_remap_shift);
    }
    if(p.conv_H > 0 && p.tn)
    {   // B is the NHWC tensor [K = images*H*W pixels, C]; the [pixels, 9*C] patch matrix is formed by the loads
        if(p.N != 9 * p.conv_C || p.K * p.conv_C * esz >= (int64_t(1) << 31) || p.conv_H > 65535 || p.conv_W > 65535
           || (p.conv_C * esz) % 16 != 0 || p.K % (static_cast<int64_t>(p.conv_H) * p.conv_W) != 0)
            return hipErrorInvalidValue;
        a.conv_H = p.conv_H; a.conv_W = p.conv_W; a.conv_Cb = static_cast<int>(p.conv_C * esz);
    }
    else if(p.conv_H > 0)
    {   // A is the NHWC tensor [M = images*H*W, C]; its 3x3 patch matrix [M, 9*C] is formed by the loads
        if(p.K != 9 * p.conv_C || plan.splits > 1 || p.M * p.conv_C * esz >= (int64_t(1) << 31)
           || p.conv_H > 65535 || p.conv_W > 65535 || (p.conv_C * esz) % 16 != 0
           || p.M % (static_cast<int64_t>(p.conv_H) * p.conv_W) != 0)
            return hipErrorInvalidValue;
        a.conv_H = p.conv_H; a.conv_W = p.conv_W; a.conv_Cb = static_cast<int>(p.conv_C * esz);
    }
    const int64_t ktiles = (a.Kb + kRowBytes - 1) / kRowBytes;
    int splits = plan.splits < 1 ? 1 : plan.splits;
    a.ktiles_per_split = static_cast<int>((ktiles + splits - 1) / splits);
    if(a.ktiles_per_split < 1) a.ktiles_per_split = 1;
    const TileShape ts = kTiles[plan.tile];
    a.tiles_m = static_cast<int>((p.M + ts.bm - 1) / ts.bm);
    a.tiles_n = static_cast<int>((p.N + ts.bn - 1) / ts.bn);
    a.group_m = kGroupM;      // (2, 4, 16 and 32 measured within noise of 8 on config 5's shapes, int8 and binary16)
    return hipSuccess;
}

// Second launch of a product in K splits: their sum and the epilogue.
static hipError_t reduce_splits(const GemmProblem& p, int splits, void* workspace, hipStream_t stream, ColumnFoldArgs* fold)
{
    const bool vec4 = p.N % 4 == 0 && ((reinterpret_cast<uintptr_t>(workspace) | reinterpret_cast<uintptr_t>(p.C)) & 15) == 0;
    int64_t    nb   = (p.M * p.N / (vec4 ? 4 : 1) + kThreads - 1) / kThreads;
    nb              = nb > 65536 ? 65536 : nb;
    if(p.out_amax_bits && nb > 1024) nb = 1024;    // at most one atomic per workgroup on one word: keep them few
    const ColumnFoldArgs beside = fold ? *fold : ColumnFoldArgs{};
    if(fold) *fold = ColumnFoldArgs{};
    auto reduce = [&](auto acc_tag, auto vec_tag, const void* ws, int32_t* dump) {
        typedef decltype(acc_tag) acc_t;
        splitk_reduce_kernel<acc_t, decltype(vec_tag)::value><<<dim3(nb + beside.blocks()), dim3(kThreads), 0, stream>>>(
            static_cast<const acc_t*>(ws), splits, p.M, p.N, p.C, p.c_dtype == kF16, p.s0, p.s1, p.col_scale, p.col_bias, dump,
            p.out_amax_bits, static_cast<int8_t*>(p.out_codes), p.out_code_inv, p.out_code_qmax, static_cast<int>(nb), beside);
    };
    if(p.prec == 8)
    {
        if(vec4) reduce(int32_t{}, std::true_type{}, workspace, p.acc_dump);
        else     reduce(int32_t{}, std::false_type{}, workspace, p.acc_dump);
    }
    else
    {
        if(vec4) reduce(float{}, std::true_type{}, workspace, nullptr);
        else     reduce(float{}, std::false_type{}, workspace, nullptr);
    }
    return hipGetLastError();
}

hipError_t launch_gemm(const GemmProblem& p, const GemmPlan& plan, void* workspace, hipStream_t stream, ColumnFoldArgs* fold)
{
    if(p.M <= 0 || p.N <= 0) return hipSuccess;
    if(p.prec == 32 && (p.conv_H > 0 || p.b_remap_C > 0)) return hipErrorInvalidValue;
    const int splits = plan.splits < 1 ? 1 : plan.splits;
    if(p.prec == 32)
    {
        const hipError_t e = launch_gemm_f32(p, plan, workspace, stream);
        return e != hipSuccess || splits == 1 ? e : reduce_splits(p, splits, workspace, stream, fold);
    }
    GemmKernelArgs   a;
    const hipError_t bad = kernel_args(p, plan, workspace, a);
    if(bad != hipSuccess) return bad;
    if(g_tile_override < 0 && g_persistent_mode != 1)
    {   // (whatever the plan holds: room for its K splits stays asked for, and unused here)
        bool             taken = false;
        const hipError_t e     = launch_gemm_rows(p, &taken, stream);
        if(taken || e != hipSuccess) return e;
    }
    if(p.conv_H > 0 && !p.tn)
    {
        bool             taken = false;
        const hipError_t e     = launch_conv3x3(p, g_tile_override, &taken, stream);
        if(taken || e != hipSuccess) return e;
    }
    if(p.conv_H > 0 && p.tn && splits > 1 && g_tile_override < 0)
    {
        hipError_t e   = hipSuccess;
        const int  own = launch_conv3x3_wgrad(p, splits, plan.us, workspace, stream, &e);
        if(own > 0) return e != hipSuccess ? e : reduce_splits(p, own, workspace, stream, fold);
    }
    // The persistent kernel is opt-in.  Its write-back of a tile overlaps the next tile's K loop, which on 32x32 instructions gained
    // 7-20 % launched alone and back to back; the present K loop leaves its wavefronts no registers for a second set of the columns'
    // fragments, and it loses there too: 16384x4096x1024 int8 75.1 us per tile, 80.5 persistent, binary16 124.4 and 127.1, 16384x1024x4096 53.0
    // and 53.5.  Inside an operator sequence its fixed tile assignment costs more: workgroups that start late, behind the tail of the
    // previous kernel, still walk their full share of tiles, while the per-tile grid is balanced by the hardware dispatcher.
    if(!p.tn && persistent_eligible(a, p.prec, plan.tile, splits)
       && g_persistent_mode == 1)
        return p.prec == 8 ? launch_persistent<I8Traits>(a, stream) : launch_persistent<F16Traits>(a, stream);
    hipError_t e = p.prec == 8 ? launch_traits<I8Traits>(plan.tile, a, splits, stream, p.tn)
                               : launch_traits<F16Traits>(plan.tile, a, splits, stream, p.tn);
    return e != hipSuccess || splits == 1 ? e : reduce_splits(p, splits, workspace, stream, fold);
}

// K tiles of a workgroup per round of 256 workgroups -> time of the compute unit that gets the first workgroup of every
// round (the hardware deals them out in order): `occ` workgroups share the unit's rate evenly, the next one starts when
// one ends.
static double unit_time(const TileModel& m, double mop, const double* rounds, int n)
{
    double left[8], us = 0.0;
    int    active = 0, next = 0;
    for(;;)
    {
        while(active < m.occ && next < n) left[active++] = rounds[next++];
        if(active == 0) return us;
        double shortest = left[0];
        for(int i = 1; i < active; ++i) shortest = left[i] < shortest ? left[i] : shortest;
        const double rate = m.r1 * active < m.rmax ? m.r1 * active : m.rmax;
        us += shortest * active * mop / rate;
        int kept = 0;
        for(int i = 0; i < active; ++i)
            if(left[i] > shortest) left[kept++] = left[i] - shortest;
        active = kept;
    }
}

// Tile on which two GEMMs share a launch (`a` first), or -1 when two launches are estimated to be about as fast: with more
// than sixteen rounds of workgroups each of them fills the chip by itself, and a long contraction unsplit beside short ones
// would outlast them.  Separate launches -> one, measured: int8 1808x1040x784 15.6 -> 12.2 us, 1024^3 10.7 -> 6.9, 512^3 6.8 -> 4.8,
// 4096x768x3072 31.5 -> 30.5; binary16 2056x1000x1032 31.0 -> 25.3, 4096x3072x768 50.3 -> 50.8 (4096x768x3072 and 4096x3072x768
// gained 5 and 9 us before the separate launches had loading wavefronts); not paired: 4096x768x768 binary16 26.1 (one launch
// 26.5), 3000x768x768 24.9 (25.1).
// How far the estimate reaches, over 146 backward passes (44 operators from 512^3 to 8192 x 1024^2, drawn evenly over the
// logarithm, both types, transposed copies and row-major, replayed from a graph; two launches against one on either tile), all on the
// tiles' form of 32x32 instructions: its rms error is 17 % for int8 and 27 % for binary16, where it is 14 % too long on average.  The choice costs 1.9 % on
// average against the best of the three and more than 10 % in ten cases (binary16 384x1744x1168 left apart, 19.5 us against
// 14.2, is the worst); it errs towards two launches: the 114 pairs run 1.48 times as fast as apart, the worst of them
// 2.4 % slower.
static double pair_us(const GemmProblem& a, const GemmProblem& b, int t, int splits)
{
    constexpr int kMaxRounds = 16;
    TileModel m = kTileModel[t];
    if(a.prec == 16) m.r1 *= t == 1 ? 0.83 : 0.6;       // a long binary16 contraction left over alone, fitted
    auto tiles  = [&](const GemmProblem& p) { return ((p.M + kTiles[t].bm - 1) / kTiles[t].bm) * ((p.N + kTiles[t].bn - 1) / kTiles[t].bn); };
    auto ktiles = [&](const GemmProblem& p, int s) { return std::ceil(std::ceil(static_cast<double>(p.K * (p.prec / 8)) / kRowBytes) / s) / tn_factor(t, p.prec, p.tn); };
    const int64_t wa = tiles(a) * splits, wgs = wa + tiles(b);
    if(wgs > kMaxRounds * kNumCu) return -1.0;
    const double ka = ktiles(a, splits), kb = ktiles(b, 1), mop = 2.0 * kTiles[t].bm * kTiles[t].bn * kRowBytes * 1e-6;
    double rounds[kMaxRounds];
    int    n = 0;
    for(int64_t at = 0; at < wgs; at += kNumCu) rounds[n++] = at < wa ? ka : kb;
    const double unit = unit_time(m, mop, rounds, n), chip = (wa * ka + (wgs - wa) * kb) * mop / m.cap;
    const double full = std::ceil(static_cast<double>(wgs) / (kNumCu * m.occ));      // rounds of co-resident workgroups
    const double us   = (unit > chip ? unit : chip) + m.ovh * (full > 1.0 ? full - 0.5 : full);
    return splits > 1 ? us + 4.0 + static_cast<double>(splits + 1) * static_cast<double>(a.M) * static_cast<double>(a.N) * 4.0 / 6.24e6 : us;
}
static int pair_tile(const GemmProblem& a, const GemmProblem& b, double separate_us)
{
    int    tile = -1;
    double best = 0.93 * separate_us;
    for(int t = 1; t < kNumTiles; ++t)
    {
        if(g_tile_override >= 0 && t != g_tile_override) continue;
        const double us = pair_us(a, b, t, 1);
        if(us >= 0.0 && us < (tile < 0 ? 1.0 : 0.95) * best) { best = us; tile = t; }      // (the smaller tile must win by 5 %)
    }
    return tile;
}
// Where the two would go apart, the first (the longer contraction) in K splits: the tile and the splits, up to as many, on which they share
// a launch all the same, with the sum of the splits behind it.  Few outputs over a long contraction leave units idle, and the parts of
// both together fill them: three launches become two.  Binary16 keeps the plan's splits, not fewer: a sum over a longer piece has more roundings
// (4096x768x3072 unsplit 59.8 -> 54.8 us, but the error of dW against 64 bits 2.4e-7 -> 4.1e-7); int8 sums are exact.  Backward passes of 64..16384 by
// 64..4096 (both types, both forms, replayed from a graph), apart -> this, us: binary16 6784x912x592 41.5 -> 31.2, 13536x1360x240 42.1 -> 37.6,
// 4224x312x160 13.5 -> 9.7, int8 15744x2288x112 32.2 -> 22.9, 14640x128x2608 54.9 -> 42.0; of 120 drawn 26 gain, 1.25 times on
// average.  The estimate does not know how the second's contraction drags on over the small tile: with
// more than 36 K tiles of it the pair may lose (binary16 3200x3656x128 30.7, 39.8 together), nor of gemm_rows_kernel
// (2112x1696x96 13.0, 20.0).
static GradientPair split_pair(const GemmProblem& a, const GemmPlan& plan_a, const GemmProblem& b, double separate_us)
{
    GradientPair pair;
    const int64_t kb = (b.K * (b.prec / 8) + kRowBytes - 1) / kRowBytes;
    if(plan_a.splits < 2 || kb > 36 || g_tile_override >= 0 || gemm_rows_takes(a) || gemm_rows_takes(b)) return pair;
    double best = separate_us;
    for(int t = 1; t < kNumTiles; ++t)
        for(int s = a.prec == 8 ? 1 : plan_a.splits; s <= plan_a.splits; ++s)
        {
            const double us = pair_us(a, b, t, s);
            if(us >= 0.0 && us < best) { best = us; pair = GradientPair{t, s}; }
        }
    return pair;
}

// The weight gradient lands in memory that the data gradient reads (a caller that stores dW over the transposed weights or
// over dY, say): fine in two launches, data gradient first, a race in one.
static bool dw_over_dx_operands(const GemmProblem& dx, const GemmProblem& dw)
{
    auto meets = [](const void* a, int64_t a_bytes, const void* b, int64_t b_bytes) {
        const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
        return a && b && x < y + static_cast<uintptr_t>(b_bytes) && y < x + static_cast<uintptr_t>(a_bytes);
    };
    const int64_t esz = dx.prec / 8, out = dw.M * dw.N;
    auto written = [&](const void* p, int64_t bytes) {
        return meets(dw.C, out * (dw.c_dtype == kF16 ? 2 : 4), p, bytes) || meets(dw.acc_dump, out * 4, p, bytes);
    };
    return written(dx.A, dx.M * dx.K * esz) || written(dx.B, dx.N * dx.K * esz) || written(dx.s0, 4) || written(dx.s1, 4)
        || written(dx.col_scale, dx.N * 4);
}

static bool dw_is_first(const GemmProblem& dx, const GemmProblem& dw) { return dw.tn || dw.K >= dx.K; }      // the longer contraction, or the row-major one

GradientPair gradient_pair(const GemmProblem& dx, const GemmPlan& plan_dx, const GemmProblem& dw, const GemmPlan& plan_dw)
{
    auto plain = [](const GemmProblem& p) {
        return (p.prec == 8 || p.prec == 16) && p.M > 0 && p.N > 0 && p.K > 0 && p.conv_H == 0 && p.b_remap_C == 0
            && !p.out_amax_bits && !p.out_codes;
    };
    if(dx.prec != dw.prec || !plain(dx) || !plain(dw) || dx.tn || g_persistent_mode == 1 || dw_over_dx_operands(dx, dw)) return GradientPair{};
    // (The estimates are the tiles', also of a product that by itself would go to gemm_rows_kernel.  One shared launch -> that kernel for
    // what it takes, replayed from a graph: 64x128x128 int8 4.2 us, apart 6.3, 512^3 4.8 and 8.1, 128x1024x2048 8.2 and 8.8;
    // binary16 4.0 and 6.1, 5.8 and 9.1, but 128x1024x2048 11.0 and 9.7, 256x1024x1024 10.8 and 9.7: the worst of 32.)
    const double       us = plan_dx.us + plan_dw.us;
    const bool         dw_first = dw_is_first(dx, dw);
    const GemmProblem &a = dw_first ? dw : dx, &b = dw_first ? dx : dw;
    GradientPair       pair;
    pair.tile = pair_tile(a, b, us);
    return pair.tile >= 0 ? pair : split_pair(a, dw_first ? plan_dw : plan_dx, b, us);
}

hipError_t launch_gradient_pair(const GemmProblem& dx, void* ws_dx, const GemmProblem& dw, void* ws_dw, const GradientPair& pair, const ColumnFoldArgs& fold, hipStream_t stream)
{
    const bool         dw_first = dw_is_first(dx, dw);
    const GemmProblem &a = dw_first ? dw : dx, &b = dw_first ? dx : dw;
    void* const        workspace = dw_first ? ws_dw : ws_dx;
    GemmPairArgs       args;
    hipError_t         e = kernel_args(a, GemmPlan{pair.tile, pair.splits, 0, 0.0}, workspace, args.g[0]);
    if(e == hipSuccess) e = kernel_args(b, GemmPlan{pair.tile, 1, 0, 0.0}, nullptr, args.g[1]);
    if(e != hipSuccess) return e;
    args.splits = pair.splits;
    args.na     = args.g[0].tiles_m * args.g[0].tiles_n * pair.splits;
    args.total  = args.na + args.g[1].tiles_m * args.g[1].tiles_n;
    if(pair.splits == 1) args.fold = fold;
    auto go = [&](auto tn, auto split) {
        constexpr bool TNA = decltype(tn)::value, SPLITA = decltype(split)::value;
        return a.prec == 8 ? launch_pair_traits<I8Traits, TNA, SPLITA>(pair.tile, args, stream) : launch_pair_traits<F16Traits, TNA, SPLITA>(pair.tile, args, stream);
    };
    constexpr std::true_type  yes{};
    constexpr std::false_type no{};
    if(pair.splits == 1) return a.tn ? go(yes, no) : go(no, no);
    e = a.tn ? go(yes, yes) : go(no, yes);
    ColumnFoldArgs beside = fold;
    return e != hipSuccess ? e : reduce_splits(a, pair.splits, workspace, stream, &beside);
}

}  // namespace qsync
