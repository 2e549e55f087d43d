// Workgroup block kernel: bf16 / fp16 rows of order n = pb * 128 with a +-1 block of order
// 32 < pb <= 256 along the strided axis (H_n = B (x) H_128, B = H_p (x) H_{2^(k-7)}; sections
// 2.3.2, 2.3.3) - e.g. 18944 = 148 * 128 with the order-148 Paley II block; also the Sylvester
// orders 2^14 and 2^15, which are too long for one wave (B = H_128, H_256).
//
// The dense block product Y1[pb x 128] = B * X[pb x 128] is a real contraction (pb adds per
// output), so it runs on the matrix cores.  NW = ceil(pb / 16) waves share a row, wave w owning
// the 16 block rows 16 w .. 16 w + 15 on input and on output:
//   phase 1  the wave loads its block rows (16-byte chunks, 4 per lane), transposes 16-bit
//            values inside each lane (v_perm_b32) so that consecutive block rows of one column are
//            adjacent, and writes them to LDS as the data operands of phase 2, one 1 KB block per
//            matrix-core instruction in lane order (no bank conflicts on either side);
//   phase 2  the wave computes its 16 output block rows for all 128 columns: 8 column tiles x
//            KK = ceil(pb / 32) contraction steps of v_mfma_f32_16x16x32_bf16, its KK operand tiles of
//            B resident in registers, the data operands read from LDS (16 bytes per lane) a few
//            instructions ahead of their use;
//   phase 3  128-point transform along the columns: three register stages, four fused DPP
//            stages, absmax; workgroup absmax through LDS;
//   phase 4  scale, round/clamp, pack; b = 4 stores dwords, b = 3 assembles the row's bytes in LDS
//            and all waves copy them out in 16-byte units.
// Column tile nt holds columns {8 c + nt}, so a lane ends up with 8 consecutive columns of 4
// block rows.  One wave per 16 block rows keeps a wave near 100 VGPRs, so two workgroups share a
// CU.  A workgroup loops over rows; barriers order the LDS reuse.
//
// Short Sylvester factors (CB < 4): n = p * 2^k with k = CB + 3 = 5 or 6 has block rows of only 32
// or 64 columns, so RPW = 128 / 2^k consecutive rows of X are laid side by side and taken in one
// pass: column group c = (row of the pass, 8-column chunk of that row).  The block product treats
// the 128 columns alike; the column transform then runs over CB lane bits only, and absmax, scale
// and the output rows are per row of the pass.  Here the block is H_p itself, of any order
// 4 <= p <= 256.
#pragma once
#include "error_grid.h"
#include "wave_common.h"

namespace rq {
namespace {

// LDS operand buffer: for every (column tile nt, contraction step kk) one 1 KB block holding the data
// operand of that matrix-core instruction in lane order - lane (g, c) finds the 8 block rows
// 32 kk + 8 g .. + 7 of column (c, nt) at byte lane * 16 of the block.  A read instruction thus takes
// 1 KB of consecutive bytes and a phase-1 write instruction (8 bytes per lane: 4 block rows) 512
// consecutive bytes: neither meets a bank conflict, with no swizzle and no padding.  (Measured with a
// read-only probe on this chip: 16-byte reads in lane order move 488 bytes per ns and CU, a layout that
// gives the 16 lanes of a DPP row 16 different 16-byte slots of a 256-byte window in scattered order only
// 375.)
template <int KK>
constexpr size_t wg_ops_bytes() { return (size_t)8 * KK * 1024; }

template <int KK>
constexpr size_t wg_lds_bytes() { return wg_ops_bytes<KK>() + (size_t)KK * 32 * 48; }

// Register budget, as waves per SIMD (512 VGPRs per SIMD lane).  The hardware deals the waves of
// successive workgroups round robin over the four SIMDs, so a CU holds 4 x this many waves:
//   KK <= 3, KK == 5  6 (80 VGPRs): several small workgroups per CU, or two of 9 - 10 waves (3 of
//            which may land on one SIMD, so 96 registers would often leave room for one only);
//   KK == 4, KK >= 6   4 (128): two workgroups of up to 8 waves, or one of up to 16.
// At 128 registers there is room for the next pass's 16 load registers, so its loads are issued one
// pass ahead (right after the barrier that ends phase 1) and their latency is covered by phases
// 2 - 4.  At 80 registers the same prefetch spills, and spill reloads wait on the same counter as the
// loads: measured slower.  (Touching one byte per 128 of the next row a pass ahead, to bring it into
// the L2 cache, measured no better than the plain loads either.)
template <int KK>
constexpr int wg_waves_per_simd(bool wide = false) { return !wide && (KK <= 3 || KK == 5) ? 6 : 4; }

// What the kernel does with the rotated row (phase 4), and the arguments that takes beyond WaveArgs:
//   kWgQuantize  codes and scale of rq_rotate_quantize;
//   kWgError     squared quantization error per clip ratio (rq_quant_error);
//   kWgRotate    the values themselves (rq_rotate; rq_dequantize_rotate, whose rows come from packed codes);
//   kWgGrid      squared quantization error at every clip ratio of a search's grid (error_grid.h), summed over the rows.
enum WgSink { kWgQuantize, kWgError, kWgRotate, kWgGrid };
struct WgNone {};
struct QeArgs {
    ClipArg clips;
    double* partial;      // [rows][number of clips]
    int max_shares;       // workgroups that may share the clip ratios of a pass (grid y; each repeats the rotation)
};
struct WgRotArgs {
    void* Y;
    int d_out;
    int64_t ld_out;
    double inv;           // 1 / sqrt(n)
    int out;              // 0 bf16, 1 fp32, 2 fp16
};
struct WgGridArgs {
    double inv_norm;      // 1 / n^2
    GbsDev* dev;
};
template <int SINK>
using WgArgs = std::conditional_t<SINK == kWgError, QeArgs, std::conditional_t<SINK == kWgRotate, WgRotArgs,
                                  std::conditional_t<SINK == kWgGrid, WgGridArgs, WgNone>>>;

// The histogram of the grid sink.  (KK == 1: two waves a pass, which take its four rows one after the other: a sixteenth of a row's
// values meet in an instruction, and the last cells' further words cost what they gain; 512 x 896, b = 4 59.0 us a search with them, 58.1
// without.  A thread's words are held in registers where its share is small enough: 21 of them, KK = 3 with b = 4, spill 18.)
template <int KK, int BITS>
using WgGrid = ErrorGrid<BITS, KK == 1 ? 1 : kGridSpread, KK < (BITS == 3 ? 3 : 5) ? 0 : 64 * (2 * KK - 1)>;

// DPP row, 8-column chunk and row of the pass of a lane, as values the compiler does not keep across the phases.
template <int CB>
__device__ __forceinline__ void wg_lane(int lane, int& g, int& cl, int& rsub) {
    asm volatile("" : "+v"(lane));
    const int cphys = lane & 15, c = (cphys & 4) ? (cphys ^ 3) : cphys;
    g = lane >> 4;
    cl = CB == 4 ? c : c & ((1 << CB) - 1);
    rsub = CB == 4 ? 0 : c >> CB;
}

// The sign a lane's values carry after the column transform (CB < 4: the first lane stage is the plain one, the fused
// ones start at the second bit).
template <int CB>
__device__ __forceinline__ float wg_flip(int cl) {
    return (__builtin_popcount(CB == 4 ? cl : cl >> 1) & 1) ? -1.0f : 1.0f;
}

// SRC: 0 = 16-bit rows of X, 3 / 4 = packed signed codes of that width (kWgRotate only): the lane's eight codes of
// a block row become fp16 integers (code_operands), the matrix cores contract them exactly, and the
// row's scale multiplies once at the end.
// WIDE: fp32 results (kWgRotate only), see phase 3; the doubles take 128 registers, 80 spill up to 37 of them (KK = 8
// spills 20 - 24 at 128).  16-bit results keep fp32 stages: the type's own rounding is all of their error (18944 wide, rows to
// bf16 1.659369867e-3 against 64 bits, 1.659369866e-3 on the general kernel with its fp64 block sums; fp16 2.0731412e-4 and
// 2.0731411e-4), and fp64 stages cost 3584 x 18944 to bf16 51 -> 81 us.
template <int KK, int BITS, bool FULL, int SINK, int CB = 4, bool F16 = false, int SRC = 0, bool WIDE = false>
__global__ __launch_bounds__(128 * KK) __attribute__((amdgpu_waves_per_eu(wg_waves_per_simd<KK>(WIDE || SINK == kWgGrid))))
void k_wg_block(RQ_WAVE_PARAMS, WgArgs<SINK> sa) {
    RQ_WAVE_ARGS(a);
    RQ_WAVE_BLOCK_ROWS(pb);
    static_assert(CB >= 2 && CB <= 4 && (CB == 4 || !FULL), "unsupported shape");
    static_assert(SRC == 0 || (SINK == kWgRotate && F16 && !FULL), "packed codes: rotation only, fp16 operands");
    constexpr bool QE = SINK == kWgError;
    constexpr int RPW = 16 >> CB;                        // rows of X per pass
    constexpr int SEG = 8 << CB;                         // columns of one block row (2^k)
    constexpr bool PF = !WIDE && SINK != kWgGrid && wg_waves_per_simd<KK>() == 4;   // loads run one pass ahead
    constexpr bool EARLY = SINK == kWgQuantize && KK == 4;   // column stages start beside the block product, see phase 2
    __shared__ float esum[QE ? 16 : 1][QE ? RPW : 1][QE ? RQ_MAX_CLIPS : 1];   // [wave][row of the pass][clip]
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    uint8_t* const ops = lds_raw;                        // [column tile][contraction step] x 1 KB, see wg_ops_bytes
    uint8_t* const stage = lds_raw + wg_ops_bytes<KK>(); // packed codes of the row (b = 3); fp32 results, 2 KB a wave
    __shared__ __attribute__((aligned(16))) float wmax[RPW * 16];   // [row of the pass][wave]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;                      // ceil(pb / 16)
    const int g = lane >> 4, cphys = lane & 15;
    const int c = (cphys & 4) ? (cphys ^ 3) : cphys;    // logical column group (8 columns)
    const int rsub = CB == 4 ? 0 : c >> CB;              // row of the pass
    const int cl = CB == 4 ? c : c & ((1 << CB) - 1);    // 8-column chunk inside that row

    u32x4 A[KK];
    if constexpr (SINK != kWgGrid) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) A[kk] = a.tiles[(wave * KK + kk) * 64 + lane];
    }
    // (uniform, but computed by vector instructions: moved to scalar registers)
    auto uniform = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
    const float c1h = uniform((float)a.c1), c1l = uniform((float)(a.c1 - (double)c1h));
    const float flip = wg_flip<CB>(cl);
    const uint32_t sg0 = (c & 1) ? 0x80000000u : 0u;

    // phase-1 geometry: lane (g, c) loads block rows 16 wave + 4 g + t, t = 0..3, at constant
    // strides from one offset.  Block rows at or beyond pb meet zero columns of B, with which an infinity of a real row would
    // make NaN: they lie beyond d and read as zero, or, where the loads do not check that (STANDIN), the last four real rows
    // are read in their place and cleared.  (Registers spilled, bounds checked by the loads and so: full rows, KK = 5, b = 3 10
    // and 0, b = 4 11 and 2; the search's passes of several rows, KK = 2 11 and 10; the other forms of several rows, KK = 5, 7 and 9.)
    constexpr bool STANDIN = SINK != kWgRotate && (FULL || (SINK == kWgGrid && CB < 4));
    const int r0 = 16 * wave + 4 * g;
    const int eoff0 = (!STANDIN || r0 < pb ? r0 : pb - 4) * SEG + cl * 8;
    // phase-1 writes: the lane's block rows 16 wave + 4 g .. + 3 are one 8-byte half of the unit that
    // reader lane (2 (wave & 1) + g / 2, c) takes in contraction step wave / 2
    uint8_t* const wr0 = ops + ((((wave >> 1) * 4 + 2 * (wave & 1) + (g >> 1)) * 16 + cphys) * 16 + (g & 1) * 8);
    const uint8_t* const rd0 = ops + lane * 16;

    u32x4 R[4];
    [[maybe_unused]] float rscale = 1.0f;               // packed codes: the row's scale
    auto load_row = [&](int64_t row) {
        const uint16_t* xr = a.X + row * a.ld;
        if constexpr (CB == 4) {
            const RowView xv = row_view(xr, a.d);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                R[t] = FULL ? load16(xr + eoff0 + t * SEG) : load_chunk(xv, eoff0 + t * SEG);
        } else {
            // the lanes of a wave read different rows: per-lane addresses, whole chunks (d % 8 == 0)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                R[t] = eoff0 + t * SEG < a.d ? load16(xr + eoff0 + t * SEG) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    // Rotation only: the rows of a pass as one buffer resource (rows beyond the end lie outside it and read as
    // zero) with 32-bit lane offsets, which leaves the registers to the transform.
    auto load_rows = [&](int64_t row0) {
        const int64_t left = a.rows - row0;
        const int live_rows = left < RPW ? (int)left : RPW;
        int gq, cq, rq;
        wg_lane<CB>(lane, gq, cq, rq);
        // block rows that do not exist: of X they lie beyond d and read as zero (their products with zero columns of B
        // would not, for infinities of real rows); of codes the last four real ones are read
        const int b0 = 16 * wave + 4 * gq, br = SRC == 0 || b0 < pb ? b0 : pb - 4;
        if constexpr (SRC != 0) {
            const int row_bytes = (SEG * SRC / 8) * pb;
            const auto rs = __builtin_amdgcn_make_buffer_rsrc(a.codes + row0 * (row_bytes / 4), 0, live_rows * row_bytes, 0x00020000);
            const CodeAt at = code_at<SRC>((br << CB) + cq);
            const uint32_t base = (uint32_t)(rq * row_bytes);
            constexpr int STEP = SEG * SRC / 8;              // bytes of a block row
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                R[t][0] = __builtin_amdgcn_raw_buffer_load_b32(rs, base + at.off0 + t * STEP, 0, 2);
                if constexpr (SRC == 3) R[t][1] = __builtin_amdgcn_raw_buffer_load_b32(rs, base + at.off1 + t * STEP, 0, 2);
            }
            const auto ss = __builtin_amdgcn_make_buffer_rsrc(a.scales + row0, 0, live_rows * 4, 0x00020000);
            R[0][2] = __builtin_amdgcn_raw_buffer_load_b32(ss, rq * 4, 0, 0);
        } else {
            const int bytes = (int)(((live_rows - 1) * a.ld + a.d) * 2);
            const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.X) + row0 * a.ld, 0, bytes, 0x00020000);
            const int base = rq * (int)a.ld;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int e = (br + t) * SEG + cq * 8;
                const uint32_t off = CB == 4 || e < a.d ? (uint32_t)(base + e) * 2u : 0x80000000u;
                R[t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 2));
            }
        }
    };
    using Grid = WgGrid<KK, BITS>;
    constexpr int SUMS = SINK == kWgGrid ? (kGridRatios - 1 + 64 * (2 * KK - 1) - 1) / (64 * (2 * KK - 1)) : 1;   // ratios of a thread
    [[maybe_unused]] double sum[SUMS];
    __shared__ uint64_t tot[SINK == kWgGrid ? 16 : 1][3];
    static_assert(SINK != kWgGrid || Grid::within_margin(1, sizeof(wmax) + sizeof(tot) + sizeof(esum)), "see grid_rows_beside");
    if constexpr (SINK == kWgGrid) {
#pragma unroll
        for (int k = 0; k < SUMS; ++k) sum[k] = 0.0;
        if (blockIdx.x == 0 && threadIdx.x == 0) sa.dev->grid_ticket = 0;
    }
    const int64_t n_pass = (a.rows + RPW - 1) / RPW;
    // CB == 4: one row per pass, uniform over the workgroup; otherwise the lane's own row, the
    // last row standing in (loads only) for rows beyond the end
    auto load_pass = [&](int64_t ps) {
        if constexpr (SINK == kWgRotate) return load_rows(ps * RPW);
        const int64_t r = ps * RPW + rsub;
        load_row(CB == 4 || r < a.rows ? r : a.rows - 1);
    };
    if constexpr (PF) load_pass(blockIdx.x);             // (the grid has no more workgroups than passes)
    // Units for block rows at or beyond 16 nw (nw odd: the upper half of the last contraction step) are never written by
    // phase 1 but are read, against zero columns of B: they hold zeros.  A pass reads the maxima of waves that do not exist, too.
    // The barrier behind the first phase 1 orders both: with the whole buffer cleared and a barrier before the first loads, 500 rows
    // of 8960 take 7.17 us and not 6.85, 300 of 18944 8.95 and not 8.76, 4096 of 8960 (b = 3) 30.0 and not 29.2.
    if (nw & 1)
        for (int i = threadIdx.x; i < 8 * 32; i += blockDim.x)
            reinterpret_cast<u32x4*>(ops)[((i >> 5) * KK + KK - 1) * 64 + 32 + (i & 31)] = u32x4{0u, 0u, 0u, 0u};
    if (threadIdx.x < RPW * 16) wmax[threadIdx.x] = 0.0f;
    for (int64_t pass = blockIdx.x; pass < n_pass; pass += gridDim.x) {
        if (!PF) load_pass(pass);
        if constexpr (SINK == kWgGrid) {
            // Beside the row in every pass: held, the tiles leave too few registers to the histogram's phases.  Spilled, held -> now: one row per
            // pass 6 - 14 -> 0 beyond blocks of 160 (0 up to there), several 17 - 35 -> 6 - 10, for blocks up to 32 28 - 32 -> 24 - 28.  A
            // search on 512 rows, b = 3, us a call: 8960 wide 46.0 -> 43.5, 18944 43.3 -> 42.3,
            // 28672 55.2 -> 51.3, 14336 (b = 4) 40.7 -> 40.3, 896 wide unchanged.
            int l = lane;
            asm volatile("" : "+v"(l));
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) A[kk] = a.tiles[(wave * KK + kk) * 64 + l];
        }
        // ---- phase 1
        if (STANDIN && 16 * wave + 16 > pb) {            // (the last wave)
#pragma unroll
            for (int t = 0; t < 4; ++t) R[t] = 16 * wave + 4 * g < pb ? R[t] : u32x4{0u, 0u, 0u, 0u};
        }
        // (4-bit codes of several rows a pass, or of blocks up to 64, are spread first and transposed like rows: us a call, so and
        // through code_operands, 3500 x 8960 23.0 and 25.3, 4000 x 8960 26.5 and 27.9, 3000 x 5120 10.4 and 10.8; the others 2000 x
        // 14336 18.0 and 17.2, 3000 x 11008 22.0 and 21.4, 2000 x 18944 26.4 and 25.9)
        constexpr bool DEAL = SRC == 3 || (SRC == 4 && CB == 4 && KK >= 3);
        if constexpr (SRC != 0) {
            rscale = __uint_as_float(R[0][2]);
            uint32_t x[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)   // (a block row is a whole number of dwords: the field's bit position is that of the chunk in it)
                x[t] = SRC == 4 ? R[t][0] : __builtin_amdgcn_alignbit(R[t][1], R[t][0], (3u * cl & 3u) * 8u);
            if constexpr (DEAL) {
                u32x2 v[8];
                code_operands<SRC, 2>(x, v);
#pragma unroll
                for (int ic = 0; ic < 8; ++ic) *reinterpret_cast<u32x2*>(wr0 + ic * (KK * 1024)) = v[ic];
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) R[t] = codes4_f16(x[t]);
            }
        }
        if constexpr (!DEAL) {
#pragma unroll
            for (int ic = 0; ic < 8; ++ic) {
                const uint32_t sel = (ic & 1) ? 0x07060302u : 0x05040100u;
                uint2 v;
                v.x = __builtin_amdgcn_perm(R[1][ic >> 1], R[0][ic >> 1], sel);
                v.y = __builtin_amdgcn_perm(R[3][ic >> 1], R[2][ic >> 1], sel);
                *reinterpret_cast<uint2*>(wr0 + ic * (KK * 1024)) = v;
            }
        }
        __syncthreads();
        if (PF && pass + gridDim.x < n_pass) load_pass(pass + gridDim.x);
        // ---- phase 2
        // Waves of another workgroup that are in their vector phases go first: a wave in here mostly waits for its
        // operand reads or for the matrix cores (4096 rows of 18944, b = 3: 52.8 -> 51.8 us; 512 MiB of 8960-wide rows,
        // b = 4 204 -> 196; 14336, 28672 and 4864 wide: no difference; the rotation, bound by its memory traffic, gains
        // nothing)
        if constexpr (SINK != kWgRotate) __builtin_amdgcn_s_setprio(0);
        f32x4 acc[8];
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        {
            // The 8 KK operand reads run DEPTH ahead of the matrix-core instructions that use them, in a ring
            // of DEPTH register quads; the contraction step is the outer loop, so that consecutive
            // instructions go to different accumulators and none waits for its predecessor's result.
            // (3 where the 80-register kernels have room for it, 2 in their padded-row and quant_error forms)
            // EARLY: column tiles 0 - 3 go over all contraction steps first, then 4 - 7, and the first two column stages
            // of tiles 0 - 3, the same additions as in phase 3, are issued between the matrix-core instructions of the others.
            // Four accumulators in turn still hide an instruction's latency.  4096 rows, on two cards: 13824 wide,
            // b = 3 37.0 -> 36.1 and 32.9 -> 32.5 us, 14336 wide, b = 4 38.0 -> 37.4 and 32.9 -> 32.6.  The forms of 80 registers spill on it (18944 wide, b = 4: 2 -> 7 registers, 4096
            // rows 55.6 -> 57.9 us, 300 rows 8.2 -> 9.3; 4864 wide 27.0 -> 27.3), and one workgroup a compute unit
            // (KK >= 6) gains nothing (28672 wide 65.3 and 65.5).
            constexpr int DEPTH = KK >= 6 ? 4 : (FULL && !QE) ? 3 : 2, ITEMS = 8 * KK;
            auto tile = [](int i) { return EARLY ? i / (4 * KK) * 4 + i % 4 : i % 8; };
            auto step = [](int i) { return EARLY ? i % (4 * KK) / 4 : i / 8; };
            auto read_item = [&](int i) { return *reinterpret_cast<const u32x4*>(rd0 + (tile(i) * KK + step(i)) * 1024); };
            u32x4 ring[DEPTH];
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) ring[i] = read_item(i);
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                __builtin_amdgcn_sched_barrier(0);
                acc[tile(i)] = mfma_pm1<F16>(A[step(i)], ring[i % DEPTH], acc[tile(i)]);
                if (i + DEPTH < ITEMS) ring[i % DEPTH] = read_item(i + DEPTH);
                if constexpr (EARLY) {
                    // additions j of 16: the pairs (0, 1), (2, 3), (0, 2), (1, 3) of four registers each
                    const int done = i - 4 * KK, of = 4 * KK - 1;
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (done >= 1 && j >= 16 * (done - 1) / of && j < 16 * done / of) {
                            constexpr int lo[4] = {0, 2, 0, 1}, hi[4] = {1, 3, 2, 3};
                            const float u = acc[lo[j / 4]][j % 4], v = acc[hi[j / 4]][j % 4];
                            acc[lo[j / 4]][j % 4] = u + v;
                            acc[hi[j / 4]][j % 4] = u - v;
                        }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- phase 3
        if constexpr (SINK != kWgRotate) __builtin_amdgcn_s_setprio(1);
        if constexpr (WIDE && SRC == 0) {
            // fp32 results of rows: the Sylvester stages and the factor in fp64, one register of the accumulators at a
            // time, so that seven stages do not each add a rounding.  Relative error against 64 bits on 18944-wide rows:
            // 6.1e-8 with fp32 stages, 2.6e-8 so (the general kernel, with fp64 block sums, 3.6e-8).  fp64 additions run at
            // the fp32 rate; the launch stays bound by its traffic (4.2 - 5.4 TB/s on 2^26 values).
            __syncthreads();                            // the operand buffer is free from here on
            int gq, cq, rq;
            wg_lane<CB>(lane, gq, cq, rq);
            const int64_t row0 = pass * RPW, left = a.rows - row0;
            const int live_rows = left < RPW ? (int)left : RPW;
            const auto ys = __builtin_amdgcn_make_buffer_rsrc(static_cast<char*>(sa.Y) + row0 * sa.ld_out * 4, 0,
                                                              (int)(((live_rows - 1) * sa.ld_out + sa.d_out) * 4), 0x00020000);
            auto sign = [&](int b) { return __builtin_bit_cast(double, make_uint2(0u, 0x3FF00000u | ((uint32_t)(cq >> b) << 31))); };
#pragma unroll
            for (int ip = 0; ip < 4; ++ip) {
                double v[8];
#pragma unroll
                for (int nt = 0; nt < 8; ++nt) v[nt] = (double)acc[nt][ip];
#pragma unroll
                for (int s = 1; s < 8; s <<= 1)
#pragma unroll
                    for (int nt = 0; nt < 8; ++nt)
                        if (!(nt & s)) {
                            const double u = v[nt], w = v[nt | s];
                            v[nt] = u + w;
                            v[nt | s] = u - w;
                        }
                float o[8];
#pragma unroll
                for (int nt = 0; nt < 8; ++nt) {
                    double x = v[nt];
                    x = fma(x, sign(0), dpp_d<kDppXor1>(x));
                    x = fma(x, sign(1), dpp_d<kDppXor2>(x));
                    if constexpr (CB >= 3) x = fma(x, sign(2), dpp_d<kDppHalfMirror>(x));
                    if constexpr (CB >= 4) x = fma(x, sign(3), dpp_d<kDppRor8>(x));
                    o[nt] = (float)(x * sa.inv);
                }
                const int ao0 = 16 * wave + 4 * ip;
                store_block_f32(reinterpret_cast<float*>(stage) + wave * 512, ((rq * 4 + gq) << CB) + cq, lane, o,
                                [&](int e, const u32x4& unit) {
                    const int rs = CB == 4 ? 0 : e / (4 * SEG), col = ao0 * SEG + (CB == 4 ? e : e % (4 * SEG));
                    const uint32_t off = CB == 4 || col < sa.d_out ? (uint32_t)(rs * (int)sa.ld_out + col) * 4u : 0x80000000u;
                    __builtin_amdgcn_raw_buffer_store_b128(unit, ys, off, 0, 2);
                });
            }
            continue;
        }
#pragma unroll
        for (int s = 1; s < 8; s <<= 1)
#pragma unroll
            for (int nt = 0; nt < 8; ++nt)
                if (!(nt & s) && !(EARLY && (nt | s) < 4)) {
                    const f32x4 u = acc[nt], v = acc[nt | s];
                    acc[nt] = u + v;
                    acc[nt | s] = u - v;
                }
        [[maybe_unused]] float m = 0.0f;
        // rotation only: nothing else of this pass needs the workgroup, the operand buffer is free from here on
        if constexpr (SINK == kWgRotate) __syncthreads();
        // the stage signs are rebuilt from the column group every pass (two instructions each) rather
        // than held in registers across phases 1 and 2
        int cs = c;
        asm volatile("" : "+v"(cs));
        float sf[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) sf[b] = __uint_as_float(0x3F800000u | ((uint32_t)(cs >> b) << 31));
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
            f32x4 v = acc[nt];
            if constexpr (CB == 4) {
                lane_stages_fused(v, sf[0], sf[1], sf[2], sf[3]);
            } else {
                lane_stage<kDppXor1>(v, sg0);
                lane_stages_tail<CB>(v, sf);
            }
            acc[nt] = v;
            if constexpr (SINK != kWgRotate) m = absmax4(m, v);
        }
        if constexpr (SINK == kWgRotate) {
            // the pass's rows of Y as one buffer resource; what lies beyond it (rows past the end, and with one
            // row per pass the columns from d_out on) is not stored
            int gq, cq, rq;
            wg_lane<CB>(lane, gq, cq, rq);
            const float sgn = wg_flip<CB>(cq);
            // (the factor is rounded once; from codes the sums are exact integers)
            const double kd = SRC ? (double)(sgn * rscale) * sa.inv : (double)sgn * sa.inv;
            const float k = (float)kd;
            const int64_t row0 = pass * RPW, left = a.rows - row0;
            const int live_rows = left < RPW ? (int)left : RPW;
            constexpr int esz = WIDE ? 4 : 2;
            const auto ys = __builtin_amdgcn_make_buffer_rsrc(static_cast<char*>(sa.Y) + row0 * sa.ld_out * esz, 0,
                                                              (int)(((live_rows - 1) * sa.ld_out + sa.d_out) * esz), 0x00020000);
#pragma unroll
            for (int ip = 0; ip < 4; ++ip) {
                const int ao0 = 16 * wave + 4 * ip;                      // first of the four output block rows of this register
                float o[8];
#pragma unroll
                for (int nt = 0; nt < 8; ++nt) o[nt] = acc[nt][ip];
                if constexpr (WIDE) {
                    // (exact integers times the scale: one rounding)
#pragma unroll
                    for (int nt = 0; nt < 8; ++nt) o[nt] = (float)((double)o[nt] * kd);
                    // block rows ao0 .. ao0 + 3 of each row of the pass are 4 SEG consecutive values
                    store_block_f32(reinterpret_cast<float*>(stage) + wave * 512, ((rq * 4 + gq) << CB) + cq, lane, o,
                                    [&](int e, const u32x4& unit) {
                        const int rs = CB == 4 ? 0 : e / (4 * SEG), col = ao0 * SEG + (CB == 4 ? e : e % (4 * SEG));
                        const uint32_t off = CB == 4 || col < sa.d_out ? (uint32_t)(rs * (int)sa.ld_out + col) * 4u : 0x80000000u;
                        __builtin_amdgcn_raw_buffer_store_b128(unit,
                                                               ys, off, 0, 2);
                    });
                } else {
#pragma unroll
                    for (int nt = 0; nt < 8; ++nt) o[nt] *= k;
                    const u32x4 unit = sa.out == 0 ? pack16<0>(o) : pack16<2>(o);
                    const int col = (ao0 + gq) * SEG + cq * 8;
                    const uint32_t off = CB == 4 || col < sa.d_out ? (uint32_t)(rq * (int)sa.ld_out + col) * 2u : 0x80000000u;
                    __builtin_amdgcn_raw_buffer_store_b128(unit,
                                                           ys, off, 0, 2);
                }
            }
            continue;
        } else {
        m = wave_absmax<CB>(m);                          // over the lanes that share the row
        if (g == 0 && cl == 0) wmax[rsub * 16 + wave] = m;
        __syncthreads();    // also: every wave is done reading this row's operands from LDS
        {
            // All waves' maxima with one LDS latency (a read per wave, each waiting for the one before it, takes nw of
            // them while the whole workgroup waits: 14336-wide rows, b = 4, 512 MiB 154 -> 145 us).  Up to four 16-byte
            // reads in flight, or, where their registers spill (KK = 5 with several rows per pass or b = 4: 80 registers for
            // 32 values and 20 of operand tiles; 8960-wide rows 196 -> 165 us), one read: the lane of chunk cl takes RPW of
            // the row's 16 slots and the lanes that share the row do the rest.  (Elsewhere the reads are the faster:
            // 4864-wide rows 148 against 151 us.)
            int gq, cq, rq;
            wg_lane<CB>(lane, gq, cq, rq);
            if constexpr (KK == 5 && (CB < 4 || BITS == 4)) {
                uint32_t u[RPW];
                __builtin_memcpy(u, &wmax[rq * 16 + cq * RPW], sizeof u);
                uint32_t mu = u[0];
#pragma unroll
                for (int i = 1; i < RPW; ++i) mu = max(mu, u[i]);
                m = __uint_as_float(lanes_max_u32<CB>(mu));
            } else {
                constexpr int NQ = (2 * KK + 3) / 4;
                f32x4 q[NQ];
#pragma unroll
                for (int i = 0; i < NQ; ++i) q[i] = *reinterpret_cast<const f32x4*>(&wmax[rq * 16 + 4 * i]);
                m = 0.0f;
#pragma unroll
                for (int i = 0; i < NQ; ++i) m = absmax4(m, q[i]);
            }
        }
        // ---- phase 4
        if constexpr (SINK == kWgGrid) {
            // one histogram: the rows of a pass one after the other
            uint64_t* const hist = reinterpret_cast<uint64_t*>(stage);
            const int NT = (int)blockDim.x, t = (int)threadIdx.x;
            for (int rs = 0; rs < RPW && pass * RPW + rs < a.rows; ++rs) {
                for (int i = t; i < Grid::WORDS / 2; i += NT) reinterpret_cast<u32x4*>(hist)[i] = u32x4{0u, 0u, 0u, 0u};
                float mr = m;
                if constexpr (RPW > 1) {
                    mr = 0.0f;
                    for (int w = 0; w < nw; ++w) mr = __builtin_fmaxf(mr, wmax[rs * 16 + w]);
                }
                const typename Grid::Scale sc = Grid::scale(mr, sa.inv_norm);
                __syncthreads();
                double q2 = 0.0;
                float fl = flip;
                asm volatile("" : "+v"(fl));             // (or the signed values are kept from row to row)
                if (RPW == 1 || rsub == rs) {
                    // (a row with an infinity or a NaN has one in every value, or its maximum is infinite: its error is NaN)
                    if (!(__builtin_fabsf(acc[0][0]) < __builtin_inff()) || !(mr < __builtin_inff())) q2 = __builtin_nan("");
#pragma unroll
                    for (int nt = 0; nt < 8; ++nt)
#pragma unroll
                        for (int ip = 0; ip < 4; ++ip) Grid::add(hist, acc[nt][ip] * fl, sc.s, q2, lane);
                }
                __syncthreads();
                q2 = Grid::finish(hist, q2, t, NT, tot);
#pragma unroll
                for (int k = 0; k < SUMS; ++k) {
                    const int c1 = 1 + t + k * NT;
                    if (c1 < kGridRatios) sum[k] += Grid::error(hist, c1, q2, sc);
                }
                __syncthreads();
            }
            continue;
        }
        if constexpr (QE) {
            const ClipView clips = clip_view(sa.clips);
            const int per = (clips.n + (int)gridDim.y - 1) / (int)gridDim.y, k0 = (int)blockIdx.y * per, k1 = k0 + per < clips.n ? k0 + per : clips.n;
            float v[32];
#pragma unroll
            for (int nt = 0; nt < 8; ++nt)
#pragma unroll
                for (int ip = 0; ip < 4; ++ip) v[nt * 4 + ip] = acc[nt][ip];
            // the sums run over the lanes that share a row of the pass: CB lane bits and the four DPP rows
            qe_candidates<32, BITS, CB>(v, m, flip, clips, k0, k1, [&](int k, float e2) {
                if (g == 0 && cl == 0) esum[wave][rsub][k] = e2;
            });
            __syncthreads();   // the next row writes esum only after two more barriers
            for (int i = threadIdx.x; i < RPW * (k1 - k0); i += blockDim.x) {
                const int rs = i / (k1 - k0), k = k0 + i - rs * (k1 - k0);
                const int64_t orow = pass * RPW + rs;
                if (orow < a.rows) {
                    float t = 0.0f;
                    for (int w = 0; w < nw; ++w) t += esum[w][rs][k];
                    const double nn = (double)pb * (double)SEG;
                    sa.partial[orow * clips.n + k] = (double)t / (nn * nn);
                }
            }
            continue;
        }
        // Where registers are tight (several rows per pass; b = 4 at KK = 2, 3) the lane's place is worked out again here, so
        // that nothing of it is held through the phases before (512 MiB of rows, b = 4: 8960 wide 229 -> 196 us, 11008 wide
        // 161 -> 151).  Elsewhere holding it is the faster: 14336 wide, b = 4 145 against 150, 18944 wide, b = 3 169 against
        // 173, 1792 wide (KK = 1) 132 against 134.
        constexpr bool AGAIN = KK > 1 && (CB < 4 || (BITS == 4 && KK <= 3));
        int gq = g, cq = cl, rq = rsub, lq = lane;
        if constexpr (AGAIN) {
            wg_lane<CB>(lane, gq, cq, rq);
            asm volatile("" : "+v"(lq));
        }
        const int64_t row = pass * RPW + rq;
        const bool live = CB == 4 || row < a.rows;
        const float fl = AGAIN ? wg_flip<CB>(cq) : flip;
        // (18944 wide, b = 4: the compiler's own order of the shift-adds needs fewer registers: 4096 rows 53 -> 51.5 us; other
        // forms are the faster with the chain, 8960 wide 170 against 179)
        constexpr bool FREE = KK == 5 && CB == 4 && BITS == 4;
        // (2^b - 1) / (clip m) from a float pair of the constant: reciprocal, Newton step, correction
        const float s = m > 0.0f ? fl * div_pair(c1h, c1l, m) : 0.0f;
        uint32_t* out = a.codes + row * (int64_t)(SEG * BITS / 32) * pb;   // used by live lanes only
#pragma unroll
        for (int ip = 0; ip < 4; ++ip) {
            const int ao = 16 * wave + 4 * ip + gq;      // output block row of this register
            const uint32_t w = Quant<BITS>::template pack8<FREE>(acc[0][ip], acc[1][ip], acc[2][ip], acc[3][ip], acc[4][ip],
                                                                 acc[5][ip], acc[6][ip], acc[7][ip], s);
            if constexpr (CB == 4) {
                const int word = ao * 16 + cq;
                if (BITS == 4) {
                    if (ao < pb) store_codes(out + word, w);
                } else {
                    stage24(stage, word, w);            // block rows >= pb land beyond the copied part
                }
            } else if (ao < pb) {
                // the pass's rows are staged one after the other, each pb * 2^CB groups of 8 codes
                if (BITS == 4) {
                    if (live) store_codes(out + (ao << CB) + cq, w);
                } else {
                    stage24(stage, ((rq * pb + ao) << CB) + cq, w);
                }
            }
        }
        if (BITS == 3 && CB < 4) {
            // as below; a wave's 16 block rows are 3 * 2^CB 16-byte units in each row of the pass
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            constexpr int UPR = 3 << CB;
            const int rs = lq / UPR;
            const int unit = UPR * wave + lq % UPR;   // the row has pb * UPR / 16 units
            const int64_t orow = pass * RPW + rs;
            if (lq < 48 && unit * 16 < pb * UPR && orow < a.rows)
                __builtin_nontemporal_store(
                    *reinterpret_cast<const u32x4*>(stage + (size_t)rs * pb * UPR + unit * 16),
                    reinterpret_cast<u32x4*>(a.codes + orow * (int64_t)(SEG * 3 / 32) * pb) + unit);
        }
        if (BITS == 3 && CB == 4) {
            // a wave's 16 block rows are 768 contiguous bytes of the packed row, written and read
            // back by the same wave: no workgroup barrier, only the wave's own LDS ordering
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int unit = 48 * wave + lq;          // 16-byte units; the row has 3 pb of them
            if (lq < 48 && unit < 3 * pb)
                __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(stage + unit * 16),
                                            reinterpret_cast<u32x4*>(out) + unit);
        }
        if (wave == 0 && gq == 0 && cq == 0 && live) a.scales[row] = (float)(a.c2 * (double)m);
        }
    }
    if constexpr (SINK == kWgGrid) {
#pragma unroll
        for (int k = 0; k < SUMS; ++k) {
            const int c1 = 1 + (int)threadIdx.x + k * (int)blockDim.x;
            if (c1 < kGridRatios) sa.dev->grid_sums[blockIdx.x][c1] = sum[k];
        }
    }
}


template <int SINK>
using WgKernel = void (*)(RQ_WAVE_PARAMS, WgArgs<SINK>);

// One launch: as many workgroups as fit the chip (registers, LDS), each looping over rows.
template <int KK, int SINK>
int wg_launch(const rq_hadamard* h, WgKernel<SINK> fn, const WaveArgs& a, int pb, int cb, size_t lds, const WgArgs<SINK>& sa,
              hipStream_t s, int waves_per_simd = wg_waves_per_simd<KK>()) {
    const int nw = (pb + 15) / 16;
    int per_cu = (int)((size_t)h->max_lds / (lds + 128));
    const int by_waves = 4 * waves_per_simd / nw;   // see the register budget note at the kernel
    if (per_cu > by_waves) per_cu = by_waves;
    if (per_cu < 1) per_cu = 1;
    const int64_t cap = (int64_t)h->num_cu * per_cu;
    const int rpw = 16 >> cb;
    const int64_t passes = (a.rows + rpw - 1) / rpw;
    unsigned shares = 1;
    if constexpr (SINK == kWgError) {
        // few rows: the clip ratios of a pass over as many workgroups as make about ten waves per compute unit (32 x 8960, 32
        // ratios: 31.9 -> 12.3 us; beyond that the repeated rotations cost more than the idle units: 512 x 5120 with four
        // shares 16.4 -> 20.4)
        const int64_t want = (int64_t)h->num_cu * 10 / (passes * nw);
        shares = (unsigned)(want < 1 ? 1 : want > sa.max_shares ? sa.max_shares : want);
    }
    const unsigned grid = (unsigned)(passes < cap ? passes : cap);
    launch_kernel(fn, dim3(grid, shares), dim3(64 * nw), lds, s, RQ_WAVE_VALUES(a, pb), sa);
    return launch_rc();
}

}  // namespace
}  // namespace rq
