// Rotation and quantization of rows whose block splits into pairs of rows: the form of the workgroup block kernel
// (wg_block_kernel.h) for many rows of n = 128 pb columns, pb = 2 hb.
//
// With a the even and b the odd block rows of a row, the blocks of order 2 (q + 1) (Paley's second construction) and the
// Kronecker products with H_2 are a butterfly over halves:
//     y_2i = e_i + f_i, y_2i+1 = e_i - f_i   with   e = C a + D b, f = C b - D a,
// C of order hb and D diagonal (-1 for the second construction, nothing for a product).  So the contraction is half as long: 16 NW
// output pairs take ceil(NW / 2) steps of 32 for each of e and f instead of NW steps for twice the rows, at one more addition
// a value.  D costs no step: where the last step is half empty (NW odd), its upper lanes read the
// wave's own 16 rows of the other half, and the operand tile has the diagonal there.
//
// A wave holds 16 rows of e and of f, 64 accumulators, and has 128 registers (four waves a SIMD).  Of five-wave workgroups a
// compute unit takes only two at a time (3 3 2 2 waves a SIMD; a third would fit, 4 4 4 3, and waits; 4096 x 18944 52 us): three
// rows share a workgroup there (47), and two where a row takes six waves.  Each row's waves meet at a barrier of their own
// (row_barrier), or the rows would load, contract and quantize in step.
//
// What bounds it: vector issue (910 instructions a wave and row, four fifths of the fullest SIMD's cycles at 16384 x 18944) at the
// clock that the power limit leaves; the matrix cores are busy 16 percent of the time, 24 in the other form.  us a call, other form -> this:
// 18944 wide, 1024 rows, b = 4 17.2 -> 15.7, 4096 rows, b = 3 52.8 -> 47.2, 10000 rows, b = 4 127.7 -> 111.2; 14336 wide, 700 rows, b = 4 9.8
// -> 8.6, 3000 rows, b = 4 28.8 -> 27.6, 10000 rows, b = 3 81.6 -> 75.2; 28672 wide, 300 rows, b = 3 13.3 -> 10.7, 1000 rows, b = 4 26.4 -> 22.9,
// 4096 rows, b = 3 82.4 -> 68.3; 2048 rows: 16384, b = 4 21.3 and 21.3, 20480, b = 3 28.2 -> 25.3, 24576, b = 4 34.2 -> 31.4, 25088, b = 4 39.7 ->
// 34.5, 32768, b = 3 45.4 -> 36.6.
// Scales against 64 bits, rms (largest), either form: 18944 wide 4.8 - 5.5e-8 (1.6e-7), 14336 4.6 - 5.4e-8 (1.8e-7).
// A row with infinities: 0 inf is NaN where an operand tile has zeros, so with a diagonal all values of the 32 block rows of an
// infinity's wave are NaN, which the maximum passes over.  Where every wave of a row has an infinity nothing else is left; the row is
// then taken a second time for the answer of the other form (infinity_signs): an infinite scale if some value is the sum of
// infinities of one sign, 0 if there is none or the row has a NaN.
#pragma once
#include "wave_common.h"

namespace rq {
namespace {

// Rows of a workgroup.
constexpr int pair_rows(int nw) { return nw == 5 ? 3 : nw == 6 ? 2 : 1; }

// LDS of a row: the operands in groups of 16 rows of a half, 512 bytes for each of the eight column tiles (lane order, as in
// the workgroup block kernel), a group of zeros where the last step's upper lanes have none, and the packed codes (b = 3).
template <int NW, bool DIAG>
constexpr size_t pair_ops_bytes() { return (size_t)(2 * NW + (!DIAG && (NW & 1) ? 1 : 0)) * 4096; }
template <int NW, bool DIAG>
constexpr size_t pair_lds_bytes() { return pair_ops_bytes<NW, DIAG>() + (size_t)NW * 32 * 48; }

// A barrier of the NW waves of a row: each counts itself in and waits until all have (`target`: the count by then).  Every
// wave of a workgroup is resident and counts itself before it waits, and a row's waves pass the same number of barriers, so
// every wait ends.
template <int NW>
__device__ __forceinline__ void row_barrier(uint32_t* count, uint32_t& target, int lane) {
    target += NW;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own LDS traffic is done
    if (lane == 0) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while ((int32_t)(__builtin_amdgcn_readfirstlane(__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) - target) < 0)
        __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");
}

// Infinities among a lane's operands (eight column tiles of 16 bytes from `at`) to 1 with their sign, everything else to 0; how many
// there were, more than a row holds for a NaN.  The sums of such rows are exact: one as large as the number of infinities has
// added them all with one sign.  (In LDS, behind the row's phase 1, which stays as it is for it.)
template <bool F16>
__device__ __forceinline__ uint32_t infinity_signs(uint8_t* at) {
    constexpr uint32_t INF = F16 ? 0x7c00u : 0x7f80u;
    uint32_t count = 0, one = F16 ? 0x3c00u : 0x3f80u, nans = 1u << 20;
    asm volatile("" : "+s"(one), "+s"(nans));            // (or both are held in vector registers for the whole launch)
#pragma unroll 1
    for (int i = 0; i < 32; ++i) {
        uint32_t* const two = reinterpret_cast<uint32_t*>(at + (i >> 2) * 512) + (i & 3);
        const uint32_t v = *two, lo = v & 0x7fffu, hi = (v >> 16) & 0x7fffu;
        *two = (v & 0x80008000u) | (lo == INF ? one : 0u) | (hi == INF ? one << 16 : 0u);
        count += (lo == INF) + (hi == INF);
        if (lo > INF || hi > INF) count |= nans;
    }
    return count;
}

// NW = ceil(hb / 16) waves a row; DIAG: D is not zero (NW odd).
template <int NW, bool DIAG, int BITS, bool F16>
__global__ __launch_bounds__(64 * NW * pair_rows(NW)) __attribute__((amdgpu_waves_per_eu(4)))
void k_wg_pair(RQ_WAVE_PARAMS) {
    RQ_WAVE_ARGS(a);
    RQ_WAVE_BLOCK_ROWS(pb);
    static_assert(!DIAG || (NW & 1), "the other half's rows take the upper half of the last step");
    constexpr int STEPS = (NW + 1) / 2, HALF = NW * 4096, ROWS = pair_rows(NW);
    constexpr bool ODD = (NW & 1) != 0;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = ROWS > 1 ? wave_all / NW : 0, wave = wave_all - sub * NW;   // row of the workgroup, wave of the row
    const int tid = threadIdx.x - sub * 64 * NW;
    uint8_t* const ops = lds_raw + sub * pair_lds_bytes<NW, DIAG>();
    uint8_t* const stage = ops + pair_ops_bytes<NW, DIAG>();
    constexpr int WM = (NW + 3) / 4 * 4;
    __shared__ __attribute__((aligned(16))) float wmax_all[ROWS * WM];
    float* const wmax = wmax_all + sub * WM;
    __shared__ uint32_t counts[ROWS];
    uint32_t target = 0;
    bool again = false;                                  // DIAG: the row is taken a second time
    __shared__ uint32_t infinities[DIAG ? ROWS : 1];     // of such a row
    auto barrier = [&] {
        if constexpr (ROWS > 1) row_barrier<NW>(&counts[sub], target, lane);
        else __syncthreads();
    };
    if constexpr (ROWS > 1) {
        if (threadIdx.x < ROWS) counts[threadIdx.x] = 0;
        __syncthreads();
    }
    const int g = lane >> 4, cphys = lane & 15;
    const int c = (cphys & 4) ? (cphys ^ 3) : cphys;     // logical column group (8 columns)

    u32x4 A[STEPS];
#pragma unroll
    for (int k = 0; k < STEPS; ++k) A[k] = a.tiles[(wave * STEPS + k) * 64 + lane];
    auto uniform = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
    const float c1h = uniform((float)a.c1), c1l = uniform((float)(a.c1 - (double)c1h));
    const float flip = (__builtin_popcount(c) & 1) ? -1.0f : 1.0f;

    // Phase 1: the lane's eight rows of one half, block rows 2 (16 wave + 8 (g >> 1) + t) + (g & 1), t = 0 .. 7, are the
    // 16 bytes that reader lane (g >> 1, c) of the group takes of each column tile.  Rows at or beyond pb lie beyond d and
    // read as zero.
    const int eoff = (32 * wave + 16 * (g >> 1) + (g & 1)) * 128 + c * 8;
    static_assert((32 * (NW - 1) + 17) * 256 + 15 * 16 < 0x10000, "bytes of the first of them");
    uint8_t* const wr0 = ops + (g & 1) * HALF + wave * 4096 + ((g >> 1) * 16 + cphys) * 16;
    const uint8_t* const rd0 = ops + (g >> 1) * 4096 + ((g & 1) * 16 + cphys) * 16;
    const uint8_t* last[2];                              // the last step's operands, NW odd
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
        last[hh] = rd0 + hh * HALF + (STEPS - 1) * 8192;
        if (ODD && g >= 2) last[hh] = ops + (DIAG ? (1 - hh) * HALF + wave * 4096 : 2 * HALF) + ((g & 1) * 16 + cphys) * 16;
    }
    if (!DIAG && ODD)
        for (int i = tid; i < 256; i += 64 * NW) reinterpret_cast<u32x4*>(ops + 2 * HALF)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid < WM) wmax[tid] = 0.0f;
    if (DIAG && tid == 0) infinities[sub] = 0;

    // (The next row's loads beside the quantizer, into the registers that it frees: no difference, 4096 x 28672, b = 3 64.6 and
    // 64.2, 2048 x 32768, b = 4 39.2 and 40.4, or slower, 4096 x 18944 44.9 and 46.1.)
    for (int64_t row = (int64_t)blockIdx.x + (int64_t)sub * gridDim.x; row < a.rows; row += again ? 0 : (int64_t)gridDim.x * ROWS) {
        const RowView xv = row_view(a.X + row * a.ld, a.d);
        u32x4 R[8];
        // (One address register for all: two block rows on, 512 bytes, as the instruction's own offset, which the range check counts
        // with the register.  The masked register is known to stay below 2^16, so that the sum may be formed in the check.)
        uint32_t off = (uint32_t)eoff * 2u;
        asm volatile("" : "+v"(off));
        off &= 0xffffu;
#pragma unroll
        for (int t = 0; t < 8; ++t) R[t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xv.rs, off + t * 512u, 0, 2));
#pragma unroll
        for (int ic = 0; ic < 8; ++ic) {
            const uint32_t sel = (ic & 1) ? 0x07060302u : 0x05040100u;
            u32x4 v;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = __builtin_amdgcn_perm(R[2 * k + 1][ic >> 1], R[2 * k][ic >> 1], sel);
            *reinterpret_cast<u32x4*>(wr0 + ic * 512) = v;
        }
        if (DIAG && __builtin_expect(again, 0)) atomicAdd(&infinities[sub], infinity_signs<F16>(wr0));
        barrier();
        // ---- phase 2: e in acc[0], f in acc[1].  (Waves in their vector phases go first, as in the workgroup block kernel.)
        __builtin_amdgcn_s_setprio(0);
        f32x4 acc[2][8];
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) acc[0][nt] = acc[1][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        {
            // Column tiles 0 - 3 of both halves go over all steps first, then 4 - 7, and the pairs and first two column stages of
            // tiles 0 - 3, the same additions as in phase 3, are issued between the matrix-core instructions of the others; eight
            // accumulators in turn, reads DEPTH ahead.  us a call, all tiles at once, two ahead -> so: 4096 x 18944, b = 3 48.6 -> 47.2,
            // 10000, b = 4 114.7 -> 111.2, 10000 x 14336 78.2 -> 75.2, 2048 x 24576 32.0 -> 31.4; 1024 x 18944 15.3 and 15.7, 28672 wide
            // 0 - 2 percent less (two or four ahead, so: 4096 x 18944, b = 4 48.5 and 47.4 where three have 47.0).
            constexpr int DEPTH = 3, ITEMS = 16 * STEPS;
            auto step = [](int i) { return i % (8 * STEPS) / 8; };
            auto tile = [](int i) { return i / (8 * STEPS) * 4 + i % 8 / 2; };
            auto read_item = [&](int i) {
                const int k = step(i), nt = tile(i), hh = i & 1;
                const uint8_t* p = ODD && k == STEPS - 1 ? last[hh] : rd0 + hh * HALF + k * 8192;
                return *reinterpret_cast<const u32x4*>(p + nt * 512);
            };
            // additions j of 48, two operations each: the pairs of tiles 0 - 3, their first column stage, their second
            auto addition = [&](int j) __attribute__((always_inline)) {
                const int r = j % 4, q = j / 4 % 4, st = j / 16 - 1;
                const int h0 = st < 0 ? 0 : q / 2, h1 = st < 0 ? 1 : q / 2;
                const int t0 = st < 0 ? q : st == 0 ? 2 * (q % 2) : q % 2, t1 = st < 0 ? q : st == 0 ? t0 + 1 : t0 + 2;
                const float u = acc[h0][t0][r], v = acc[h1][t1][r];
                acc[h0][t0][r] = u + v;
                acc[h1][t1][r] = u - v;
            };
            u32x4 minus = A[STEPS - 1];                  // the last step's tile for f
            if constexpr (DIAG) {
                uint32_t flip_d = g >= 2 ? 0x80008000u : 0u;
                asm volatile("" : "+v"(flip_d));         // (or the tile is held from pass to pass, and four registers spill)
#pragma unroll
                for (int k = 0; k < 4; ++k) minus[k] ^= flip_d;
            }
            u32x4 ring[DEPTH];
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) ring[i] = read_item(i);
            auto item = [&](int i) __attribute__((always_inline)) {
                __builtin_amdgcn_sched_barrier(0);
                const int k = step(i), nt = tile(i), hh = i & 1;
                acc[hh][nt] = mfma_pm1<F16>(DIAG && hh && k == STEPS - 1 ? minus : A[k], ring[i % DEPTH], acc[hh][nt]);
                if (i + DEPTH < ITEMS) ring[i % DEPTH] = read_item(i + DEPTH);
            };
#pragma unroll
            for (int i = 0; i < ITEMS / 2; ++i) item(i);
            item(ITEMS / 2);
#pragma unroll
            for (int i = 1; i < ITEMS / 2; ++i) {
                constexpr int OF = ITEMS / 2 - 1;
                item(ITEMS / 2 + i);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (48 * (i - 1) / OF + j < 48 * i / OF) addition(48 * (i - 1) / OF + j);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- phase 3: what is left of the pairs and column stages, the row's maximum
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int nt = 4; nt < 8; ++nt) {
            const f32x4 u = acc[0][nt], v = acc[1][nt];
            acc[0][nt] = u + v;
            acc[1][nt] = u - v;
        }
        float m = 0.0f;
        int cs = c;
        asm volatile("" : "+v"(cs));                     // (the signs are worked out again in every pass)
        float sf[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) sf[b] = __uint_as_float(0x3F800000u | ((uint32_t)(cs >> b) << 31));
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
            for (int s = 1; s < 8; s <<= 1)
#pragma unroll
                for (int nt = 0; nt < 8; ++nt)
                    if (!(nt & s) && (nt | s) >= 4) {
                        const f32x4 u = acc[hh][nt], v = acc[hh][nt | s];
                        acc[hh][nt] = u + v;
                        acc[hh][nt | s] = u - v;
                    }
#pragma unroll
            for (int nt = 0; nt < 8; ++nt) {
                f32x4 v = acc[hh][nt];
                lane_stages_fused(v, sf[0], sf[1], sf[2], sf[3]);
                acc[hh][nt] = v;
                m = absmax4(m, v);
            }
        }
        m = wave_absmax<4>(m);
        if (lane == 0) wmax[wave] = !DIAG || m > 0.0f ? m : acc[0][0][0];   // (0, or NaN of a wave that has nothing else)
        barrier();    // also: every wave is done reading this row's operands
        [[maybe_unused]] float first;
        {
            f32x4 q[WM / 4];
#pragma unroll
            for (int i = 0; i < WM / 4; ++i) q[i] = *reinterpret_cast<const f32x4*>(&wmax[4 * i]);
            m = 0.0f;
#pragma unroll
            for (int i = 0; i < WM / 4; ++i) m = absmax4(m, q[i]);
            first = q[0][0];
        }
        // ---- phase 4
        float s = 0.0f;
        bool lost = false;                               // (the row's: all of its waves see the same maxima)
        if (m > 0.0f) s = flip * div_pair(c1h, c1l, m);
        else if (DIAG) lost = __builtin_amdgcn_readfirstlane(first != first);
        if (DIAG && __builtin_expect(again, 0)) s = __builtin_nanf("");   // (the row's codes stay those of NaN)
        // the row's codes as a buffer resource: block rows at or beyond pb lie outside it and are not stored
        const auto out = __builtin_amdgcn_make_buffer_rsrc(a.codes + row * (int64_t)(4 * BITS) * pb, 0, 16 * BITS * pb, 0x00020000);
        const int r0 = 32 * wave + 2 * g;
#pragma unroll
        for (int ip = 0; ip < 4; ++ip)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {             // block row r0 + 8 ip + hh (the two halves of a cache line one after the other)
                const f32x4(&v)[8] = acc[hh];
                const uint32_t w = Quant<BITS>::pack8(v[0][ip], v[1][ip], v[2][ip], v[3][ip], v[4][ip], v[5][ip], v[6][ip], v[7][ip], s);
                if (BITS == 4)
                    __builtin_amdgcn_raw_buffer_store_b32(w, out, r0 * 64 + c * 4 + (8 * ip + hh) * 64, 0, 2);
                else
                    stage24(stage, r0 * 16 + c + (8 * ip + hh) * 16, w);
            }
        if (BITS == 3) {
            // a wave's 32 block rows are 1536 consecutive bytes, written and read back by the same wave
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int at = 1536 * wave + 16 * lane;
            __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(stage + at), out, at, 0, 2);
            if (lane < 32) __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(stage + at + 1024), out, at + 1024, 0, 2);
        }
        if (tid == 0) {
            if (DIAG && __builtin_expect(again, 0)) {
                m = m == (float)infinities[sub] ? __builtin_inff() : 0.0f;
                infinities[sub] = 0;                     // (counted in again two barriers from here at the earliest)
            }
            a.scales[row] = (float)(a.c2 * (double)m);
        }
        if constexpr (DIAG) again = lost && !again;
    }
}

}  // namespace
}  // namespace rq
