// Rotation-free quantizers for short groups of values (head rows).
// First the asymmetric quantizer in groups of 128 values (section 5.1, the KV-cache setting, for
// a tensor whose rotation is fused into the producing weights - the value cache): per group
// lo = clip * min, hi = clip * max, Delta = (hi - lo) / (2^b - 1), code = clamp(rne((x - lo) / Delta),
// 0, 2^b - 1).  A group is the 16 lanes of a DPP row, 8 values per lane; a wave takes four groups
// per pass.  The extremes cross the 16 lanes with four DPP steps; the codes are taken in fp32 as
// in the rotating kernels (centred on the value that maps to the middle code), and - since
// un-rotated inputs can sit exactly on rounding ties - every value whose fp32 quotient is within 2e-5
// of a tie (wider for a group that lies far from zero, where fp32 places the centre less well) is
// retaken with the exact fp64 quotient.
#include "wave_common.h"

namespace rq {
namespace {

// Eight values as they are stored.  DT: 0 bf16, 1 fp32, 2 fp16.  ALIGNED: 16-byte loads (X 16-byte aligned, ld a multiple of
// 8 / 4).
template <int DT>
struct Raw8 { uint32_t w[DT == 1 ? 8 : 4]; };
template <int DT, bool ALIGNED>
__device__ __forceinline__ Raw8<DT> load_raw8(const void* X, int64_t idx) {
    Raw8<DT> r;
    if constexpr (ALIGNED) {
        const u32x4* p = reinterpret_cast<const u32x4*>(static_cast<const char*>(X) + idx * (DT == 1 ? 4 : 2));
#pragma unroll
        for (int h = 0; h < (DT == 1 ? 2 : 1); ++h) {
            const u32x4 a = __builtin_nontemporal_load(p + h);
#pragma unroll
            for (int i = 0; i < 4; ++i) r.w[4 * h + i] = a[i];
        }
    } else if constexpr (DT == 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) r.w[i] = static_cast<const uint32_t*>(X)[idx + i];
    } else {
        const uint16_t* p = static_cast<const uint16_t*>(X) + idx;
#pragma unroll
        for (int i = 0; i < 4; ++i) r.w[i] = (uint32_t)p[2 * i] | ((uint32_t)p[2 * i + 1] << 16);
    }
    return r;
}
template <int DT>
__device__ __forceinline__ void to_float8(const Raw8<DT>& r, float (&x)[8]) {
    if constexpr (DT == 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = __uint_as_float(r.w[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (DT == 2) {
                x[2 * i] = (float)__builtin_bit_cast(_Float16, (uint16_t)r.w[i]);
                x[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(r.w[i] >> 16));
            } else {
                x[2 * i] = __uint_as_float(r.w[i] << 16);
                x[2 * i + 1] = __uint_as_float(r.w[i] & 0xffff0000u);
            }
        }
    }
}

// Minima and maxima of four passes over the 16 lanes of a DPP row: lane c of the row ends with those of pass c mod 4.  The first
// two steps merge passes two and two while they cross the lane bits that name them.  (Assembly: the compiler does not fold a
// DPP operand into a float min / max, and first passes each operand through a canonicalizing max.  The s_nop keep two wait
// states between a vector write of a register and a DPP read of it.)
__device__ __forceinline__ void row_min_max4(const float (&mn)[4], const float (&mx)[4], int lane, float& lo, float& hi) {
    const bool b0 = lane & 1, b1 = lane & 2;
    float n0 = b0 ? mn[1] : mn[0], n1 = b0 ? mn[3] : mn[2], x0 = b0 ? mx[1] : mx[0], x1 = b0 ? mx[3] : mx[2];
    asm("s_nop 1\n\t"
        "v_min_f32_dpp %0, %4, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %5, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %2, %6, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %3, %7, %3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
        : "+&v"(n0), "+&v"(n1), "+&v"(x0), "+&v"(x1)
        : "v"(b0 ? mn[0] : mn[1]), "v"(b0 ? mn[2] : mn[3]), "v"(b0 ? mx[0] : mx[1]), "v"(b0 ? mx[2] : mx[3]));
    lo = b1 ? n1 : n0;
    hi = b1 ? x1 : x0;
    asm("s_nop 1\n\t"
        "v_min_f32_dpp %0, %2, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %3, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_min_f32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %1, %1 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_min_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1"
        : "+&v"(lo), "+&v"(hi)
        : "v"(b1 ? n0 : n1), "v"(b1 ? x0 : x1));
}
// Lane u of each quad to all four.
template <int U>
__device__ __forceinline__ float quad_lane(float x) { return __uint_as_float(dpp_u<0x55 * U>(__float_as_uint(x))); }

// max |y_k| of eight floats as three-operand instructions with magnitude operands
__device__ __forceinline__ float absmax8(const float (&y)[8]) {
    float m;
    asm("v_max3_f32 %0, |%1|, |%2|, |%3|\n\t"
        "v_max3_f32 %0, %0, |%4|, |%5|\n\t"
        "v_max3_f32 %0, %0, |%6|, |%7|\n\t"
        "v_max_f32 %0, %0, |%8|"
        : "=&v"(m)
        : "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]), "v"(y[4]), "v"(y[5]), "v"(y[6]), "v"(y[7]));
    return m;
}

// Bound: vector issue on large tensors (262 144 waves: port 89 % busy, 430 instructions a wave, 574 before); 16 376 waves are a
// few rounds and leave it half idle (51 %).
// A wave takes four passes of four groups; extremes, multiplier, centre, tie window and results of its
// sixteen groups are worked out once, lane c of a DPP row for pass c mod 4, and go back to the lanes of a pass with one quad
// permutation each; sixteen groups that lie one behind the other (ld = d) are read from one address.  bf16, b = 3, before (all of
// it once a pass and by every lane, a 64-bit address for each load) -> now: 262 016 groups 17.0 -> 16.1 us (15.6 since
// the arguments come in registers and the loop's step is hidden, see wave_common.h), 1 048 576 63.3 ->
// 55.7 (5.2 -> 5.9 TB/s); b = 4, 2 097 152 groups 125 -> 110.
template <int BITS, int DT, bool ALIGNED>
__global__ __launch_bounds__(64) void k_plain_asym(const void* X, int64_t n_groups, int gpr, int gpr_shift, uint32_t gpr_magic, int64_t ld, double clip,
                                                   uint32_t* codes, float* scales, float* mins) {
    constexpr int U = 4;
    constexpr double kL = (double)((1 << BITS) - 1);
    constexpr double kMid = (double)(1 << (BITS - 1)) / kL;     // centre of the code range
    const int lane = threadIdx.x;
    const int g = lane >> 4, c = lane & 15;
    constexpr float kMidF = (float)kMid;
    const float c1f = (float)(kL / clip), clipf = (float)clip;
    // a wave takes U passes of four groups per iteration, all loads issued before the first is used
    for (int64_t g0 = (int64_t)blockIdx.x * (4 * U); g0 < n_groups; g0 = next_item<false, kMostGroups * 4 * U>(g0)) {
        Raw8<DT> raw[U];
        const int left = n_groups - g0 < 4 * U ? (int)(n_groups - g0) : 4 * U;
        if (left == 4 * U && ld == (int64_t)gpr * 128) {
            // sixteen consecutive groups: one base, one lane offset
#pragma unroll
            for (int u = 0; u < U; ++u)
                raw[u] = load_raw8<DT, ALIGNED>(static_cast<const char*>(X) + g0 * (128 * (DT == 1 ? 4 : 2)), u * 512 + lane * 8);
        } else {
            // uniform over the wave, so scalar work - but a 64-bit scalar division is a hundred instructions:
            // a shift where gpr is a power of two (the usual widths), else a 32-bit division if that will do
            int64_t row0;
            if (gpr_shift >= 0) row0 = g0 >> gpr_shift;
            else if (n_groups <= 0xffffffffll) row0 = (uint32_t)g0 / (uint32_t)gpr;
            else row0 = g0 / gpr;
            const uint32_t rem0 = (uint32_t)(g0 - row0 * gpr);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int gi = u * 4 + g;
                // (row, group of the row) from the iteration's uniform split plus a small offset, whose
                // quotient by gpr is a multiply-high with ceil(2^32 / gpr): exact while offset * gpr < 2^32
                const uint32_t off = rem0 + (uint32_t)(gi < left ? gi : left - 1);
                const uint32_t k = gpr == 1 ? off : __umulhi(off, gpr_magic);
                const int64_t row = row0 + k;
                const uint32_t gc = off - k * (uint32_t)gpr;
                raw[u] = load_raw8<DT, ALIGNED>(X, row * ld + (int64_t)gc * 128 + c * 8);
            }
        }
        // outputs of the iteration: a base in scalar registers plus per-lane offsets
        uint32_t* const cbase = codes + g0 * (4 * BITS);
        const uint32_t code_off = (uint32_t)(g * (4 * BITS) + (BITS == 4 ? c : (c >> 2) * 3 + (c & 3))) * 4u;
        uint32_t* const out0 = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(cbase) + code_off);
        float x[U][8], mn, mx;
        {
            float n[U], m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                to_float8<DT>(raw[u], x[u]);
                n[u] = min8(x[u]);
                m[u] = max8(x[u]);
            }
            row_min_max4(n, m, lane, mn, mx);
        }
        // Group parameters in fp32.  What they cost the pre-round value t in accuracy: the range r
        // and the multiplier s (reciprocal plus one Newton step) about 3e-7 relative, |t - mid| <= 8;
        // the centre about 2.5 ulp, which in units of t is 3e-7 |cen| s - small for a group that
        // straddles zero, unbounded for a narrow group far from it.  Both go into the tie window, so
        // a group whose offset swamps its range is simply taken in fp64 throughout.
        const float r = mx - mn;
        const bool flat = !(r > 0.0f);
        float q = __builtin_amdgcn_rcpf(r);
        q = fmaf(fmaf(-r, q, 1.0f), q, q);
        const float s4 = flat ? 0.0f : c1f * q;
        const float cen4 = clipf * fmaf(r, kMidF, mn);
        // (a range whose reciprocal is subnormal - the reciprocal instruction returns zero for it -
        // or so small that s overflows leaves no window at all, nor does a flat group, which takes code 0)
        const float thr4 = (r < 4e37f && s4 < 1e30f && !flat) ? fmaf(-3e-7f * __builtin_fabsf(cen4), s4, 0.49998f) : -1.0f;
        {
            float delta = clipf * r * (float)(1.0 / kL);            // each factor good to 6e-8
            if (!(r < 3e38f)) {                                     // max - min beyond fp32
                float mx_here = mx;
                asm volatile("" : "+v"(mx_here));
                delta = (float)((clip * (double)mx_here - clip * (double)mn) * (1.0 / kL));
            }
            const int gs = c * 4 + g;                               // lane c < U: group of pass c
            if (c < U && gs < left) {
                scales[g0 + gs] = delta;
                mins[g0 + gs] = clipf * mn;
            }
        }
        auto pass = [&](auto which) {
            constexpr int u = decltype(which)::value;
            const float s = quad_lane<u>(s4), cen = quad_lane<u>(cen4), thr = quad_lane<u>(thr4);
            float v[8], e[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float dx = x[u][k] - cen;
                v[k] = fmaf(dx, s, Quant<BITS>::kBias);
                e[k] = fmaf(dx, s, Quant<BITS>::kBias - v[k]);     // t - round(t)
            }
            // near a rounding tie: the definition itself, in fp64 and with its two divisions (an exact tie
            // turns on their last bit), for that value only; one test per lane and pass guards the lot
            const bool near = !(absmax8(e) <= thr);
            if (__builtin_amdgcn_ballot_w64(near) != 0) {
                // (the whole wave is here: the extremes come from other lanes)
                float mn_here = quad_lane<u>(mn), mx_here = quad_lane<u>(mx);
                asm volatile("" : "+v"(mn_here), "+v"(mx_here));   // keeps the fp64 work inside the branch
                if (near) {
                    if (!(mx_here - mn_here > 0.0f)) {
#pragma unroll
                        for (int k = 0; k < 8; ++k) v[k] = Quant<BITS>::kMagic;
                    } else {
                        const double lo64 = clip * (double)mn_here, hi64 = clip * (double)mx_here;
                        const double delta64 = (hi64 - lo64) / kL;
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            if (!(__builtin_fabsf(e[k]) <= thr))
                                v[k] = Quant<BITS>::kMagic + (float)fmin(fmax(rint(((double)x[u][k] - lo64) / delta64), 0.0), kL);
                    }
                }
            }
            const uint32_t w = Quant<BITS>::join(v);
            const bool live = u * 4 + g < left;
            if (BITS == 4) {
                if (live) store_codes(out0 + u * (16 * BITS), w);
            } else {
                const int qpos = c & 3;
                const uint32_t dw = merge24<false>(w, qpos);
                if (live && qpos < 3) store_codes(out0 + u * (16 * BITS), dw);
            }
        };
        pass(std::integral_constant<int, 0>{});
        pass(std::integral_constant<int, 1>{});
        pass(std::integral_constant<int, 2>{});
        pass(std::integral_constant<int, 3>{});
    }
}

// Per-token symmetric quantizer (section 2.1) for short rows, d <= 8 LPR <= 512 - head rows that arrive
// already rotated: LPR = 16, 32 or 64 lanes hold a row, 8 values each, so a wave takes 4, 2 or 1 rows
// per pass and U passes per iteration.  Same scheme as above without the offset: absmax over the row's
// lanes (bit patterns of non-negative floats order like unsigned integers), s = (2^b - 1) / (clip amax)
// in fp32, codes by one fused multiply-add, values within 2e-5 of a tie retaken from the exact fp64
// quotient x / Delta.
template <int BITS, int DT, int LPR, int U>
__global__ __launch_bounds__(64) void k_plain_short(const void* X, int64_t rows, int d, int64_t ld, double clip,
                                                    uint32_t* codes, float* scales) {
    constexpr double kL = (double)((1 << BITS) - 1);
    constexpr int RPP = 64 / LPR;                                 // rows per pass
    constexpr float kQmin = -(float)(1 << (BITS - 1)), kQmax = (float)((1 << (BITS - 1)) - 1);
    const int lane = threadIdx.x;
    const int sr = lane / LPR, c = lane % LPR;
    const bool has = c * 8 < d;                                   // d is a multiple of 32: whole quads of lanes
    const int row_dwords = d * BITS / 32;
    const float c1f = (float)(kL / clip), clipf = (float)clip;
    for (int64_t r0 = (int64_t)blockIdx.x * (RPP * U); r0 < rows; r0 = next_item<false, kMostGroups * RPP * U>(r0)) {
        float x[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t row = r0 + u * RPP + sr;
            const int64_t rl = row < rows ? row : rows - 1;
            if (has) to_float8<DT>(load_raw8<DT, true>(X, rl * ld + c * 8), x[u]);
            else
#pragma unroll
                for (int k = 0; k < 8; ++k) x[u][k] = 0.0f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t row = r0 + u * RPP + sr;
            const bool live = row < rows && has;
            uint32_t mi = __float_as_uint(absmax8(x[u]));
            mi = max(mi, dpp_u<kDppXor1>(mi));
            mi = max(mi, dpp_u<kDppXor2>(mi));
            mi = max(mi, dpp_u<kDppHalfMirror>(mi));
            mi = max(mi, dpp_u<kDppRor8>(mi));
            if constexpr (LPR >= 32) {                            // DPP rows 0 | 1 and 2 | 3
                const auto a = __builtin_amdgcn_permlane16_swap(mi, mi, false, false);
                mi = max((uint32_t)a[0], (uint32_t)a[1]);
            }
            if constexpr (LPR == 64) {
                const auto b = __builtin_amdgcn_permlane32_swap(mi, mi, false, false);
                mi = max((uint32_t)b[0], (uint32_t)b[1]);
            }
            const float m = __uint_as_float(mi);
            const bool flat = !(m > 0.0f);
            float q = __builtin_amdgcn_rcpf(m);
            q = fmaf(fmaf(-m, q, 1.0f), q, q);
            const float s = flat ? 0.0f : c1f * q;
            // (no window where the reciprocal of amax is subnormal or s overflows: fp64 throughout)
            const float thr = (m < 4e37f && s < 1e30f) ? 0.49998f : -1.0f;
            float v[8], e[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                v[k] = fmaf(x[u][k], s, Quant<BITS>::kBias);
                e[k] = fmaf(x[u][k], s, Quant<BITS>::kBias - v[k]);     // t - round(t)
            }
            const float emax = absmax8(e);
            if (!(emax <= thr) && !flat) {
                float m_here = m;
                asm volatile("" : "+v"(m_here));                  // keeps the fp64 work inside the branch
                const double delta64 = clip * (double)m_here / kL;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (!(__builtin_fabsf(e[k]) <= thr))
                        v[k] = Quant<BITS>::kBias + fminf(fmaxf((float)rint((double)x[u][k] / delta64), kQmin), kQmax);
            }
            const uint32_t w = Quant<BITS>::join(v) ^ Quant<BITS>::msb();
            uint32_t* out = codes + row * (int64_t)row_dwords;
            if (BITS == 4) {
                if (live) store_codes(out + c, w);
            } else {
                const int qpos = c & 3;
                const uint32_t dw = merge24<false>(w, qpos);
                if (live && qpos < 3) store_codes(out + (c >> 2) * 3 + qpos, dw);
            }
            if (live && c == 0) scales[row] = clipf * m * (float)(1.0 / kL);
        }
    }
}

template <int DT, int LPR>
void launch_short(int bits, hipStream_t s, const void* X, int64_t rows, int d, int64_t ld, double clip,
                  uint32_t* codes, float* scales) {
    constexpr int U = 4;
    const int64_t iters = (rows + (64 / LPR) * U - 1) / ((64 / LPR) * U);
    const dim3 grid = item_groups(iters);
    if (bits == 4) launch_kernel((k_plain_short<4, DT, LPR, U>), grid, dim3(64), 0, s, X, rows, d, ld, clip, codes, scales);
    else launch_kernel((k_plain_short<3, DT, LPR, U>), grid, dim3(64), 0, s, X, rows, d, ld, clip, codes, scales);
}

template <int DT>
void launch_short_dt(int bits, hipStream_t s, const void* X, int64_t rows, int d, int64_t ld, double clip,
                     uint32_t* codes, float* scales) {
    if (d <= 128) launch_short<DT, 16>(bits, s, X, rows, d, ld, clip, codes, scales);
    else if (d <= 256) launch_short<DT, 32>(bits, s, X, rows, d, ld, clip, codes, scales);
    else launch_short<DT, 64>(bits, s, X, rows, d, ld, clip, codes, scales);
}

template <int DT>
void launch_dt(bool aligned, int bits, dim3 grid, hipStream_t s, const void* X, int64_t n_groups, int gpr,
               int64_t ld, double clip, uint32_t* codes, float* scales, float* mins) {
    const int gpr_shift = (gpr & (gpr - 1)) == 0 ? __builtin_ctz((unsigned)gpr) : -1;
    const uint32_t gpr_magic = (uint32_t)((((uint64_t)1 << 32) + gpr - 1) / gpr);   // gpr >= 2 where it is used
    auto go = [&](auto kernel) { launch_kernel(kernel, grid, dim3(64), 0, s, X, n_groups, gpr, gpr_shift, gpr_magic, ld, clip, codes, scales, mins); };
    if (aligned) {
        if (bits == 4) go(k_plain_asym<4, DT, true>); else go(k_plain_asym<3, DT, true>);
    } else {
        if (bits == 4) go(k_plain_asym<4, DT, false>); else go(k_plain_asym<3, DT, false>);
    }
}

}  // namespace

int plain_quantize_asym(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                        uint32_t* codes, float* scales, float* mins, hipStream_t s) {
    const int gpr = d / RQ_GROUP;
    const int64_t n_groups = rows * gpr;
    const int64_t passes = (n_groups + 15) / 16;          // 4 groups x 4 passes per wave iteration
    const dim3 grid = item_groups(passes);
    const int esz = dtype == RQ_F32 ? 4 : 2;
    const bool aligned = (reinterpret_cast<uintptr_t>(X) & 15) == 0 && (ld * esz) % 16 == 0;
    if (dtype == RQ_BF16) launch_dt<0>(aligned, bits, grid, s, X, n_groups, gpr, ld, (double)clip, codes, scales, mins);
    else if (dtype == RQ_F32) launch_dt<1>(aligned, bits, grid, s, X, n_groups, gpr, ld, (double)clip, codes, scales, mins);
    else launch_dt<2>(aligned, bits, grid, s, X, n_groups, gpr, ld, (double)clip, codes, scales, mins);
    return launch_rc();
}

bool plain_short_supports(const void* X, int dtype, int d, int64_t ld) {
    const int esz = dtype == RQ_F32 ? 4 : 2;
    return d <= 512 && d % 32 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0 && (ld * esz) % 16 == 0;
}

int plain_short_quantize(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                         uint32_t* codes, float* scales, hipStream_t s) {
    if (dtype == RQ_BF16) launch_short_dt<0>(bits, s, X, rows, d, ld, (double)clip, codes, scales);
    else if (dtype == RQ_F32) launch_short_dt<1>(bits, s, X, rows, d, ld, (double)clip, codes, scales);
    else launch_short_dt<2>(bits, s, X, rows, d, ld, (double)clip, codes, scales);
    return launch_rc();
}

}  // namespace rq
