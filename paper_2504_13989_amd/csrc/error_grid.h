// Quantization error of a rotated row at every clip ratio m / 512, m = 1 .. 511, at once (sections 2.1, 3.1).
//
// A value y of a row with absolute maximum a takes code q = min(round(|y| / Delta), Q), Q = 2^(b-1) - 1, one more for
// negative y, at Delta = (m / 512) a / (2^b - 1).  In units u = |y| 1024 (2^b - 1) / a of half the finest Delta,
//     q = #{ j in 1 .. Q : u >= (2 j - 1) m }   (+ 1 where y < 0 and u >= (2 Q + 1) m):
// every threshold of every ratio is an integer.  So the row's values go into a histogram of unit cells - a count and the
// sum of u in each -, suffix sums turn it into counts and sums beyond every threshold, and with A = sum of q u and
// B = sum of q^2 = sum over j of (2 j - 1) #{ u >= (2 j - 1) m } the error of ratio m is
//     sum (u - 2 m q)^2 = sum u^2 - 4 m A + 4 m^2 B:
// a value costs one LDS addition (two if negative) whatever the number of ratios, where evaluating a ratio costs five
// vector operations a value.  (At a threshold itself both codes have the same error, so rounding there does not matter.)
//
// u is kept in fixed point, V = u 2^FRAC < 2^28, the fp32 product rounded to an integer: sums and counts are exact
// integers, the result does not depend on the order of the additions, and the three terms, which cancel to 1 / 250 of the
// first, are formed in fp64 (relative error of a search's values against 64 bits, rms: normal rows 2.2e-8 - 1.1e-7, heavy
// tails with outliers 2.4e-8 - 2.1e-7, at most 4.3e-7; with fp32 sums of squares 2.2e-8 - 1.3e-7, 2.5e-8 - 2.4e-7 and
// 6.1e-7; a row whose energy is in one value has that value's rounding, 1.8e-8 - 1.2e-7 and 1.8e-8 - 1.0e-7).  A cell is
// one 64-bit word, the count in the upper 16 bits (at most 2^15 values a row) and the sum of V (below 2^43) under it, so a
// value is one ds_add_u64.  The last threshold, which only negative values have, has a histogram of its own in cells of 2 Q
// + 1 units: 25 KB in all for b = 3, 57 KB for b = 4, where two signed histograms would take 50 and 115.
//
// The last cell of either histogram takes whatever lies beyond every threshold: a sixth of a normal row, most of a row that
// an outlier channel makes bimodal.  Lanes that add to one address are served one after the other, so these two cells have
// sixteen words each; a suffix sum over them is that of one cell.  A search on heavy-tailed rows, us a call: 512 x 4096
// 28.6 -> 23.5, 1024 x 3584 38.2 -> 31.9, 300 x 8192 33.9 -> 26.4, 512 x 8960 43.5 -> 36.1, 512 x 14336 (b = 4) 45.3 -> 34.8, 512 x 18944
// 52.6 -> 37.1; normal rows, 512 x 4096 25.1 -> 23.6.  (The lanes' shares summed in registers and added once a wave: 25.4, 35.1, -, 46,
// 40.7, 43.3; normal rows 25.4.)
#pragma once
#include "search_state.h"
#include "wave_common.h"

namespace rq {
namespace {

// THREADS: the fewest threads that share a row, where the kernel knows it (finish then keeps a thread's share of the words in
// registers; FINE and COARSE are whole shares, the words added to them stay zero).
template <int BITS, int SPREAD = kGridSpread, int THREADS = 0>
struct ErrorGrid {
    static constexpr int LEVELS = (1 << BITS) - 1, Q = (1 << (BITS - 1)) - 1, FRAC = BITS == 3 ? 15 : 14;
    static constexpr int LAST = 2 * Q + 1;                           // units a step of the last threshold
    static constexpr int CELLS = grid_cells(BITS);
    // a thread's words of either histogram: odd, so that consecutive lanes start in different banks
    static constexpr int share(int words) { return THREADS ? ((words + THREADS - 1) / (THREADS ? THREADS : 1)) | 1 : 1; }
    static constexpr int SHARE_A = share(CELLS + SPREAD - 1), SHARE_B = share(kGridRatios + SPREAD - 1);
    static constexpr int FINE = (CELLS + SPREAD - 1 + SHARE_A - 1) / SHARE_A * SHARE_A;   // words of the histograms
    static constexpr int COARSE = (kGridRatios + SPREAD - 1 + SHARE_B - 1) / SHARE_B * SHARE_B;
    static constexpr int WORDS = (FINE + COARSE + 1) / 2 * 2;        // (cleared by 16 bytes)
    static_assert(WORDS <= grid_words(BITS) + 2 * (SPREAD - 1) + SHARE_A + SHARE_B && SPREAD <= kGridSpread && (SPREAD & (SPREAD - 1)) == 0, "see search_rule.h");
    static constexpr size_t bytes() { return (size_t)WORDS * sizeof(uint64_t); }
    // whether `rows` histograms and `arrays` bytes of static arrays keep to what grid_rows_beside allows for
    static constexpr bool within_margin(int rows, size_t arrays) {
        return rows * (bytes() - sizeof(uint64_t) * grid_words(BITS)) + arrays <= kGridMargin;
    }
    static constexpr float kTiny = 1e-30f;                           // rows below it: their squares are zero in fp32

    // What scales a row: V = |y| s.  A row of zeros has s = 0.
    struct Scale {
        float s;
        double step, back;                                           // Delta in V's units at m = 1, what takes sums of V^2 to y^2
    };
    static __device__ __forceinline__ Scale scale(float amax, double inv_norm) {
        constexpr double units = (double)(2 * kGridRatios) * LEVELS * (1 << FRAC);
        if (!(amax >= kTiny)) return Scale{0.0f, 0.0, 0.0};
        const float s = (float)(units / (double)amax);
        const double ds = (double)s;
        return Scale{s, 2.0 * (1 << FRAC) * (ds * (double)amax / units), inv_norm / (ds * ds)};
    }

    // One value (y with its sign) into the histogram; q2 accumulates V^2.
    static __device__ __forceinline__ void add(uint64_t* hist, float y, float s, double& q2, int lane) {
        // (the bound holds by itself in a finite row; it is for infinities and NaN, whose conversion is undefined: the minimum of a
        // NaN and a number is the number)
        const uint32_t v = (uint32_t)__builtin_rintf(__builtin_fminf(__builtin_fabsf(y) * s, 0x1p28f));
        q2 = fma((double)v, (double)v, q2);
        const uint32_t u = v >> FRAC;
        const unsigned long long word = (1ull << 48) | v;
        auto* const h = reinterpret_cast<unsigned long long*>(hist);
        const uint32_t top = (uint32_t)(CELLS - 1 + (lane & (SPREAD - 1)));      // (any of the last cell's words will do)
        if (u > 0) atomicAdd(h + min(u, top), word);
        if (y < 0.0f && u >= (uint32_t)LAST) {
            // u / LAST by multiplication: exact for the u there are (up to 2^(b + 10))
            const uint32_t c = BITS == 3 ? (u * 9363u) >> 16 : (u * 34953u) >> 19;
            atomicAdd(h + FINE + min(c, top - (uint32_t)(CELLS - kGridRatios)), word);
        }
    }

    // Sum of h[base, end), a thread's share of the words, and its suffix sums given the sum beyond it; eight LDS reads in
    // flight at a time.
    static constexpr int kBatch = 8;
    static __device__ __forceinline__ uint64_t chunk_sum(const uint64_t* h, int base, int end) {
        uint64_t s = 0;
        for (int i = base; i < end; i += kBatch) {
            uint64_t x[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) x[k] = h[min(i + k, end - 1)];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) s += i + k < end ? x[k] : 0;
        }
        return s;
    }
    static __device__ __forceinline__ void chunk_suffix(uint64_t* h, int base, int end, uint64_t beyond) {
        for (int i = end - 1; i >= base; i -= kBatch) {
            uint64_t x[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) x[k] = h[max(i - k, base)];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                beyond += x[k];
                if (i - k >= base) h[i - k] = beyond;
            }
        }
    }
    static __device__ __forceinline__ uint64_t lane_u64(uint64_t x, int lane) {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), lane) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
    }
    template <int SHL>
    static __device__ __forceinline__ uint64_t row_shl(uint64_t x) {
        return ((uint64_t)dpp_u<0x100 + SHL>((uint32_t)(x >> 32)) << 32) | dpp_u<0x100 + SHL>((uint32_t)x);
    }
    // Sum over this lane and those above it; `all`: over the wave.
    static __device__ __forceinline__ uint64_t lanes_from(uint64_t s, int lane, uint64_t& all) {
        s += row_shl<1>(s);
        s += row_shl<2>(s);
        s += row_shl<4>(s);
        s += row_shl<8>(s);
        const uint64_t t3 = lane_u64(s, 48), t2 = t3 + lane_u64(s, 32), t1 = t2 + lane_u64(s, 16);
        all = t1 + lane_u64(s, 0);
        return s + (lane < 16 ? t1 : lane < 32 ? t2 : lane < 48 ? t3 : 0);
    }
    static __device__ __forceinline__ double lanes_sum(double x) {
        x += dpp_d<kDppXor1>(x);
        x += dpp_d<kDppXor2>(x);
        x += dpp_d<kDppHalfMirror>(x);
        x += dpp_d<kDppRor8>(x);
        auto at = [&](int lane) { return __longlong_as_double((long long)lane_u64((uint64_t)__double_as_longlong(x), lane)); };
        return (at(0) + at(16)) + (at(32) + at(48));
    }

    // The histogram of a row to suffix sums, by the NT threads (whole waves, numbered by t) that share it, and the row's
    // sum of V^2 from the threads' q2.  `tot`: three words of LDS for each wave of the row.  Every thread of the workgroup calls it.
    static __device__ __forceinline__ double finish(uint64_t* hist, double q2, int t, int NT, uint64_t (*tot)[3]) {
        if constexpr (THREADS != 0) return finish_known(hist, q2, t, NT >> 6, tot);
        const int lane = t & 63, wave = t >> 6, nw = NT >> 6;
        // (odd shares: consecutive lanes then start in different banks)
        asm volatile("" : "+v"(t));
        const int ca = ((FINE + NT - 1) / NT) | 1, cb = ((COARSE + NT - 1) / NT) | 1;
        const int a0 = min(t * ca, FINE), a1 = min(a0 + ca, FINE);
        const int b0 = min(t * cb, COARSE), b1 = min(b0 + cb, COARSE);
        uint64_t* const coarse = hist + FINE;
        const uint64_t sa = chunk_sum(hist, a0, a1), sb = chunk_sum(coarse, b0, b1);
        uint64_t all_a, all_b, xa = lanes_from(sa, lane, all_a) - sa, xb = lanes_from(sb, lane, all_b) - sb;
        q2 = lanes_sum(q2);
        if (lane == 0) {
            tot[wave][0] = all_a;
            tot[wave][1] = all_b;
            tot[wave][2] = (uint64_t)__double_as_longlong(q2);
        }
        __syncthreads();
        q2 = 0.0;
        for (int w = 0; w < nw; ++w) {
            if (w > wave) {
                xa += tot[w][0];
                xb += tot[w][1];
            }
            q2 += __longlong_as_double((long long)tot[w][2]);
        }
        chunk_suffix(hist, a0, a1, xa);
        chunk_suffix(coarse, b0, b1, xb);
        __syncthreads();
        return q2;
    }

    // The same where at least THREADS threads, at most 64 more, share the row: a thread's words stay in registers between the two
    // passes over them, and their number needs no bounds in a loop.  The vector port bounds it (four waves a SIMD): about 200
    // instructions a wave where the general form has 450; 512 x 4096 2.9 -> 1.7 us of a search's 23.  us a search: 512 x 4096 23.1
    // -> 22.4, 1000 x 2048 (b = 4) 30.6 -> 28.4, 1000 x 3584 (b = 4) 34.2 -> 32.0, in the workgroup block kernel 512 x 18944 37.0 -> 34.6,
    // 512 x 8960 36.4 -> 33.5, 200 x 4864 31.0 -> 28.6, 300 x 28672 (b = 4) 47.6 -> 44.0.
    static __device__ __forceinline__ double finish_known(uint64_t* hist, double q2, int t, int nw, uint64_t (*tot)[3]) {
        static_assert(THREADS % 64 == 0 && THREADS * SHARE_A >= FINE && THREADS * SHARE_B >= COARSE, "every word is a thread's");
        const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
        const bool has_a = t < FINE / SHARE_A, has_b = t < COARSE / SHARE_B;
        uint64_t* const a = hist + t * SHARE_A;
        uint64_t* const b = hist + FINE + t * SHARE_B;
        uint64_t x[SHARE_A] = {}, y[SHARE_B] = {};
        if (has_a) {
#pragma unroll
            for (int k = 0; k < SHARE_A; ++k) x[k] = a[k];
        }
        if (has_b) {
#pragma unroll
            for (int k = 0; k < SHARE_B; ++k) y[k] = b[k];
        }
        q2 = lanes_sum(q2);
#pragma unroll
        for (int k = SHARE_A - 2; k >= 0; --k) x[k] += x[k + 1];
#pragma unroll
        for (int k = SHARE_B - 2; k >= 0; --k) y[k] += y[k + 1];
        uint64_t all_a, all_b, xa = lanes_from(x[0], lane, all_a) - x[0], xb = lanes_from(y[0], lane, all_b) - y[0];
        if (lane == 0) {
            tot[wave][0] = all_a;
            tot[wave][1] = all_b;
            tot[wave][2] = (uint64_t)__double_as_longlong(q2);
        }
        __syncthreads();
        q2 = 0.0;
#pragma unroll
        for (int w = 0; w <= THREADS / 64; ++w) {
            if (w >= nw) break;
            if (w > wave) {
                xa += tot[w][0];
                xb += tot[w][1];
            }
            q2 += __longlong_as_double((long long)tot[w][2]);
        }
        if (has_a) {
#pragma unroll
            for (int k = 0; k < SHARE_A; ++k) a[k] = x[k] + xa;
        }
        if (has_b) {
#pragma unroll
            for (int k = 0; k < SHARE_B; ++k) b[k] = y[k] + xb;
        }
        __syncthreads();
        return q2;
    }

    // The row's error at ratio m (over n^2, as `scale` was given it) from the suffix sums.
    static __device__ __forceinline__ double error(const uint64_t* hist, int m, double q2, const Scale& sc) {
        asm volatile("" : "+v"(m));                                  // (or the addresses of all ratios are kept from row to row)
        constexpr uint64_t kSum = (1ull << 48) - 1;
        uint64_t x = hist[FINE + m], a = x & kSum;
        uint32_t b = (uint32_t)LAST * (uint32_t)(x >> 48);
#pragma unroll
        for (int j = 1; j <= Q; ++j) {
            x = hist[(2 * j - 1) * m];
            a += x & kSum;
            b += (uint32_t)(2 * j - 1) * (uint32_t)(x >> 48);
        }
        const double delta = sc.step * (double)m;
        return fma(delta, fma(delta, (double)b, -2.0 * (double)a), q2) * sc.back;
    }
};

}  // namespace
}  // namespace rq
