// Rotations of a row into registers that more than one kernel is built on: a long Sylvester row split over the waves of
// a workgroup, and a Paley-block row (blocks up to 32 x 128) on one wave.
#pragma once
#include "wave_common.h"

namespace rq {
namespace {

// The rotation of a row split over S waves: wave `seg` gets output segment seg of the row, T / S register sets of
// values that carry the lane's sign (split_flip); returns the segment's absmax over the lane.
template <int T, bool FULL, int S, bool F16>
__device__ __forceinline__ float split_rotate_row(const WaveArgs& a, int64_t row, int seg, int c, int chunk, const u32x4& A0,
                                                  const u32x4& A1, f32x4 (&acc)[T / S][2]) {
    constexpr int TS = T / S;
    // operand tiles per input segment: negated where H_S[seg][sp] = -1 (Sylvester sign; bit 15 is the
    // sign of a bf16 and of an fp16 alike)
    u32x4 P0[S], P1[S];
#pragma unroll
    for (int sp = 0; sp < S; ++sp) {
        const uint32_t sg = (__builtin_popcount(seg & sp) & 1) ? 0x80008000u : 0u;
        const u32x4 sgn = {sg, sg, sg, sg};
        P0[sp] = A0 ^ sgn;
        P1[sp] = A1 ^ sgn;
    }
    float sf[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) sf[b] = ((c >> b) & 1) ? -1.0f : 1.0f;
    const uint16_t* xr = a.X + row * a.ld;
    const RowView xv = row_view(xr, a.d);
    // all T loads of the row first (see k_wave_sylvester); plain (cached) loads: the S waves of the
    // workgroup read the same lines
    u32x4 raw[TS][S];
#pragma unroll
    for (int t = 0; t < TS; ++t)
#pragma unroll
        for (int sp = 0; sp < S; ++sp) {
            const int e0 = ((sp * TS + t) * 64 + chunk) * 8;
            raw[t][sp] = FULL ? *reinterpret_cast<const u32x4*>(xr + e0) : load_chunk(xv, e0);
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < TS; ++t) {
        acc[t][0] = f32x4{0.f, 0.f, 0.f, 0.f};
        acc[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sp = 0; sp < S; ++sp) {
            acc[t][0] = mfma_pm1<F16>(P0[sp], raw[t][sp], acc[t][0]);
            acc[t][1] = mfma_pm1<F16>(P1[sp], raw[t][sp], acc[t][1]);
        }
    }
#pragma unroll
    for (int s = 1; s < TS; s <<= 1)
#pragma unroll
        for (int t = 0; t < TS; ++t)
            if (!(t & s))
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 u = acc[t][h], v = acc[t | s][h];
                    acc[t][h] = u + v;
                    acc[t | s][h] = u - v;
                }
    float m = 0.0f;
#pragma unroll
    for (int t = 0; t < TS; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x4 v = acc[t][h];
            if (TS == 1) {                               // straight from the matrix cores: see lane_stages_tail
                const uint32_t sg0 = (c & 1) ? 0x80000000u : 0u;
                lane_stage<kDppXor1>(v, sg0);
                lane_stages_tail<4>(v, sf);
            } else {
                lane_stages_fused(v, sf[0], sf[1], sf[2], sf[3]);
            }
            acc[t][h] = v;
            m = absmax4(m, v);
        }
    return m;
}
// The sign a lane's values carry after split_rotate_row.
template <int T, int S>
__device__ __forceinline__ float split_flip(int c) {
    return (__builtin_popcount(T == S ? c >> 1 : c) & 1) ? -1.0f : 1.0f;
}

// The rotation of one row for the block kernels: loads, block product on the matrix cores, the
// 128-point transform along the columns.  y[column i][j]: register j = 4 h + ip holds block rows
// 4 j .. 4 j + 3 (one per DPP row g); only the NV = ceil(pb / 4) registers that hold real block rows
// are carried.  Values carry the lane's flip sign (see lane_stages_fused).  Returns the row's absmax.
// SRC = 3, 4: the row comes from packed signed codes of that width (a.codes) as exact fp16 integers.
// SPREAD (4-bit codes): each row's codes are spread to fp16 first and then transposed like rows, not dealt out by code_operands.
template <bool FULL, int NV, bool F16 = false, int SRC = 0, bool SPREAD = false>
__device__ __forceinline__ float block_rotate_row(const WaveArgs& a, int64_t row, int e_base, const u32x4& A0,
                                              const u32x4& A1, const float (&sf)[4], float (&y)[8][NV]) {
    constexpr int NH1 = NV > 4 ? NV - 4 : 0;              // live registers of the second half
    constexpr int NH0 = NV > 4 ? 4 : NV;
    u32x4 R[8], bm[8];
    if constexpr (SRC != 0) {
        constexpr int STEP = 16 * SRC;                   // bytes of a block row
        const int row_bytes = STEP * (a.d >> 7);
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(a.codes + row * (row_bytes / 4), 0, row_bytes, 0x00020000);
        const CodeAt at = code_at<SRC>(e_base >> 3);
        uint32_t lo[8], hi[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            lo[t] = __builtin_amdgcn_raw_buffer_load_b32(rs, at.off0 + t * STEP, 0, 2);
            if constexpr (SRC == 3) hi[t] = __builtin_amdgcn_raw_buffer_load_b32(rs, at.off1 + t * STEP, 0, 2);
        }
        __builtin_amdgcn_sched_barrier(0);               // every load is issued before the first wait
        if constexpr (SRC == 3) {
#pragma unroll
            for (int t = 0; t < 8; ++t) lo[t] = __builtin_amdgcn_alignbit(hi[t], lo[t], at.sh);
        }
        if constexpr (SPREAD) {
#pragma unroll
            for (int t = 0; t < 8; ++t) R[t] = codes4_f16(lo[t]);
        } else {
            code_operands<SRC, 4>(lo, bm);
        }
    } else {
        const uint16_t* xr = a.X + row * a.ld + e_base;
        const RowView xv = row_view(a.X + row * a.ld, a.d);
#pragma unroll
        for (int t = 0; t < 8; ++t)
            R[t] = FULL ? load16(xr + t * 128) : load_chunk(xv, e_base + t * 128);
    }
    if constexpr (SRC == 0 || SPREAD) {
#pragma unroll
        for (int ic = 0; ic < 8; ++ic) {
            const uint32_t sel = (ic & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                bm[ic][w] = __builtin_amdgcn_perm(R[2 * w + 1][ic >> 1], R[2 * w][ic >> 1], sel);
        }
    }
#pragma unroll
    for (int ic = 0; ic < 8; ++ic) {
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        const f32x4 d0 = mfma_pm1<F16>(A0, bm[ic], z);
#pragma unroll
        for (int j = 0; j < NH0; ++j) y[ic][j] = d0[j];
        if constexpr (NH1 > 0) {
            const f32x4 d1 = mfma_pm1<F16>(A1, bm[ic], z);
#pragma unroll
            for (int j = 0; j < NH1; ++j) y[ic][4 + j] = d1[j];
        }
    }
#pragma unroll
    for (int s = 1; s < 8; s <<= 1)
#pragma unroll
        for (int ic = 0; ic < 8; ++ic)
            if (!(ic & s))
#pragma unroll
                for (int j = 0; j < NV; ++j) {
                    const float u = y[ic][j], v = y[ic | s][j];
                    y[ic][j] = u + v;
                    y[ic | s][j] = u - v;
                }
    float m = 0.0f;
#pragma unroll
    for (int ic = 0; ic < 8; ++ic) {
        fused_group<NH0>(&y[ic][0], sf);
        if constexpr (NH1 > 0) fused_group<NH1>(&y[ic][4], sf);
#pragma unroll
        for (int j = 0; j < NV; ++j) m = __builtin_fmaxf(m, __builtin_fabsf(y[ic][j]));
    }
    return wave_absmax<4>(m);
}

// A Sylvester row of 512 T values over W waves, T / W register sets each.
template <int T, int W_, bool F16>
struct SylvesterRows {
    static constexpr int W = W_, NVAL = T / W * 8;
    static __device__ __forceinline__ float rotate(const WaveArgs& a, int, int64_t row, int seg, int lane, float (&v)[NVAL], float* flip) {
        const int g = lane >> 4, cphys = lane & 15, c = (cphys & 4) ? (cphys ^ 3) : cphys;
        const u32x4 A0 = a.tiles[lane], A1 = a.tiles[64 + lane];
        f32x4 acc[T / W][2];
        const float m = split_rotate_row<T, false, W, F16>(a, row, seg, c, (g << 4) + c, A0, A1, acc);
#pragma unroll
        for (int t = 0; t < T / W; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[(t * 2 + h) * 4 + i] = acc[t][h][i];
        *flip = split_flip<T, W>(c);
        return wave_absmax<4>(m);
    }
};
// A row of a block order, pb <= 32: W waves with 16 output block rows each.
template <int W_, bool F16>
struct BlockRows {
    static constexpr int W = W_, NVAL = 32;
    static __device__ __forceinline__ float rotate(const WaveArgs& a, int pb, int64_t row, int seg, int lane, float (&v)[NVAL], float* flip) {
        const int g = lane >> 4, cphys = lane & 15, c = (cphys & 4) ? (cphys ^ 3) : cphys;
        const u32x4 A = a.tiles[seg * 64 + lane];
        float sf[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) sf[b] = ((c >> b) & 1) ? -1.0f : 1.0f;
        const int base_g = 8 * g < pb - 8 ? 8 * g : pb - 8;
        float y[8][4];
        const float m = block_rotate_row<false, 4, F16>(a, row, base_g * 128 + c * 8, A, A, sf, y);
#pragma unroll
        for (int ic = 0; ic < 8; ++ic)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[ic * 4 + j] = y[ic][j];
        *flip = (__builtin_popcount(c) & 1) ? -1.0f : 1.0f;
        return m;
    }
};

}  // namespace
}  // namespace rq
