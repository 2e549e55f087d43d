// Rotation alone for the orders of the workgroup block kernel (wg_block_kernel.h): rq_rotate - offline fusion of
// the wide weights, the online rotation of rows that are not quantized, the inverse with the transposed block's
// operand tiles - and rq_dequantize_rotate, whose rows come from packed codes.
// Bound: the kernel's vector and matrix-core issue, as for the quantizing form, less the absmax, the quantizer and one
// of the two barriers.
#include "wg_block_kernel.h"

namespace rq {
namespace {

// fp32 results pass through 2 KB of LDS per wave (store_block_f32)
template <int KK>
size_t rot_lds_bytes(int out) { return wg_ops_bytes<KK>() + (out == 1 ? (size_t)KK * 2 * 2048 : 0); }

template <int KK, bool F16, int SRC, bool WIDE>
WgKernel<kWgRotate> pick_shape(int cb) {
    if (cb == 4) {
        if constexpr (KK >= 2) return k_wg_block<KK, 4, false, kWgRotate, 4, F16, SRC, WIDE>;
        return nullptr;
    }
    if (cb == 3) return k_wg_block<KK, 4, false, kWgRotate, 3, F16, SRC, WIDE>;
    return cb == 2 ? k_wg_block<KK, 4, false, kWgRotate, 2, F16, SRC, WIDE> : nullptr;
}

// src: 0 rows of X, 3 / 4 packed codes of that width.
template <int KK, bool WIDE>
WgKernel<kWgRotate> pick_kernel(int src, int cb, bool f16) {
    if (src == 4) return pick_shape<KK, true, 4, WIDE>(cb);
    if (src == 3) return pick_shape<KK, true, 3, WIDE>(cb);
    return f16 ? pick_shape<KK, true, 0, WIDE>(cb) : pick_shape<KK, false, 0, WIDE>(cb);
}

template <int KK>
bool prepare_kk() {
    if (rot_lds_bytes<KK>(1) <= 48 * 1024) return true;
    for (int src : {0, 3, 4})
        for (int cb = 2; cb <= 4; ++cb)
            for (int f16 = 0; f16 < 2; ++f16) {
                for (WgKernel<kWgRotate> fn : {pick_kernel<KK, false>(src, cb, f16 != 0), pick_kernel<KK, true>(src, cb, f16 != 0)})
                    if (fn && hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                  (int)rot_lds_bytes<KK>(1)) != hipSuccess)
                        return false;
            }
    return true;
}

template <int KK>
int launch_kk(const rq_hadamard* h, const WaveArgs& w, int src, int pb, int cb, const WgRotArgs& o, hipStream_t s) {
    const bool wide = o.out == 1;
    WgKernel<kWgRotate> fn = wide ? pick_kernel<KK, true>(src, cb, w.f16) : pick_kernel<KK, false>(src, cb, w.f16);
    if (!fn) return RQ_ERR_NO_ORDER;
    return wg_launch<KK, kWgRotate>(h, fn, w, pb, cb, rot_lds_bytes<KK>(o.out), o, s, wg_waves_per_simd<KK>(wide));
}

int launch(const rq_hadamard* h, const WaveArgs& w, int src, int pb, int cb, const WgRotArgs& o, hipStream_t s) {
    switch ((pb + 31) / 32) {
        case 1: return launch_kk<1>(h, w, src, pb, cb, o, s);
        case 2: return launch_kk<2>(h, w, src, pb, cb, o, s);
        case 3: return launch_kk<3>(h, w, src, pb, cb, o, s);
        case 4: return launch_kk<4>(h, w, src, pb, cb, o, s);
        case 5: return launch_kk<5>(h, w, src, pb, cb, o, s);
        case 6: return launch_kk<6>(h, w, src, pb, cb, o, s);
        case 7: return launch_kk<7>(h, w, src, pb, cb, o, s);
        case 8: return launch_kk<8>(h, w, src, pb, cb, o, s);
        default: return RQ_ERR_NO_ORDER;
    }
}

WgRotArgs rot_args(const RowArgs& a, const OutArgs& o) {
    return WgRotArgs{o.Y, o.d_out, o.ld_out, 1.0 / std::sqrt((double)a.n),
                     o.dtype == RQ_BF16 ? 0 : o.dtype == RQ_F32 ? 1 : 2};
}

// (a pass takes up to four rows through 32-bit byte offsets)
bool out_ok(const OutArgs& o) {
    if (o.ld_out > (1 << 26)) return false;
    if ((reinterpret_cast<uintptr_t>(o.Y) & 15) != 0 || (o.d_out & 7) != 0) return false;
    return o.dtype == RQ_F32 ? (o.ld_out & 3) == 0 : (o.ld_out & 7) == 0;
}

}  // namespace

bool wg_rotate_prepare(int pb) {
    switch ((pb + 31) / 32) {
        case 1: return prepare_kk<1>();
        case 2: return prepare_kk<2>();
        case 3: return prepare_kk<3>();
        case 4: return prepare_kk<4>();
        case 5: return prepare_kk<5>();
        case 6: return prepare_kk<6>();
        case 7: return prepare_kk<7>();
        case 8: return prepare_kk<8>();
        default: return false;
    }
}

bool wg_rotate_supports(const rq_hadamard* h, const RowArgs& a, const OutArgs& o) {
    return wg_block_supports(h, a) && a.ld <= (1 << 26) && out_ok(o);
}

int wg_rotate(const rq_hadamard* h, const RowArgs& a, int transpose, const OutArgs& o, hipStream_t s) {
    int pb, cb;
    if (!wg_shape(a, &pb, &cb)) return RQ_ERR_NO_ORDER;
    const bool f16 = a.dtype == RQ_F16;
    const void* tiles = transpose ? (f16 ? h->d_tiles_t_f16 : h->d_tiles_t) : (f16 ? h->d_tiles_f16 : h->d_tiles);
    WaveArgs w{static_cast<const uint16_t*>(a.X), a.rows, a.d, a.ld, static_cast<const u32x4*>(tiles), nullptr, nullptr, 0.0, 0.0};
    w.f16 = f16;
    return launch(h, w, 0, pb, cb, rot_args(a, o), s);
}

bool wg_dequant_rotate_supports(const rq_hadamard* h, const RowArgs& a, const float* mins, const OutArgs& o) {
    int pb, cb;
    return h->device >= 0 && h->d_tiles && h->wg_ok && !mins && wg_shape(a, &pb, &cb) && out_ok(o);
}

int wg_dequant_rotate(const rq_hadamard* h, const RowArgs& a, const uint32_t* codes, const float* scales, int transpose,
                      const OutArgs& o, hipStream_t s) {
    int pb, cb;
    if (!wg_shape(a, &pb, &cb)) return RQ_ERR_NO_ORDER;
    WaveArgs w{nullptr, a.rows, a.n, a.n, static_cast<const u32x4*>(transpose ? h->d_tiles_t_f16 : h->d_tiles_f16),
               const_cast<uint32_t*>(codes), const_cast<float*>(scales), 0.0, 0.0};
    w.f16 = true;
    return launch(h, w, a.bits, pb, cb, rot_args(a, o), s);
}

}  // namespace rq
