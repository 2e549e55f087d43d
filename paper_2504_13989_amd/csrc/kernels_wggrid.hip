// Rows of the workgroup block kernel (wg_block_kernel.h) for the grid form of the clip search (kernels_gridsearch.hip).
#include "wg_block_kernel.h"

namespace rq {
namespace {

template <int KK, int BITS, bool F16>
WgKernel<kWgGrid> pick_shape(int cb) {
    if (cb == 4) {
        if constexpr (KK >= 2) return k_wg_block<KK, BITS, false, kWgGrid, 4, F16>;
        return nullptr;
    }
    if (cb == 3) return k_wg_block<KK, BITS, false, kWgGrid, 3, F16>;
    return cb == 2 ? k_wg_block<KK, BITS, false, kWgGrid, 2, F16> : nullptr;
}

template <int KK>
WgKernel<kWgGrid> pick_kernel(int bits, int cb, bool f16) {
    if (bits == 4) return f16 ? pick_shape<KK, 4, true>(cb) : pick_shape<KK, 4, false>(cb);
    return f16 ? pick_shape<KK, 3, true>(cb) : pick_shape<KK, 3, false>(cb);
}

template <int KK>
int launch_kk(const rq_hadamard* h, const WaveArgs& w, int bits, int pb, int cb, int* groups, const WgGridArgs& g, hipStream_t s) {
    WgKernel<kWgGrid> fn = pick_kernel<KK>(bits, cb, w.f16);
    if (!fn) return RQ_ERR_NO_ORDER;
    const size_t lds = wg_ops_bytes<KK>() + (bits == 4 ? WgGrid<KK, 4>::bytes() : WgGrid<KK, 3>::bytes());
    if (!allow_lds(fn, lds)) return RQ_ERR_NO_ORDER;
    const int rpw = 16 >> cb, cus = h->num_cu < kGridGroups ? h->num_cu : kGridGroups;
    const int64_t passes = (w.rows + rpw - 1) / rpw;
    *groups = (int)(passes < cus ? passes : cus);
    launch_kernel(fn, dim3((unsigned)*groups), dim3((unsigned)(64 * ((pb + 15) / 16))), lds, s, RQ_WAVE_VALUES(w, pb), g);
    return launch_rc();
}

}  // namespace

size_t wg_grid_ops_bytes(int pb) { return (size_t)((pb + 31) / 32) * wg_ops_bytes<1>(); }

int wg_grid_rows(const rq_hadamard* h, const RowArgs& a, GbsDev* dev, int* groups, hipStream_t s) {
    int pb, cb;
    if (!wg_shape(a, &pb, &cb)) return RQ_ERR_NO_ORDER;
    const bool f16 = a.dtype == RQ_F16;
    WaveArgs w{static_cast<const uint16_t*>(a.X), a.rows, a.d, a.ld,
               static_cast<const u32x4*>(f16 ? h->d_tiles_f16 : h->d_tiles), nullptr, nullptr, 0.0, 0.0};
    w.f16 = f16;
    const WgGridArgs g{1.0 / ((double)a.n * (double)a.n), dev};
    switch ((pb + 31) / 32) {
        case 1: return launch_kk<1>(h, w, a.bits, pb, cb, groups, g, s);
        case 2: return launch_kk<2>(h, w, a.bits, pb, cb, groups, g, s);
        case 3: return launch_kk<3>(h, w, a.bits, pb, cb, groups, g, s);
        case 4: return launch_kk<4>(h, w, a.bits, pb, cb, groups, g, s);
        case 5: return launch_kk<5>(h, w, a.bits, pb, cb, groups, g, s);
        case 6: return launch_kk<6>(h, w, a.bits, pb, cb, groups, g, s);
        case 7: return launch_kk<7>(h, w, a.bits, pb, cb, groups, g, s);
        case 8: return launch_kk<8>(h, w, a.bits, pb, cb, groups, g, s);
        default: return RQ_ERR_NO_ORDER;
    }
}

}  // namespace rq
