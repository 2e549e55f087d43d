// Launches of the workgroup block kernel (wg_block_kernel.h) that quantize rows or evaluate their quantization
// error, and the block's operand tiles.
#include "wg_block_kernel.h"

namespace rq {
namespace {

template <int KK, int BITS, int SINK, bool F16>
WgKernel<SINK> pick_shape(bool full, int cb) {
    if (cb == 4) {
        if constexpr (KK >= 2) return full ? k_wg_block<KK, BITS, true, SINK, 4, F16> : k_wg_block<KK, BITS, false, SINK, 4, F16>;
        return nullptr;
    }
    if (cb == 3) return k_wg_block<KK, BITS, false, SINK, 3, F16>;
    return cb == 2 ? k_wg_block<KK, BITS, false, SINK, 2, F16> : nullptr;
}

// The kernel instance for a launch, or nullptr when the combination is not built: cb = 4 needs
// KK >= 2 (smaller blocks have the one-wave kernel).
template <int KK, int SINK>
WgKernel<SINK> pick_kernel(int bits, bool full, int cb, bool f16) {
    if (bits == 4) return f16 ? pick_shape<KK, 4, SINK, true>(full, cb) : pick_shape<KK, 4, SINK, false>(full, cb);
    if (bits == 3) return f16 ? pick_shape<KK, 3, SINK, true>(full, cb) : pick_shape<KK, 3, SINK, false>(full, cb);
    return nullptr;
}

template <int KK, int SINK>
int launch_kk(const rq_hadamard* h, const WaveArgs& a, int bits, int pb, int cb, hipStream_t s, const WgArgs<SINK>& sa) {
    WgKernel<SINK> fn = pick_kernel<KK, SINK>(bits, cb == 4 && a.d == 128 * pb, cb, a.f16);
    if (!fn) return RQ_ERR_NO_ORDER;
    return wg_launch<KK, SINK>(h, fn, a, pb, cb, wg_lds_bytes<KK>(), sa, s);
}

template <int KK, int SINK>
bool prepare_sink() {
    for (int bits = 3; bits <= 4; ++bits)
        for (int full = 0; full < 2; ++full)
            for (int cb = 2; cb <= 4; ++cb)
                for (int f16 = 0; f16 < 2; ++f16) {
                    WgKernel<SINK> fn = pick_kernel<KK, SINK>(bits, full != 0, cb, f16 != 0);
                    if (fn && hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                  (int)wg_lds_bytes<KK>()) != hipSuccess)
                        return false;
                }
    return true;
}

template <int KK>
bool prepare_kk() {
    return wg_lds_bytes<KK>() <= 48 * 1024 || (prepare_sink<KK, kWgQuantize>() && prepare_sink<KK, kWgError>());
}

}  // namespace

// Operand tiles of the zero-padded block `bm` (order pb): [wave][kk][lane] x 16 bytes, wave <
// ceil(pb/16), kk < ceil(pb/32); operand lane (gA, mm) of (wave, kk) holds block row
// 16 wave + 4 (mm & 3) + (mm >> 2) at the contraction slots a = 32 kk + 8 gA + i.  Those of the pair form follow.
std::vector<uint32_t> wg_block_tiles(const std::vector<int8_t>& bm, int pb) {
    const int NW = (pb + 15) / 16, KK = (pb + 31) / 32;
    std::vector<uint32_t> t((size_t)NW * KK * 64 * 4, 0u);
    for (int w = 0; w < NW; ++w)
        for (int kk = 0; kk < KK; ++kk)
            for (int lane = 0; lane < 64; ++lane) {
                const int gA = lane >> 4, mm = lane & 15;
                const int ao = 16 * w + 4 * (mm & 3) + (mm >> 2);
                for (int i = 0; i < 8; ++i) {
                    const int ai = 32 * kk + 8 * gA + i;
                    uint32_t v = 0;
                    if (ao < pb && ai < pb) v = bm[(size_t)ao * pb + ai] > 0 ? 0x3F80u : 0xBF80u;
                    t[(((size_t)w * KK + kk) * 64 + lane) * 4 + (i >> 1)] |= v << ((i & 1) * 16);
                }
            }
    const std::vector<uint32_t> pairs = wg_pair_tiles(bm, pb);
    t.insert(t.end(), pairs.begin(), pairs.end());
    return t;
}

bool wg_block_prepare(int pb) {
    if (!wg_rotate_prepare(pb)) return false;
    wg_pair_prepare(pb);
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

// Shape of a launch: block order and lane bits of the column transform (4: block rows of 128
// columns; 3, 2: block rows of 64 / 32 columns, several rows of X per pass).  False when the order
// is not served by this kernel.
bool wg_shape(const RowArgs& a, int* pb, int* cb) {
    if (a.p == 1) {
        // Sylvester orders beyond the one-wave kernel (2^14, 2^15): the block is H_128 / H_256 itself
        if (a.log2m < 14 || a.log2m > 15) return false;
        *pb = 1 << (a.log2m - 7);
        *cb = 4;
        return true;
    }
    if (a.log2m >= 7) {
        *pb = a.p << (a.log2m - 7);
        *cb = 4;
        return *pb > 32 && *pb <= 256;
    }
    *pb = a.p;
    *cb = a.log2m - 3;
    return a.log2m >= 5 && a.p >= 4 && a.p <= 256;
}

bool wg_block_supports(const rq_hadamard* h, const RowArgs& a, bool quant_error) {
    (void)quant_error;                                  // both forms cover the same shapes
    int pb, cb;
    if (h->device < 0 || !h->d_tiles || !h->wg_ok || !wg_shape(a, &pb, &cb)) return false;
    if (a.dtype != RQ_BF16 && !(a.dtype == RQ_F16 && h->d_tiles_f16)) return false;
    if ((reinterpret_cast<uintptr_t>(a.X) & 15) != 0 || (a.ld & 7) != 0 || (a.d & 7) != 0) return false;
    return true;
}

template <int SINK>
static int launch_by_kk(const rq_hadamard* h, const WaveArgs& w, int bits, int pb, int cb, hipStream_t s,
                        const WgArgs<SINK>& sa) {
    switch ((pb + 31) / 32) {
        case 1: return launch_kk<1, SINK>(h, w, bits, pb, cb, s, sa);
        case 2: return launch_kk<2, SINK>(h, w, bits, pb, cb, s, sa);
        case 3: return launch_kk<3, SINK>(h, w, bits, pb, cb, s, sa);
        case 4: return launch_kk<4, SINK>(h, w, bits, pb, cb, s, sa);
        case 5: return launch_kk<5, SINK>(h, w, bits, pb, cb, s, sa);
        case 6: return launch_kk<6, SINK>(h, w, bits, pb, cb, s, sa);
        case 7: return launch_kk<7, SINK>(h, w, bits, pb, cb, s, sa);
        case 8: return launch_kk<8, SINK>(h, w, bits, pb, cb, s, sa);
        default: return RQ_ERR_NO_ORDER;
    }
}

int wg_block_quant_error(const rq_hadamard* h, const RowArgs& a, const ClipArg& clips, int max_clips, double* partial,
                         hipStream_t s) {
    int pb, cb;
    if (!wg_shape(a, &pb, &cb)) return RQ_ERR_NO_ORDER;
    const bool f16 = a.dtype == RQ_F16;
    WaveArgs w{static_cast<const uint16_t*>(a.X), a.rows, a.d, a.ld,
               static_cast<const u32x4*>(f16 ? h->d_tiles_f16 : h->d_tiles), nullptr, nullptr, 0.0, 0.0};
    w.f16 = f16;
    QeArgs qe;
    qe.clips = clips;
    qe.partial = partial;
    qe.max_shares = (max_clips + 3) / 4;                 // (ratios are taken four at a time)
    return launch_by_kk<kWgError>(h, w, a.bits, pb, cb, s, qe);
}

int wg_block_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                             float* scales, hipStream_t s) {
    int pb, cb;
    if (!wg_shape(a, &pb, &cb)) return RQ_ERR_NO_ORDER;
    const bool f16 = a.dtype == RQ_F16;
    const double lvl = (double)((1 << a.bits) - 1);
    WaveArgs w{static_cast<const uint16_t*>(a.X), a.rows, a.d, a.ld,
               static_cast<const u32x4*>(f16 ? h->d_tiles_f16 : h->d_tiles), codes, scales,
               lvl / (double)clip, (double)clip / (std::sqrt((double)a.n) * lvl)};
    w.f16 = f16;
    return launch_by_kk<kWgQuantize>(h, w, a.bits, pb, cb, s, WgNone{});
}

}  // namespace rq
