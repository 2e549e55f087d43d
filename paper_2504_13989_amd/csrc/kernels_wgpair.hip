// Launches of the pair form of the workgroup block kernel (wg_pair_kernel.h), and its operand tiles.
#include "wg_pair_kernel.h"

namespace rq {
namespace {

using PairKernel = void (*)(RQ_WAVE_PARAMS);

// The forms that are built are those that are faster than the workgroup block kernel, four to eight waves a row (figures in
// wg_pair_kernel.h).  Three are slower: 6000 rows, b = 3, 9728 wide 35.9 there and 39.3 us so, 10240 wide 38.6 and 40.4.
template <int NW, bool DIAG>
PairKernel pick(int bits, bool f16) {
    if (bits == 4) return f16 ? k_wg_pair<NW, DIAG, 4, true> : k_wg_pair<NW, DIAG, 4, false>;
    if (bits == 3) return f16 ? k_wg_pair<NW, DIAG, 3, true> : k_wg_pair<NW, DIAG, 3, false>;
    return nullptr;
}

struct PairForm {
    PairKernel kernel = nullptr;
    int waves = 0, rows = 0;    // of a row, rows of a workgroup
    size_t lds = 0;             // of a workgroup
};

template <int NW, bool DIAG = false>
PairForm form(int bits, bool f16) {
    return PairForm{pick<NW, DIAG>(bits, f16), NW, pair_rows(NW), pair_rows(NW) * pair_lds_bytes<NW, DIAG>()};
}

PairForm pair_form(int pb, bool diag, int bits, bool f16) {
    const int nw = (pb + 31) / 32;
    if (diag) return nw == 5 ? form<5, true>(bits, f16) : nw == 7 ? form<7, true>(bits, f16) : PairForm{};
    switch (nw) {
        case 4: return form<4>(bits, f16);
        case 5: return form<5>(bits, f16);
        case 6: return form<6>(bits, f16);
        case 7: return form<7>(bits, f16);
        case 8: return form<8>(bits, f16);
        default: return PairForm{};
    }
}

// Whether an order's block of 128-column rows is made of pairs, and whether with a diagonal: a product with H_2, or Paley's second
// construction itself (build_block).
bool in_pairs(const Factorisation& f, bool* diag) {
    *diag = f.log2m == 7 && f.kind == 2;
    return f.log2m > 7 || *diag;
}
bool in_pairs(int pb, bool* diag) {
    Factorisation f;
    return factor_order(128 * pb, &f) && in_pairs(f, diag);
}

}  // namespace

// Operand tiles of the zero-padded halves: [wave][step][lane] x 16 bytes; operand lane (gA, mm) holds C's row 16 wave + 4
// (mm & 3) + (mm >> 2) at the contraction slots 32 step + 8 gA + i.  With a diagonal (a cell of the block's diagonal is not a multiple of
// H_2) the lanes gA >= 2 of the last step hold that row of D at the columns 16 wave + 8 (gA - 2) + i.  Nothing for other blocks.
std::vector<uint32_t> wg_pair_tiles(const std::vector<int8_t>& bm, int pb) {
    const int hb = pb / 2, NW = (hb + 15) / 16, STEPS = (NW + 1) / 2;
    bool diag;
    if (NW < 4 || !in_pairs(pb, &diag)) return {};
    // [[1, 1], [1, -1]] [[x, y], [-y, x]] is the cell of a pair of rows and of columns
    auto x_of = [&](int i, int j) { return (bm[(size_t)2 * i * pb + 2 * j] + bm[(size_t)(2 * i + 1) * pb + 2 * j]) / 2; };
    auto y_of = [&](int i, int j) { return (bm[(size_t)2 * i * pb + 2 * j + 1] + bm[(size_t)(2 * i + 1) * pb + 2 * j + 1]) / 2; };
    std::vector<uint32_t> t((size_t)NW * STEPS * 64 * 4, 0u);
    for (int w = 0; w < NW; ++w)
        for (int k = 0; k < STEPS; ++k)
            for (int lane = 0; lane < 64; ++lane) {
                const int gA = lane >> 4, mm = lane & 15;
                const int i = 16 * w + 4 * (mm & 3) + (mm >> 2);
                const bool other = diag && k == STEPS - 1 && gA >= 2;
                for (int b = 0; b < 8; ++b) {
                    const int j = other ? 16 * w + 8 * (gA - 2) + b : 32 * k + 8 * gA + b;
                    if (i >= hb || j >= hb) continue;
                    const int v = !other ? x_of(i, j) : i == j ? y_of(i, i) : 0;
                    const uint32_t u = v > 0 ? 0x3F80u : v < 0 ? 0xBF80u : 0u;
                    t[(((size_t)w * STEPS + k) * 64 + lane) * 4 + (b >> 1)] |= u << ((b & 1) * 16);
                }
            }
    return t;
}

size_t wg_pair_tiles_at(int pb) { return (size_t)((pb + 15) / 16) * ((pb + 31) / 32) * 64; }

// (A form whose LDS a device does not have is not launched there, see wg_pair_pays; the workgroup block kernel serves its rows.)
void wg_pair_prepare(int pb) {
    bool diag;
    if (!in_pairs(pb, &diag)) return;
    for (int k = 0; k < 4; ++k) {
        const PairForm f = pair_form(pb, diag, 3 + (k & 1), k & 2);
        if (f.kernel) (void)allow_lds(f.kernel, f.lds);
    }
}

// Few rows leave compute units with a row or two, whose latency the longer waves make longer: up to there the workgroup
// block kernel is the faster, or as fast.  us a call there and here, two rows a unit (512 rows, b = 3): 14336 wide 6.05 and 6.46, 16384
// 6.47 and 6.83, 18944 8.79 and 8.84, 20480 9.15 and 9.00; beyond (520 rows, b = 4) 6.98 and 7.11, 7.67 and 7.44, 11.03 and 9.91, 11.55
// and 10.07, 640 rows 7.59 and 7.35, 8.63 and 7.76, 11.54 and 10.69, 12.08 and 11.07.  From six waves a row on, where the other kernel
// has one workgroup on a unit, the line is at one row a unit (b = 3): 256 rows 24576 wide 6.34 and 6.78, 28672 8.08 and 7.08; 264 rows
// 24576 9.11 and 8.43, 28672 11.61 and 9.43, 32768 12.76 and 9.82.
bool wg_pair_pays(const rq_hadamard* h, const RowArgs& a) {
    int pb, cb;
    bool diag;
    if (!wg_shape(a, &pb, &cb) || cb != 4 || !in_pairs(h->f, &diag)) return false;
    const PairForm f = pair_form(pb, diag, a.bits, a.dtype == RQ_F16);
    if (!f.kernel || f.lds + 256 > (size_t)h->max_lds) return false;
    return a.rows > (int64_t)h->num_cu * ((pb + 31) / 32 >= 6 ? 1 : 2);
}

int wg_pair_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes, float* scales, hipStream_t s) {
    const bool f16 = a.dtype == RQ_F16;
    int pb, cb;
    bool diag;
    if (!wg_shape(a, &pb, &cb) || cb != 4 || !in_pairs(h->f, &diag)) return RQ_ERR_NO_ORDER;
    const PairForm f = pair_form(pb, diag, a.bits, f16);
    if (!f.kernel) return RQ_ERR_NO_ORDER;
    const double lvl = (double)((1 << a.bits) - 1);
    const WaveArgs w{static_cast<const uint16_t*>(a.X), a.rows, a.d, a.ld,
                     static_cast<const u32x4*>(f16 ? h->d_tiles_f16 : h->d_tiles) + wg_pair_tiles_at(pb), codes, scales,
                     lvl / (double)clip, (double)clip / (std::sqrt((double)a.n) * lvl)};
    // as many workgroups as fit the chip, each looping over rows
    const int by_lds = (int)((size_t)h->max_lds / (f.lds + 256)), by_waves = 16 / (f.waves * f.rows);
    const int64_t cap = (int64_t)h->num_cu * (by_lds < by_waves ? by_lds : by_waves);
    launch_kernel(f.kernel, dim3((unsigned)(a.rows < cap ? a.rows : cap)), dim3(64 * f.waves * f.rows), f.lds, s, RQ_WAVE_VALUES(w, pb));
    return launch_rc();
}

}  // namespace rq
