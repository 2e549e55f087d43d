// The clip-ratio search of Algorithm 1 (section 4.1) in its grid form: every probe of a search down to a bracket of 1 / 256
// is a multiple of 1 / 512 (a probe halves the wider of the two gaps beside the best point, so no gap gets to a quarter of
// the bracket or below), and the error of a row at all 511 ratios costs little more than the rotation (error_grid.h).  One
// kernel passes over the rows once and leaves each workgroup's sums, a second adds them up and walks the search; nothing
// is evaluated twice and no step waits for another.
// Bound: latency (vector port 26 - 43 % busy).  512 x 4096, b = 3, by time stamps in the kernels: 9 us in the first (a workgroup's
// rows there and rotated 1.5 after its start, the maximum 1, the additions of two rows a compute unit 1.8, the passes over the
// histogram 1.7, sums out 0.9; the first workgroup starts 2 before most others, as the chip has been idle), 1.5 between the kernels, 5.5
// in the second (1 MB of sums 1.5, the count of the workgroups 1, totals back 0.6, the walk 1.2, results over the bus 0.7).
// The totals reduced inside the waves and both loads of the means at once: no difference (22.9 and 22.45 - 23.0).
// A search, us a call, resident or batched form -> grid form, normal rows (heavy-tailed ones within 3 %): 512 x 4096 45 -> 22,
// 512 x 8192 58 -> 25, 512 x 3584 44 -> 23, 512 x 5120 81 -> 28, 512 x 14336 121 -> 28, 512 x 18944 153 -> 33, 512 x 896 59 -> 46.
#include "error_grid.h"
#include "row_rotation.h"

namespace rq {
namespace {

// Rows held in registers, eight waves a row, `conc` rows (one or two) a workgroup at a time, each with a histogram of its
// own.  Where a row is rotated by fewer waves, W, all eight repeat the rotation and share the values: the additions and
// the passes over the histogram take longer than the rotation, and LDS (57 KB a row for b = 4) leaves no room for more
// rows in their place (one row a wave: 2048 x 1024, b = 4 65 us a search, 512 x 4096 on four waves a row 26.7).
constexpr int kRowThreads = 512;
template <typename Rows, int BITS>
__global__ __launch_bounds__(1024) void k_grid_rows(WaveArgs a, int pb, int conc, double inv_norm, GbsDev* dev) {
    constexpr int W = Rows::W, NVAL = Rows::NVAL, NT = kRowThreads, SHARES = NT / 64 / W;
    using Grid = ErrorGrid<BITS, kGridSpread, NT>;
    static_assert(NT >= kGridRatios - 1, "a ratio a thread");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    __shared__ float wmax[16];
    __shared__ uint64_t tot[2][8][3];
    static_assert(Grid::within_margin(2, sizeof(wmax) + sizeof(tot)), "see grid_rows_beside");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rsub = wave >> 3, seg = wave % W, share = (wave & 7) / W, t = tid - rsub * NT;
    uint64_t* const hist = reinterpret_cast<uint64_t*>(lds) + (size_t)rsub * Grid::WORDS;
    if (blockIdx.x == 0 && tid == 0) dev->grid_ticket = 0;
    double sum = 0.0;
    for (int64_t row0 = (int64_t)blockIdx.x * conc; row0 < a.rows; row0 += (int64_t)gridDim.x * conc) {
        for (int i = t; i < Grid::WORDS / 2; i += NT) reinterpret_cast<u32x4*>(hist)[i] = u32x4{0u, 0u, 0u, 0u};
        const int64_t row = row0 + rsub;
        const bool live = row < a.rows;
        float v[NVAL], flip = 1.0f, m = 0.0f;
        int l = lane;
        // (rows of 8192: the operand tiles' address held from row to row is two registers too many)
        if constexpr (Rows::NVAL == 32 && W == 4) asm volatile("" : "+v"(l));
        if (live) {
            m = Rows::rotate(a, pb, row, seg, l, v, &flip);
        } else {
#pragma unroll
            for (int i = 0; i < NVAL; ++i) v[i] = 0.0f;
        }
        if (lane == 0) wmax[wave] = m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < W; ++w) m = __builtin_fmaxf(m, wmax[rsub * 8 + w]);
        const typename Grid::Scale sc = Grid::scale(m, inv_norm);
        // a row with an infinity or a NaN has one in every value, or its maximum is infinite: its error is NaN
        double q2 = !(__builtin_fabsf(v[0]) < __builtin_inff()) || !(m < __builtin_inff()) ? __builtin_nan("") : 0.0;
#pragma unroll
        for (int i = 0; i < NVAL; ++i)
            if (i % SHARES == share) Grid::add(hist, v[i] * flip, sc.s, q2, l);
        __syncthreads();
        q2 = Grid::finish(hist, q2, t, NT, tot[rsub]);
        if (t > 0 && t < kGridRatios) sum += Grid::error(hist, t, q2, sc);
        __syncthreads();
    }
    // the rows a workgroup took side by side
    double* const part = reinterpret_cast<double*>(lds);
    if (rsub == 1) part[t] = sum;
    __syncthreads();
    if (rsub == 0) dev->grid_sums[blockIdx.x][t] = conc > 1 ? sum + part[t] : sum;
}

// Totals over the workgroups, eight ratios a workgroup, then, in the workgroup that is last, the search.
constexpr int kWalkThreads = 256, kWalkRatios = 8;
__global__ __launch_bounds__(kWalkThreads) void k_grid_walk(GbsDev* dev, GbsOut* out, int groups, int64_t rows, double eps, int max_evals) {
    __shared__ double part[kWalkThreads];
    __shared__ float mean[kGridRatios];
    __shared__ float trace_clips[256], trace_mse[256];
    __shared__ uint32_t came;
    __shared__ int n_evals;
    const int tid = threadIdx.x, c = blockIdx.x * kWalkRatios + (tid & (kWalkRatios - 1));
    constexpr int LANES = kWalkThreads / kWalkRatios, U = kGridGroups / LANES;
    double v[U], s = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int g = tid / kWalkRatios + u * LANES;
        v[u] = dev->grid_sums[g < groups ? g : 0][c];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s += tid / kWalkRatios + u * LANES < groups ? v[u] : 0.0;
    part[tid] = s;
    for (int h = kWalkThreads / 2; h >= kWalkRatios; h >>= 1) {
        __syncthreads();
        if (tid < h) part[tid] += part[tid + h];
    }
    // Totals go past the L2 (agent scope), are there before the workgroup counts itself, and are read past it by the last
    // one: no fence, which would write the L2 back.
    if (tid < 64) {
        if (tid < kWalkRatios) __hip_atomic_store(&dev->grid_totals[c], part[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (tid == 0) came = __hip_atomic_fetch_add(&dev->grid_ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (came != gridDim.x - 1) return;
    for (int i = tid; i < kGridRatios; i += kWalkThreads)
        mean[i] = (float)(__hip_atomic_load(&dev->grid_totals[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) / (double)rows);
    __syncthreads();
    auto put = [](auto* to, auto x) { __hip_atomic_store(to, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); };
    if (tid == 0) {
        // GbsState in units of 1 / kGridRatios
        constexpr float unit = 1.0f / kGridRatios;
        const int most = (int)fmin(eps * kGridRatios, (double)kGridRatios);      // brackets of at most so many units end the search
        int left = 0, right = kGridRatios, best = kGridRatios / 2, side = 0, evals = 1;
        float fm = mean[best];
        trace_clips[0] = (float)best * unit;
        trace_mse[0] = fm;
        // The probe to come and the two that may follow it, whose values are read while its own is compared: a step after the
        // other, each waiting for a value out of LDS, is 1.7 us for 16 steps, this about 1.2 (512 x 3584 23.4 -> 23.2 us a search,
        // 64 x 2048 19.3 -> 19.1, 512 x 4096 22.3 -> 22.1).  Six steps at a time with a path a lane: 2.1, most of it instructions fetched for one use.
        int x = (left + best) >> 1;
        float fb = mean[x], fw = fb;
        bool better = true;                              // which of the two x is
#pragma unroll 2
        while (right - left > most && evals < max_evals) {
            const int bl = side ? best : left, br = side ? right : best, wl = side ? left : x, wr = side ? x : right;
            const int xb = ((side ? bl : br) + x) >> 1, xw = ((side ? wl : wr) + best) >> 1;
            const float nb = mean[xb], nw = mean[xw];
            const float fx = better ? fb : fw;
            trace_clips[evals] = (float)x * unit;
            trace_mse[evals++] = fx;
            better = fx < fm;
            left = better ? bl : wl;
            right = better ? br : wr;
            best = better ? x : best;
            fm = better ? fx : fm;
            x = better ? xb : xw;
            fb = nb;
            fw = nw;
            side ^= 1;
        }
        put(&out->clip, (float)best * unit);
        put(&out->mse, fm);
        put(&out->evals, evals);
        n_evals = evals;
    }
    __syncthreads();
    if (tid >= 64) return;
    for (int i = tid; i < n_evals; i += 64) {
        put(&out->trace_clips[i], trace_clips[i]);
        put(&out->trace_mse[i], trace_mse[i]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the flag when the results have arrived
    if (tid == 0) put(&out->done, 1);
}

template <typename Rows, int BITS>
int launch_rows(const rq_hadamard* h, const RowArgs& a, const WaveArgs& w, int pb, int* groups, GbsDev* dev, hipStream_t s) {
    using Grid = ErrorGrid<BITS, kGridSpread, kRowThreads>;
    const int cus = h->num_cu < kGridGroups ? h->num_cu : kGridGroups;
    const int conc = a.rows > cus ? grid_rows_beside(BITS, h->max_lds) : 1;
    const int64_t passes = (a.rows + conc - 1) / conc;
    *groups = (int)(passes < cus ? passes : cus);
    void (*const fn)(WaveArgs, int, int, double, GbsDev*) = k_grid_rows<Rows, BITS>;
    const size_t lds = (size_t)conc * Grid::bytes();
    if (!allow_lds(fn, lds)) return RQ_ERR_NO_ORDER;
    launch_kernel(fn, dim3((unsigned)*groups), dim3((unsigned)(kRowThreads * conc)), lds, s, w, pb, conc,
                  1.0 / ((double)a.n * (double)a.n), dev);
    return launch_rc();
}

template <int BITS, bool F16>
int rows_pass(const rq_hadamard* h, const RowArgs& a, const WaveArgs& w, int* groups, GbsDev* dev, hipStream_t s) {
    const int pb = a.p > 1 ? a.p << (a.log2m - 7) : 0;
    if (a.p > 1) return pb <= 16 ? launch_rows<BlockRows<1, F16>, BITS>(h, a, w, pb, groups, dev, s)
                                 : launch_rows<BlockRows<2, F16>, BITS>(h, a, w, pb, groups, dev, s);
    switch (a.log2m) {
        case 10: return launch_rows<SylvesterRows<2, 1, F16>, BITS>(h, a, w, pb, groups, dev, s);
        case 11: return launch_rows<SylvesterRows<4, 2, F16>, BITS>(h, a, w, pb, groups, dev, s);
        case 12: return launch_rows<SylvesterRows<8, 4, F16>, BITS>(h, a, w, pb, groups, dev, s);
        case 13: return launch_rows<SylvesterRows<16, 4, F16>, BITS>(h, a, w, pb, groups, dev, s);
        default: return RQ_ERR_NO_ORDER;
    }
}

}  // namespace

// Brackets down to 2 / kGridRatios, see above, where the search is long enough (search_rule.h).
bool gbs_grid_supports(const rq_hadamard* h, const RowArgs& a, double eps, int steps) {
    if (eps < 2.0 / kGridRatios) return false;
    const int cus = h->num_cu < kGridGroups ? h->num_cu : kGridGroups;
    GridCase c{a.rows, a.n, a.bits, cus, a.p == 1, grid_rows_beside(a.bits, h->max_lds), gbs_row_waves(h, a), 0, 0};
    if (c.waves == 0) {
        int pb, cb;
        if (wave_quant_error_supports(h, a) || !wg_block_supports(h, a, true) || !wg_shape(a, &pb, &cb)) return false;
        c.beside = grid_rows_beside(a.bits, h->max_lds, (int64_t)wg_grid_ops_bytes(pb));
        c.rows_per_pass = 16 >> cb;
        c.threads = 64 * ((pb + 15) / 16);
    }
    return gbs_grid_pays(c, steps);
}

int gbs_grid(const rq_hadamard* h, const RowArgs& a, GbsDev* dev, GbsOut* out, double eps, int max_evals, hipStream_t s) {
    const bool f16 = a.dtype == RQ_F16;
    WaveArgs w{static_cast<const uint16_t*>(a.X), a.rows, a.d, a.ld,
               static_cast<const u32x4*>(f16 ? h->d_tiles_f16 : h->d_tiles), nullptr, nullptr, 0.0, 0.0};
    w.f16 = f16;
    int groups = 0;
    const int rc = gbs_row_waves(h, a) == 0 ? wg_grid_rows(h, a, dev, &groups, s) : a.bits == 4 ? (f16 ? rows_pass<4, true>(h, a, w, &groups, dev, s) : rows_pass<4, false>(h, a, w, &groups, dev, s))
                               : (f16 ? rows_pass<3, true>(h, a, w, &groups, dev, s) : rows_pass<3, false>(h, a, w, &groups, dev, s));
    if (rc != RQ_OK) return rc;
    launch_kernel(k_grid_walk, dim3(kGridRatios / kWalkRatios), dim3(kWalkThreads), 0, s, dev, out, groups, a.rows, eps, max_evals);
    return launch_rc();
}

}  // namespace rq
