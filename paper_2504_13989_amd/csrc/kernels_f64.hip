// rotate_quantize for fp32 rows: the row is transformed and quantized in fp64 (log2 n fp32 stages on 24-bit inputs move
// a value by up to 2e-7 of its size, enough to push one code in a million across a rounding boundary), orders
// p * 2^k with 2^k >= 32 and p = 1 or a block order of at most 256 (sections 2.1, 2.3, 3.1, 4.2).
//
// fp64 adds run at the rate of fp32 ones on this chip, so the vector ALU is not what a row costs; the passes over LDS
// are.  A thread therefore takes 16 values through four butterfly stages in registers at a time (radix 16), and
// the first group of stages works on the values as they come from memory, the last one ends in the
// quantizer: an order of 2^12 crosses LDS twice.
//   first    2^R1 values per item, a stride of 2^(k - R1) apart, from memory (coalesced, zero beyond d); R1 takes up
//            what 4 does not divide of k;
//   block    (p > 1) outputs 16 part .. + 15 of a column per thread: one LDS read and 16 fused multiply-adds with
//            +-1.0 in scalar registers (the wave's part is uniform; its signs come as one bit mask per input row);
//   middle   16 values a stride of 16 apart (orders with k >= 10; twice for 2^14);
//   last     16 consecutive values: absmax over the row, scale, codes, 8 or 6 bytes per thread.
// LDS holds the rows of the workgroup with one value of padding after every 16: the last stage reads 16 consecutive
// values per lane, which without it would put all lanes on the same banks.  Rows shorter than 1024 values share a
// workgroup (RW rows).
// Measured against one 256-thread workgroup per row with an LDS pass and a barrier for each stage (the general
// kernel): 64 x 256 5.5 -> 2.9 us, 783 x 8192 66 -> 12.6 us, 1257 x 896 17.8 -> 10.6 us.  The loads go through one
// buffer resource per workgroup: as predicated loads they came out as sixteen branches, each waiting for memory
// (64 x 256 then took 4.6 us, 783 x 8192 28 us).
#include "wave_common.h"

namespace rq {
namespace {

struct F64Args {
    const float* X;
    int64_t rows;
    int d;
    int64_t ld;
    int p;
    const uint32_t* signs;    // [part][input block row]: bit q set where output row 16 part + q takes it negated
    uint32_t* codes;
    float* scales;
    double clip, c2;          // c2 = 1 / (sqrt(n) (2^b - 1))
};

// How the k stages fall on the passes: R1 in the first, 4 in each of MIDS middle ones and in the last.
constexpr int f64_mids(int k) { return k <= 9 ? 0 : k <= 13 ? 1 : 2; }
constexpr int f64_r1(int k) { return k - 4 - 4 * f64_mids(k); }
// Rows of a workgroup: at least one wave at 16 values per thread; block orders have at least 64 columns.
constexpr int f64_rw(int k, bool block) { return block ? (k < 6 ? 2 : 1) : k < 10 ? 1 << (10 - k) : 1; }

__device__ __forceinline__ int pad(int i) { return i + (i >> 4); }

template <int R>
__device__ __forceinline__ void butterflies(double (&v)[1 << R]) {
#pragma unroll
    for (int s = 1; s < (1 << R); s <<= 1)
#pragma unroll
        for (int i = 0; i < (1 << R); ++i)
            if (!(i & s)) {
                const double x = v[i], y = v[i | s];
                v[i] = x + y;
                v[i | s] = x - y;
            }
}

template <int K, bool BLOCK, int BITS>
__global__ __launch_bounds__(1024) void k_f64_rows(F64Args a) {
    constexpr int R1 = f64_r1(K), MIDS = f64_mids(K), RW = f64_rw(K, BLOCK), M = 1 << K;
    extern __shared__ __attribute__((aligned(16))) double buf[];
    __shared__ unsigned long long smax[RW];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int n = BLOCK ? a.p * M : M;
    const int64_t row0 = group_index() * RW;
    if (row0 >= a.rows) return;                           // whole workgroup
    if (tid < RW) smax[tid] = 0ull;
    // the sign masks of this wave's part, one lane an input block row, on their way while the row comes in
    constexpr int LOG2C = K < 6 ? 6 : K;                  // columns of the workgroup (a wave has one part)
    const int part = BLOCK ? __builtin_amdgcn_readfirstlane(tid >> LOG2C) : 0;
    [[maybe_unused]] uint32_t masks = 0;
    if constexpr (BLOCK) masks = (tid & 63) < a.p ? a.signs[part * a.p + (tid & 63)] : 0u;
    {
        constexpr int NV = 1 << R1, ITEMS = R1 >= 4 ? 1 : 16 >> R1, SH = K - R1;
        const int per_row = n >> R1, total = RW * per_row;
        float x[ITEMS][NV];
        auto place = [&](int it, int* rs) {               // row of the workgroup and first position of an item
            *rs = !BLOCK ? it >> (K - R1) : RW == 2 && it >= per_row;
            const int rem = it - *rs * per_row;
            return ((rem >> SH) << K) | (rem & ((1 << SH) - 1));
        };
        // the workgroup's rows as one buffer resource: reads beyond it (columns from d on of the last row, rows past
        // the end) return zero without a branch, so that all loads are in flight together
        const int64_t left = a.rows - row0;
        const int live_rows = left < RW ? (int)left : RW;
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.X) + row0 * a.ld, 0,
                                                            (int)(((live_rows - 1) * a.ld + a.d) * 4), 0x00020000);
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int it = tid + i * nt;
            int rs;
            const int j0 = place(it, &rs);
            const uint32_t base = (uint32_t)(rs * (int)a.ld + j0) * 4u;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                uint32_t off = base + (uint32_t)(v << SH) * 4u;
                if (RW > 1 && j0 + (v << SH) >= a.d) off = 0x80000000u;
                if (BLOCK && it >= total) off = 0x80000000u;
                x[i][v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 2));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int it = tid + i * nt;
            if (it < total) {
                int rs;
                const int j0 = place(it, &rs);
                double* const at = buf + pad(rs * n + j0);            // (a stride of 16 or more: padding is linear in k)
                double v[NV];
#pragma unroll
                for (int k = 0; k < NV; ++k) v[k] = (double)x[i][k];
                butterflies<R1>(v);
#pragma unroll
                for (int k = 0; k < NV; ++k) at[k * (17 << (SH - 4))] = v[k];
            }
        }
    }
    __syncthreads();
    if constexpr (BLOCK) {
        const int col = tid & ((1 << LOG2C) - 1);
        double* const at = buf + pad((col >> K) * n + (col & (M - 1)));
        constexpr int STEP = 17 << (K - 4);               // from block row to block row
        double acc[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] = 0.0;
        for (int b0 = 0; b0 < a.p; b0 += 64) {
            if (b0) masks = b0 + (tid & 63) < a.p ? a.signs[part * a.p + b0 + (tid & 63)] : 0u;
            const int nb = a.p - b0 < 64 ? a.p - b0 : 64;             // a multiple of 4, as p is
            for (int b = 0; b < nb; b += 4) {
                double x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = at[(b0 + b + u) * STEP];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t m = __builtin_amdgcn_readlane(masks, b + u);
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const uint32_t hi = 0x3FF00000u | ((m << (31 - q)) & 0x80000000u);
                        acc[q] = fma(__builtin_bit_cast(double, (uint64_t)hi << 32), x[u], acc[q]);
                    }
                }
            }
        }
        __syncthreads();                                  // every input of the product has been read
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if (16 * part + q < a.p) at[(16 * part + q) * STEP] = acc[q];
        __syncthreads();
    }
    const int items = RW * n >> 4;                        // at most one per thread
#pragma unroll
    for (int mid = MIDS; mid > 0; --mid) {
        if (tid < items) {
            const int sh = 4 * mid;
            double* const at = buf + pad(((tid >> sh) << (sh + 4)) | (tid & ((1 << sh) - 1)));
            double v[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) v[k] = at[k * (17 << (sh - 4))];
            butterflies<4>(v);
#pragma unroll
            for (int k = 0; k < 16; ++k) at[k * (17 << (sh - 4))] = v[k];
        }
        __syncthreads();
    }
    const int per_row = n >> 4;
    const int rs = !BLOCK ? tid >> (K - 4) : RW == 2 && tid >= per_row, t_in_row = tid - rs * per_row;
    const bool live = tid < items && row0 + rs < a.rows;
    double y[16];
    if (live) {
#pragma unroll
        for (int k = 0; k < 16; ++k) y[k] = buf[tid * 17 + k];
        butterflies<4>(y);
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) y[k] = 0.0;
    }
    double m = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) m = fmax(m, fabs(y[k]));
    // a row is a multiple of 8 threads
    for (int s = 1; s < 8; s <<= 1) m = fmax(m, __shfl_xor(m, s, 64));
    if ((tid & 7) == 0 && live) atomicMax(&smax[rs], (unsigned long long)__double_as_longlong(m));
    __syncthreads();
    if (!live) return;
    m = __longlong_as_double((long long)smax[rs]);
    constexpr double kLvl = (double)((1 << BITS) - 1);
    constexpr double kMax = (double)((1 << (BITS - 1)) - 1), kMin = -(double)(1 << (BITS - 1));
    const double s = m > 0.0 ? kLvl / (a.clip * m) : 0.0;
    uint64_t w = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        // rounded to the nearest-even integer by the addition: its low bits are the code
        const double t = fmin(fmax(y[k] * s, kMin), kMax) + 6755399441055744.0;            // 1.5 * 2^52
        w |= (uint64_t)((uint32_t)__double_as_longlong(t) & ((1u << BITS) - 1u)) << (BITS * k);
    }
    typedef uint32_t u32_any __attribute__((aligned(2)));
    uint8_t* out = reinterpret_cast<uint8_t*>(a.codes) + (row0 + rs) * (int64_t)(n / 8 * BITS) + t_in_row * (2 * BITS);
    *reinterpret_cast<u32_any*>(out) = (uint32_t)w;
    if constexpr (BITS == 4) *reinterpret_cast<u32_any*>(out + 4) = (uint32_t)(w >> 32);
    else *reinterpret_cast<uint16_t*>(out + 4) = (uint16_t)(w >> 32);
    if (t_in_row == 0) a.scales[row0 + rs] = (float)(a.clip * m * a.c2);
}

struct Shape {
    int threads, rw;
    size_t lds;
};

// Workgroup of an order: 16 values per thread; block orders have 16 outputs of a column per thread in the block
// stage (columns x parts threads).
bool shape_of(const rq_hadamard* h, Shape* s) {
    const int n = h->f.n, p = h->f.p, k = h->f.log2m;
    if (p == 1 ? k < 7 || k > 14 : k < 5 || k > 9 || p % 4 != 0 || p > kMaxPaleyOrder) return false;
    s->rw = f64_rw(k, p > 1);
    s->threads = p == 1 ? s->rw * n / 16 : ((p + 15) / 16) << (k < 6 ? 6 : k);
    s->lds = (size_t)s->rw * n * 17 / 16 * sizeof(double);
    return s->threads <= 1024 && s->lds + 512 <= (size_t)h->max_lds;
}

using Kernel = void (*)(F64Args);

template <bool BLOCK>
Kernel pick(int k, int bits) {
    auto of = [&](auto kc) -> Kernel {
        constexpr int K = decltype(kc)::value;
        if constexpr (BLOCK ? K >= 5 && K <= 9 : K >= 7)
            return bits == 4 ? k_f64_rows<K, BLOCK, 4> : k_f64_rows<K, BLOCK, 3>;
        else
            return nullptr;
    };
    switch (k) {
        case 5: return of(std::integral_constant<int, 5>{});
        case 6: return of(std::integral_constant<int, 6>{});
        case 7: return of(std::integral_constant<int, 7>{});
        case 8: return of(std::integral_constant<int, 8>{});
        case 9: return of(std::integral_constant<int, 9>{});
        case 10: return of(std::integral_constant<int, 10>{});
        case 11: return of(std::integral_constant<int, 11>{});
        case 12: return of(std::integral_constant<int, 12>{});
        case 13: return of(std::integral_constant<int, 13>{});
        case 14: return of(std::integral_constant<int, 14>{});
        default: return nullptr;
    }
}
Kernel pick(int k, bool block, int bits) { return block ? pick<true>(k, bits) : pick<false>(k, bits); }

}  // namespace

// Sign masks of the block stage: [part][input row], 16 output rows to a part.
std::vector<uint32_t> f64_block_signs(const std::vector<int8_t>& block, int p) {
    const int parts = (p + 15) / 16;
    std::vector<uint32_t> t((size_t)parts * p, 0u);
    for (int a = 0; a < p; ++a)
        for (int b = 0; b < p; ++b)
            if (block[(size_t)a * p + b] < 0) t[(size_t)(a / 16) * p + b] |= 1u << (a % 16);
    return t;
}

// Set-up: whether the order's rows fit, and the kernels' LDS limit.
bool f64_prepare(const rq_hadamard* h) {
    Shape s;
    if (!shape_of(h, &s)) return false;
    for (int bits = 3; bits <= 4; ++bits)
        if (s.lds > 48 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(pick(h->f.log2m, h->f.p > 1, bits)),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)s.lds) != hipSuccess)
            return false;
    return true;
}

bool f64_rows_supports(const rq_hadamard* h, const RowArgs& a) {
    return h->device >= 0 && h->f64_ok && a.dtype == RQ_F32 && a.ld <= (1 << 26);     // (32-bit offsets inside a workgroup's rows)
}

int f64_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes, float* scales, hipStream_t s) {
    Shape sh;
    if (!shape_of(h, &sh)) return RQ_ERR_NO_ORDER;
    const int64_t groups = (a.rows + sh.rw - 1) / sh.rw;
    if (groups > 0x7fffffffLL) return RQ_ERR_ARG;
    const F64Args f{static_cast<const float*>(a.X), a.rows, a.d, a.ld, a.p, static_cast<const uint32_t*>(h->d_signs), codes,
                    scales, (double)clip,
                    1.0 / (std::sqrt((double)a.n) * (double)((1 << a.bits) - 1))};
    launch_kernel(pick(a.log2m, a.p > 1, a.bits), group_grid(groups, sh.threads), dim3(sh.threads), sh.lds, s, f);
    return launch_rc();
}

}  // namespace rq
