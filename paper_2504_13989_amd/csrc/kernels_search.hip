// The clip-ratio search of Algorithm 1 (section 4.1) on the device, in the three forms that serve what the grid form
// (kernels_gridsearch.hip) does not: brackets below 1 / 256, other row formats and orders, searches of few steps, many short rows.
//
// Batches (any tensor): between the batches of objective values a search
// needs (one quant_error pass each), a kernel of one workgroup averages the batch, walks the search with it and writes
// the clip ratios of the next batch to device memory, where the next pass reads them.  The host enqueues all of it and
// waits once; a trip to the host between the batches cost about 8 us each, as much as a pass on a small tensor.
// Resident (tensors that fit the chip's registers): one launch.  Stepped: the resident form's steps as a launch each,
// where that cannot run; which of the two a call takes depends on what else the device is doing, so they compute the same
// values bit for bit.
//
// The probes are taken in the listing's order, but evaluated ahead of time in batches: where a probe lies depends only
// on the outcomes of the comparisons before it, so one batch covers every probe the next `depth` steps can ask for, a
// binary tree over those outcomes.  The sequence of probes is that of the one-at-a-time loop.
#include <mutex>

#include "row_rotation.h"
#include "search_state.h"

namespace rq {

// Probe of node i (1 .. 2^depth - 1) of the tree below `st`, in heap order (children 2 i for "better", 2 i + 1 for "not
// better"); false where the search ends before it gets there.
__host__ __device__ inline bool gbs_node(GbsState st, double eps, int depth, int i, double* x) {
    bool live = st.width() > eps;
    for (int b = depth - 2; b >= 0; --b)
        if (i >> (b + 1)) {                               // below the node's leading bit
            st.next(st.probe(), !((i >> b) & 1));
            live = live && st.width() > eps;
        }
    *x = st.probe();
    return live;
}

namespace {

constexpr int kStepThreads = 1024;

// partial: [count] sums per clip ratio, `stride` rows apart, in rows of as many values as the batch has clip ratios.
// What the kernel costs is latency: it is one workgroup in the middle of a chain of launches.  All loads of a thread are
// issued before the first wait, every lane of the first wave works out its own node of the tree, and host memory is
// written once, at the end of the search (a store over the bus holds the end of the kernel up).
__global__ __launch_bounds__(kStepThreads) void k_gbs_step(GbsDev* state, GbsOut* out, int first, double eps, int depth, int max_evals,
                                                           double levels, const double* partial, int64_t rows, int64_t count,
                                                           int64_t stride) {
    __shared__ double part[kStepThreads];
    __shared__ float value[RQ_MAX_CLIPS];
    __shared__ double node_x[RQ_MAX_CLIPS];
    __shared__ int node_slot[RQ_MAX_CLIPS];
    __shared__ GbsState next_st;
    __shared__ int n_evals, finished;
    const int tid = threadIdx.x, lane = tid & 63;
    if (!first && state->done) return;                    // a batch enqueued beyond the end of the search
    const int nodes = 1 << depth;
    const GbsState st0 = first ? gbs_start() : state->st;
    const float fm0 = first ? 0.0f : state->fm;
    const int evals0 = first ? 0 : state->evals;
    const int lead = first ? 1 : 0;                       // the starting point leads the first batch
    // (every wave works the tree out for itself: the batch's size is needed at once)
    double x;
    const bool live = gbs_node(st0, eps, depth, lane, &x) && lane >= 1 && lane < nodes;
    const uint64_t mask = __ballot(live);
    const int n = lead + __popcll(mask);
    if (tid < 64) {
        node_x[lane] = x;
        node_slot[lane] = lead + __popcll(mask & ((1ull << lane) - 1ull));
    }
    int kp = 1;
    while (kp < n) kp <<= 1;
    {
        // consecutive threads read consecutive values: clip ratio tid % kp of row tid / kp, a fixed order of summation
        const int k = tid & (kp - 1), lanes = kStepThreads / kp;
        const int kc = k < n ? k : n - 1;
        double acc = 0.0;
        constexpr int U = 8;
        for (int64_t r0 = tid / kp; r0 < count; r0 += (int64_t)U * lanes) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t r = r0 + (int64_t)u * lanes;
                v[u] = partial[(r < count ? r : count - 1) * stride * n + kc];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) acc += r0 + (int64_t)u * lanes < count ? v[u] : 0.0;
        }
        part[tid] = acc;
        for (int s = kStepThreads / 2; s >= kp; s >>= 1) {
            __syncthreads();
            if (tid < s) part[tid] += part[tid + s];
        }
        if (tid < n) value[tid] = (float)(part[tid] / (double)rows);
        __syncthreads();
    }
    if (tid == 0) {
        GbsState st = st0;
        float fm = fm0;
        int evals = evals0;
        auto record = [&](float c, float v) {
            state->trace_clips[evals] = c;
            state->trace_mse[evals] = v;
            ++evals;
        };
        if (first) {
            fm = value[0];
            record((float)st.best, fm);
        }
        int idx = 1;
        for (int lvl = 0; lvl < depth && st.width() > eps && evals < max_evals; ++lvl) {
            const double p = node_x[idx];
            const float fx = value[node_slot[idx]];
            record((float)p, fx);
            const bool better = fx < fm;
            if (better) fm = fx;
            st.next(p, better);
            idx = 2 * idx + (better ? 0 : 1);
        }
        finished = st.width() <= eps || evals >= max_evals;
        n_evals = evals;
        next_st = st;
        state->st = st;
        state->fm = fm;
        state->evals = evals;
        state->done = finished;
        if (first && !finished) out->done = 0;
        if (finished) {
            state->clips.n = 0;
            out->clip = (float)st.best;
            out->mse = fm;
            out->evals = evals;
        }
    }
    __syncthreads();
    if (finished) {
        // (the trace was written by this workgroup: visible to it after the barrier)
        if (tid < n_evals) {
            out->trace_clips[tid] = state->trace_clips[tid];
            out->trace_mse[tid] = state->trace_mse[tid];
        }
        if (tid == 0) out->done = 1;                      // (the host reads the results after the stream is done)
        return;
    }
    if (tid < 64) {
        const bool more = gbs_node(next_st, eps, depth, lane, &x) && lane >= 1 && lane < nodes;
        const uint64_t m = __ballot(more);
        if (more) state->clips.set(__popcll(m & ((1ull << lane) - 1ull)), (float)x, levels);
        if (tid == 0) state->clips.n = __popcll(m);
    }
}

// ---------------------------------------------------------------------------------------------
// Resident form: the tensor is rotated once, into the registers of as many waves as hold it, and stays there for the
// whole search - one launch.  Each step looks three probes ahead (seven clip ratios, with the starting point eight at
// first); the workgroups' sums meet through a small exchange buffer in device memory, and every workgroup averages all
// of them in the same order and so takes the same decisions.  A step costs the arithmetic of its ratios and one
// exchange between the workgroups (about 3 us, whence three probes a step); the batched form pays two launches and a
// repeated rotation for four steps.
//
// Exchange: a sum travels in one 64-bit word, the upper 48 bits of the fp64 value (rounded to nearest: 37 significant
// bits, where the fp32 sums of the waves it is made of have 24) and the number of the step below them, so that a word is
// its own flag.  (Whole values in two words are twice the traffic: 512 x 4096 46 -> 57 us.)  Two sets of words
// alternate, which is enough, because a workgroup that is two steps ahead has seen every other one publish the step
// between.  At most one workgroup per compute unit is launched, so all are resident together unless other work holds
// the chip; a workgroup that waits longer than wait_ticks gives the search up (everyone does in the end), and the host
// takes the stepped form: the same kernel, which leaves its sums in the workspace and returns after each step; the next
// launch picks them up (512 x 4096: 65 us).
constexpr int kMaxGroups = 1024;
constexpr uint64_t kWaitTicks = 30000;                    // of the 100 MHz clock: 300 us, a hundred times a step
constexpr int kAhead = kStepsAhead, kSlots = 1 << kAhead;  // probes a step looks ahead, clip ratios of a step

struct ResidentArgs {
    GbsOut* out;
    uint64_t* exchange;       // [2][kMaxGroups][kSlots]
    uint32_t epoch;           // 16-bit number of the first step; no word in the buffer has it or one of the next 255
    double eps, levels;
    int max_evals;
    int rows_per_group;
    uint64_t wait_ticks;
    // stepped form
    GbsCarry* carry;          // [2], taken in turn
    double* sums;             // [2][workgroups][kSlots]
    uint32_t step;
};

template <typename Rows, int BITS, bool STEPPED>
__global__ __launch_bounds__(1024) void k_gbs_resident(WaveArgs a, int pb, double inv_norm, ResidentArgs r) {
    constexpr int W = Rows::W, NVAL = Rows::NVAL;
    __shared__ float wmax[16];
    __shared__ __attribute__((aligned(16))) float esum[kSlots][16];      // [slot][wave], zero beyond the waves there are
    __shared__ __attribute__((aligned(16))) double gsum[kSlots][16];
    __shared__ int gave_up;
    __shared__ float trace_clips[STEPPED ? 1 : 256], trace_mse[STEPPED ? 1 : 256];    // (kept by the first workgroup)
    const int tid = threadIdx.x, lane = tid & 63, nt = (int)blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rsub = wave / W, seg = wave - rsub * W;
    const int64_t row = (int64_t)blockIdx.x * r.rows_per_group + rsub;
    const bool live = row < a.rows;
    float v[NVAL], flip = 1.0f;
    float m = 0.0f;
    if (live) {
        m = Rows::rotate(a, pb, row, seg, lane, v, &flip);
    } else {
#pragma unroll
        for (int i = 0; i < NVAL; ++i) v[i] = 0.0f;
    }
    if (lane == 0) wmax[wave] = m;
    for (int i = tid; i < kSlots * 16; i += nt) {
        esum[i >> 4][i & 15] = 0.0f;
        gsum[i >> 4][i & 15] = 0.0;
    }
    if (tid == 0) gave_up = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < W; ++w) m = __builtin_fmaxf(m, wmax[rsub * W + w]);
    const double inv_m = m > 0.0f ? 1.0 / (double)m : 0.0, inv_rows = 1.0 / (double)a.rows;
    const double m_over_levels = (double)m / r.levels;
    const int words = (int)gridDim.x * kSlots;
    auto put = [](auto* to, auto x) { __hip_atomic_store(to, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); };

    GbsState st = gbs_start();
    float fm = 0.0f;
    int evals = 0;

    // The sums of this workgroup's rows at the clip ratios of a step, one thread a ratio: returned to the first kSlots.
    auto evaluate = [&](bool first) -> uint64_t {
        // the step's clip ratios, one lane a slot (first step: the starting point, then nodes 1 .. 7; later nodes 1 .. 7); a
        // slot the search cannot reach repeats the best point
        const int node = (lane & (kSlots - 1)) + (first ? 0 : 1);
        double x = st.best;
        bool reach = node == 0;
        if (node >= 1 && node < kSlots) {
            double p;
            reach = gbs_node(st, r.eps, kAhead, node, &p);
            if (reach) x = p;
        }
        const uint32_t wanted = (uint32_t)__ballot(reach) & ((1u << kSlots) - 1u);
        const double cf = (double)(float)x;
        const float s_slot = (float)(r.levels / cf * inv_m), d_slot = (float)(cf * m_over_levels);
        constexpr float kQmax = (float)((1 << (BITS - 1)) - 1), kQmin = -(float)(1 << (BITS - 1));
        // four slots at a time (independent chains); the last step of a search often wants only the first
#pragma unroll
        for (int k0 = 0; k0 < kSlots; k0 += 4) {
            if (!(wanted >> k0 & 15u)) continue;
            float sk[4], ndk[4], e2[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                sk[k] = flip * __uint_as_float((uint32_t)__builtin_amdgcn_readlane(__float_as_uint(s_slot), k0 + k));
                ndk[k] = -flip * __uint_as_float((uint32_t)__builtin_amdgcn_readlane(__float_as_uint(d_slot), k0 + k));
                e2[k] = 0.0f;
            }
#pragma unroll
            for (int i = 0; i < NVAL; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(v[i] * sk[k]), kQmin, kQmax);
                    const float e = fmaf(q, ndk[k], v[i]);
                    e2[k] = fmaf(e, e, e2[k]);
                }
#pragma unroll
            for (int k = 0; k < 4; ++k) e2[k] += dpp_f<kDppXor1>(e2[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) e2[k] += dpp_f<kDppXor2>(e2[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) e2[k] += dpp_f<kDppHalfMirror>(e2[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) e2[k] += dpp_f<kDppRor8>(e2[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                e2[k] = rows_sum(e2[k]);
                if (lane == k) esum[k0 + k][wave] = e2[k];
            }
        }
        __syncthreads();
        double t = 0.0;
        if (tid < kSlots) {
#pragma unroll
            for (int w = 0; w < 16; ++w) t += (double)esum[tid][w];
        }
        // the bits a sum has in the exchange, in both forms
        return ((uint64_t)__double_as_longlong(t * inv_norm) + 0x8000u) & ~0xffffull;
    };
    // Everyone's sums, in a fixed order: fetch(i0, value) gives the thread the sums i0, i0 + nt, i0 + 2 nt, i0 + 3 nt (those
    // there are) or returns false.  Consecutive lanes read consecutive sums (reading a workgroup's sums one after the
    // other in a lane multiplied the traffic by eight: 7 us a step).  Then the search takes the step's decisions.
    auto decide = [&](bool first, auto fetch) {
        double f = 0.0;
        bool lost = false;
        for (int i0 = tid; i0 < words && !lost; i0 += 4 * nt) {
            double value[4];
            lost = !fetch(i0, value);
#pragma unroll
            for (int u = 0; u < 4; ++u) f += i0 + u * nt < words ? value[u] : 0.0;
        }
        if (lost) gave_up = 1;
        for (int sh = kSlots; sh < 64; sh <<= 1) f += __shfl_xor(f, sh, 64);
        if (lane < kSlots) gsum[lane][wave] = f;
        __syncthreads();
        if (gave_up) return false;                        // the whole workgroup; the others run into the same limit
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) t += gsum[lane & (kSlots - 1)][w];
        const float mean = (float)(t * inv_rows);         // lane k: the objective at slot k
        auto value = [&](int slot) {
            return __uint_as_float((uint32_t)__builtin_amdgcn_readlane(__float_as_uint(mean), __builtin_amdgcn_readfirstlane(slot)));
        };
        auto record = [&](float c, float f1) {
            if (blockIdx.x == 0 && tid == 0) {
                if constexpr (STEPPED) {
                    put(&r.out->trace_clips[evals], c);
                    put(&r.out->trace_mse[evals], f1);
                } else {
                    trace_clips[evals] = c;
                    trace_mse[evals] = f1;
                }
            }
            ++evals;
        };
        const int lead = first ? 1 : 0;
        if (first) {
            fm = value(0);
            record((float)st.best, fm);
        }
        int at = 1;
        for (int lvl = 0; lvl < kAhead && st.width() > r.eps && evals < r.max_evals; ++lvl) {
            const double p = st.probe();
            const float fx = value(at - 1 + lead);
            record((float)p, fx);
            const bool better = fx < fm;
            if (better) fm = fx;
            st.next(p, better);
            at = 2 * at + (better ? 0 : 1);
        }
        return true;
    };
    auto over = [&] { return st.width() <= r.eps || evals >= r.max_evals; };
    // Results to host memory by one wave, the flag when they have arrived there.
    auto finish = [&] {
        if (blockIdx.x != 0 || wave != 0) return;
        if constexpr (!STEPPED)
            for (int i = lane; i < evals; i += 64) {
                put(&r.out->trace_clips[i], trace_clips[i]);
                put(&r.out->trace_mse[i], trace_mse[i]);
            }
        if (lane == 0) {
            put(&r.out->clip, (float)st.best);
            put(&r.out->mse, fm);
            put(&r.out->evals, evals);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) put(&r.out->done, 1);
    };

    if constexpr (STEPPED) {
        const uint32_t step = r.step;
        const bool keeps = blockIdx.x == 0 && tid == 0;
        GbsCarry* const next = r.carry + (step & 1);
        if (step > 0) {
            const GbsCarry last = r.carry[(step - 1) & 1];
            bool done = last.done;                        // (a launch enqueued beyond the end of the search)
            if (!done) {
                st = last.st;
                fm = last.fm;
                evals = last.evals;
                const double* const from = r.sums + (size_t)((step - 1) & 1) * words;
                decide(step == 1, [&](int i0, double (&value)[4]) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) value[u] = from[i0 + u * nt < words ? i0 + u * nt : i0];
                    return true;
                });
                done = over();
                if (done) finish();
            }
            if (done) {
                if (keeps) next->done = 1;
                return;
            }
        } else if (keeps) {
            put(&r.out->done, 0);
        }
        if (keeps) *next = GbsCarry{st, fm, evals, 0};
        const uint64_t sum = evaluate(step == 0);
        if (tid < kSlots) r.sums[(size_t)(step & 1) * words + blockIdx.x * kSlots + tid] = __longlong_as_double((long long)sum);
    } else {
        for (uint32_t step = 0;; ++step) {
            const uint64_t sum = evaluate(step == 0), tag = (r.epoch + step) & 0xffffu;
            uint64_t* const set = r.exchange + (size_t)(step & 1) * kMaxGroups * kSlots;
            if (tid < kSlots)
                __hip_atomic_store(set + (size_t)blockIdx.x * kSlots + tid, sum | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t began = wall_clock64();
            const bool met = decide(step == 0, [&](int i0, double (&value)[4]) {
                for (;;) {
                    uint64_t w[4];
                    bool ready = true;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        w[u] = __hip_atomic_load(set + (i0 + u * nt < words ? i0 + u * nt : i0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int u = 0; u < 4; ++u) ready = ready && (w[u] & 0xffffull) == tag;
#pragma unroll
                    for (int u = 0; u < 4; ++u) value[u] = __longlong_as_double((long long)(w[u] & ~0xffffull));
                    if (ready) return true;
                    if (wall_clock64() - began > r.wait_ticks) return false;
                }
            });
            if (!met) return;
            if (over()) break;
        }
        finish();
    }
}

// Waves per row of the resident form, 0 where the order has none.
int resident_waves(const RowArgs& a) {
    if (a.p == 1) return a.log2m == 10 ? 1 : a.log2m == 11 ? 2 : a.log2m == 12 || a.log2m == 13 ? 4 : 0;
    return (a.p << (a.log2m - 7)) <= 16 ? 1 : 2;
}

template <int BITS, bool F16, bool STEPPED>
int launch_resident(const RowArgs& a, const WaveArgs& w, double inv_norm, const ResidentArgs& r, dim3 grid, dim3 block, hipStream_t s) {
    const int pb = a.p > 1 ? a.p << (a.log2m - 7) : 0;
    auto go = [&](auto kernel) { launch_kernel(kernel, grid, block, 0, s, w, pb, inv_norm, r); };
    if (a.p > 1) {
        if (pb <= 16) go(k_gbs_resident<BlockRows<1, F16>, BITS, STEPPED>); else go(k_gbs_resident<BlockRows<2, F16>, BITS, STEPPED>);
    } else {
        switch (a.log2m) {
            case 10: go(k_gbs_resident<SylvesterRows<2, 1, F16>, BITS, STEPPED>); break;
            case 11: go(k_gbs_resident<SylvesterRows<4, 2, F16>, BITS, STEPPED>); break;
            case 12: go(k_gbs_resident<SylvesterRows<8, 4, F16>, BITS, STEPPED>); break;
            case 13: go(k_gbs_resident<SylvesterRows<16, 4, F16>, BITS, STEPPED>); break;
            default: return RQ_ERR_NO_ORDER;
        }
    }
    return launch_rc();
}

// Grid, block and what both forms share of the arguments.
template <bool STEPPED>
int resident_launch(const rq_hadamard* h, const RowArgs& a, ResidentArgs r, hipStream_t s) {
    const int w = resident_waves(a);
    const int groups = h->num_cu < kMaxGroups ? h->num_cu : kMaxGroups;
    const int per = (int)((a.rows + groups - 1) / groups);
    const bool f16 = a.dtype == RQ_F16;
    WaveArgs wa{static_cast<const uint16_t*>(a.X), a.rows, a.d, a.ld,
                static_cast<const u32x4*>(f16 ? h->d_tiles_f16 : h->d_tiles), nullptr, nullptr, 0.0, 0.0};
    wa.f16 = f16;
    r.levels = (double)((1 << a.bits) - 1);
    r.rows_per_group = per;
    const double inv_norm = 1.0 / ((double)a.n * (double)a.n);
    const dim3 grid((unsigned)((a.rows + per - 1) / per)), block((unsigned)(64 * per * w));
    if (f16)
        return a.bits == 4 ? launch_resident<4, true, STEPPED>(a, wa, inv_norm, r, grid, block, s)
                           : launch_resident<3, true, STEPPED>(a, wa, inv_norm, r, grid, block, s);
    return a.bits == 4 ? launch_resident<4, false, STEPPED>(a, wa, inv_norm, r, grid, block, s)
                       : launch_resident<3, false, STEPPED>(a, wa, inv_norm, r, grid, block, s);
}

}  // namespace

int gbs_row_waves(const rq_hadamard* h, const RowArgs& a) { return wave_quant_error_supports(h, a) ? resident_waves(a) : 0; }

bool gbs_resident_supports(const rq_hadamard* h, const RowArgs& a) {
    const int w = gbs_row_waves(h, a);
    if (w == 0) return false;
    const int groups = h->num_cu < kMaxGroups ? h->num_cu : kMaxGroups;
    return a.rows <= (int64_t)groups * (16 / w);          // 16 waves per compute unit
}

size_t gbs_exchange_bytes() { return (size_t)2 * kMaxGroups * kSlots * sizeof(uint64_t); }

int gbs_resident(const rq_hadamard* h, const RowArgs& a, GbsOut* out, uint64_t* exchange, uint32_t epoch, double eps, int max_evals,
                 bool wait, hipStream_t s) {
    ResidentArgs r{};
    r.out = out;
    r.exchange = exchange;
    r.epoch = epoch;
    r.eps = eps;
    r.max_evals = max_evals;
    r.wait_ticks = wait ? kWaitTicks : 0;
    return resident_launch<false>(h, a, r, s);
}

// (a workgroup has a row at least, and the workspace of a search 8 values a row or more: room for two sets of kSlots sums
// needs 16, which it has wherever the resident form applies)
int gbs_stepped(const rq_hadamard* h, const RowArgs& a, GbsDev* state, GbsOut* out, double* sums, double eps, int max_evals, int steps,
                hipStream_t s) {
    ResidentArgs r{};
    r.out = out;
    r.eps = eps;
    r.max_evals = max_evals;
    r.carry = state->carry;
    r.sums = sums;
    // a launch for every kAhead steps of the search, and one that takes the last decisions
    const int launches = (steps > 0 ? (steps + kAhead - 1) / kAhead : 1) + 1;
    int rc = RQ_OK;
    for (int i = 0; i < launches && rc == RQ_OK; ++i) {
        r.step = (uint32_t)i;
        rc = resident_launch<true>(h, a, r, s);
    }
    return rc;
}

size_t gbs_state_bytes() { return sizeof(GbsDev); }
GbsDev* gbs_state_at(GbsDev* base, int slot) { return base + slot; }

static __device__ GbsDev g_states[kSearchSlots];
static __device__ GbsOut g_outs[kSearchSlots];

SearchMemory search_memory(int dev) {
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static SearchMemory found[kMaxDevices];
    if (dev < 0 || dev >= kMaxDevices) return SearchMemory{};
    std::lock_guard<std::mutex> hold(lock);
    if (found[dev].state) return found[dev];
    int cur = -1;
    void *state = nullptr, *out = nullptr;
    if (hipGetDevice(&cur) == hipSuccess && cur == dev && hipGetSymbolAddress(&state, HIP_SYMBOL(g_states)) == hipSuccess &&
        hipGetSymbolAddress(&out, HIP_SYMBOL(g_outs)) == hipSuccess)
        found[dev] = SearchMemory{static_cast<GbsDev*>(state), static_cast<GbsOut*>(out)};
    (void)hipGetLastError();
    return found[dev];
}
const ClipList* gbs_state_clips(const GbsDev* state) { return &state->clips; }

void gbs_first_batch(double eps, int depth, int bits, ClipList* out) {
    const double levels = (double)((1 << bits) - 1);
    const GbsState st = gbs_start();
    out->n = 0;
    out->set(out->n++, (float)st.best, levels);
    double x;
    for (int i = 1; i < (1 << depth); ++i)
        if (gbs_node(st, eps, depth, i, &x)) out->set(out->n++, (float)x, levels);
}

int gbs_step(GbsDev* state, GbsOut* out, bool first, double eps, int depth, int max_evals, int bits, const double* partial,
             int64_t rows, int64_t count, int64_t stride, hipStream_t s) {
    launch_kernel(k_gbs_step, dim3(1), dim3(kStepThreads), 0, s, state, out, first ? 1 : 0, eps, depth, max_evals,
                  (double)((1 << bits) - 1), partial, rows, count, stride);
    return launch_rc();
}

}  // namespace rq
