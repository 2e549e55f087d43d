// C ABI: argument validation, handle management and kernel dispatch.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "rotq_internal.h"
#include "search_rule.h"

namespace {

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

int check_rows(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d, int64_t ld,
               int bits) {
    if (!h) return RQ_ERR_ARG;
    if (dtype != RQ_BF16 && dtype != RQ_F32 && dtype != RQ_F16) return RQ_ERR_ARG;
    if (rows < 0 || d < 1 || d > h->f.n || ld < d) return RQ_ERR_ARG;
    if (bits != 3 && bits != 4) return RQ_ERR_ARG;
    // with no rows nothing is read or written through X / codes / scales: they may be NULL
    if (rows > 0 && (!X || !aligned(X, dtype == RQ_F32 ? 4 : 2))) return RQ_ERR_ARG;
    return RQ_OK;
}

bool clip_ok(float c) { return c > 0.0f && c <= 1.0f; }   // false for NaN

// variants that only searches know, see rq_hadamard_set_variant
constexpr int kSearchStepped = 5, kSearchNoWait = 6, kSearchUnpinned = 7;

// records which kernel family a call chose (diagnostic; the handle's only field written after build)
void note(const rq_hadamard_t* h, const char* name) { h->last_kernel.store(name, std::memory_order_relaxed); }

rq::RowArgs row_args(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d,
                     int64_t ld, int bits) {
    return rq::RowArgs{X, dtype, rows, d, ld, h->f.n, h->f.p, h->f.log2m, h->d_block, bits};
}

// The device tables of a handle, gathered on the host and uploaded together.
struct TableSet {
    struct Slot { void** where; size_t offset; };
    std::vector<uint32_t> words;
    std::vector<Slot> slots;
    void add(void** where, const std::vector<uint32_t>& t) {
        slots.push_back(Slot{where, words.size()});
        words.insert(words.end(), t.begin(), t.end());
        words.resize((words.size() + 63) / 64 * 64, 0u);             // 256-byte steps
    }
    void share(void** where, void** with) {
        for (const Slot& s : slots)
            if (s.where == with) {
                slots.push_back(Slot{where, s.offset});
                return;
            }
    }
    bool upload(void** pool) {
        const size_t bytes = words.size() * sizeof(uint32_t);
        if (hipMalloc(pool, bytes) != hipSuccess) return false;
        if (hipMemcpy(*pool, words.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipFree(*pool);
            return false;
        }
        for (const Slot& s : slots) *s.where = static_cast<uint32_t*>(*pool) + s.offset;
        return true;
    }
};

// What a search needs besides the caller's workspace: its state on the device, and its results in pinned host memory the
// device writes (`out`) or, where there is none, in device memory (`out` is null) from where they are copied.
struct SearchMem {
    int slot;                 // of the device's static memory; negative: `own` holds the state and the results
    rq::GbsDev* state;
    rq::GbsOut* out;
    rq::GbsOut* out_dev;
    void* own;
};

// Searches under way on a device.  The states and the results' device copies are static device arrays, as the scratch of
// rq_quant_error_noalloc is; the pinned memory (33 KB) and the resident form's exchange buffers (256 KB) are allocated by
// the first search on a device that wants them and, like the arrays, stay until the process ends: a handle built for one
// search pays for neither.  (Exchange buffers in a static array cost a search of 512 x 4096 rows 48.6 us instead of
// 45.5.)  Constant-initialised, so there is nothing to construct.
constexpr int kMaxDevices = 64;
struct SearchDevice {
    uint32_t used;            // slots in use, one bit each
    bool resident;            // a resident search is under way: one at a time, since two of them could each keep the
                              // other's workgroups from running (a second one takes the batched form)
    uint64_t* exchange;       // of the resident form: two buffers, taken in turn
    uint32_t epoch;           // first step number that is not in them
    int turn;                 // buffer of the next search
    int unclear;              // buffers to be cleared before use, one bit each
    rq::GbsOut *out, *out_dev;
};
static_assert(rq::kSearchSlots <= 32, "one bit each");
std::mutex g_search_lock;
SearchDevice g_search[kMaxDevices];

// Numbers a search takes for its steps, as many as the most steps of any search.  They have 16 bits.
constexpr uint32_t kSteps = 256, kStepNumbers = 1u << 16;

// The turn of the resident form on a device, where it is wanted and its buffers can be had.
class ResidentTurn {
    SearchDevice* mine_ = nullptr;
public:
    ResidentTurn(int device, bool wanted) {
        if (!wanted || device >= kMaxDevices) return;
        std::lock_guard<std::mutex> hold(g_search_lock);
        SearchDevice& d = g_search[device];
        if (d.resident) return;
        if (!d.exchange) {
            void* p = nullptr;
            int cur = -1;
            if (hipGetDevice(&cur) != hipSuccess || cur != device || hipMalloc(&p, 2 * rq::gbs_exchange_bytes()) != hipSuccess) {
                (void)hipGetLastError();
                return;
            }
            d.exchange = static_cast<uint64_t*>(p);
            d.epoch = 1;                                  // (0 is what a cleared buffer holds)
            d.unclear = 3;
        }
        mine_ = &d;
        mine_->resident = true;
    }
    ~ResidentTurn() {
        if (!mine_) return;
        std::lock_guard<std::mutex> hold(g_search_lock);
        mine_->resident = false;
    }
    ResidentTurn(const ResidentTurn&) = delete;
    ResidentTurn& operator=(const ResidentTurn&) = delete;
    explicit operator bool() const { return mine_; }
    SearchDevice* operator->() const { return mine_; }    // (only the turn's holder touches the exchange)
};

int take_search_mem(int device, bool pinned, SearchMem* m) {
    const rq::SearchMemory st = rq::search_memory(device);
    if (!st.state) return RQ_ERR_HIP;
    int slot = -1;
    rq::GbsOut *out = nullptr, *out_dev = nullptr;
    {
        std::lock_guard<std::mutex> hold(g_search_lock);
        SearchDevice& d = g_search[device];
        for (int i = 0; i < rq::kSearchSlots && slot < 0; ++i)
            if (!(d.used >> i & 1u)) slot = i;
        if (slot >= 0) d.used |= 1u << slot;
        if (slot >= 0 && pinned && !d.out) {
            void *host = nullptr, *dev = nullptr;
            if (hipHostMalloc(&host, rq::kSearchSlots * sizeof(rq::GbsOut), hipHostMallocMapped | hipHostMallocPortable) == hipSuccess &&
                hipHostGetDevicePointer(&dev, host, 0) == hipSuccess && dev) {
                d.out = static_cast<rq::GbsOut*>(host);
                d.out_dev = static_cast<rq::GbsOut*>(dev);
            } else {
                if (host) (void)hipHostFree(host);
                (void)hipGetLastError();
            }
        }
        if (pinned) out = d.out, out_dev = d.out_dev;
    }
    if (slot >= 0) {
        *m = SearchMem{slot, rq::gbs_state_at(st.state, slot), out ? out + slot : nullptr, out ? out_dev + slot : st.out + slot, nullptr};
        return RQ_OK;
    }
    void* own = nullptr;                                  // more searches at once than there are slots
    if (hipMalloc(&own, rq::gbs_state_bytes() + sizeof(rq::GbsOut)) != hipSuccess) {
        (void)hipGetLastError();
        return RQ_ERR_HIP;
    }
    *m = SearchMem{-1, static_cast<rq::GbsDev*>(own), nullptr,
                   reinterpret_cast<rq::GbsOut*>(static_cast<char*>(own) + rq::gbs_state_bytes()), own};
    return RQ_OK;
}

void give_search_mem(int device, const SearchMem& m) {
    if (m.own) (void)hipFree(m.own);
    if (m.slot < 0) return;
    std::lock_guard<std::mutex> hold(g_search_lock);
    g_search[device].used &= ~(1u << m.slot);
}
}  // namespace

extern "C" {

int rq_hadamard_build(int n, rq_hadamard_t** out) {
    if (!out || n < 32) return RQ_ERR_ARG;
    if (n % 8 != 0) return RQ_ERR_NO_ORDER;     // packed rows are whole bytes for 3 and 4 bits
    rq::Factorisation f;
    if (!rq::factor_order(n, &f)) return RQ_ERR_NO_ORDER;
    rq_hadamard* h = new (std::nothrow) rq_hadamard;
    if (!h) return RQ_ERR_NOMEM;
    h->f = f;
    try {
        h->block = rq::build_block(f);
    } catch (const std::bad_alloc&) {
        delete h;
        return RQ_ERR_NOMEM;
    }
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count == 0) {
        (void)hipGetLastError();
        *out = h;   // host-only handle
        return RQ_OK;
    }
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
        delete h;
        return RQ_ERR_HIP;
    }
    h->max_lds = (int)prop.sharedMemPerBlock;
    h->num_cu = prop.multiProcessorCount;
    // every table goes to the device in one allocation and one copy; a slot may share another's table
    TableSet tables;
    void* d_block = nullptr;
    const bool sylv = f.p == 1 && f.log2m >= 7 && f.log2m <= 13;
    // block orders of the block kernels; the Sylvester orders 2^14, 2^15 ride along with p = 1
    const bool blk = (f.p > 1 && f.log2m >= 7 && (f.p << (f.log2m - 7)) <= 256) ||
                     (f.p == 1 && (f.log2m == 14 || f.log2m == 15));
    const bool blk_short = f.p > 1 && (f.log2m == 5 || f.log2m == 6) && f.p <= 256;   // block rows of 32 / 64
    const bool dense = !sylv && !blk && !blk_short && n <= 4096;
    // tiles of a block in both 16-bit encodings, and those of its transpose (Paley I blocks are not symmetric)
    auto add_block = [&](const std::vector<int8_t>& bm, int pb, std::vector<uint32_t> (*make)(const std::vector<int8_t>&, int)) {
        const std::vector<uint32_t> tiles = make(bm, pb);
        tables.add(&h->d_tiles, tiles);
        tables.add(&h->d_tiles_f16, rq::tiles_to_f16(tiles));
        std::vector<int8_t> bt((size_t)pb * pb);
        for (int i = 0; i < pb; ++i)
            for (int j = 0; j < pb; ++j) bt[(size_t)i * pb + j] = bm[(size_t)j * pb + i];
        if (bt == bm) {
            tables.share(&h->d_tiles_t, &h->d_tiles);
            tables.share(&h->d_tiles_t_f16, &h->d_tiles_f16);
        } else {
            const std::vector<uint32_t> tt = make(bt, pb);
            tables.add(&h->d_tiles_t, tt);
            tables.add(&h->d_tiles_t_f16, rq::tiles_to_f16(tt));
        }
    };
    try {
        std::vector<uint32_t> block_words((h->block.size() + 3) / 4);
        std::memcpy(block_words.data(), h->block.data(), h->block.size());
        tables.add(&d_block, block_words);
        if (f.p > 1 && f.log2m >= 5 && f.p <= rq::kMaxPaleyOrder) tables.add(&h->d_signs, rq::f64_block_signs(h->block, f.p));
        if (sylv) {
            const std::vector<uint32_t> tiles = rq::wave_sylvester_tiles();
            tables.add(&h->d_tiles, tiles);
            tables.add(&h->d_tiles_f16, rq::tiles_to_f16(tiles));
        } else if (dense) {
            std::vector<int8_t> hm((size_t)n * n);
            if (rq_hadamard_dense(h, hm.data()) != RQ_OK) {
                delete h;
                return RQ_ERR_ARG;
            }
            tables.add(&h->d_tiles, rq::dense_block_tiles(hm, n));
            h->dense_ok = true;
        } else if (blk_short) {
            add_block(h->block, f.p, rq::wg_block_tiles);
            h->wg_ok = rq::wg_block_prepare(f.p);
        } else if (blk) {
            // block of the strided axis: H_p (x) H_{2^(k-7)}, index a * 2^(k-7) + (high bits of c)
            const int e = 1 << (f.log2m - 7), pb = f.p * e;
            std::vector<int8_t> bm((size_t)pb * pb);
            for (int i = 0; i < pb; ++i)
                for (int j = 0; j < pb; ++j)
                    bm[(size_t)i * pb + j] = (int8_t)(h->block[(size_t)(i / e) * f.p + j / e] *
                                                      rq::sylvester_entry(i % e, j % e));
            add_block(bm, pb, pb <= 32 ? rq::wave_block_tiles : rq::wg_block_tiles);
            if (pb > 32) h->wg_ok = rq::wg_block_prepare(pb);
            if (pb > 32 && pb <= 64) {
                // these blocks also have a one-wave kernel (rotate_quantize), with operand tiles of its own
                const std::vector<uint32_t> t2 = rq::wave_block2_tiles(bm, pb);
                tables.add(&h->d_tiles2, t2);
                tables.add(&h->d_tiles2_f16, rq::tiles_to_f16(t2));
            }
        }
    } catch (const std::bad_alloc&) {
        delete h;
        return RQ_ERR_NOMEM;
    }
    if (!tables.upload(&h->d_tables)) {
        delete h;
        return RQ_ERR_HIP;
    }
    h->d_block = static_cast<int8_t*>(d_block);
    h->device = dev;
    h->generic_ok = rq::generic_prepare(h);
    h->f64_ok = h->generic_f64_ok && rq::f64_prepare(h);
    // set-up time is when the addresses of the static arrays on this device are asked for; a failure only makes
    // rq_quant_error_noalloc or the searches return RQ_ERR_HIP
    (void)rq::static_scratch(dev);
    (void)rq::search_memory(dev);
    *out = h;
    return RQ_OK;
}

void rq_hadamard_free(rq_hadamard_t* h) {
    if (!h) return;
    if (h->d_tables) (void)hipFree(h->d_tables);
    delete h;
}

int rq_hadamard_info(const rq_hadamard_t* h, int* n, int* p, int* kind, int* q, int* log2m) {
    if (!h) return RQ_ERR_ARG;
    if (n) *n = h->f.n;
    if (p) *p = h->f.p;
    if (kind) *kind = h->f.kind;
    if (q) *q = h->f.q;
    if (log2m) *log2m = h->f.log2m;
    return RQ_OK;
}

int rq_hadamard_dense(const rq_hadamard_t* h, int8_t* host_out) {
    if (!h || !host_out || h->f.n > 8192) return RQ_ERR_ARG;
    const int n = h->f.n, p = h->f.p, m = 1 << h->f.log2m;
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j)
            host_out[(size_t)i * n + j] = (int8_t)(h->block[(size_t)(i / m) * p + (j / m)] *
                                                   rq::sylvester_entry(i % m, j % m));
    return RQ_OK;
}

int rq_next_order(int d, int* n_out) {
    if (d < 1 || !n_out) return RQ_ERR_ARG;
    for (int64_t n = ((int64_t)d + 31) / 32 * 32; n <= (1 << 30); n += 32) {
        rq::Factorisation f;
        if (rq::factor_order((int)n, &f) && f.log2m >= 5 && f.p <= rq::kMaxPaleyOrder) {
            *n_out = (int)n;
            return RQ_OK;
        }
    }
    return RQ_ERR_NO_ORDER;
}

int rq_hadamard_set_variant(rq_hadamard_t* h, int variant) {
    if (!h || variant < 0 || variant > 7) return RQ_ERR_ARG;
    h->variant = variant == 1 ? 1 : 0;
    h->search = variant > 4 ? variant : 0;
    h->split = variant == 2 ? -1 : variant == 3 ? 2 : variant == 4 ? 4 : 0;
    return RQ_OK;
}

const char* rq_hadamard_last_kernel(const rq_hadamard_t* h) {
    return h ? h->last_kernel.load(std::memory_order_relaxed) : "";
}

int rq_rotate_quantize(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d,
                       int64_t ld, int bits, float clip, void* codes, float* scales, void* stream) {
    int rc = check_rows(h, X, dtype, rows, d, ld, bits);
    if (rc != RQ_OK) return rc;
    if (!clip_ok(clip)) return RQ_ERR_ARG;
    if (rows == 0) return RQ_OK;
    if (!codes || !scales || !aligned(codes, 4) || !aligned(scales, 4)) return RQ_ERR_ARG;
    if (h->device < 0) return RQ_ERR_HIP;
    const rq::RowArgs a = row_args(h, X, dtype, rows, d, ld, bits);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (h->variant == 0 && rq::wave_supports(h, a)) {
        note(h, "wave_sylvester");
        return rq::wave_rotate_quantize(h, a, clip, static_cast<uint32_t*>(codes), scales, s);
    }
    if (h->variant == 0 && rq::wave_block_supports(h, a)) {
        note(h, "wave_block");
        return rq::wave_block_rotate_quantize(h, a, clip, static_cast<uint32_t*>(codes), scales, s);
    }
    if (h->variant == 0 && rq::wave_block2_supports(h, a)) {
        note(h, "wave_block");
        return rq::wave_block2_rotate_quantize(h, a, clip, static_cast<uint32_t*>(codes), scales, s);
    }
    if (h->variant == 0 && rq::wg_block_supports(h, a)) {
        if (rq::wg_pair_pays(h, a)) {
            note(h, "wg_block_pair");
            return rq::wg_pair_rotate_quantize(h, a, clip, static_cast<uint32_t*>(codes), scales, s);
        }
        note(h, "wg_block");
        return rq::wg_block_rotate_quantize(h, a, clip, static_cast<uint32_t*>(codes), scales, s);
    }
    if (h->variant == 0 && rq::dense_block_supports(h, a)) {
        note(h, "dense_block");
        return rq::dense_block_rotate_quantize(h, a, clip, static_cast<uint32_t*>(codes), scales, s);
    }
    if (h->variant == 0 && rq::f64_rows_supports(h, a)) {
        note(h, "f64_rows");
        return rq::f64_rotate_quantize(h, a, clip, static_cast<uint32_t*>(codes), scales, s);
    }
    if (!rq::generic_supports(h)) return RQ_ERR_NO_ORDER;
    note(h, "generic_lds");
    return rq::generic_rotate_quantize(h, a, clip, static_cast<uint32_t*>(codes), scales, s);
}

int rq_rotate_quantize_asym(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d,
                            int64_t ld, int bits, float clip, void* codes, float* scales,
                            float* mins, void* stream) {
    int rc = check_rows(h, X, dtype, rows, d, ld, bits);
    if (rc != RQ_OK) return rc;
    if (!clip_ok(clip) || h->f.n % RQ_GROUP != 0) return RQ_ERR_ARG;
    if (rows == 0) return RQ_OK;
    if (!codes || !scales || !mins || !aligned(codes, 4) || !aligned(scales, 4) || !aligned(mins, 4))
        return RQ_ERR_ARG;
    if (h->device < 0) return RQ_ERR_HIP;
    const rq::RowArgs a = row_args(h, X, dtype, rows, d, ld, bits);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (h->variant == 0 && rq::wave_asym_supports(h, a)) {
        note(h, "wave_short_asym");
        return rq::wave_rotate_quantize_asym(h, a, clip, static_cast<uint32_t*>(codes), scales, mins, s);
    }
    if (!rq::generic_supports(h)) return RQ_ERR_NO_ORDER;
    note(h, "generic_lds_asym");
    return rq::generic_rotate_quantize_asym(h, a, clip, static_cast<uint32_t*>(codes), scales, mins, s);
}

int rq_stream_reference(const void* X, int64_t rows, int n, int64_t ld, int bits, void* codes,
                        float* scales, void* stream) {
    if (rows < 0 || n < 512 || n > 8192 || n % 512 != 0 || ld < n || ld % 8 != 0 || (bits != 3 && bits != 4))
        return RQ_ERR_ARG;
    if (rows == 0) return RQ_OK;
    if (!X || !codes || !scales || !aligned(X, 16) || !aligned(codes, 4) || !aligned(scales, 4)) return RQ_ERR_ARG;
    return rq::stream_reference(X, rows, n, ld, bits, static_cast<uint32_t*>(codes), scales,
                                static_cast<hipStream_t>(stream));
}

int rq_quantize(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                void* codes, float* scales, void* stream) {
    if (dtype != RQ_BF16 && dtype != RQ_F32 && dtype != RQ_F16) return RQ_ERR_ARG;
    if (rows < 0 || d < 32 || d % 32 != 0 || ld < d) return RQ_ERR_ARG;
    if (bits != 3 && bits != 4) return RQ_ERR_ARG;
    if (!clip_ok(clip)) return RQ_ERR_ARG;
    if (rows == 0) return RQ_OK;
    if (!X || !aligned(X, dtype == RQ_F32 ? 4 : 2)) return RQ_ERR_ARG;
    if (!codes || !scales || !aligned(codes, 4) || !aligned(scales, 4)) return RQ_ERR_ARG;
    if (rq::plain_wave_short_supports(X, dtype, d, ld))     // head rows of 128 / 256 / 512: the short-row passes
        return rq::plain_wave_short_quantize(X, dtype, rows, d, ld, bits, clip, static_cast<uint32_t*>(codes), scales,
                                             static_cast<hipStream_t>(stream));
    if (rq::plain_short_supports(X, dtype, d, ld))          // other short rows: several rows per wave
        return rq::plain_short_quantize(X, dtype, rows, d, ld, bits, clip, static_cast<uint32_t*>(codes), scales,
                                        static_cast<hipStream_t>(stream));
    if (rq::plain_wave_supports(X, dtype, d, ld))
        return rq::plain_wave_quantize(X, dtype, rows, d, ld, bits, clip, static_cast<uint32_t*>(codes), scales,
                                       static_cast<hipStream_t>(stream));
    return rq::plain_quantize(X, dtype, rows, d, ld, bits, clip, static_cast<uint32_t*>(codes), scales,
                              static_cast<hipStream_t>(stream));
}

int rq_quantize_asym(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                     void* codes, float* scales, float* mins, void* stream) {
    if (dtype != RQ_BF16 && dtype != RQ_F32 && dtype != RQ_F16) return RQ_ERR_ARG;
    if (rows < 0 || d < RQ_GROUP || d % RQ_GROUP != 0 || ld < d) return RQ_ERR_ARG;
    if (bits != 3 && bits != 4) return RQ_ERR_ARG;
    if (!clip_ok(clip)) return RQ_ERR_ARG;
    if (rows == 0) return RQ_OK;
    if (!X || !aligned(X, dtype == RQ_F32 ? 4 : 2)) return RQ_ERR_ARG;
    if (!codes || !scales || !mins || !aligned(codes, 4) || !aligned(scales, 4) || !aligned(mins, 4)) return RQ_ERR_ARG;
    return rq::plain_quantize_asym(X, dtype, rows, d, ld, bits, clip, static_cast<uint32_t*>(codes), scales, mins,
                                   static_cast<hipStream_t>(stream));
}

int rq_rotate(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d, int64_t ld,
              int transpose, void* Y, int out_dtype, int d_out, int64_t ld_out, void* stream) {
    int rc = check_rows(h, X, dtype, rows, d, ld, 4);
    if (rc != RQ_OK) return rc;
    if (out_dtype != RQ_BF16 && out_dtype != RQ_F32 && out_dtype != RQ_F16) return RQ_ERR_ARG;
    if (d_out < 1 || d_out > h->f.n || ld_out < d_out || (transpose != 0 && transpose != 1))
        return RQ_ERR_ARG;
    if (rows == 0) return RQ_OK;
    if (!Y || !aligned(Y, out_dtype == RQ_F32 ? 4 : 2)) return RQ_ERR_ARG;
    if (h->device < 0) return RQ_ERR_HIP;
    const rq::RowArgs a = row_args(h, X, dtype, rows, d, ld, 4);
    const rq::OutArgs o{Y, out_dtype, d_out, ld_out};
    if (h->variant == 0 && rq::wave_rotate_supports(h, a, o)) {      // Sylvester orders: H is symmetric
        note(h, "wave_rotate");
        return rq::wave_rotate(h, a, o, static_cast<hipStream_t>(stream));
    }
    if (h->variant == 0 && rq::wave_block_rotate_supports(h, a, o)) {
        note(h, "wave_block_rotate");
        return rq::wave_block_rotate(h, a, transpose, o, static_cast<hipStream_t>(stream));
    }
    if (h->variant == 0 && rq::wg_rotate_supports(h, a, o)) {
        note(h, "wg_block_rotate");
        return rq::wg_rotate(h, a, transpose, o, static_cast<hipStream_t>(stream));
    }
    if (!rq::generic_supports(h)) return RQ_ERR_NO_ORDER;
    note(h, "generic_rotate");
    return rq::generic_rotate(h, a, transpose, o, static_cast<hipStream_t>(stream));
}

int rq_dequantize_rotate(const rq_hadamard_t* h, const void* codes, const float* scales,
                         const float* mins, int64_t rows, int bits, int transpose, void* Y,
                         int out_dtype, int d_out, int64_t ld_out, void* stream) {
    if (!h || rows < 0 || (bits != 3 && bits != 4)) return RQ_ERR_ARG;
    if (out_dtype != RQ_BF16 && out_dtype != RQ_F32 && out_dtype != RQ_F16) return RQ_ERR_ARG;
    if (d_out < 1 || d_out > h->f.n || ld_out < d_out || (transpose != 0 && transpose != 1))
        return RQ_ERR_ARG;
    if (mins && h->f.n % RQ_GROUP != 0) return RQ_ERR_ARG;
    if (rows == 0) return RQ_OK;
    if (!codes || !scales || !Y || !aligned(codes, 4) || !aligned(scales, 4) || !aligned(mins, 4) ||
        !aligned(Y, out_dtype == RQ_F32 ? 4 : 2))
        return RQ_ERR_ARG;
    if (h->device < 0) return RQ_ERR_HIP;
    const rq::RowArgs a = row_args(h, nullptr, RQ_F32, rows, h->f.n, h->f.n, bits);
    const rq::OutArgs o{Y, out_dtype, d_out, ld_out};
    if (h->variant == 0 && rq::wave_dequant_rotate_supports(h, a, mins, o)) {   // Sylvester orders: H is symmetric
        note(h, "wave_dequant_rotate");
        return rq::wave_dequant_rotate(h, a, static_cast<const uint32_t*>(codes), scales, mins, o,
                                       static_cast<hipStream_t>(stream));
    }
    if (h->variant == 0 && rq::wave_block_dequant_rotate_supports(h, a, mins, o)) {
        note(h, "wave_block_dequant_rotate");
        return rq::wave_block_dequant_rotate(h, a, static_cast<const uint32_t*>(codes), scales, transpose, o,
                                             static_cast<hipStream_t>(stream));
    }
    if (h->variant == 0 && rq::wg_dequant_rotate_supports(h, a, mins, o)) {
        note(h, "wg_block_dequant_rotate");
        return rq::wg_dequant_rotate(h, a, static_cast<const uint32_t*>(codes), scales, transpose, o,
                                     static_cast<hipStream_t>(stream));
    }
    if (!rq::generic_supports(h)) return RQ_ERR_NO_ORDER;
    note(h, "generic_dequant_rotate");
    return rq::generic_dequant_rotate(h, a, static_cast<const uint32_t*>(codes), scales, mins, transpose,
                                      o, static_cast<hipStream_t>(stream));
}

static int dequantize_impl(const rq_hadamard_t* h, const void* codes, const float* scales, const float* mins,
                           bool asym, int64_t rows, int bits, float* Y, void* stream) {
    if (!h || rows < 0 || (bits != 3 && bits != 4)) return RQ_ERR_ARG;
    if (asym && h->f.n % RQ_GROUP != 0) return RQ_ERR_ARG;
    if (rows == 0) return RQ_OK;
    if (!codes || !scales || !Y || (asym && !mins)) return RQ_ERR_ARG;
    if (!aligned(codes, 4) || !aligned(scales, 4) || !aligned(mins, 4) || !aligned(Y, 4)) return RQ_ERR_ARG;
    if (h->device < 0) return RQ_ERR_HIP;
    note(h, "dequantize");
    return rq::dequantize_rows(static_cast<const uint32_t*>(codes), scales, asym ? mins : nullptr, rows, h->f.n,
                               bits, Y, static_cast<hipStream_t>(stream));
}

int rq_dequantize(const rq_hadamard_t* h, const void* codes, const float* scales, int64_t rows, int bits,
                  float* Y, void* stream) {
    return dequantize_impl(h, codes, scales, nullptr, false, rows, bits, Y, stream);
}

int rq_dequantize_asym(const rq_hadamard_t* h, const void* codes, const float* scales, const float* mins,
                       int64_t rows, int bits, float* Y, void* stream) {
    return dequantize_impl(h, codes, scales, mins, true, rows, bits, Y, stream);
}

int rq_expand_limit(int n, int bits, int bits_reduced, int64_t* d_max) {
    if (!d_max || n < 1 || bits_reduced < 1 || bits_reduced > bits || bits > 64) return RQ_ERR_ARG;
    *d_max = ((int64_t)n * (bits - bits_reduced)) / bits_reduced;
    return RQ_OK;
}

size_t rq_quant_error_workspace(int64_t rows, int n_clips) {
    if (rows < 0 || n_clips < 1 || n_clips > RQ_MAX_CLIPS) return 0;
    size_t r = rows > 0 ? (size_t)rows : 1;
    return r * (size_t)n_clips * sizeof(double);
}

}  // extern "C"

// The pass over the rows of a quant_error evaluation: partial[rows][number of clips].
static int quant_error_rows(const rq_hadamard_t* h, const rq::RowArgs& a, const rq::ClipArg& cl, int max_clips, double* partial,
                            bool asym, hipStream_t s) {
    if (asym) {
        if (h->variant == 0 && a.rows > 0 && rq::wave_asym_supports(h, a)) {
            note(h, "wave_quant_error_asym");
            return rq::wave_quant_error_asym(h, a, cl, max_clips, partial, s);
        }
        if (!rq::generic_supports(h)) return RQ_ERR_NO_ORDER;
        note(h, "generic_lds_asym");
        return rq::generic_quant_error_asym(h, a, cl, partial, s);
    }
    if (h->variant == 0 && a.rows > 0 && rq::wave_quant_error_supports(h, a)) {
        note(h, "wave_quant_error");
        return rq::wave_quant_error(h, a, cl, max_clips, partial, s);
    }
    if (h->variant == 0 && a.rows > 0 && rq::wg_block_supports(h, a, true)) {
        note(h, "wg_block_quant_error");
        return rq::wg_block_quant_error(h, a, cl, max_clips, partial, s);
    }
    if (!rq::generic_supports(h)) return RQ_ERR_NO_ORDER;
    note(h, "generic_lds");
    return rq::generic_quant_error(h, a, cl, partial, s);
}

int rq::quant_error_impl(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d,
                         int64_t ld, int bits, const float* clips, int n_clips, float* mse,
                         void* workspace, size_t workspace_bytes, void* stream, bool asym) {
    int rc = check_rows(h, X, dtype, rows, d, ld, bits);
    if (rc != RQ_OK) return rc;
    if (asym && h->f.n % RQ_GROUP != 0) return RQ_ERR_ARG;
    if (!clips || n_clips < 1 || n_clips > RQ_MAX_CLIPS) return RQ_ERR_ARG;
    if (!mse || !aligned(mse, 4) || !workspace || !aligned(workspace, 8)) return RQ_ERR_ARG;
    if (workspace_bytes < rq_quant_error_workspace(rows, n_clips)) return RQ_ERR_ARG;
    rq::ClipArg cl;
    std::memset(&cl, 0, sizeof cl);
    cl.list.n = n_clips;
    for (int k = 0; k < n_clips; ++k) {
        if (!clip_ok(clips[k])) return RQ_ERR_ARG;
        cl.list.set(k, clips[k], (double)((1 << bits) - 1));
    }
    if (h->device < 0) return RQ_ERR_HIP;
    const rq::RowArgs a = row_args(h, X, dtype, rows, d, ld, bits);
    hipStream_t s = static_cast<hipStream_t>(stream);
    double* partial = static_cast<double*>(workspace);
    rc = quant_error_rows(h, a, cl, n_clips, partial, asym, s);
    if (rc != RQ_OK) return rc;
    return rq::reduce_partials(partial, rows, n_clips, mse, s);
}

extern "C" {

int rq_quant_error(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d,
                   int64_t ld, int bits, const float* clips, int n_clips, float* mse,
                   void* workspace, size_t workspace_bytes, void* stream) {
    return rq::quant_error_impl(h, X, dtype, rows, d, ld, bits, clips, n_clips, mse, workspace, workspace_bytes,
                            stream, false);
}

int rq_quant_error_asym(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d,
                        int64_t ld, int bits, const float* clips, int n_clips, float* mse,
                        void* workspace, size_t workspace_bytes, void* stream) {
    return rq::quant_error_impl(h, X, dtype, rows, d, ld, bits, clips, n_clips, mse, workspace, workspace_bytes,
                                stream, true);
}

size_t rq_gbs_workspace(int64_t rows) {
    if (rows < 0) return 0;
    // the order is not known here: with the smallest one (32) more than 2^22 / 32 rows always take 3 steps
    const int cands = rows * 32 <= rq::kGbsSmall ? 32 : 8;
    const size_t q = rq_quant_error_workspace(rows, cands);
    return q ? q + 256 : 0;
}

static int gbs_impl(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d, int64_t ld,
                    int bits, float eps, int max_evals, void* workspace, size_t workspace_bytes,
                    void* stream, float* clip_out, float* mse_out, float* trace_clips,
                    float* trace_mse, int* n_evals, bool asym) {
    int rc = check_rows(h, X, dtype, rows, d, ld, bits);
    if (rc != RQ_OK) return rc;
    if (asym && h->f.n % RQ_GROUP != 0) return RQ_ERR_ARG;
    if (rows < 1 || !(eps > 0.0f) || max_evals < 1 || max_evals > 256) return RQ_ERR_ARG;
    if (!clip_out || !mse_out || !workspace || !aligned(workspace, 8)) return RQ_ERR_ARG;
    if (workspace_bytes < rq_gbs_workspace(rows)) return RQ_ERR_ARG;
    if (h->device < 0) return RQ_ERR_HIP;
    double* partial = static_cast<double*>(workspace);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const rq::RowArgs a = row_args(h, X, dtype, rows, d, ld, bits);
    SearchMem mem;
    rc = take_search_mem(h->device, h->search != kSearchUnpinned, &mem);
    if (rc != RQ_OK) return rc;
    auto finish = [&](int code, const rq::GbsOut* o) {
        if (code == RQ_OK) {
            *clip_out = o->clip;
            *mse_out = o->mse;
            if (trace_clips) std::memcpy(trace_clips, o->trace_clips, sizeof(float) * (size_t)o->evals);
            if (trace_mse) std::memcpy(trace_mse, o->trace_mse, sizeof(float) * (size_t)o->evals);
            if (n_evals) *n_evals = o->evals;
        }
        give_search_mem(h->device, mem);
        return code;
    };
    if (mem.out) mem.out->done = 0;
    const volatile int* done = mem.out ? &mem.out->done : nullptr;
    const int steps = rq::gbs_most_steps((double)eps, max_evals - 1);
    const bool in_registers = !asym && h->variant == 0 && rq::gbs_resident_supports(h, a);
    // after the last launch: the results, copied back where they are in device memory
    auto collect = [&](int code) {
        rq::GbsOut copied;
        const rq::GbsOut* result = mem.out;
        if (code == RQ_OK && !mem.out) {
            result = &copied;
            if (hipMemcpyAsync(&copied, mem.out_dev, sizeof copied, hipMemcpyDeviceToHost, s) != hipSuccess) code = RQ_ERR_HIP;
        }
        if (hipStreamSynchronize(s) != hipSuccess && code == RQ_OK) code = RQ_ERR_HIP;
        return finish(code == RQ_OK && !result->done ? RQ_ERR_HIP : code, result);
    };
    // The result arrives in host memory before the runtime reports the stream done: worth about 5 us to look there.
    auto watch = [&] {
        const auto began = std::chrono::steady_clock::now();
        for (int spin = 1; !*done; ++spin) {
            __builtin_ia32_pause();
            if (spin % 256 == 0 && std::chrono::steady_clock::now() - began > std::chrono::microseconds(500)) break;
        }
        if (!*done && hipStreamSynchronize(s) != hipSuccess) return false;
        std::atomic_thread_fence(std::memory_order_acquire);
        return true;
    };
    const int form = h->search;
    // (a variant that names one of the forms below takes it)
    const bool named = in_registers && (form == kSearchStepped || form == kSearchNoWait);
    if (!asym && h->variant == 0 && !named && rq::gbs_grid_supports(h, a, (double)eps, steps)) {
        rc = rq::gbs_grid(h, a, mem.state, mem.out_dev, (double)eps, max_evals, s);
        if (rc != RQ_ERR_NO_ORDER) {                         // (nothing launched: the forms below need less LDS)
            note(h, "grid_search");
            if (rc == RQ_OK && done && !watch()) rc = RQ_ERR_HIP;
            if (rc == RQ_OK && done && *done) return finish(RQ_OK, mem.out);
            return collect(rc);
        }
        rc = RQ_OK;
    }
    // (without pinned memory there is no result to look for while the stream is busy: the stepped form)
    if (const ResidentTurn turn{h->device, in_registers && mem.out && form != kSearchStepped}) {
        if (turn->epoch + kSteps > kStepNumbers) {           // the numbers start again
            turn->epoch = 1;
            turn->unclear = 3;
        }
        // Searches take the buffers in turn: the host goes on when the result has arrived, and a workgroup of this
        // search may then still be reading the last step's words.  A buffer is cleared when its own turn has come, and counts
        // as cleared once a search has come through on it (on a stream under capture nothing has run).
        const int b = turn->turn;
        uint64_t* const buf = turn->exchange + b * (rq::gbs_exchange_bytes() / sizeof(uint64_t));
        if ((turn->unclear >> b & 1) && hipMemsetAsync(buf, 0, rq::gbs_exchange_bytes(), s) != hipSuccess)
            return finish(RQ_ERR_HIP, nullptr);
        rc = rq::gbs_resident(h, a, mem.out_dev, buf, turn->epoch, (double)eps, max_evals, form != kSearchNoWait, s);
        turn->epoch += kSteps;
        turn->turn ^= 1;
        if (rc != RQ_OK) return finish(rc, nullptr);
        if (!watch()) return finish(RQ_ERR_HIP, nullptr);
        if (*done) {
            turn->unclear &= ~(1 << b);
            note(h, "gbs_resident");
            return finish(RQ_OK, mem.out);
        }
        // other work kept part of the search from running: the stepped form needs no two workgroups at one time
    }
    if (in_registers) {
        note(h, "gbs_stepped");
        return collect(rq::gbs_stepped(h, a, mem.state, mem.out_dev, partial, (double)eps, max_evals, steps, s));
    }
    const auto [batches, depth] = rq::gbs_batches(rows, h->f.n, steps);
    const int most = 1 << depth;                             // clip ratios of a batch
    rq::ClipArg cl;
    std::memset(&cl, 0, sizeof cl);
    rq::gbs_first_batch((double)eps, depth, bits, &cl.list);
    for (int b = 0; b < batches && rc == RQ_OK && !(done && *done); ++b) {
        const bool first = b == 0;
        if (!first) cl.dev = rq::gbs_state_clips(mem.state);
        int64_t count = 0, stride = 0;
        rc = quant_error_rows(h, a, cl, most, partial, asym, s);
        if (rc == RQ_OK) rc = rq::reduce_chunks(partial, rows, first ? cl.list.n : most, cl.dev, &count, &stride, s);
        if (rc == RQ_OK)
            rc = rq::gbs_step(mem.state, mem.out_dev, first, (double)eps, depth, max_evals, bits, partial, rows, count, stride, s);
    }
    return collect(rc);
}

int rq_gbs_search(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d, int64_t ld,
                  int bits, float eps, int max_evals, void* workspace, size_t workspace_bytes,
                  void* stream, float* clip_out, float* mse_out, float* trace_clips,
                  float* trace_mse, int* n_evals) {
    return gbs_impl(h, X, dtype, rows, d, ld, bits, eps, max_evals, workspace, workspace_bytes, stream,
                    clip_out, mse_out, trace_clips, trace_mse, n_evals, false);
}

int rq_gbs_search_asym(const rq_hadamard_t* h, const void* X, int dtype, int64_t rows, int d, int64_t ld,
                       int bits, float eps, int max_evals, void* workspace, size_t workspace_bytes,
                       void* stream, float* clip_out, float* mse_out, float* trace_clips,
                       float* trace_mse, int* n_evals) {
    return gbs_impl(h, X, dtype, rows, d, ld, bits, eps, max_evals, workspace, workspace_bytes, stream,
                    clip_out, mse_out, trace_clips, trace_mse, n_evals, true);
}

const char* rq_strerror(int code) {
    switch (code) {
        case RQ_OK: return "ok";
        case RQ_ERR_ARG: return "invalid argument";
        case RQ_ERR_NO_ORDER: return "no supported Hadamard order";
        case RQ_ERR_HIP: return "HIP failure or handle without device tables";
        case RQ_ERR_NOMEM: return "out of host memory";
        case RQ_ERR_TOO_LARGE: return "input larger than the static scratch buffer of the no-allocation call";
        default: return "unknown error";
    }
}

}  // extern "C"
