// Internal declarations shared by the C ABI layer and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <tuple>
#include <utility>
#include <vector>

#include "../../include/rotq.h"
#include "hadamard.h"

struct rq_hadamard {
    rq::Factorisation f;
    std::vector<int8_t> block;       // host copy of H_p, row-major p x p
    int device = -1;                 // device the tables live on; -1 = host-only handle
    void* d_tables = nullptr;        // the one device allocation all tables below lie in
    int8_t* d_block = nullptr;       // device copy of `block`
    void* d_tiles = nullptr;         // device MFMA operand tiles of the block stage (bf16)
    void* d_tiles_f16 = nullptr;     // the same tiles encoded in fp16 (not the dense-block kernel's)
    void* d_tiles_t = nullptr;       // operand tiles of the transposed block (rotations with transpose = 1), bf16
    void* d_tiles_t_f16 = nullptr;   // and fp16; those of the block itself where it is symmetric
    void* d_signs = nullptr;         // sign masks of the block for the fp64 kernel of fp32 rows
    void* d_tiles2 = nullptr;        // blocks of 33 .. 64: operand tiles of the one-wave kernel (d_tiles holds the
    void* d_tiles2_f16 = nullptr;    // workgroup kernel's), bf16 and fp16
    int max_lds = 0;                 // bytes of LDS one workgroup may use on `device`
    int num_cu = 0;
    bool wg_ok = false;              // the workgroup block kernel is usable for this order
    bool dense_ok = false;           // d_tiles holds the whole matrix for the dense-block kernel
    bool generic_ok = false;         // the general LDS kernel can hold a row of this order
    bool generic_f64_ok = false;     // ... and an fp64 copy of it (how fp32 rows are quantized)
    bool f64_ok = false;             // fp32 rows of this order have the fp64 kernel of their own
    // test / measurement hook (rq_hadamard_set_variant); atomic so that a hot-path call on another
    // thread reads a whole value
    std::atomic<int> variant{0};     // 0 auto, 1 general LDS kernel
    std::atomic<int> split{0};       // long Sylvester rows: 0 auto, 2 / 4 waves per row, -1 never split
    std::atomic<int> search{0};      // variants of the searches only: 0 auto, 5 .. 7 see rq_hadamard_set_variant
    // diagnostic only: name of the kernel family the most recent hot-path call chose.  The hot-path
    // calls take the handle as const and may run on several host threads at once, hence atomic.
    mutable std::atomic<const char*> last_kernel{""};
};

namespace rq {

// Launch of a kernel: the runtime call itself, without the round trip of the launch syntax through the runtime's
// configuration stack (3.4 -> 3.2 us of host time per launch).  Launchers end with launch_rc().
inline thread_local bool launch_failed = false;              // a launch of this thread has, since launch_rc() was last asked
template <typename... P, typename... A>
inline void launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t s, A&&... args) {
    std::tuple<P...> values{static_cast<P>(std::forward<A>(args))...};
    std::apply([&](auto&... v) {
        void* ptrs[] = {static_cast<void*>(&v)...};
        if (hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, s) != hipSuccess) launch_failed = true;
    }, values);
}
// (asking the runtime for its last error would cost every call 0.04 us)
inline int launch_rc() {
    if (!launch_failed) return RQ_OK;
    launch_failed = false;
    (void)hipGetLastError();                                  // reported here, not left for others to find
    return RQ_ERR_HIP;
}

// Leave for a kernel to take that much dynamic LDS; false where the device has none for it.
template <typename... P>
inline bool allow_lds(void (*kernel)(P...), size_t lds) {
    if (lds <= 48 * 1024 || hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                (int)lds) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Grid of `groups` workgroups (fewer than 2^35) of a kernel that takes one item each, numbered by group_index()
// (wave_common.h): a dimension holds fewer than 2^32 threads (beyond that the launch keeps the remainder, without
// an error).
inline dim3 group_grid(int64_t groups, int threads) {
    const int64_t most = ((int64_t)1 << 31) / threads;
    return groups <= most ? dim3((unsigned)groups) : dim3((unsigned)most, (unsigned)((groups + most - 1) / most));
}

struct RowArgs {
    const void* X;
    int dtype;
    int64_t rows;
    int d;
    int64_t ld;
    int n, p, log2m;
    const int8_t* block;
    int bits;
};

struct OutArgs {
    void* Y;          // rows x d_out results, fp32, bf16 or fp16
    int dtype;
    int d_out;
    int64_t ld_out;
};

struct ClipList {
    float v[RQ_MAX_CLIPS];
    // row-independent factors of the candidate scales, formed once in fp64: levels / clip and clip / levels,
    // levels = 2^b - 1
    double lvl_over_clip[RQ_MAX_CLIPS];
    double clip_over_lvl[RQ_MAX_CLIPS];
    int n;
    __host__ __device__ void set(int k, float clip, double levels) {
        v[k] = clip;
        lvl_over_clip[k] = levels / (double)clip;
        clip_over_lvl[k] = (double)clip / levels;
    }
};
// The clip ratios of a launch: those handed over with it, or a list in device memory that an earlier kernel on the
// stream wrote (the search, whose next ratios depend on values only the device has seen).
struct ClipArg {
    ClipList list;
    const ClipList* dev;
};

// General LDS kernels: one workgroup per row, any supported order that fits in LDS.
// Return RQ_OK / RQ_ERR_*.
int generic_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                            float* scales, hipStream_t s);
// quant_error: the row kernels fill partial[rows][number of clips]; `max_clips` bounds that number for the launch
// where only the device knows it.  reduce_partials then averages over rows.
int generic_quant_error(const rq_hadamard* h, const RowArgs& a, const ClipArg& clips, double* partial, hipStream_t s);
int generic_rotate_quantize_asym(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                                 float* scales, float* mins, hipStream_t s);
// Rotation with a floating-point result (H_n or H_n^T), from rows or from packed codes.
int generic_rotate(const rq_hadamard* h, const RowArgs& a, int transpose, const OutArgs& o,
                   hipStream_t s);
int generic_dequant_rotate(const rq_hadamard* h, const RowArgs& a, const uint32_t* codes,
                           const float* scales, const float* mins, int transpose, const OutArgs& o,
                           hipStream_t s);
// Rotation-free per-token quantizer (any d that is a multiple of 32).
int plain_quantize(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                   uint32_t* codes, float* scales, hipStream_t s);
// The same on the wave path: bf16 / fp16 rows up to 20480 wide, 16-byte aligned.
bool plain_wave_supports(const void* X, int dtype, int d, int64_t ld);
int plain_wave_quantize(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                        uint32_t* codes, float* scales, hipStream_t s);
// The same on head rows of 128 / 256 / 512 16-bit values: the short-row passes of the rotating kernels with the
// identity on the matrix cores.
bool plain_wave_short_supports(const void* X, int dtype, int d, int64_t ld);
int plain_wave_short_quantize(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                              uint32_t* codes, float* scales, hipStream_t s);
bool generic_supports(const rq_hadamard* h);
bool generic_prepare(rq_hadamard* h);

// Wave-per-row kernels (bf16 / fp16 rows, Sylvester orders 128 .. 8192, 16-byte aligned rows).
std::vector<uint32_t> wave_sylvester_tiles();
// The +-1 entries of a bf16 operand table re-encoded as IEEE fp16.
std::vector<uint32_t> tiles_to_f16(const std::vector<uint32_t>& bf16_tiles);
bool wave_supports(const rq_hadamard* h, const RowArgs& a);
int wave_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                         float* scales, hipStream_t s);
// Asymmetric group-128 variant on the wave path: bf16 / fp16 rows of order 128 (one group per row).
bool wave_asym_supports(const rq_hadamard* h, const RowArgs& a);
int wave_rotate_quantize_asym(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                              float* scales, float* mins, hipStream_t s);
bool wave_quant_error_supports(const rq_hadamard* h, const RowArgs& a);
int wave_quant_error(const rq_hadamard* h, const RowArgs& a, const ClipArg& clips, int max_clips,
                     double* partial, hipStream_t s);
int wave_quant_error_asym(const rq_hadamard* h, const RowArgs& a, const ClipArg& clips, int max_clips, double* partial,
                          hipStream_t s);
int generic_quant_error_asym(const rq_hadamard* h, const RowArgs& a, const ClipArg& clips, double* partial, hipStream_t s);
int reduce_partials(double* partial, int64_t rows, int n_clips, float* mse, hipStream_t s);
// First level of that reduction for many rows: sums over chunks of rows, each left in the chunk's own first row of
// `partial`.  Returns the number of sums per clip ratio and their distance in rows; RQ_OK or an error.
int reduce_chunks(double* partial, int64_t rows, int n_clips, const ClipList* dev, int64_t* count, int64_t* stride, hipStream_t s);
// Block kernel: bf16 / fp16 rows, n = pb * 128 with a +-1 block of order pb <= 32 (Paley (x) small
// Sylvester) on the matrix cores.
std::vector<uint32_t> wave_block_tiles(const std::vector<int8_t>& bm, int pb);
bool wave_block_supports(const rq_hadamard* h, const RowArgs& a);
int wave_block_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                               float* scales, hipStream_t s);

// Rotation alone for those orders (H_n, or H_n^T with the transposed block's tiles).
bool wave_block_rotate_supports(const rq_hadamard* h, const RowArgs& a, const OutArgs& o);
int wave_block_rotate(const rq_hadamard* h, const RowArgs& a, int transpose, const OutArgs& o, hipStream_t s);
// Packed per-token codes back to rows for those orders.
bool wave_block_dequant_rotate_supports(const rq_hadamard* h, const RowArgs& a, const float* mins, const OutArgs& o);
int wave_block_dequant_rotate(const rq_hadamard* h, const RowArgs& a, const uint32_t* codes, const float* scales, int transpose,
                              const OutArgs& o, hipStream_t s);

// One-wave block kernel for blocks of 33 .. 64 (n <= 8192): bf16 / fp16 rows, 16-byte aligned.
std::vector<uint32_t> wave_block2_tiles(const std::vector<int8_t>& bm, int pb);
bool wave_block2_supports(const rq_hadamard* h, const RowArgs& a);
int wave_block2_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                                float* scales, hipStream_t s);

// Rotation-free asymmetric group-128 quantizer: any input type; 16-byte loads when the rows allow.
bool plain_short_supports(const void* X, int dtype, int d, int64_t ld);
int plain_short_quantize(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                         uint32_t* codes, float* scales, hipStream_t s);
int plain_quantize_asym(const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits, float clip,
                        uint32_t* codes, float* scales, float* mins, hipStream_t s);

// Rotation alone on the wave path: 16-bit rows of Sylvester order 128 .. 8192, 16-byte aligned rows in and out.
bool wave_rotate_supports(const rq_hadamard* h, const RowArgs& a, const OutArgs& o);
int wave_rotate(const rq_hadamard* h, const RowArgs& a, const OutArgs& o, hipStream_t s);
// Packed codes (+ scales, + mins when a row is one group of 128) to rows in the original basis on the
// wave path: Sylvester orders 128 .. 8192.
bool wave_dequant_rotate_supports(const rq_hadamard* h, const RowArgs& a, const float* mins, const OutArgs& o);
int wave_dequant_rotate(const rq_hadamard* h, const RowArgs& a, const uint32_t* codes, const float* scales,
                        const float* mins, const OutArgs& o, hipStream_t s);

// Dense-block kernel: bf16 / fp16 rows, any order n <= 4096 that the wave kernels do not serve (the whole
// matrix on the matrix cores), e.g. 1544 as one Paley block.
std::vector<uint32_t> dense_block_tiles(const std::vector<int8_t>& hm, int n);
bool dense_block_supports(const rq_hadamard* h, const RowArgs& a);
int dense_block_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                                float* scales, hipStream_t s);

// fp32 rows, quantized in fp64: orders p * 2^k with 2^k >= 32.
std::vector<uint32_t> f64_block_signs(const std::vector<int8_t>& block, int p);
bool f64_prepare(const rq_hadamard* h);
bool f64_rows_supports(const rq_hadamard* h, const RowArgs& a);
int f64_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes, float* scales, hipStream_t s);

// Workgroup block kernel: bf16 or fp16 rows, n = pb * 128 with 32 < pb <= 256 (e.g. 18944 = 148 * 128),
// or n = p * 64 / p * 32 with 4 <= p <= 256 (several rows per pass).
std::vector<uint32_t> wg_block_tiles(const std::vector<int8_t>& bm, int pb);
bool wg_block_prepare(int pb);
// Shape of a launch of that kernel: block order and lane bits of the column transform; false when it does not serve the order.
bool wg_shape(const RowArgs& a, int* pb, int* cb);
// Its form for many rows whose block splits into pairs of rows (wg_pair_kernel.h): rq_rotate_quantize only.
// Its operand tiles lie behind the others' (at wg_pair_tiles_at, in units of 16 bytes) where the block is large enough.
std::vector<uint32_t> wg_pair_tiles(const std::vector<int8_t>& bm, int pb);
size_t wg_pair_tiles_at(int pb);
void wg_pair_prepare(int pb);
bool wg_pair_pays(const rq_hadamard* h, const RowArgs& a);   // (of a call that wg_block_supports)
int wg_pair_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes, float* scales, hipStream_t s);
// Rotation alone on it, from rows or from packed per-token codes; with transpose the transposed block's tiles.
bool wg_rotate_prepare(int pb);
bool wg_rotate_supports(const rq_hadamard* h, const RowArgs& a, const OutArgs& o);
int wg_rotate(const rq_hadamard* h, const RowArgs& a, int transpose, const OutArgs& o, hipStream_t s);
bool wg_dequant_rotate_supports(const rq_hadamard* h, const RowArgs& a, const float* mins, const OutArgs& o);
int wg_dequant_rotate(const rq_hadamard* h, const RowArgs& a, const uint32_t* codes, const float* scales, int transpose,
                      const OutArgs& o, hipStream_t s);
bool wg_block_supports(const rq_hadamard* h, const RowArgs& a, bool quant_error = false);
int wg_block_rotate_quantize(const rq_hadamard* h, const RowArgs& a, float clip, uint32_t* codes,
                             float* scales, hipStream_t s);
int wg_block_quant_error(const rq_hadamard* h, const RowArgs& a, const ClipArg& clips, int max_clips, double* partial,
                         hipStream_t s);

// One step of the clip search on the device (kernels_search.hip): the batch of objective values in `partial` is
// averaged, the search walks on with them and leaves its next batch of clip ratios in *state.
struct GbsDev;
struct GbsOut {               // host memory the device writes (pinned, mapped)
    float clip, mse;          // the best point and its objective
    int evals;
    int done;                 // set last
    float trace_clips[256], trace_mse[256];
};
size_t gbs_state_bytes();
GbsDev* gbs_state_at(GbsDev* base, int slot);
// The static device memory of the searches on device `dev` (null pointers when it cannot be resolved; as
// static_scratch, to be asked for first with that device current): kSearchSlots states and results.
constexpr int kSearchSlots = 16;
struct SearchMemory {
    GbsDev* state;
    GbsOut* out;
};
SearchMemory search_memory(int dev);
const ClipList* gbs_state_clips(const GbsDev* state);
// The first batch of a search, `depth` steps ahead: the starting point and every probe those steps can ask for.
void gbs_first_batch(double eps, int depth, int bits, ClipList* out);
// Waves that hold a row in their registers, 0 where none do.
int gbs_row_waves(const rq_hadamard* h, const RowArgs& a);
// The whole search in one launch, for tensors whose rows the chip holds that way all at once; false where it does not.  (`wait`
// false: a workgroup that finds another's sums missing gives the search up at once, for tests.)
bool gbs_resident_supports(const rq_hadamard* h, const RowArgs& a);
size_t gbs_exchange_bytes();
int gbs_resident(const rq_hadamard* h, const RowArgs& a, GbsOut* out, uint64_t* exchange, uint32_t epoch, double eps, int max_evals,
                 bool wait, hipStream_t s);
// The same steps, a launch each, for searches of up to `steps` steps after the starting point; `sums` is the workspace.
int gbs_stepped(const rq_hadamard* h, const RowArgs& a, GbsDev* state, GbsOut* out, double* sums, double eps, int max_evals, int steps,
                hipStream_t s);
// The grid form: those rows or the workgroup block kernel's, brackets down to 1 / 256, where it is the faster one for a search
// of up to `steps` steps; rows of the latter.
bool gbs_grid_supports(const rq_hadamard* h, const RowArgs& a, double eps, int steps);
int gbs_grid(const rq_hadamard* h, const RowArgs& a, GbsDev* dev, GbsOut* out, double eps, int max_evals, hipStream_t s);
// (RQ_ERR_NO_ORDER with nothing launched: the kernels' LDS cannot be had)
int wg_grid_rows(const rq_hadamard* h, const RowArgs& a, GbsDev* dev, int* groups, hipStream_t s);
size_t wg_grid_ops_bytes(int pb);                            // LDS of the operand buffer of a block of that order
int gbs_step(GbsDev* state, GbsOut* out, bool first, double eps, int depth, int max_evals, int bits, const double* partial,
             int64_t rows, int64_t count, int64_t stride, hipStream_t s);

// The shared body of rq_quant_error / rq_quant_error_asym (argument checks, dispatch, reduction).
int quant_error_impl(const rq_hadamard* h, const void* X, int dtype, int64_t rows, int d, int64_t ld, int bits,
                     const float* clips, int n_clips, float* mse, void* workspace, size_t workspace_bytes,
                     void* stream, bool asym);

// Device address of the library's static scratch array on device `dev`; the first call for a device must
// be made with that device current (rq_hadamard_build does so).  nullptr when it cannot be resolved.
void* static_scratch(int dev);

// Codes (+ scales, + mins) to values in the rotated domain, no rotation.
int dequantize_rows(const uint32_t* codes, const float* scales, const float* mins, int64_t rows, int n, int bits,
                    float* Y, hipStream_t s);

// Traffic-only reference kernel (measurement aid): rows of n = 512 T 16-bit values.
int stream_reference(const void* X, int64_t rows, int n, int64_t ld, int bits, uint32_t* codes, float* scales,
                     hipStream_t s);

}  // namespace rq
