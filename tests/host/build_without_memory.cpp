// rq_hadamard_build with every host allocation failing in turn: compiled with rotq_api.cpp and hadamard.cpp against stand-ins
// for the device runtime and the kernels' table builders.  Each failure has to come back as RQ_ERR_NOMEM, with
// nothing thrown and no host or device memory left behind.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "../../paper_2504_13989_amd/csrc/rotq_internal.h"

namespace {
long g_until = -1;          // allocations until one fails; negative: never
long g_live = 0, g_device = 0;
void* allocate(size_t n) {
    if (g_until == 0) return nullptr;
    if (g_until > 0) --g_until;
    ++g_live;
    return std::malloc(n ? n : 1);
}
std::vector<uint32_t> table() { return std::vector<uint32_t>(100, 1u); }
}  // namespace

void* operator new(size_t n) {
    void* p = allocate(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return allocate(n); }
void operator delete(void* p) noexcept {
    if (p) --g_live;
    std::free(p);
}
void operator delete(void* p, size_t) noexcept { operator delete(p); }

// the device runtime
extern "C" {
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    p->sharedMemPerBlock = 160 * 1024;
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return ++g_device, *p = std::malloc(n), hipSuccess; }
hipError_t hipFree(void* p) { return --g_device, std::free(p), hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

// the kernels' side of a handle
namespace rq {
std::vector<uint32_t> wave_sylvester_tiles() { return table(); }
std::vector<uint32_t> tiles_to_f16(const std::vector<uint32_t>& t) { return t; }
std::vector<uint32_t> wave_block_tiles(const std::vector<int8_t>&, int) { return table(); }
std::vector<uint32_t> wave_block2_tiles(const std::vector<int8_t>&, int) { return table(); }
std::vector<uint32_t> wg_block_tiles(const std::vector<int8_t>&, int) { return table(); }
std::vector<uint32_t> dense_block_tiles(const std::vector<int8_t>&, int) { return table(); }
std::vector<uint32_t> f64_block_signs(const std::vector<int8_t>&, int) { return table(); }
bool wg_block_prepare(int) { return true; }
bool generic_prepare(rq_hadamard*) { return true; }
bool f64_prepare(const rq_hadamard*) { return true; }
void* static_scratch(int) { return nullptr; }
SearchMemory search_memory(int) { return SearchMemory{}; }
}  // namespace rq

int main() {
    int bad = 0;
    for (int n : {32, 40, 96, 128, 896, 1544, 3584, 4096, 4864, 7680, 18944, 32768}) {
        rq_hadamard_t* h = nullptr;
        long failures = 0;
        for (long k = 0;; ++k) {
            const long live = g_live, device = g_device;
            g_until = k;
            int rc;
            try {
                rc = rq_hadamard_build(n, &h);
            } catch (...) {
                rc = 1;
            }
            const bool ran_out = g_until == 0;
            g_until = -1;
            if (rc == RQ_OK) {
                rq_hadamard_free(h);
                if (!ran_out || g_live != live || g_device != device) break;
                continue;                                 // (the allocation after the last one would have failed)
            }
            ++failures;
            if (rc != RQ_ERR_NOMEM || g_live != live || g_device != device) {
                std::printf("n=%d allocation %ld: rc %d, %ld host and %ld device blocks left\n", n, k, rc, g_live - live,
                            g_device - device);
                ++bad;
                if (rc == 1) g_live = live, g_device = device;
            }
        }
        if (failures < 3) std::printf("n=%d: only %ld allocations\n", n, failures), ++bad;
    }
    std::printf("%s\n", bad ? "failed" : "ok");
    return bad != 0;
}
