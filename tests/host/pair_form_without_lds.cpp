// The workgroup block kernel on a device without the LDS of its pair form: compiled with the host side of the launches against
// stand-ins for the device runtime, which grant a kernel 160 KB and then 64 (for blocks of 148 and 160 the block kernel takes up to 60
// KB, its pair form 142 and 154).  A line each: order, whether the block kernel is usable, whether the pair form takes 4096 rows.
#include <cstdio>

#include "../../paper_2504_13989_amd/csrc/rotq_internal.h"

namespace {
size_t g_grants = 0, g_most = 0;
}

extern "C" {
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int value) {
    if ((size_t)value > g_most) return hipErrorInvalidValue;
    return ++g_grants, hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}

int main() {
    for (const size_t most : {(size_t)160 * 1024, (size_t)64 * 1024}) {
        g_most = most;
        for (const int n : {148 * 128, 160 * 128}) {
            rq_hadamard h;
            if (!rq::factor_order(n, &h.f)) return 1;
            h.device = 0;
            h.num_cu = 256;
            h.max_lds = (int)most;
            h.wg_ok = rq::wg_block_prepare(n / 128);
            rq::RowArgs a{};
            a.rows = 4096;
            a.n = a.d = n;
            a.ld = n;
            a.p = h.f.p;
            a.log2m = h.f.log2m;
            a.bits = 3;
            a.dtype = RQ_BF16;
            std::printf("%d %d %d\n", n, h.wg_ok ? 1 : 0, rq::wg_pair_pays(&h, a) ? 1 : 0);
        }
    }
    return g_grants ? 0 : 1;
}
