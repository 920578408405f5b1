// Scratch of a context after a larger field, or created for one: calls on
// smaller fields allocate nothing (the stub runtime of hip_stub.cpp; device
// allocations are counted by wrapping hipMalloc at link time).  Exit status 0
// = no allocation.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../../include/fz.h"
#include "../../paper_2509_20563_amd/csrc/fz_kernels.h"

extern "C" int hipstub_errors();

static int g_mallocs = 0;
extern "C" hipError_t __real_hipMalloc(void** p, size_t n);
extern "C" hipError_t __wrap_hipMalloc(void** p, size_t n) {
    g_mallocs++;
    return __real_hipMalloc(p, n);
}

namespace fz {
// the launch's count of groups
uint32_t encode_groups(uint32_t ntiles) {
    const uint32_t T = encode_tiles(ntiles);
    return (ntiles + T - 1) / T;
}
}  // namespace fz

// One compression and decompression of n values; the allocations they made.
static int call(fz_ctx* c, uint64_t n, uint32_t pred) {
    fz_params p;
    memset(&p, 0, sizeof(p));
    p.ndim = 1;
    p.dims[0] = n;
    p.dims[1] = p.dims[2] = 1;
    p.eb_mode = FZ_EB_REL;
    p.eb = 1e-3;
    p.pred = pred;
    p.radius = 512;
    float* x = nullptr;
    uint8_t* out = nullptr;
    const uint64_t cap = fz_compress_bound(&p);
    __real_hipMalloc((void**)&x, 4 * n);
    __real_hipMalloc((void**)&out, cap);
    uint64_t bytes = 0;
    const int before = g_mallocs;
    int rc = fz_compress(c, &p, x, out, cap, &bytes, nullptr);
    if (rc == FZ_OK) rc = fz_decompress(c, out, bytes, out, x, n, nullptr);
    const int made = g_mallocs - before;
    hipFree(x);
    hipFree(out);
    if (rc != FZ_OK) {
        printf("call on %llu values: status %d\n", (unsigned long long)n, rc);
        return 1000;
    }
    return made;
}

int main() {
    int bad = 0;
    const uint64_t tile = 2048;
    // larger field, then smaller ones, in tiles of 2048 values
    const uint32_t seq[][4] = {{256, 255, 200, 1}, {300, 255, 256, 64}, {1000, 255, 130, 999},
                               {6144, 6143, 3500, 255}, {7000, 6143, 6144, 5000}};
    for (const auto& s : seq)
        for (int up_front = 0; up_front < 2; up_front++) {
            fz_ctx* c = nullptr;
            if (fz_ctx_create(&c, 0, up_front ? s[0] * tile : 0) != FZ_OK) return 2;
            if (!up_front) call(c, s[0] * tile, FZ_PRED_LORENZO1);
            for (int k = 1; k < 4; k++) {
                const int made = call(c, s[k] * tile - 7, FZ_PRED_LORENZO1);
                if (made) {
                    printf("%u tiles after %u%s: %d allocations\n", s[k], s[0], up_front ? " (max_elems)" : "", made);
                    bad++;
                }
            }
            fz_ctx_destroy(c);
        }
    for (uint32_t n = 1, most = 0; n < 50000; n++) {
        if (fz::encode_groups(n) > most) most = fz::encode_groups(n);
        if (fz::encode_descriptors(n) < most || fz::encode_descriptors(n) > n) bad++;
    }
    printf("%d calls allocated, %d stub errors\n", bad, hipstub_errors());
    return bad || hipstub_errors() ? 1 : 0;
}
