// Test infrastructure: workspace sizes and layer creation on the host.  The two
// device queries that they make are answered here (this program's definitions
// come before the HIP runtime's), so it runs without a GPU and launches
// nothing.  tests/test_workspace.py builds it against the library.
#include <stdint.h>
#include <stdio.h>

#include <initializer_list>

#include "../include/ffsl.h"

extern "C" int hipGetDevice(int *dev) {
    *dev = 0;
    return 0;
}
extern "C" int hipDeviceGetAttribute(int *value, int, int) {
    *value = 256;   // compute units
    return 0;
}

static int failures = 0;

static int create(int64_t L, int d, int k, int vt, int B, int nnz, size_t bytes, bool unfused) {
    void *p = (void *)(uintptr_t)(1u << 20);   // never dereferenced
    float *f = (float *)p;
    ffsl_layer *h = nullptr;
    const int rc = ffsl_create_layer_ex(&h, L, d, k, vt, FFSL_IDX_I32, p, p, f, f, f, f, f, unfused ? f : nullptr,
                                        unfused ? f : nullptr, p, bytes, B, nnz);
    if (h) ffsl_destroy_layer(h);
    return rc;
}

int main() {
    const int64_t Ls[] = {1, 4096, 30938, 131072, 262145, 1048576, 3145728};
    const struct {
        int d, k;
    } widths[] = {{32, 3},    {128, 16},  {128, 32},  {768, 32},  {768, 64},   {768, 128},  {832, 31},  {1151, 64},
                  {2048, 64}, {2303, 64}, {2304, 64}, {4607, 32}, {4608, 128}, {16384, 16}};
    const int Bs[] = {1, 16, 17, 32, 64, 65, 128, 1024};
    const int nnzs[] = {0, 100, 40000};
    for (int64_t L : Ls)
        for (auto &w : widths)
            for (int B : Bs)
                for (int nnz : nnzs) {
                    const size_t any = ffsl_workspace_bytes(L, w.d, w.k, B, nnz);
                    for (int vt : {(int)FFSL_F32, (int)FFSL_BF16})
                        for (bool unfused : {false, true}) {
                            const size_t typed = ffsl_workspace_bytes_ex(L, w.d, w.k, vt, B, nnz);
                            const bool ok = typed > 0 && create(L, w.d, w.k, vt, B, nnz, any, unfused) == FFSL_OK &&
                                            create(L, w.d, w.k, vt, B, nnz, typed, unfused) == FFSL_OK &&
                                            create(L, w.d, w.k, vt, B, nnz, typed - 1, unfused) == FFSL_EINVAL;
                            if (!ok) {
                                printf("FAIL L=%lld d=%d k=%d B=%d nnz=%d type=%d: %zu bytes without a type, %zu with it (%s)\n",
                                       (long long)L, w.d, w.k, B, nnz, vt, any, typed, ffsl_last_error());
                                ++failures;
                            }
                        }
                }
    printf("workspace driver: %d failures\n", failures);
    return failures == 0 ? 0 : 1;
}
