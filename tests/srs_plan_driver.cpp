// Host-only (igemm_plan.cpp, no HIP): the kernel that the automatic plan of one
// block of the int16-output update takes. Arguments: element bytes, m, n, k,
// lda, ldb. Prints "<kernel> <vec_a> <workgroups>".
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include "igemm_internal.h"
using namespace igemm;
int main(int argc, char **argv) {
    if (argc != 7) return 2;
    int64_t v[6];
    for (int i = 0; i < 6; ++i) v[i] = std::atoll(argv[i + 1]);
    const void *p = (const void *)(uintptr_t)0x10000;
    igemm_plan plan;
    if (make_srs_plan((int)v[0], v[1], v[2], v[3], p, v[4], p, v[5], v[2], 256, -1, &plan) !=
        IGEMM_OK)
        return 1;
    std::printf("%s %d %lld\n", kKernels[plan.kernel].name, plan.vec_a, (long long)plan.grid);
    return 0;
}
