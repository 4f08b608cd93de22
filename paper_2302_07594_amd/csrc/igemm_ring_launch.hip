// Launches of the ring kernel (igemm_ring.h).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "igemm.h"
#include "igemm_internal.h"
#include "igemm_ring.h"

namespace igemm {
namespace {

int launch(const igemm_plan &p, int64_t m, int64_t n, int64_t k, const void *A, int64_t lda,
           const void *B, int64_t ldb, int32_t *C, int64_t ldc, const ConvGeom *g, int epi_kind,
           int epi, void *stream) {
    const bool reg = p.vec_a == 0;
    const void *fn = kKernels[p.kernel].es == 2
                         ? ring_i16(p.kernel, g != nullptr, epi_kind)
                         : ring_i8(p.kernel, g != nullptr, reg, epi_kind,
                                   p.grid <= num_cu_of_current_device());
    if (fn == nullptr) return IGEMM_EINVAL;
    int mi = (int)m, ni = (int)n, ki = (int)k, kc = (int)p.k_chunk;
    int tm = (int)((m + p.bm - 1) / p.bm), tn = (int)((n + p.bn - 1) / p.bn);
    ConvGeom gg = {};
    if (g != nullptr) gg = *g;
    void *args[] = {(void *)&A,  (void *)&lda, (void *)&B,  (void *)&ldb, (void *)&C,
                    (void *)&ldc, (void *)&mi, (void *)&ni, (void *)&ki,  (void *)&kc,
                    (void *)&tm, (void *)&tn,  (void *)&gg, (void *)&epi};
    hipError_t e = hipLaunchKernel(fn, dim3((unsigned)p.grid), dim3((unsigned)p.threads), args, 0,
                                   (hipStream_t)stream);
    return e == hipSuccess ? IGEMM_OK : IGEMM_EHIP;
}

}  // namespace

int launch_ring(const igemm_plan &p, int64_t m, int64_t n, int64_t k, const void *A, int64_t lda,
                const void *B, int64_t ldb, int32_t *C, int64_t ldc, const ConvGeom *g,
                void *stream) {
    return launch(p, m, n, k, A, lda, B, ldb, C, ldc, g,
                  p.split > 1 ? ring::EPI_ATOMIC : ring::EPI_ADD, 0, stream);
}

int launch_ring_srs(const igemm_plan &p, int64_t m, int64_t n, int64_t k, const void *A,
                    int64_t lda, const void *B, int64_t ldb, int16_t *C, int64_t ldc, int shift,
                    int round_half_up, void *stream) {
    if (p.split != 1) return IGEMM_EINVAL;
    return launch(p, m, n, k, A, lda, B, ldb, (int32_t *)C, ldc, nullptr, ring::EPI_SRS,
                  (shift & 0xff) | (round_half_up ? 0x100 : 0), stream);
}

}  // namespace igemm
