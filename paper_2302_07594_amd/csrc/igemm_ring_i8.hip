// Instantiations of the ring kernel: int8 operands.
#include "igemm_ring.h"

namespace igemm {
using namespace ring;

// k-tiles of 128, so that a row of A is a whole 128-byte line per request; two
// workgroups per compute unit. By DMA four waves: 128 x 128 tiles in 64 x 64, two
// 32 KB stages, 64 x 128 tiles in 32 x 64, three 24 KB stages. Through registers
// eight waves of half the columns and two stages: they read more from LDS but
// cover each other's waits for loads and stores (when chosen, operands in the
// caches: 777 x 1111 x 2049 14.4 us against 16.5, 1000 x 3001 x 1777 20.4 against
// 23.1; by DMA 1024 x 4096 x 4096 36.3 against 35.2). Through registers 128 x 128
// tiles need more than the 128 registers of two workgroups: a grid of one
// workgroup per unit at most takes them (ROCC 1; 1000 x 3001 x 1777 25.8 us
// against 28.4, operands not cached), a larger one spills two to six (2048 x 4096
// x 4096 53.5 against 57.3).
template <int BM, int BN, int WM, int WN, int NST, int ROCC>
static const void *pick_i8(bool conv, bool reg, int epi) {
#define IGEMM_R(am, rg, ep)                                                                  \
    (const void *)&igemm_ring<1, BM, BN, WM, rg ? WN / 2 : WN, 128, rg ? 2 : NST, rg ? ROCC : 2, \
                              am, rg, ep>
    if (conv) {
        if (epi == EPI_SRS) return nullptr;
        if (reg) return epi == EPI_ATOMIC ? IGEMM_R(1, true, EPI_ATOMIC) : IGEMM_R(1, true, EPI_ADD);
        return epi == EPI_ATOMIC ? IGEMM_R(1, false, EPI_ATOMIC) : IGEMM_R(1, false, EPI_ADD);
    }
    if (reg)
        return epi == EPI_SRS      ? IGEMM_R(0, true, EPI_SRS)
               : epi == EPI_ATOMIC ? IGEMM_R(0, true, EPI_ATOMIC)
                                   : IGEMM_R(0, true, EPI_ADD);
    return epi == EPI_SRS      ? IGEMM_R(0, false, EPI_SRS)
           : epi == EPI_ATOMIC ? IGEMM_R(0, false, EPI_ATOMIC)
                               : IGEMM_R(0, false, EPI_ADD);
#undef IGEMM_R
}

const void *ring_i8(int id, bool conv, bool reg, int epi, bool one_per_cu) {
    switch (id) {
        case K_I8_RING_128x128:
            if (reg && one_per_cu) return pick_i8<128, 128, 64, 64, 2, 1>(conv, true, epi);
            return pick_i8<128, 128, 64, 64, 2, 2>(conv, reg, epi);
        case K_I8_RING_64x128: return pick_i8<64, 128, 32, 64, 3, 2>(conv, reg, epi);
        default: return nullptr;
    }
}

}  // namespace igemm
