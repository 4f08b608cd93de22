// Instantiations of the ring kernel: int8 operands.
#include "igemm_ring.h"

namespace igemm {
using namespace ring;

// k-tiles of 128, so that a row of A is a whole 128-byte line per request. 128
// x 128 tiles, four waves of 64 x 64, two 32 KB stages; 64 x 128 tiles, four
// waves of 32 x 64, three 24 KB stages by DMA, two through registers; two
// workgroups per compute unit.
template <int BM, int BN, int WM, int WN, int NST>
static const void *pick_i8(bool conv, bool reg, int epi) {
#define IGEMM_R(am, rg, ep) \
    (const void *)&igemm_ring<1, BM, BN, WM, WN, 128, rg ? 2 : NST, 2, am, rg, ep>
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

const void *ring_i8(int id, bool conv, bool reg, int epi) {
    switch (id) {
        case K_I8_RING_128x128: return pick_i8<128, 128, 64, 64, 2>(conv, reg, epi);
        case K_I8_RING_64x128: return pick_i8<64, 128, 32, 64, 3>(conv, reg, epi);
        default: return nullptr;
    }
}

}  // namespace igemm
