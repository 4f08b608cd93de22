// Instantiations of the ring kernel: int16 operands.
#include "igemm_ring.h"

namespace igemm {
using namespace ring;

// Through registers only (the limb split happens there). 128 x 128 tiles, eight
// waves of 64 x 32, two 32 KB stages, one workgroup per compute unit; 64 x 64
// tiles, four waves of 32 x 32, two 16 KB stages, three workgroups.
template <int BM, int BN, int WM, int WN, int OCC>
static const void *pick_i16(bool conv, int epi) {
#define IGEMM_R(am, ep) (const void *)&igemm_ring<2, BM, BN, WM, WN, 64, 2, OCC, am, true, ep>
    if (conv)
        return epi == EPI_SRS      ? nullptr
               : epi == EPI_ATOMIC ? IGEMM_R(1, EPI_ATOMIC)
                                   : IGEMM_R(1, EPI_ADD);
    return epi == EPI_SRS      ? IGEMM_R(0, EPI_SRS)
           : epi == EPI_ATOMIC ? IGEMM_R(0, EPI_ATOMIC)
                               : IGEMM_R(0, EPI_ADD);
#undef IGEMM_R
}

const void *ring_i16(int id, bool conv, int epi) {
    switch (id) {
        case K_I16_RING_128x128: return pick_i16<128, 128, 64, 32, 1>(conv, epi);
        case K_I16_RING_64x64: return pick_i16<64, 64, 32, 32, 3>(conv, epi);
        default: return nullptr;
    }
}

}  // namespace igemm
