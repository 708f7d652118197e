// Activation-resident kernel: 3x3 windows with per-pixel scales, 8-bit codes (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

const void *hq_resident_bytes(int out, int ks) {
    constexpr int KIND = kResBytes;
#define HQ_RES(O) \
    if (out == O) return ks == 1 ? reinterpret_cast<const void *>(resident_kernel<O, KIND, 1>) \
                       : ks == 2 ? reinterpret_cast<const void *>(resident_kernel<O, KIND, 2>) \
                                 : reinterpret_cast<const void *>(resident_kernel<O, KIND, 3>);
    HQ_RES(kOutF16)
    HQ_RES(kOutF32)
    HQ_RES(kOutI32)
#undef HQ_RES
    return nullptr;
}
