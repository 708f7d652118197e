// Activation-resident kernel: 3x3 windows with per-pixel scales, 8-bit codes (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

HQ_RESIDENT_FORM(hq_resident_bytes, kResBytes, HQ_RESIDENT_WHOLE, HQ_RESIDENT_WHOLE, HQ_RESIDENT_WHOLE)
