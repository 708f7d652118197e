// Activation-resident kernel: 3x3 windows with per-pixel scales, fp16 results and integer sums (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

HQ_RESIDENT_FORM(hq_resident_pertap, kResPerTap, HQ_RESIDENT_WHOLE, HQ_RESIDENT_NONE, HQ_RESIDENT_WHOLE)
