// Activation-resident kernel: 3x3 windows with one scale (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

HQ_RESIDENT_FORM(hq_resident_sum, kResSum, HQ_RESIDENT_WHOLE, HQ_RESIDENT_WHOLE, HQ_RESIDENT_WHOLE)
