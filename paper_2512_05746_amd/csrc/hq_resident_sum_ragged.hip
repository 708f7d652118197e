// Activation-resident kernel: 3x3 windows with one scale, channel counts that are no multiple of 64 (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

HQ_RESIDENT_FORM(hq_resident_sum_ragged, kResSum, HQ_RESIDENT_TAIL, HQ_RESIDENT_TAIL, HQ_RESIDENT_TAIL)
