// Activation-resident kernel: 3x3 windows with per-pixel scales, channel counts that are no multiple of 64 (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

HQ_RESIDENT_FORM(hq_resident_wholetaps_ragged, kResWholeTaps, HQ_RESIDENT_TAIL, HQ_RESIDENT_TAIL, HQ_RESIDENT_NONE)
