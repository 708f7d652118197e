// Activation-resident kernel: 3x3 windows with per-pixel scales, fp32 results and fp16 ones of ragged channels (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

HQ_RESIDENT_FORM(hq_resident_wholetaps, kResWholeTaps, HQ_RESIDENT_FORM_OUT, HQ_RESIDENT_FORM_OUT, HQ_RESIDENT_NONE)
