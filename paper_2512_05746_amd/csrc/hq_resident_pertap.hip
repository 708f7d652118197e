// Activation-resident kernel: 3x3 windows with per-pixel scales (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

HQ_RESIDENT_FORM(hq_resident_pertap, kResPerTap)
