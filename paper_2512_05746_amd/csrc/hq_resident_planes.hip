// Activation-resident kernel: 3x3 windows with one scale, activations as three digit planes (hq_resident_kernel.h).
#include "hq_resident_kernel.h"

HQ_RESIDENT_FORM(hq_resident_planes, kResPlanes, HQ_RESIDENT_WHOLE, HQ_RESIDENT_WHOLE, HQ_RESIDENT_WHOLE)
