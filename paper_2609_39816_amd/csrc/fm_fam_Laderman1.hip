// Generated by gen_patterns.py: the specialized kernels of the Laderman1
// family.  Do not edit by hand.
#include "fm_device.h"
#include "fm_direct.h"
#include "fm_joint.h"

namespace fm {
FM_DEFINE_FAMILY(Laderman1)
FM_DEFINE_DIRECT(Laderman1)
FM_DEFINE_JOINT(Laderman1)
}  // namespace fm
