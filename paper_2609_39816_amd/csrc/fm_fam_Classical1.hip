// Generated by gen_patterns.py: the specialized kernels of the Classical1
// family.  Do not edit by hand.
#include "fm_device.h"
#include "fm_direct.h"
#include "fm_joint.h"

namespace fm {
FM_DEFINE_FAMILY(Classical1)
FM_DEFINE_DIRECT(Classical1)
FM_DEFINE_JOINT(Classical1)
}  // namespace fm
