// Generated by gen_patterns.py: the specialized kernels of the Strassen3
// family.  Do not edit by hand.
#include "fm_device.h"
#include "fm_direct.h"
#include "fm_joint.h"

namespace fm {
FM_DEFINE_FAMILY(Strassen3)
FM_DEFINE_DIRECT(Strassen3)
FM_DEFINE_JOINT(Strassen3)
}  // namespace fm
