// Generated by gen_patterns.py: the specialized kernels of the Strassen2
// family.  Do not edit by hand.
#include "fm_device.h"
#include "fm_direct.h"
#include "fm_joint.h"

namespace fm {
FM_DEFINE_FAMILY(Strassen2)
FM_DEFINE_DIRECT(Strassen2)
FM_DEFINE_JOINT(Strassen2)
}  // namespace fm
