// Generated by gen_patterns.py: the specialized kernels of the DenseR7G2
// family.  Do not edit by hand.
#include "fm_device.h"
#include "fm_direct.h"
#include "fm_joint.h"

namespace fm {
FM_DEFINE_FAMILY(DenseR7G2)
FM_DEFINE_DIRECT(DenseR7G2)
FM_DEFINE_JOINT(DenseR7G2)
}  // namespace fm
