// Generated by gen_patterns.py: the specialized kernels of the DenseR23G3
// family.  Do not edit by hand.
#include "fm_device.h"
#include "fm_direct.h"
#include "fm_joint.h"

namespace fm {
FM_DEFINE_FAMILY(DenseR23G3)
FM_DEFINE_DIRECT(DenseR23G3)
FM_DEFINE_JOINT(DenseR23G3)
}  // namespace fm
