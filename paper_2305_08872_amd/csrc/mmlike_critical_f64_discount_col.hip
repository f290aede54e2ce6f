// DISCOUNT in fp64 by critical values (mmlike_critical_f64_impl.h), threshold operand form "col".
#include "mmlike_critical_f64_impl.h"

namespace amulet {
template hipError_t launch_mmlike_critical_f64<1, 0>(const MmlikeArgsF64 &, int, hipStream_t);
}
