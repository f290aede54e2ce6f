// COUNT in fp64 by critical values (mmlike_critical_f64_impl.h).
#include "mmlike_critical_f64_impl.h"

namespace amulet {
template hipError_t launch_mmlike_critical_f64<3, 0>(const MmlikeArgsF64 &, int, hipStream_t);
template hipError_t launch_mmlike_critical_f64<3, 1>(const MmlikeArgsF64 &, int, hipStream_t);
template hipError_t launch_mmlike_critical_f64<3, 2>(const MmlikeArgsF64 &, int, hipStream_t);
}
