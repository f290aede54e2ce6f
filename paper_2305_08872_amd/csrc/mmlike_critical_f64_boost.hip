// BOOST in fp64 by a clamp (mmlike_critical_f64_impl.h).
#include "mmlike_critical_f64_impl.h"

namespace amulet {
template hipError_t launch_mmlike_critical_f64<2, 0>(const MmlikeArgsF64 &, int, hipStream_t);
template hipError_t launch_mmlike_critical_f64<2, 1>(const MmlikeArgsF64 &, int, hipStream_t);
template hipError_t launch_mmlike_critical_f64<2, 2>(const MmlikeArgsF64 &, int, hipStream_t);
}
