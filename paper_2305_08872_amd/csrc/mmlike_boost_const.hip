// BOOST on the vector ALU and the matrix cores, one threshold.
#include "mmlike_boost_impl.h"

namespace amulet {
template hipError_t launch_mmlike_boost<THRES_CONST>(const MmlikeArgs &, hipStream_t);
}
