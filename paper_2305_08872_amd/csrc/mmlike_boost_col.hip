// BOOST on the vector ALU and the matrix cores, thres[j].
#include "mmlike_boost_impl.h"

namespace amulet {
template hipError_t launch_mmlike_boost<THRES_COL>(const MmlikeArgs &, hipStream_t);
}
