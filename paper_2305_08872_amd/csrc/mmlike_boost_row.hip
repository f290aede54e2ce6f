// BOOST on the vector ALU and the matrix cores, thres[i].
#include "mmlike_boost_impl.h"

namespace amulet {
template hipError_t launch_mmlike_boost<THRES_ROW>(const MmlikeArgs &, hipStream_t);
}
