// The FP32 (mixed form) instances of the resident CG solves, compiled apart from the FP64 ones.
#include "resident_kernel.h"

namespace gspm {

template bool resident_fits<float>(ResArgs &, int, bool, size_t, int);
template int launch_resident<float>(const ResArgs &, int, bool, hipStream_t);

}  // namespace gspm
