// The FP64 instances of the resident CG solves, compiled apart from the FP32 ones.
#include "resident_kernel.h"

namespace gspm {

template bool resident_fits<double>(ResArgs &, int, bool, size_t, int);
template int launch_resident<double>(const ResArgs &, int, bool, hipStream_t);

}  // namespace gspm
