// The rank-8 scan for float32 queries.
#include "scan_quad.h"

namespace locks {
template hipError_t launch_scan_quad<float>(const ScanArgs&, int, int, int, hipStream_t);
}
