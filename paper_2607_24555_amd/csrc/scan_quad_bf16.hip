// The rank-8 scan for bfloat16 queries.
#include "scan_quad.h"

namespace locks {
template hipError_t launch_scan_quad<uint16_t>(const ScanArgs&, int, int, int, hipStream_t);
}
