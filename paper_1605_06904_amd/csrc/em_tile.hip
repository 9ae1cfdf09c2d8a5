// EM of sixteen models per workgroup: OOPS and ZOOPS.
#include "em_tile.h"

namespace pm {
int launch_em_tile(const EmArgs &a, hipStream_t st) { return launch_tile<false>(a, st); }
}  // namespace pm
