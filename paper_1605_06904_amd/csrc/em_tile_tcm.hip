// EM of sixteen models per workgroup: TCM.
#include "em_tile.h"

namespace pm {
int launch_em_tile_tcm(const EmArgs &a, hipStream_t st) { return launch_tile<true>(a, st); }
}  // namespace pm
