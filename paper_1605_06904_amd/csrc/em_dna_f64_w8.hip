// EM of DNA models with a workgroup per model: FP64, eight waves.
#include "em_dna.h"

namespace pm {
int launch_em_dna_f64_w8(const EmArgs &a, size_t lds, hipStream_t st) { return launch_positions<double, 8>(a, lds, st); }
}  // namespace pm
