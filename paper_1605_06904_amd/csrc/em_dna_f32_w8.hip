// EM of DNA models with a workgroup per model: FP32, eight waves.
#include "em_dna.h"

namespace pm {
int launch_em_dna_f32_w8(const EmArgs &a, size_t lds, hipStream_t st) { return launch_positions<float, 8>(a, lds, st); }
}  // namespace pm
