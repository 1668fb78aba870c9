// The launches per draft position for float32 heads, sampled.
#include "draft_step.hpp"

namespace dls {
template hipError_t launch_step<float, bf16_t, true>(const DraftArgs&, hipStream_t);
template hipError_t launch_step<float, float, true>(const DraftArgs&, hipStream_t);
}  // namespace dls
