// The launches per draft position for bf16 heads, greedy.
#include "draft_step.hpp"

namespace dls {
template hipError_t launch_step<bf16_t, bf16_t, false>(const DraftArgs&, hipStream_t);
template hipError_t launch_step<bf16_t, float, false>(const DraftArgs&, hipStream_t);
}  // namespace dls
