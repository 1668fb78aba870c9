// Host side of the launches per draft position: the workspace layout and the dispatch to the
// instantiations (one translation unit per head type and decoding mode, built in parallel).
#include "draft_step.hpp"

namespace dls {

#define DLS_STEP(WT, LT)                                                       \
  extern template hipError_t launch_step<WT, LT, false>(const DraftArgs&, hipStream_t); \
  extern template hipError_t launch_step<WT, LT, true>(const DraftArgs&, hipStream_t);
DLS_STEP(bf16_t, bf16_t)
DLS_STEP(bf16_t, float)
DLS_STEP(float, bf16_t)
DLS_STEP(float, float)
#undef DLS_STEP

namespace {
size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

template <typename WT, typename LT>
hipError_t launch_mode(const DraftArgs& a, hipStream_t st) {
  return a.smp.inv_temp != 0.f ? launch_step<WT, LT, true>(a, st) : launch_step<WT, LT, false>(a, st);
}
}  // namespace

DraftLayout draft_layout(const dls_local_head& h, int32_t batch, int32_t B) {
  (void)B;
  DraftLayout L;
  const bool markov = h.kind == DLS_HEAD_MARKOV;
  // one workgroup per CU; small vocabularies: one operand tile per wave
  L.groups = (int)std::min<int64_t>(kMaxG, ((int64_t)h.V + 127) / 128);
  size_t o = 0;
  L.off_h0 = o; o = align256(o + (size_t)batch * h.H * 4);
  L.off_h1 = o; o = align256(o + (size_t)batch * h.H * 4);
  L.off_rho = o; o = align256(o + (markov ? 0 : (size_t)batch * h.r * 4));
  // argmax keys (8 bytes) and partials (28): two sets for a Markov head
  L.off_part = o; o = align256(o + (size_t)(markov ? 2 : 1) * batch * L.groups * 36);
  L.total = o;
  return L;
}

hipError_t launch_draft(const DraftArgs& a, hipStream_t st) {
  if (!a.prep && small_head(a.head, a.batch, a.B)) return launch_small(a, st);
  if (a.head.dtype == DLS_BF16)
    return a.long_dtype == DLS_BF16 ? launch_mode<bf16_t, bf16_t>(a, st) : launch_mode<bf16_t, float>(a, st);
  return a.long_dtype == DLS_BF16 ? launch_mode<float, bf16_t>(a, st) : launch_mode<float, float>(a, st);
}

}  // namespace dls
