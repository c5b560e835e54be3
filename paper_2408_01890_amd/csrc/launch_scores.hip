// Instantiations of the CONCAT scores kernel.
#include "host.h"

namespace lisa {

namespace {
template <int HBI, int FS, int HBO, bool TILED = false>
int launch_scores_mfma_t(const lisa_desc* d, const ScoresMfmaArgs& a, hipStream_t st) {
  const int lds = scores_mfma_lds<HBI, FS, HBO>(d->H);
  auto kern = d->act == LISA_ACT_SILU ? k_lisa_scores_mfma<HBI, FS, HBO, 1, TILED>
                                      : k_lisa_scores_mfma<HBI, FS, HBO, 0, TILED>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return hip_fail(e);
  // one workgroup per compute unit, each with an equal run of the tiles
  const long long total = a.tiles_b * a.B;
  dim3 grid((unsigned)std::min<long long>(total, kComputeUnits));
  StageScope prof("k_lisa_scores_mfma", st);
  kern<<<grid, 512, lds, st>>>(a);
  return check_launch();
}
}  // namespace

// The weights as the kernel that launch_scores_mfma_kernel() chooses has them.
FfnImage scores_mfma_image(const lisa_desc* d, const void* w1, const void* w2) {
  const int HBO = d->H <= 16 ? 1 : d->H <= 32 ? 2 : 3;
  return FfnImage{(const bf16_t*)w1, (const bf16_t*)w2, nullptr, 2 * d->H, d->F, d->H, HBO, d->F > 128 ? 8 : 4, HBO, 1, d->H, 0};
}

int launch_scores_mfma_kernel(const lisa_desc* d, const ScoresMfmaArgs& a, hipStream_t st) {
  const bool wide = d->F > 128;
  if (d->score_tiled) {                                      // (concat_tiled_ok: up to 32 heads)
    if (d->H <= 16)
      return wide ? launch_scores_mfma_t<2, 8, 1, true>(d, a, st) : launch_scores_mfma_t<2, 4, 1, true>(d, a, st);
    return wide ? launch_scores_mfma_t<4, 8, 2, true>(d, a, st) : launch_scores_mfma_t<4, 4, 2, true>(d, a, st);
  }
  if (d->H <= 16) return wide ? launch_scores_mfma_t<2, 8, 1>(d, a, st) : launch_scores_mfma_t<2, 4, 1>(d, a, st);
  if (d->H <= 32) return wide ? launch_scores_mfma_t<4, 8, 2>(d, a, st) : launch_scores_mfma_t<4, 4, 2>(d, a, st);
  return wide ? launch_scores_mfma_t<6, 8, 3>(d, a, st) : launch_scores_mfma_t<6, 4, 3>(d, a, st);
}

}  // namespace lisa
