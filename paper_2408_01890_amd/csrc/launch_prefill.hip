// Instantiations of the fused prefill kernel.  Compiled once per LISA_PART.
#include "host.h"

namespace lisa {

template <int NG, int FS, int HPW, int NW, int ACT, int RS, int SHG = 0, bool FTRIM = false>
int launch_prefill_fused_t(const lisa_desc* d, const PrefillArgs& a, hipStream_t st) {
  constexpr int GH = NW * HPW, H = NG * GH;
  typedef MfmaFfn<(H + 15) / 16, FS, (GH + 15) / 16> Ffn;
  // (all heads in one workgroup: the A_{n-1} piece is double buffered and doubles as A_n staging)
  constexpr bool XSTG = NG == 1 && HPW == 4;
  constexpr size_t lds = XSTG ? (size_t)2 * H * PF_XS_HEAD + (size_t)GH * PF_YS_HEAD + Ffn::kStageBytes
                              : (size_t)H * PF_XS_HEAD + (size_t)GH * PF_YS_HEAD + Ffn::kStageBytes +
                                    (size_t)GH * RS * PF_AS_HEAD;
  static_assert(lds <= 160 * 1024, "LDS of one compute unit");
  auto kern = k_lisa_prefill_fused<NG, FS, HPW, NW, ACT, RS, SHG, FTRIM>;
  if constexpr (ACT == 0 && !XSTG && RS <= 2)
    if (a.tiled && a.scores) kern = k_lisa_prefill_fused<NG, FS, HPW, NW, ACT, RS, SHG, FTRIM, true>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return hip_fail(e);
  const long long units = (long long)((a.Lq + PF_ROWS * RS - 1) / (PF_ROWS * RS)) * a.split;
  const long long chunks = ((a.pair ? (units + 1) / 2 : units) + a.chunk - 1) / a.chunk * a.B;
  const long long wgs = (chunks + 7) / 8 * 8 * a.chunk * NG;
  if (wgs > 0x7fffffffLL) return LISA_ERR_UNSUPPORTED;
  StageScope prof("k_lisa_prefill_fused", st);
  kern<<<dim3((unsigned)wgs), NW * 64, lds, st>>>(a);
  return check_launch();
}

template <int NG, int HPW, int NW, int ACT, int RS, int SHG = 0>
int launch_prefill_fused_act(const lisa_desc* d, const PrefillArgs& a, hipStream_t st) {
  if constexpr (ACT == 2) {                                  // (F = 2 H)
    constexpr int H = NG * NW * HPW, FS = (2 * H + 31) / 32;
    if constexpr (RS == 1 || FS > 1) return launch_prefill_fused_t<NG, FS, HPW, NW, 2, RS, SHG, (RS == 2 && 2 * H <= 32 * FS - 16)>(d, a, st);
    else return LISA_ERR_UNSUPPORTED;                        // (prefill_slices_ok)
  } else if constexpr (RS > 1) {                             // row slices: 33..96 hidden units (prefill_slices_ok)
    if ((d->F + 31) / 32 == 2) return launch_prefill_fused_t<NG, 2, HPW, NW, ACT, RS, SHG>(d, a, st);
    // (two slices, 65..80 hidden units: the last block of 16 is padding)
    if (RS == 2 && d->F <= 80) return launch_prefill_fused_t<NG, 3, HPW, NW, ACT, RS, SHG, true>(d, a, st);
    return launch_prefill_fused_t<NG, 3, HPW, NW, ACT, RS, SHG>(d, a, st);
  } else {
    switch ((d->F + 31) / 32) {
      case 1: return launch_prefill_fused_t<NG, 1, HPW, NW, ACT, 1, SHG>(d, a, st);
      case 2: return launch_prefill_fused_t<NG, 2, HPW, NW, ACT, 1, SHG>(d, a, st);
      case 3: return launch_prefill_fused_t<NG, 3, HPW, NW, ACT, 1, SHG>(d, a, st);
      default: return launch_prefill_fused_t<NG, 4, HPW, NW, ACT, 1, SHG>(d, a, st);
    }
  }
}
template <int NG, int HPW, int NW, int ACT>
int launch_prefill_fused_slices(const lisa_desc* d, const PrefillArgs& a, int slices, hipStream_t st) {
  if constexpr (ACT != 1) {
    if (HPW == 1 && slices == 4) return launch_prefill_fused_act<NG, 1, NW, ACT, 4>(d, a, st);
    if (HPW == 1 && slices == 2) return launch_prefill_fused_act<NG, 1, NW, ACT, 2>(d, a, st);
  }
  // the heads of a wave share their key/value head: one operand set for all of them
  constexpr int HS = HPW == 3 ? 2 : HPW;                     // (no shared form of the 24-head kernel)
  if constexpr (HPW > 1 && HPW != 3)
    if ((d->H / d->Hkv) % HPW == 0) return launch_prefill_fused_act<NG, HS, NW, ACT, 1, HS>(d, a, st);
  return launch_prefill_fused_act<NG, HPW, NW, ACT, 1>(d, a, st);
}
template <int NG, int HPW, int NW>
int launch_prefill_fused_fs(const lisa_desc* d, const PrefillArgs& a, int slices, hipStream_t st) {
  // (a test per tile of a flag instead of a form of its own: 1.2 % of the LLaMA3-8B and LLaMA2-13B shapes)
  if (a.pass_through) return launch_prefill_fused_slices<NG, HPW, NW, 2>(d, a, slices, st);
  return d->act == LISA_ACT_SILU ? launch_prefill_fused_slices<NG, HPW, NW, 1>(d, a, slices, st)
                                 : launch_prefill_fused_slices<NG, HPW, NW, 0>(d, a, slices, st);
}

#if LISA_PART == 0
template int launch_prefill_fused_fs<1, 1, 8>(const lisa_desc*, const PrefillArgs&, int, hipStream_t);
template int launch_prefill_fused_fs<2, 1, 8>(const lisa_desc*, const PrefillArgs&, int, hipStream_t);
#elif LISA_PART == 1
template int launch_prefill_fused_fs<1, 2, 8>(const lisa_desc*, const PrefillArgs&, int, hipStream_t);
template int launch_prefill_fused_fs<1, 3, 8>(const lisa_desc*, const PrefillArgs&, int, hipStream_t);
#elif LISA_PART == 2
template int launch_prefill_fused_fs<4, 1, 8>(const lisa_desc*, const PrefillArgs&, int, hipStream_t);
template int launch_prefill_fused_fs<5, 1, 8>(const lisa_desc*, const PrefillArgs&, int, hipStream_t);
#elif LISA_PART == 3
template int launch_prefill_fused_fs<1, 4, 8>(const lisa_desc*, const PrefillArgs&, int, hipStream_t);
#elif LISA_PART == 4
template int launch_prefill_fused_fs<2, 2, 8>(const lisa_desc*, const PrefillArgs&, int, hipStream_t);
#endif

}  // namespace lisa
