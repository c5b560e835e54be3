// Instantiations of the split-context decode kernel.
#include "host.h"

namespace lisa {

namespace {
template <int LISA_MODE, int HB, int FS, int ACT = 0>
int launch_decode_part_dk(const lisa_desc* d, const DecodeArgs& a, size_t lds, hipStream_t st) {
  dim3 grid(a.n_chunk, d->B);
  if (a.cmb_units > 0) lds = std::max<size_t>(lds, 4608);   // (the combine units use the same LDS)
  auto kern = d->d_k == 128 ? k_decode_part<LISA_MODE, HB, FS, 128, ACT> : k_decode_part<LISA_MODE, HB, FS, 64, ACT>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return hip_fail(e);
  }
  StageScope prof(LISA_MODE == 3 ? "k_decode_part_share" : LISA_MODE ? "k_decode_part_lisa" : "k_decode_part_std", st);
  kern<<<grid, DEC_THREADS, lds, st>>>(a);
  return check_launch();
}

// CONCAT form: HBI blocks of 16 FFN inputs (2H of them), hidden width by thirds of the range
template <int HBI, int ACT>
int launch_decode_concat_act(const lisa_desc* d, const DecodeArgs& a, size_t lds, hipStream_t st) {
  if (d->F <= 64) return launch_decode_part_dk<2, HBI, 2, ACT>(d, a, lds, st);
  if (d->F <= 128) return launch_decode_part_dk<2, HBI, 4, ACT>(d, a, lds, st);
  return launch_decode_part_dk<2, HBI, 8, ACT>(d, a, lds, st);
}
template <int HBI>
int launch_decode_concat_fs(const lisa_desc* d, const DecodeArgs& a, size_t lds, hipStream_t st) {
  return d->act == LISA_ACT_SILU ? launch_decode_concat_act<HBI, 1>(d, a, lds, st)
                                 : launch_decode_concat_act<HBI, 0>(d, a, lds, st);
}

template <int HB, int ACT>
int launch_decode_lisa_act(const lisa_desc* d, const DecodeArgs& a, size_t lds, hipStream_t st) {
  switch ((d->F + 31) / 32) {
    case 1: return launch_decode_part_dk<1, HB, 1, ACT>(d, a, lds, st);
    case 2: return launch_decode_part_dk<1, HB, 2, ACT>(d, a, lds, st);
    case 3: return launch_decode_part_dk<1, HB, 3, ACT>(d, a, lds, st);
    default: return launch_decode_part_dk<1, HB, 4, ACT>(d, a, lds, st);
  }
}
template <int HB>
int launch_decode_lisa_fs(const lisa_desc* d, const DecodeArgs& a, size_t lds, hipStream_t st) {
  return d->act == LISA_ACT_SILU ? launch_decode_lisa_act<HB, 1>(d, a, lds, st)
                                 : launch_decode_lisa_act<HB, 0>(d, a, lds, st);
}
}  // namespace

// The partial pass of a decode step over a.n_chunk chunks: picks the instantiation and its LDS size.
int launch_decode_part(const lisa_desc* d, bool lisa_layer, DecodeArgs a, hipStream_t st) {
  size_t lds = (size_t)d->H * DEC_CK * sizeof(float);
  if (lisa_layer && d->mix == LISA_MIX_SHARE) {
    a.scale = 0.f;
    return launch_decode_part_dk<3, 1, 1>(d, a, lds, st);
  } else if (lisa_layer && d->mix == LISA_MIX_CONCAT) {
    const int hbi = d->H <= 16 ? 2 : d->H <= 32 ? 4 : 6, fs = d->F <= 64 ? 2 : d->F <= 128 ? 4 : 8;
    const int ks1 = (hbi + 1) / 2, hbo = (hbi + 1) / 2;
    lds += (size_t)((d->H * d->r + 3) & ~3) * sizeof(float) + (size_t)(2 * fs * ks1 + hbo * fs) * 1024;
    a.scale = pick_scale(d->delta_scale, d->r);
    return hbi == 2   ? launch_decode_concat_fs<2>(d, a, lds, st)
         : hbi == 4 ? launch_decode_concat_fs<4>(d, a, lds, st)
                    : launch_decode_concat_fs<6>(d, a, lds, st);
  } else if (lisa_layer) {
    // + q_lr [H][r] as float + the FFN weights in MFMA operand order (mfma_ffn.h: kStageBytes)
    const int hb = (d->H + 15) / 16, fs = (d->F + 31) / 32, ks1 = (hb + 1) / 2;
    lds += (size_t)((d->H * d->r + 3) & ~3) * sizeof(float) + (size_t)(2 * fs * ks1 + hb * fs) * 1024;
    a.scale = pick_scale(d->delta_scale, d->r);
    switch ((d->H + 15) / 16) {
      case 1: return launch_decode_lisa_fs<1>(d, a, lds, st);
      case 2: return launch_decode_lisa_fs<2>(d, a, lds, st);
      case 3: return launch_decode_lisa_fs<3>(d, a, lds, st);
      default: return launch_decode_lisa_fs<4>(d, a, lds, st);
    }
  } else {
    a.scale = pick_scale(d->std_scale, d->d_k);
    return launch_decode_part_dk<0, 1, 1>(d, a, lds, st);
  }
}

}  // namespace lisa
