// float32 prefill layers on the kernels of kernels_f32.h: which shapes they take, and the launches.
#include "host.h"
#include "kernels_f32.h"

namespace lisa {

bool f32_attn_ok(const lisa_desc* d) {
  return d->dtype == LISA_F32 && d->Lq > 1 && (d->d_k == 64 || d->d_k == 128);
}

namespace {
int launch_attn(const lisa_desc* d, const F32AttnArgs& a, bool given, const char* name, hipStream_t st) {
  dim3 grid((d->Lq + 15) / 16, d->H, d->B);
  StageScope prof(name, st);
  if (d->d_k == 64) {
    if (given) k_f32_attn<1, true><<<grid, 256, 0, st>>>(a);
    else k_f32_attn<1, false><<<grid, 256, 0, st>>>(a);
  } else {
    if (given) k_f32_attn<2, true><<<grid, 256, 0, st>>>(a);
    else k_f32_attn<2, false><<<grid, 256, 0, st>>>(a);
  }
  return check_launch();
}
F32AttnArgs attn_args(const lisa_desc* d) {
  F32AttnArgs a{};
  a.H = d->H; a.Hkv = d->Hkv; a.Lq = d->Lq; a.Lk = d->Lk; a.causal = d->causal;
  a.scale = pick_scale(d->std_scale, d->d_k);
  return a;
}
}  // namespace

int run_f32_std(const lisa_desc* d, const void* q, const void* k, const void* v, void* scores, void* out,
                hipStream_t st) {
  F32AttnArgs a = attn_args(d);
  a.q = (const float*)q; a.k = (const float*)k; a.v = (const float*)v;
  a.scores = (float*)scores; a.out = (float*)out;
  return launch_attn(d, a, false, "k_f32_attn", st);
}

int run_f32_softmax_v(const lisa_desc* d, const void* scores, const void* v, void* out, hipStream_t st) {
  F32AttnArgs a = attn_args(d);
  a.given = (const float*)scores; a.v = (const float*)v; a.out = (float*)out;
  return launch_attn(d, a, true, "k_f32_softmax_v", st);
}

bool f32_scores_ok(const lisa_desc* d) {
  return d->dtype == LISA_F32 && d->Lq > 1 && d->mix == LISA_MIX_ADD && (d->act == LISA_ACT_RELU || d->act == LISA_ACT_SILU) &&
         d->H <= 32 && f32_scores_lds(d->H <= 8 ? 8 : d->H <= 16 ? 16 : 32, d->F) <= 64 * 1024;
}

int run_f32_scores(const lisa_desc* d, const void* q_lr, const void* k_lr, const void* prev, const void* w1,
                   const void* w2, void* scores, hipStream_t st) {
  F32ScoresArgs a{};
  a.q_lr = (const float*)q_lr; a.k_lr = (const float*)k_lr; a.prev = (const float*)prev;
  a.w1 = (const float*)w1; a.w2 = (const float*)w2; a.scores = (float*)scores;
  a.H = d->H; a.Hkv = d->Hkv; a.Lq = d->Lq; a.Lk = d->Lk; a.r = d->r; a.F = d->F; a.causal = d->causal;
  a.dscale = pick_scale(d->delta_scale, d->r);
  // a tile per workgroup until there are several workgroups per compute unit, then runs of tiles that share
  // the staged weights
  const int kt = (d->Lk + 15) / 16, rbs = (d->Lq + 15) / 16;
  a.tiles = (int)std::min<long long>(16, std::max<long long>(1, (long long)kt * rbs * d->B / (16 * kComputeUnits)));
  dim3 grid((kt + a.tiles - 1) / a.tiles, rbs, d->B);
  const int lds = f32_scores_lds(d->H <= 8 ? 8 : d->H <= 16 ? 16 : 32, d->F);
  StageScope prof("k_f32_lisa_scores", st);
  const bool silu = d->act == LISA_ACT_SILU;
  if (d->H <= 8) {
    if (silu) k_f32_lisa_scores<8, 1><<<grid, 256, lds, st>>>(a);
    else k_f32_lisa_scores<8, 0><<<grid, 256, lds, st>>>(a);
  } else if (d->H <= 16) {
    if (silu) k_f32_lisa_scores<16, 1><<<grid, 256, lds, st>>>(a);
    else k_f32_lisa_scores<16, 0><<<grid, 256, lds, st>>>(a);
  } else {
    if (silu) k_f32_lisa_scores<32, 1><<<grid, 256, lds, st>>>(a);
    else k_f32_lisa_scores<32, 0><<<grid, 256, lds, st>>>(a);
  }
  return check_launch();
}

}  // namespace lisa
