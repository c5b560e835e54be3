// Prefill layers in float32 arithmetic on the kernels of kernels_f32.h: which shapes they take, and the launches.
#include "host.h"
#include "kernels_f32.h"

namespace lisa {

// The order of k_f32_attn's workgroups: 0 = a head's row blocks one after the other, 1 = by length, 2 = by length, every other 256
// backwards.  A launch that fits the compute units needs no division to find its place (0.25 us).  By length all heads'
// K and V are in use at a time: where these are few an XCD has several row blocks of each that walk its tiles side by
// side, of many heads an L2 of 4 MB holds too little of any.  Standard layer, order 0 / 2 in us, heads in all, width 64: 128 heads, 512
// tokens (4096 workgroups) 115 / 78, 1500 (12032) 525 / 598; 156, 200 (2028) 21.9 / 20.7, 410 (4056) 60 / 69, 900 (8892) 272 / 390;
// 512, 600 (19456) 411 / 560; width 128: 96, 1000 (6048) 392 / 347, 1500 (9024) 783 / 747; 256, 128 (2048) 46.7 / 43.5, 200 (3328)
// 81.8 / 82.5, 700 (11264) 503 / 649, 1000 (16128) 974 / 1295.  One or two row blocks: little to order, and the divisions cost more
// (bf16, 1000 sequences of 9 tokens, 216 / 225; 8 x 17 tokens of 32 heads of 128 7.6 / 8.2).
int f32_attn_order(const lisa_desc* d, int n_rows, int parts) {
  const long long blocks = (n_rows + 15) / 16, heads = (long long)d->H * d->B, wgs = blocks * parts * heads;
  if (wgs <= kComputeUnits) return 1;
  return blocks > 2 && wgs <= (heads <= 128 ? 36 : 8) * kComputeUnits ? 2 : 0;
}

bool f32_attn_ok(const lisa_desc* d) { return d->Lq > 1 && d->dtype == LISA_F32 && (d->d_k == 64 || d->d_k == 128); }

namespace {
template <typename T, typename S, int NDK>
int launch_attn(const lisa_desc* d, F32AttnArgs<T, S> a, hipStream_t st) {
  const long long wgs = (long long)((a.n_rows + 15) / 16) * a.parts * d->H * d->B;
  // Eight waves where rows are long and workgroups few: the chain of a wave's tiles bounds them, with scores given (no K stream
  // beside it) up to four workgroups per compute unit.  float32, 8 heads of 64, four / eight waves in us: scores given, 430 tokens
  // 12.1 / 10.2, 2 x 504 14.2 / 10.9, 3 x 504 15.1 / 13.9, 3 x 700 (1056 workgroups) 19.8 / 20.2, 128 tokens 7.2 / 7.8; scores made,
  // 430 tokens (216) 14.8 / 13.4, 700 (352) 19.4 / 19.2, 2 x 504 (512) 16.7 / 17.7.
  const bool wide = sizeof(T) == 4 && a.out && d->Lk > 256 && wgs <= (a.given ? 4 : 1) * kComputeUnits;
  a.order = f32_attn_order(d, a.n_rows, a.parts);
  const int blocks = a.blocks = (a.n_rows + 15) / 16 * a.parts;
  const dim3 grid = a.order == 0 ? dim3(blocks, d->H, d->B) : a.order == 1 ? dim3(d->H, d->B, blocks) : dim3((unsigned)wgs);
  StageScope prof(a.given ? "k_f32_softmax_v" : "k_f32_attn", st);
  auto kern = a.given ? k_f32_attn<T, S, NDK, true, 4> : k_f32_attn<T, S, NDK, false, 4>;
  if constexpr (sizeof(T) == 4)
    if (wide) kern = a.given ? k_f32_attn<T, S, NDK, true, 8> : k_f32_attn<T, S, NDK, false, 8>;
  kern<<<grid, wide ? 512 : 256, 0, st>>>(a);
  return check_launch();
}

// `given`: scores of the rows row0 .. row0 + n_rows - 1 to take instead of q k^T
template <typename T, typename S>
int run_attn(const lisa_desc* d, const void* q, const void* k, const void* given, int row0, int n_rows, const void* v,
             void* scores, void* out, hipStream_t st) {
  F32AttnArgs<T, S> a{};
  a.q = (const T*)q; a.k = (const T*)k; a.v = (const T*)v; a.given = (const float*)given;
  a.scores = (S*)scores; a.out = out;
  a.B = d->B; a.H = d->H; a.Hkv = d->Hkv; a.Lq = d->Lq; a.Lk = d->Lk; a.causal = d->causal;
  a.out_f32 = d->out_f32 || d->dtype == LISA_F32;
  a.row0 = row0; a.n_rows = n_rows;
  // Scores only: nothing to merge, so few row blocks of many keys are spread until there is a workgroup per
  // compute unit, two tiles per wave at least (2 rows, 3000 keys, 8 heads of 64: 24.7 us in one workgroup per head,
  // 5.9 spread, 11.2 on the generic kernel; two per compute unit cost 13 % at 700 rows, 4 heads).
  const long long blocks = (long long)((n_rows + 15) / 16) * d->H * d->B;
  a.parts = out ? 1 : (int)std::max<long long>(1, std::min<long long>((d->Lk + 127) / 128, kComputeUnits / blocks));
  a.scale = pick_scale(d->std_scale, d->d_k);
  if constexpr (sizeof(T) == 4)
    if (d->d_k == 64) return launch_attn<T, S, 1>(d, a, st);
  return launch_attn<T, S, 2>(d, a, st);
}
}  // namespace

int run_f32_attn(const lisa_desc* d, const void* q, const void* k, const void* v, const float* given, int row0, int n_rows,
                 void* scores, void* out, hipStream_t st) {
  return d->dtype == LISA_F32 ? run_attn<float, float>(d, q, k, given, row0, n_rows, v, scores, out, st)
                              : run_attn<bf16_t, half_t>(d, q, k, given, row0, n_rows, v, scores, out, st);
}

// bf16: the float32 scores pass through the workspace a chunk of query rows at a time, 256 MB of them (what the
// last-level cache holds), at least one block of 16 rows.
int f32_chunk_rows(const lisa_desc* d) {
  const size_t row = (size_t)d->B * d->H * d->Lk * sizeof(float);
  const size_t rows = std::max<size_t>(16, (((size_t)256 << 20) / row) & ~(size_t)15);
  return (int)std::min<size_t>(rows, (size_t)d->Lq);
}
size_t f32_chunk_bytes(const lisa_desc* d) {
  return round_up((size_t)d->B * d->H * f32_chunk_rows(d) * d->Lk * sizeof(float), 256);
}

namespace {
int scores_heads(int H) { return H <= 8 ? 8 : H <= 16 ? 16 : H <= 32 ? 32 : 40; }
int scores_lds(const lisa_desc* d) { return f32_scores_lds(scores_heads(d->H), d->F, d->mix == LISA_MIX_CONCAT); }
}  // namespace

bool f32_scores_ok(const lisa_desc* d) {
  if (d->Lq == 1 || (d->act != LISA_ACT_RELU && d->act != LISA_ACT_SILU)) return false;
  if (d->dtype == LISA_F32) return d->mix == LISA_MIX_ADD && d->H <= 32 && scores_lds(d) <= 64 * 1024;
  return bf16_ragged_rows(d) && (d->mix == LISA_MIX_ADD || d->mix == LISA_MIX_CONCAT) && d->H <= 40 &&
         scores_lds(d) <= 160 * 1024;
}

namespace {
template <typename T, typename S, int HT, bool CONCAT>
int launch_scores_t(const lisa_desc* d, const F32ScoresArgs<T, S>& a, dim3 grid, hipStream_t st) {
  const int lds = f32_scores_lds(HT, d->F, CONCAT);
  auto kern = d->act == LISA_ACT_SILU ? k_f32_lisa_scores<T, S, HT, 1, CONCAT> : k_f32_lisa_scores<T, S, HT, 0, CONCAT>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return hip_fail(e);
  }
  StageScope prof("k_f32_lisa_scores", st);
  kern<<<grid, 256, lds, st>>>(a);
  return check_launch();
}

template <typename T, typename S, bool CONCAT>
int run_scores(const lisa_desc* d, const void* q_lr, const void* k_lr, const void* prev, const void* w1,
               const void* w2, void* scores, float* exact, int row0, int n_rows, hipStream_t st) {
  F32ScoresArgs<T, S> a{};
  a.q_lr = (const T*)q_lr; a.k_lr = (const T*)k_lr; a.prev = (const S*)prev;
  a.w1 = (const T*)w1; a.w2 = (const T*)w2; a.scores = (S*)scores; a.exact = exact;
  a.H = d->H; a.Hkv = d->Hkv; a.Lq = d->Lq; a.Lk = d->Lk; a.r = d->r; a.F = d->F; a.causal = d->causal;
  a.row0 = row0; a.n_rows = n_rows;
  a.dscale = pick_scale(d->delta_scale, d->r);
  // a tile per workgroup until there are several workgroups per compute unit (16; bf16, whose larger weights are
  // converted as they are staged: 6), then runs of tiles that share the staged weights
  const int kt = (d->Lk + 15) / 16, rbs = (n_rows + 15) / 16;
  const int wgs = (sizeof(T) == 4 ? 16 : 6) * kComputeUnits;
  a.tiles = (int)std::min<long long>(16, std::max<long long>(1, (long long)kt * rbs * d->B / wgs));
  dim3 grid((kt + a.tiles - 1) / a.tiles, rbs, d->B);
  switch (scores_heads(d->H)) {
    case 8: return launch_scores_t<T, S, 8, CONCAT>(d, a, grid, st);
    case 16: return launch_scores_t<T, S, 16, CONCAT>(d, a, grid, st);
    case 32: return launch_scores_t<T, S, 32, CONCAT>(d, a, grid, st);
    default:
      if constexpr (sizeof(T) == 2) return launch_scores_t<T, S, 40, CONCAT>(d, a, grid, st);
      return LISA_ERR_UNSUPPORTED;                           // (f32_scores_ok)
  }
}
}  // namespace

int run_f32_scores(const lisa_desc* d, const void* q_lr, const void* k_lr, const void* prev, const void* w1,
                   const void* w2, void* scores, float* exact, int row0, int n_rows, hipStream_t st) {
  auto* run = d->dtype == LISA_F32           ? run_scores<float, float, false>
              : d->mix == LISA_MIX_CONCAT ? run_scores<bf16_t, half_t, true>
                                          : run_scores<bf16_t, half_t, false>;
  return run(d, q_lr, k_lr, prev, w1, w2, scores, exact, row0, n_rows, st);
}

}  // namespace lisa
