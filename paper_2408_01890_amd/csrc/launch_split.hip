// Prefill layers of bf16 operands in float32 arithmetic on the kernels of kernels_split.h: which shapes they take, and the
// launches.
#include "host.h"
#include "kernels_split.h"

namespace lisa {

// Row-major score rows of a length that the bf16 and half kernels do not take.
bool bf16_ragged_rows(const lisa_desc* d) {
  return d->dtype == LISA_BF16 && d->d_k == 128 && !score_rows_aligned(d);
}

// 32-bit offsets inside two heads of a score tensor; eight elements of a row to read at least.
static bool split_sizes_ok(const lisa_desc* d) {
  return d->Lk >= 8 && (long long)(d->Lq + 16) * (d->Lk + PF_TK) < (1LL << 30);
}

bool split_attn_ok(const lisa_desc* d) { return bf16_ragged_rows(d) && d->Lq > 1; }

namespace {
int split_heads(int H) { return H <= 8 ? 8 : H <= 16 ? 16 : H <= 32 ? 32 : 40; }
template <int HT, bool CONCAT>
int keys_of(int F) {                                         // 16-key blocks per tile, 0: does not fit the LDS
  return SplitScoresGeo<HT, CONCAT, 2>::lds(F) <= 160 * 1024   ? 2
         : SplitScoresGeo<HT, CONCAT, 1>::lds(F) <= 160 * 1024 ? 1
                                                               : 0;
}
int split_keys(const lisa_desc* d) {
  const bool cc = d->mix == LISA_MIX_CONCAT;
  switch (split_heads(d->H)) {
    case 8: return cc ? keys_of<8, true>(d->F) : keys_of<8, false>(d->F);
    case 16: return cc ? keys_of<16, true>(d->F) : keys_of<16, false>(d->F);
    case 32: return cc ? keys_of<32, true>(d->F) : keys_of<32, false>(d->F);
    // (40 heads, CONCAT: the operands of two 16-key blocks do not fit the register file)
    default: return cc ? std::min(1, keys_of<40, true>(d->F)) : keys_of<40, false>(d->F);
  }
}
}  // namespace

// The float32 scores pass through the workspace in tiles, a chunk of query rows at a time: 256 MB (what the last-level cache
// holds) with the padded operands behind them, at least one block of 16 rows.  Operands that would take more than half of that
// (B H L around 1 M) leave the chunks too few rows: those calls keep the float32 kernel, which reads the operands as they are.
// Both sides, split / float32 kernel in ms: 32 heads, 28 x 1025 tokens (112 MB of operands) 3.57 / 5.17, 33 x 1025 (132 MB, chunks
// of 16 rows) 5.66 / 6.48, 40 x 1025 6.56 / 7.90; 8 KV heads, 48 x 1025 (120 MB) 6.36 / 8.64, 64 x 1025 (160 MB) 7.85 / 13.7; short
// rows lose beyond the line, 32 heads, 700 x 33 (153 MB) 0.67 / 0.56, 8 heads, 3000 x 33 (164 MB) 0.75 / 0.58, 16 heads,
// 650 x 129 (213 MB) 1.50 / 1.38.  (Long ones would still gain 13 - 43 % there.)
namespace {
constexpr size_t kSplitBudget = (size_t)256 << 20;
size_t split_row_bytes(const lisa_desc* d) {
  return (size_t)d->B * d->H * ((d->Lk + PF_TK - 1) / PF_TK * PF_TK) * sizeof(float);
}
struct SplitWs {
  size_t qp, kp, total;
  int Lqp, Lkp;
};
SplitWs split_ws(const lisa_desc* d, size_t rows) {
  SplitWs w;
  w.Lqp = (d->Lq + PF_ROWS - 1) / PF_ROWS * PF_ROWS;
  w.Lkp = (d->Lk + 63) / 64 * 64;
  w.qp = rows * split_row_bytes(d);
  w.kp = w.qp + round_up((size_t)d->B * d->H * w.Lqp * 32 * 2, 256);
  w.total = w.kp + round_up((size_t)d->B * d->Hkv * w.Lkp * 32 * 2, 256);
  return w;
}
SplitWs split_ws(const lisa_desc* d) { return split_ws(d, (size_t)(split_chunk_rows(d) + 15) / 16 * 16); }
}  // namespace

// Scores of few or short rows, which the float32 kernel makes sooner: it needs no launch that pads the operands (3 us), its
// tiles of 16 x 16 are half as large, and several workgroups share a compute unit.  What it does per tile costs more, about
// in proportion to heads x hidden units.  Both sides in us, split / float32 kernel, ADD unless said:
//   a tile per compute unit at most: 8 heads, 129 tokens, F = 32, 16.5 / 13.3, CONCAT, F = 48, 20.8 / 14.5; 16 heads 17.5 / 15;
//   32 heads, CONCAT, F = 16, 23.8 / 20.5, but F = 64 beyond the line 23.6 / 24.5; 8 heads, 401 tokens, F = 128, 27.2 / 30.5;
//   rows of one 16-key tile: 1000 x 9 tokens, 8 heads, F = 32, 83 / 51 (softmax included, which is the float32 kernel's then);
//   32 heads, F = 96, 280 / 187, one sequence of 9, F = 64, 18.3 / 20; CONCAT, F = 256, 133 / 168 (300 x 9);
//   rows up to 64 keys: 8 heads, 100 x 33, F = 32, 35.5 / 29.7, 16 heads, F = 96, 57.4 / 61.4; 8 heads, 300 x 65, F = 32, 117 / 154;
//   9 rows of 33 keys, CONCAT, F = 32: 12 heads, 1000 sequences, 160 / 133, 32 heads, 300, 118 / 100, 100, 58 / 59;
//   a second round of a few tiles: 16 heads, 30 x 65, CONCAT, F = 48, 44.5 / 33.6; 100 x 65 59 / 62;
//   chunks of one block of rows, which the operands leave room for: 32 heads, 1000 x 33, F = 32, 904 / 724; 300 x 33 209 / 215.
static bool f32_scores_win(const lisa_desc* d) {
  const bool concat = d->mix == LISA_MIX_CONCAT;
  const int heads = split_heads(d->H), work = heads * d->F;
  if (!f32_scores_ok(d)) return false;
  if (d->Lk <= 16) return heads <= 16 || work <= 1024 || (d->B >= 16 && d->F <= (heads > 32 ? 64 : concat ? 128 : 256));
  const long long rbs = (d->Lq + 15) / 16;
  if (d->B * rbs * ((d->Lk + 15) / 16) <= kComputeUnits) return heads <= 16 ? work <= 4096 : heads == 32 && work <= 512;
  if (d->Lk > 128) return false;
  if (d->Lk <= 64 && work <= 2560 && split_chunk_rows(d) < std::min(d->Lq, 32)) return true;
  if (heads > 32) return false;
  long long t32 = d->causal ? 0 : rbs * ((d->Lk + 31) / 32);  // tiles of 32 keys
  if (d->causal)
    for (int i = 0; i < d->Lq; i += 16) t32 += split_scores_tiles(i, d->Lq, d->Lq, d->Lk, 1, 32);
  t32 *= d->B;
  if (t32 > kComputeUnits && t32 <= kComputeUnits * 19 / 16) return work <= (heads <= 16 ? 4096 : 1024);
  if (heads == 8) return (d->Lk <= 64 || (rbs == 1 && (concat || t32 <= 3 * kComputeUnits))) && (d->F <= 64 || (d->F <= 128 && t32 <= 3 * kComputeUnits));
  return rbs == 1 && d->Lk <= 48 && d->F <= 64 && (heads == 16 || t32 > kComputeUnits);
}

bool split_scores_ok(const lisa_desc* d) {
  if (!split_attn_ok(d) || !split_sizes_ok(d) || (d->act != LISA_ACT_RELU && d->act != LISA_ACT_SILU)) return false;
  if (d->mix != LISA_MIX_ADD && d->mix != LISA_MIX_CONCAT) return false;
  if (d->H > 40 || d->r > 32) return false;
  if (split_ws(d, 0).total > kSplitBudget / 2 || split_ws(d, 16).total > kSplitBudget) return false;
  return split_keys(d) > 0 && !f32_scores_win(d);
}

int split_chunk_rows(const lisa_desc* d) {
  const size_t rows = std::max<size_t>(16, ((kSplitBudget - split_ws(d, 0).total) / split_row_bytes(d)) & ~(size_t)15);
  return (int)std::min<size_t>(rows, (size_t)d->Lq);
}
namespace {
// The weights as k_split_scores has them, behind the padded operands (and outside the budget: it decides the rows of a chunk).
FfnImage split_image(const lisa_desc* d, const void* w1, const void* w2) {
  const int HT = split_heads(d->H), KSA = (HT + 31) / 32;
  const bool cc = d->mix == LISA_MIX_CONCAT;
  return FfnImage{(const bf16_t*)w1, (const bf16_t*)w2, nullptr, cc ? 2 * d->H : d->H, d->F, d->H, cc ? 2 * KSA : KSA,
                  (d->F + 31) / 32, (HT + 15) / 16, 1, d->H, KSA};
}
}  // namespace
size_t split_bytes(const lisa_desc* d) { return split_ws(d).total + split_image(d, nullptr, nullptr).bytes(); }

namespace {
long long tiles_of(const lisa_desc* d, const SplitScoresArgs& a, int tk) {
  long long n = 0;
  for (int i = a.row0; i < a.row0 + a.n_rows; i += 16)
    n += split_scores_tiles(i, a.row0 + a.n_rows, d->Lq, d->Lk, d->causal, tk);
  return n;
}
// Tiles of 16 keys in place of 32: a workgroup is done with one in 0.6 - 0.9 of the time, which pays where there are no more than
// one and a half times as many rounds of them, in one or two rounds (beyond, wider rows of the tensors count).  32 and 40 heads, 32 /
// 16 keys in us: CONCAT, 64 -> 256 -> 32, 150 tokens 27.6 / 18.2, 333 30.9 / 23.1, 2 x 345 (2 / 3 rounds) 51.4 / 37.8; ADD, 32 heads,
// 250 tokens 16.1 / 13.7, 40 heads 20.3 / 17.0, 3 x 182 rows of 371 keys (2 / 3) 44.3 / 41.3; on the other side (1 / 2) CONCAT, 421
// tokens 33.0 / 35.1, ADD, 40 heads, 2 x 130 rows of 430 keys 25.1 / 30.4.
bool small_tiles_win(const lisa_desc* d, const SplitScoresArgs& a) {
  auto rounds = [&](int tk) { return (tiles_of(d, a, tk) * a.B + kComputeUnits - 1) / kComputeUnits; };
  const long long r = rounds(32);
  return d->H > 16 && r <= 2 && 2 * rounds(16) <= 3 * r;
}
template <int HT, bool CONCAT, int TKB>
int launch_scores_t(const lisa_desc* d, SplitScoresArgs& a, hipStream_t st) {
  typedef SplitScoresGeo<HT, CONCAT, TKB> Geo;
  const int lds = Geo::lds(d->F);
  auto kern = d->act == LISA_ACT_SILU ? k_split_scores<HT, 1, CONCAT, TKB> : k_split_scores<HT, 0, CONCAT, TKB>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return hip_fail(e);
  a.tiles_b = tiles_of(d, a, Geo::TK);
  const long long wgs = std::min<long long>(kComputeUnits, a.tiles_b * a.B);
  StageScope prof("k_split_scores", st);
  kern<<<(unsigned)wgs, 512, lds, st>>>(a);
  return check_launch();
}
template <int HT>
int launch_scores_h(const lisa_desc* d, SplitScoresArgs& a, hipStream_t st) {
  const int kb = split_keys(d) == 2 && small_tiles_win(d, a) ? 1 : split_keys(d);
  if (d->mix == LISA_MIX_CONCAT) {
    if constexpr (HT < 40)
      if (kb == 2) return launch_scores_t<HT, true, 2>(d, a, st);
    return launch_scores_t<HT, true, 1>(d, a, st);
  }
  return kb == 2 ? launch_scores_t<HT, false, 2>(d, a, st) : launch_scores_t<HT, false, 1>(d, a, st);
}
}  // namespace

// Q_LR, K_LR and the weights into the workspace as the scores kernel reads them.
int run_split_prepare(const lisa_desc* d, const void* q_lr, const void* k_lr, const void* w1, const void* w2, void* workspace,
                      hipStream_t st) {
  const SplitWs w = split_ws(d);
  char* ws = (char*)workspace;
  const size_t rows = (size_t)d->B * d->H * w.Lqp + (size_t)d->B * d->Hkv * w.Lkp;
  FfnImage img = split_image(d, w1, w2);
  img.out = (unsigned short*)(ws + w.total);
  StageScope prof("k_prepare_prefill", st);
  k_prepare_prefill<true><<<(unsigned)((rows + 63) / 64 + (img.pieces() + 255) / 256), 256, 0, st>>>(
      (const bf16_t*)q_lr, (const bf16_t*)k_lr, nullptr, (bf16_t*)(ws + w.qp), (bf16_t*)(ws + w.kp), nullptr, d->B, d->H, d->Hkv,
      d->Lq, d->Lk, w.Lqp, w.Lkp, d->r, 0, img);
  return check_launch();
}

int run_split_scores(const lisa_desc* d, const void* prev, void* scores, void* workspace, int row0, int n_rows, hipStream_t st) {
  const SplitWs w = split_ws(d);
  SplitScoresArgs a{};
  a.qp = (const bf16_t*)((char*)workspace + w.qp); a.kp = (const bf16_t*)((char*)workspace + w.kp);
  a.exact = (float*)workspace; a.Lqp = w.Lqp; a.Lkp = w.Lkp;
  a.prev = (const half_t*)prev; a.scores = (half_t*)scores;
  a.w = (const unsigned short*)((char*)workspace + w.total);
  a.B = d->B; a.H = d->H; a.Hkv = d->Hkv; a.Lq = d->Lq; a.Lk = d->Lk; a.F = d->F; a.causal = d->causal;
  a.row0 = row0; a.n_rows = n_rows;
  a.dscale = pick_scale(d->delta_scale, d->r);
  switch (split_heads(d->H)) {
    case 8: return launch_scores_h<8>(d, a, st);
    case 16: return launch_scores_h<16>(d, a, st);
    case 32: return launch_scores_h<32>(d, a, st);
    default: return launch_scores_h<40>(d, a, st);
  }
}

// A launch of one block of 16 rows that see few keys leaves most of k_split_attn's four waves and half of their 32 rows
// without work, and its 70 KB of LDS two workgroups per compute unit; the float32 kernel's are half as large.  Both sides,
// 1000 sequences of 32 heads, split / float32 kernel: scores given, 9 tokens 229 / 154 us, 15 rows of 31 keys 309 / 283, of 33
// 320 / 286, 9 rows of 65 331 / 325; scores made, 9 tokens 286 / 213, 16 rows of 31 keys 341 / 322, 9 rows of 65 331 / 448,
// and with 2000 workgroups in place of 32000 23 / 27; scores alone, 9 tokens 85 / 72, 16 rows of 17 keys 97 / 115.
static bool f32_attn_takes(const lisa_desc* d, bool given, bool given_tiled, int row0, int n_rows, bool with_v) {
  const int last = row0 + n_rows - 1, keys = d->causal ? std::min(d->Lk, last + 1 + d->Lk - d->Lq) : d->Lk;
  if (n_rows > 16 || given_tiled) return false;
  return keys <= (given ? 48 : with_v && (long long)d->B * d->H >= 16384 ? 32 : 16);
}

// The order of k_split_attn's workgroups: 1 = row groups of all sequences by length, 0 = sequence by sequence.
// By length where all workgroups run at once (two per compute unit, whose pair is then a long and a short one), where rows are
// short, and where one and a half to two rounds of them come from three sequences or more.  Between these the first round's
// shortest groups end together and the second round starts with all that is left; beyond them an XCD's L2 would hold the K and V of all
// sequences at a time, not of one.  And only where a prompt's row groups differ in length: rows behind as many keys or more are
// about equally long (softmax of 2 x 509 rows behind 1022 keys 69.6 us, by length 70.9).
// Standard layer, sequence by sequence / by length in us: 2 x 201 tokens of 32 heads (448 workgroups) 13.3 / 10.9, 4 x 333 of 8 (352)
// 15.2 / 12.6, 2 x 265 of 32 (576) 15.2 / 17.0, 2 x 301 of 32 (640) 19.0 / 21.0; short rows, 8 x 65 of 32 (768) 15.3 / 12.6, 4 x 99 of 40 (640)
// 14.4 / 12.3; 4 x 777 of 8 (800) 33.7 / 30.1, 16 x 201 of 8 (896) 20.9 / 18.8, 5 x 227 of 24 (960) 23 / 21; 3 x 301 of 40 (1200) 26 / 28,
// 16 x 129 rows of 229 keys, 32 heads (2560) 54.6 / 62.4, 8 x 777 of 40 (8000) 257 / 322, 32 x 777 of 40 1000 / 1705.
int split_attn_order(const lisa_desc* d, int n_rows, int parts) {
  const long long groups = (n_rows + SP_ROWS - 1) / SP_ROWS, wgs = groups * parts * d->H * d->B;
  if (d->Lk - d->Lq >= d->Lq) return 0;
  if (wgs <= 2 * kComputeUnits || (groups <= 4 && wgs <= 5 * kComputeUnits)) return 1;
  return groups >= 6 && d->B >= 3 && wgs >= 3 * kComputeUnits && wgs <= 4 * kComputeUnits;
}

int run_split_attn(const lisa_desc* d, const void* q, const void* k, const void* v, const float* given, bool given_tiled,
                   int row0, int n_rows, void* scores, void* out, hipStream_t st) {
  if (f32_attn_takes(d, given, given_tiled, row0, n_rows, out)) return run_f32_attn(d, q, k, v, given, row0, n_rows, scores, out, st);
  SplitAttnArgs a{};
  a.q = (const bf16_t*)q; a.k = (const bf16_t*)k; a.v = (const bf16_t*)v; a.given = given;
  a.scores = (half_t*)scores; a.out = out;
  a.H = d->H; a.Hkv = d->Hkv; a.Lq = d->Lq; a.Lk = d->Lk; a.causal = d->causal; a.out_f32 = d->out_f32;
  a.row0 = row0; a.n_rows = n_rows; a.given_tiled = given_tiled;
  a.scale = pick_scale(d->std_scale, d->d_k);
  const int groups = (n_rows + SP_ROWS - 1) / SP_ROWS;
  // scores only: few row groups of many keys are spread until there is a workgroup per compute unit, two tiles per wave
  // at least
  a.parts = out ? 1 : (int)std::max<long long>(1, std::min<long long>((d->Lk + 8 * SP_TK - 1) / (8 * SP_TK),
                                                                      kComputeUnits / ((long long)groups * d->H * d->B)));
  a.by_length = split_attn_order(d, n_rows, a.parts);
  const dim3 grid = a.by_length ? dim3(d->H, d->B, groups * a.parts) : dim3(d->H, groups * a.parts, d->B);
  StageScope prof(given ? "k_split_softmax_v" : "k_split_attn", st);
  if (given) k_split_attn<true, true><<<grid, 256, 0, st>>>(a);
  else if (out) k_split_attn<true, false><<<grid, 256, 0, st>>>(a);
  else k_split_attn<false, false><<<grid, 256, 0, st>>>(a);
  return check_launch();
}

}  // namespace lisa
