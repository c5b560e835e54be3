// Decode stacks by data flow, and single layers on the same kernels (kernels_stack.h): which calls take that
// way, their workspace, their launches.
#include "host.h"
#include "kernels_stack.h"

namespace lisa {

namespace {

// Query heads per wave of k_stack_pv, and its form: four waves that stream, or sixteen with everything in flight
// where `layers` of them are fewer workgroups than compute units.
int pv_heads(const lisa_desc* d) {
  const int group = d->H / d->Hkv;
  return group % 4 == 0 ? 4 : group % 2 == 0 ? 2 : 1;
}
int pv_spans(const lisa_desc* d) { return (d->Lk + stack_pv_keys(d->d_k) - 1) / stack_pv_keys(d->d_k); }
int pv_batches(const lisa_desc* d, int layers) {
  return (long long)layers * d->B * (d->H / pv_heads(d)) * pv_spans(d) >= kComputeUnits ? 4 : 1;
}

constexpr size_t kStackGroupBytes = (size_t)128 << 20;

struct GroupWs {
  size_t s, part_o, part_ml, done, w, total;   // byte offsets
  int layers, w_elems, n_span, Lp;
};

GroupWs group_ws(const lisa_desc* d) {
  GroupWs g;
  const int hb = (d->H + 15) / 16, ks = (hb + 1) / 2, fs = (d->F + 31) / 32;
  g.Lp = (d->Lk + 15) / 16 * 16;
  g.n_span = pv_spans(d);
  g.w_elems = (2 * fs * ks + hb * fs) * 512;
  const size_t s1 = (size_t)d->B * 16 * hb * g.Lp * sizeof(float);
  const size_t units = (size_t)d->B * g.n_span * d->H;
  const size_t o1 = units * d->d_k * sizeof(float), ml1 = units * 2 * sizeof(float), w1 = (size_t)g.w_elems * 2;
  // Layers per group: the whole stack while its scratch stays small, else as many as 128 MB hold, so
  // that what one launch leaves for the next stays in the last-level cache; four at least.
  g.layers = (int)std::min<size_t>(STK_MAXL, std::max<size_t>(4, kStackGroupBytes / (s1 + o1 + ml1 + w1)));
  g.s = 0;
  g.part_o = round_up(g.s + g.layers * s1, 256);
  g.part_ml = round_up(g.part_o + g.layers * o1, 256);
  g.done = round_up(g.part_ml + g.layers * ml1, 256);
  g.w = round_up(g.done + (size_t)g.layers * d->B * d->H * sizeof(unsigned), 256);
  g.total = round_up(g.w + g.layers * w1, 256);
  return g;
}

template <int HB, int ACT>
int launch_chain_act(const StackChainArgs& a, hipStream_t st) {
  dim3 grid((a.d.Lk + STK_PB - 1) / STK_PB, a.d.B, a.n_seg);
  switch ((a.d.F + 31) / 32) {
    case 1: k_stack_chain<HB, 1, ACT><<<grid, 64, 0, st>>>(a); break;
    case 2: k_stack_chain<HB, 2, ACT><<<grid, 64, 0, st>>>(a); break;
    case 3: k_stack_chain<HB, 3, ACT><<<grid, 64, 0, st>>>(a); break;
    default: k_stack_chain<HB, 4, ACT><<<grid, 64, 0, st>>>(a); break;
  }
  return check_launch();
}
template <int HB>
int launch_chain_hb(const StackChainArgs& a, int act, hipStream_t st) {
  return act == LISA_ACT_SILU ? launch_chain_act<HB, 1>(a, st) : launch_chain_act<HB, 0>(a, st);
}
int launch_chain(const StackChainArgs& a, int act, hipStream_t st) {
  StageScope prof("k_stack_chain", st);
  switch ((a.d.H + 15) / 16) {
    case 1: return launch_chain_hb<1>(a, act, st);
    case 2: return launch_chain_hb<2>(a, act, st);
    case 3: return launch_chain_hb<3>(a, act, st);
    default: return launch_chain_hb<4>(a, act, st);
  }
}

template <int DK, int NB>
int launch_pv_nb(const StackPvArgs& a, int gq, dim3 grid, hipStream_t st) {
  StageScope prof("k_stack_pv", st);
  if (gq == 4) k_stack_pv<DK, 4, NB><<<grid, 1024 / NB, 0, st>>>(a);
  else if (gq == 2) k_stack_pv<DK, 2, NB><<<grid, 1024 / NB, 0, st>>>(a);
  else k_stack_pv<DK, 1, NB><<<grid, 1024 / NB, 0, st>>>(a);
  return check_launch();
}
int launch_pv(const lisa_desc* d, StackPvArgs& a, int n_layers, hipStream_t st) {
  const int gq = pv_heads(d), nb = pv_batches(d, n_layers);
  const dim3 grid(a.d.n_span * (d->H / d->Hkv / gq), d->Hkv * d->B, n_layers);
  if (d->d_k == 128) return nb == 4 ? launch_pv_nb<128, 4>(a, gq, grid, st) : launch_pv_nb<128, 1>(a, gq, grid, st);
  return nb == 4 ? launch_pv_nb<64, 4>(a, gq, grid, st) : launch_pv_nb<64, 1>(a, gq, grid, st);
}

// For launches of k_stack_pv without counters (see the rule in run_stack_chained).
int launch_stack_combine(const lisa_desc* d, const StackCombineArgs& a, int n_layers, hipStream_t st) {
  dim3 grid(d->H, d->B, n_layers);
  StageScope prof("k_stack_combine", st);
  if (d->d_k == 128) {
    if (d->out_f32) k_stack_combine<float, 128><<<grid, 256, 0, st>>>(a);
    else k_stack_combine<bf16_t, 128><<<grid, 256, 0, st>>>(a);
  } else {
    if (d->out_f32) k_stack_combine<float, 64><<<grid, 256, 0, st>>>(a);
    else k_stack_combine<bf16_t, 64><<<grid, 256, 0, st>>>(a);
  }
  return check_launch();
}

KeyStrides cache_strides(const lisa_desc* d, int width, int cap) {
  KeyStrides s;
  s.t = 1; s.j = width; s.h = (long long)cap * width; s.b = s.h * d->Hkv;
  return s;
}
KeyStrides klr_strides(const lisa_desc* d) {
  KeyStrides s = cache_strides(d, d->r, d->Lmax);
  if (d->kcache_dim_major) s.j = 1, s.t = d->Lmax;
  return s;
}

template <int HBI, int FS, int HBO, bool CONCAT>
int launch_decode_scores_t(const lisa_desc* d, const DecodeScoresArgs& a, hipStream_t st) {
  typedef MfmaFfn<HBI, FS, HBO> Ffn;
  const int lds = decode_scores_lds(d->H, d->r, Ffn::kStageBytes);
  auto kern = d->act == LISA_ACT_SILU ? k_decode_scores<HBI, FS, HBO, 1, CONCAT> : k_decode_scores<HBI, FS, HBO, 0, CONCAT>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return hip_fail(e);
  }
  StageScope prof("k_decode_scores", st);
  kern<<<dim3((d->Lk + DS_KEYS - 1) / DS_KEYS, d->B), 256, lds, st>>>(a);
  return check_launch();
}
template <int HBI, int HBO>
int launch_decode_concat(const lisa_desc* d, const DecodeScoresArgs& a, hipStream_t st) {
  if (d->F <= 64) return launch_decode_scores_t<HBI, 2, HBO, true>(d, a, st);
  if (d->F <= 128) return launch_decode_scores_t<HBI, 4, HBO, true>(d, a, st);
  return launch_decode_scores_t<HBI, 8, HBO, true>(d, a, st);
}
template <int HB>
int launch_decode_add(const lisa_desc* d, const DecodeScoresArgs& a, hipStream_t st) {
  switch ((d->F + 31) / 32) {
    case 1: return launch_decode_scores_t<HB, 1, HB, false>(d, a, st);
    case 2: return launch_decode_scores_t<HB, 2, HB, false>(d, a, st);
    case 3: return launch_decode_scores_t<HB, 3, HB, false>(d, a, st);
    default: return launch_decode_scores_t<HB, 4, HB, false>(d, a, st);
  }
}
int launch_decode_scores(const lisa_desc* d, const DecodeScoresArgs& a, hipStream_t st) {
  if (d->mix == LISA_MIX_CONCAT)
    return d->H <= 16 ? launch_decode_concat<2, 1>(d, a, st) : d->H <= 32 ? launch_decode_concat<4, 2>(d, a, st)
                                                                          : launch_decode_concat<6, 3>(d, a, st);
  switch ((d->H + 15) / 16) {
    case 1: return launch_decode_add<1>(d, a, st);
    case 2: return launch_decode_add<2>(d, a, st);
    case 3: return launch_decode_add<3>(d, a, st);
    default: return launch_decode_add<4>(d, a, st);
  }
}

// Shape of the module's weights in operand order (the instantiation launch_decode_scores picks).
FfnOperands operand_shape(const lisa_desc* d) {
  FfnOperands w{};
  const bool concat = d->mix == LISA_MIX_CONCAT;
  w.Din = concat ? 2 * d->H : d->H;
  w.F = d->F;
  w.HO = d->H;
  w.HBO = concat ? (d->H <= 16 ? 1 : d->H <= 32 ? 2 : 3) : (d->H + 15) / 16;
  w.KS = concat ? w.HBO : (w.HBO + 1) / 2;
  w.FS = !concat ? (d->F + 31) / 32 : d->F <= 64 ? 2 : d->F <= 128 ? 4 : 8;
  return w;
}

struct SingleWs {
  size_t s, part_o, part_ml, done, w, total;
  int n_span, Lp;
};
SingleWs single_ws(const lisa_desc* d) {
  SingleWs w;
  w.Lp = (d->Lk + 15) / 16 * 16;
  w.n_span = pv_spans(d);
  const size_t units = (size_t)d->B * w.n_span * d->H;
  w.s = 0;
  w.part_o = round_up((size_t)d->B * ((d->H + 15) / 16 * 16) * w.Lp * sizeof(float), 256);
  w.part_ml = round_up(w.part_o + units * d->d_k * sizeof(float), 256);
  w.done = round_up(w.part_ml + units * 2 * sizeof(float), 256);
  w.w = round_up(w.done + (size_t)d->B * d->H * sizeof(unsigned), 256);
  w.total = round_up(w.w + (size_t)operand_shape(d).pieces() * 16, 256);
  return w;
}
StackDims single_dims(const lisa_desc* d, const SingleWs& w, void* workspace) {
  char* ws = (char*)workspace;
  StackDims dims{};
  dims.B = d->B; dims.H = d->H; dims.Hp = (d->H + 15) / 16 * 16; dims.Hkv = d->Hkv; dims.Lk = d->Lk; dims.Lp = w.Lp;
  dims.r = d->r; dims.F = d->F; dims.n_span = w.n_span;
  dims.s = (float*)(ws + w.s);
  dims.part_o = (float*)(ws + w.part_o);
  dims.part_ml = (float*)(ws + w.part_ml);
  dims.done = (unsigned*)(ws + w.done);
  return dims;
}

}  // namespace

// ADD-form modules with the two-layer FFN whose weights the chain can hold; every standard and
// direct-sharing layer of a bf16 stack with d_k = 64 or 128.
bool stack_chained_ok(const lisa_desc* d) {
  if (d->dtype != LISA_BF16 || (d->d_k != 64 && d->d_k != 128) || d->H > 64) return false;
  if (d->mix != LISA_MIX_ADD || (d->act != LISA_ACT_RELU && d->act != LISA_ACT_SILU)) return false;
  if (d->F > 128 || d->r > 64) return false;
  const long long blocks = (long long)d->B * ((d->Lk + STK_CK - 1) / STK_CK) * d->H * STK_MAXL;   // grid limits
  return blocks < (1LL << 31);
}

// Fewer layers per group at a longer context may take less than more of them at a shorter one: from there on
// at least what any group of more than four layers takes, so that a workspace for the longest
// context fits the shorter ones.
size_t stack_chained_bytes(const lisa_desc* d) {
  const GroupWs g = group_ws(d);
  if (g.layers == STK_MAXL) return g.total;
  return std::max(g.total, kStackGroupBytes + (size_t)STK_MAXL * d->B * d->H * sizeof(unsigned) + 5 * 256);
}

// rows: two half rows [B,H,Lk], used in turn where a row passes from one group of layers to the next
int run_stack_chained(const lisa_desc* d, const lisa_stack_layer* layers, int n_layers, void* const rows[2],
                      void* workspace, hipStream_t st) {
  const GroupWs gw = group_ws(d);
  char* ws = (char*)workspace;
  StackDims dims{};
  dims.B = d->B; dims.H = d->H; dims.Hp = (d->H + 15) / 16 * 16; dims.Hkv = d->Hkv; dims.Lk = d->Lk; dims.Lp = gw.Lp; dims.r = d->r; dims.F = d->F;
  dims.n_span = gw.n_span;
  dims.s = (float*)(ws + gw.s);
  dims.part_o = (float*)(ws + gw.part_o);
  dims.part_ml = (float*)(ws + gw.part_ml);
  dims.done = (unsigned*)(ws + gw.done);
  dims.w = (unsigned short*)(ws + gw.w);
  dims.w_elems = gw.w_elems;
  const KeyStrides klr = klr_strides(d);
  const half_t* carried = nullptr;                           // A of the last producing layer of the group before
  int parity = 0;
  for (int n0 = 0; n0 < n_layers; n0 += gw.layers) {
    const int n1 = std::min(n_layers, n0 + gw.layers);
    int last_producer = -1;                                  // its row is wanted by the next group
    if (n1 < n_layers && layers[n1].kind != LISA_LAYER_STD)
      for (int n = n0; n < n1; ++n)
        if (layers[n].kind != LISA_LAYER_SHARE) last_producer = n;
    half_t* carry_out = nullptr;
    if (last_producer >= 0) {
      const lisa_stack_layer& ly = layers[last_producer];
      carry_out = (half_t*)(ly.score_row ? ly.score_row : rows[parity]);
      parity ^= 1;
    }
    auto row_of = [&](int n) { return n == last_producer ? carry_out : (half_t*)layers[n].score_row; };
    StackScoresArgs sa{};
    StackChainArgs ca{};
    StackPvArgs pa{};
    StackCombineArgs ma{};
    sa.d = ca.d = pa.d = ma.d = dims;
    sa.kstd = pa.vs = cache_strides(d, d->d_k, d->Lmax);
    sa.klr = klr;
    sa.std_scale = pick_scale(d->std_scale, d->d_k);
    sa.delta_scale = pick_scale(d->delta_scale, d->r);
    ca.from_row = pa.from_row = carried;
    pa.out_f32 = d->out_f32;
    for (int kind = LISA_LAYER_STD; kind <= LISA_LAYER_LISA; ++kind)
      for (int n = n0; n < n1; ++n) {
        const lisa_stack_layer& ly = layers[n];
        if (ly.kind != kind) continue;
        const int i = sa.n_std + sa.n_lisa;
        sa.slot[i] = (n - n0);
        sa.q[i] = (const bf16_t*)ly.q;
        sa.k[i] = (const bf16_t*)ly.k_cache;
        sa.w1[i] = (const bf16_t*)ly.w1;
        sa.w2[i] = (const bf16_t*)ly.w2;
        ++(kind == LISA_LAYER_STD ? sa.n_std : sa.n_lisa);
      }
    int src = -1, n_chain = 0;                               // slot of the scores the next layer shares
    bool run = false;                                        // a chain segment is open
    for (int n = n0; n < n1; ++n) {
      const lisa_stack_layer& ly = layers[n];
      const int i = n - n0;
      if (ly.kind == LISA_LAYER_STD) {
        src = i;
        run = false;
      } else if (ly.kind == LISA_LAYER_LISA) {
        if (!run) {
          ca.first[ca.n_seg] = n_chain;
          ca.from[ca.n_seg] = src;
          ++ca.n_seg;
          run = true;
        }
        ca.slot[n_chain] = i;
        ++n_chain;
        ++ca.count[ca.n_seg - 1];
        src = i;
      }
      pa.src[i] = src;
      pa.slot[i] = ma.slot[i] = i;
      pa.share[i] = ly.kind == LISA_LAYER_SHARE;
      pa.v[i] = (const bf16_t*)ly.v_cache;
      pa.row[i] = row_of(n);
      pa.out[i] = ma.out[i] = ly.out;
    }
    int rc;
    if (sa.n_std + sa.n_lisa > 0) {
      const bool vec = klr.j == 1 && klr.t % 8 == 0 && klr.h % 8 == 0 && klr.b % 8 == 0;
      const int kpw = vec ? 512 : 64;                        // keys per wave of the a_delta part
      sa.std_blocks = d->B * d->Hkv * ((d->Lk + STK_CK - 1) / STK_CK);
      sa.n_done = (n1 - n0) * d->B * d->H;
      sa.delta_blocks = d->B * ((d->Hkv + 3) / 4) * ((d->Lk + kpw - 1) / kpw);
      sa.w_blocks = (gw.w_elems / 8 + 255) / 256;
      const unsigned grid = sa.n_std * sa.std_blocks + sa.n_lisa * (sa.delta_blocks + sa.w_blocks);
      StageScope prof("k_stack_scores", st);
      if (d->d_k == 128) k_stack_scores<128><<<grid, 256, 0, st>>>(sa);
      else k_stack_scores<64><<<grid, 256, 0, st>>>(sa);
      if ((rc = check_launch())) return rc;
    }
    if (n_chain && (rc = launch_chain(ca, d->act, st))) return rc;
    // Who merges the splits: the last workgroup of an output where there are few (no launch more), a launch of
    // its own behind the long stream, where every workgroup that waits for its stores and the counter
    // keeps the next one's loads out: 16 users at 4096 tokens, 32 layers, 4732 us with the counters, 4394 without
    // (one user at 1023, 2048 workgroups: 83 with them, 81.5 with the launch).  So the line is that of the form of
    // k_stack_pv: fewer workgroups than compute units keep the counters.  A group of direct-sharing layers alone
    // has no launch in front that clears them.
    const bool merge = gw.n_span > 1 && (sa.n_std + sa.n_lisa == 0 || pv_batches(d, n1 - n0) == 4);
    if (merge) pa.d.done = nullptr;
    if ((rc = launch_pv(d, pa, n1 - n0, st))) return rc;
    if (merge && (rc = launch_stack_combine(d, ma, n1 - n0, st))) return rc;
    if (carry_out) carried = carry_out;
    // (a group of direct-sharing layers alone passes on what it was given)
  }
  return LISA_OK;
}

// ---- single layers ------------------------------------------------------------------------------------
// k_decode_part, a workgroup per (sequence, 128 keys) that makes everything of it in one launch, reads V once per
// query head, stages the module's weights in every workgroup and waits for them before its keys; this path needs
// none of that, but passes A_n through memory as float32 between its launches, 8 bytes per head and key.
// Where query heads share a key/value head, for direct sharing and for the CONCAT form it was the faster one at
// every size measured (LLaMA3-8B heads, 16 users, 6000 tokens, ADD 70 against 106 us; CONCAT, LLaMA2-7B, 16 users,
// 4096 tokens 124 against 142).  With a key/value head per query head those 8 bytes count once there are enough
// units of 128 keys to keep k_decode_part at the memory's rate:
//   3/2 per compute unit in standard layers, which stage no weights (LLaMA2-7B heads, 320 units 124 against
//   134 - 142 us, 432 units 165 against 151, 736 units 279 - 290 against 259), and with ADD modules of narrow layers,
//   where a launch more costs as much (32 heads of 64, 320 units 55 - 59 against 58 - 60, 448 units 71 - 77
//   against 68; 8 heads of 128, 448 units 36 against 31);
//   5/2 with ADD modules of wider ones (LLaMA2-7B, 576 units 130 - 138 against 145, 736 units 171 - 181 against 167).
// The scratch has to fit the buffer of lisa_attn_decode_static (about 900 units of 32 heads).
bool decode_spread_fits(const lisa_desc* d) { return single_ws(d).total <= kDecodeSpreadMaxBytes; }
bool decode_spread_ok(const lisa_desc* d, bool lisa_layer) {
  if (!decode_spread_fits(d)) return false;
  if (d->H != d->Hkv || (lisa_layer && d->mix != LISA_MIX_ADD)) return true;
  const long long units = (long long)d->B * ((d->Lk + DEC_CK - 1) / DEC_CK);
  return units < (lisa_layer && d->H * d->d_k >= 3072 ? kComputeUnits * 5 / 2 : kComputeUnits * 3 / 2);
}
size_t decode_spread_bytes(const lisa_desc* d) { return single_ws(d).total; }

// Where the module's weights go in operand order; a launch in front of the step may write them
// (DecodeArgs::w_ready).
FfnOperands decode_spread_operands(const lisa_desc* d, const bf16_t* w1, const bf16_t* w2, void* workspace) {
  FfnOperands w = operand_shape(d);
  w.w1 = w1;
  w.w2 = w2;
  w.out = (unsigned short*)((char*)workspace + single_ws(d).w);
  return w;
}

int run_decode_spread(const lisa_desc* d, bool lisa_layer, const DecodeArgs& da, void* out, void* workspace,
                      hipStream_t st) {
  const SingleWs w = single_ws(d);
  const StackDims dims = single_dims(d, w, workspace);
  const bool share = lisa_layer && d->mix == LISA_MIX_SHARE;
  int rc;
  if (!lisa_layer) {
    StackScoresArgs a{};
    a.d = dims;
    a.kstd = da.ks;
    a.std_scale = pick_scale(d->std_scale, d->d_k);
    a.n_std = 1;
    a.q[0] = da.q;
    a.k[0] = da.kc;
    a.std_blocks = d->B * d->Hkv * ((d->Lk + STK_CK - 1) / STK_CK);
    a.n_done = d->B * d->H;
    StageScope prof("k_stack_scores", st);
    if (d->d_k == 128) k_stack_scores<128><<<a.std_blocks, 256, 0, st>>>(a);
    else k_stack_scores<64><<<a.std_blocks, 256, 0, st>>>(a);
    if ((rc = check_launch())) return rc;
  } else if (!share) {
    DecodeScoresArgs a{};
    a.d = dims;
    a.ks = da.ks;
    a.q = da.q; a.k = da.kc; a.prev = da.prev;
    a.w = (const unsigned short*)((char*)workspace + w.w);
    if (!da.w_ready) {
      const FfnOperands fo = decode_spread_operands(d, da.w1, da.w2, workspace);
      StageScope prof("k_ffn_operands", st);
      k_ffn_operands<<<(fo.pieces() + 255) / 256, 256, 0, st>>>(fo);
      if ((rc = check_launch())) return rc;
    }
    a.scale = pick_scale(d->delta_scale, d->r);
    a.pass_through = da.pass_through;
    a.n_done = d->B * d->H;
    if ((rc = launch_decode_scores(d, a, st))) return rc;
  }
  StackPvArgs pa{};
  pa.d = dims;
  pa.vs = da.vs;
  pa.out_f32 = d->out_f32;
  pa.src[0] = share ? -1 : 0;
  pa.from_row = da.prev;
  pa.v[0] = da.vc;
  pa.row[0] = da.row_out;
  pa.out[0] = out;
  if (share) pa.d.done = nullptr;
  if ((rc = launch_pv(d, pa, 1, st))) return rc;
  if (share && w.n_span > 1) {
    StackCombineArgs ma{};
    ma.d = dims;
    ma.out[0] = out;
    rc = launch_stack_combine(d, ma, 1, st);
  }
  return rc;
}

}  // namespace lisa
