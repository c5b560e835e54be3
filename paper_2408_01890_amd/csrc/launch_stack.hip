// Decode stacks by data flow (kernels_stack.h): which stacks take that way, its workspace, its launches.
#include "host.h"
#include "kernels_stack.h"

namespace lisa {

namespace {

struct GroupWs {
  size_t s, part_o, part_ml, w, total;   // byte offsets
  int layers, w_elems, n_chunk, Lp;
};

GroupWs group_ws(const lisa_desc* d) {
  GroupWs g;
  const int hb = (d->H + 15) / 16, ks = (hb + 1) / 2, fs = (d->F + 31) / 32;
  g.Lp = (d->Lk + 15) / 16 * 16;
  g.n_chunk = (d->Lk + STK_CK - 1) / STK_CK;
  g.w_elems = (2 * fs * ks + hb * fs) * 512;
  const size_t s1 = (size_t)d->B * 16 * hb * g.Lp * sizeof(float);
  const size_t units = (size_t)d->B * g.n_chunk * d->H;
  const size_t o1 = units * d->d_k * sizeof(float), ml1 = units * 2 * sizeof(float), w1 = (size_t)g.w_elems * 2;
  // Layers per group: the whole stack while its scratch stays small, else as many as 128 MB hold, so
  // that what one launch leaves for the next stays in the last-level cache; four at least.
  g.layers = (int)std::min<size_t>(STK_MAXL, std::max<size_t>(4, ((size_t)128 << 20) / (s1 + o1 + ml1 + w1)));
  g.s = 0;
  g.part_o = round_up(g.s + g.layers * s1, 256);
  g.part_ml = round_up(g.part_o + g.layers * o1, 256);
  g.w = round_up(g.part_ml + g.layers * ml1, 256);
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

template <int DK>
int launch_pv(StackPvArgs& a, int n_layers, hipStream_t st) {
  const int group = a.d.H / a.d.Hkv, gq = group % 4 == 0 ? 4 : group % 2 == 0 ? 2 : 1;
  a.blocks = (a.d.B * a.d.Hkv * (group / gq) * a.d.n_chunk + 3) / 4;
  StageScope prof("k_stack_pv", st);
  const unsigned grid = (unsigned)(n_layers * a.blocks);
  if (gq == 4) k_stack_pv<DK, 4><<<grid, 256, 0, st>>>(a);
  else if (gq == 2) k_stack_pv<DK, 2><<<grid, 256, 0, st>>>(a);
  else k_stack_pv<DK, 1><<<grid, 256, 0, st>>>(a);
  return check_launch();
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

size_t stack_chained_bytes(const lisa_desc* d) { return group_ws(d).total; }

// rows: two half rows [B,H,Lk], used in turn where a row passes from one group of layers to the next
int run_stack_chained(const lisa_desc* d, const lisa_stack_layer* layers, int n_layers, void* const rows[2],
                      void* workspace, hipStream_t st) {
  const GroupWs gw = group_ws(d);
  char* ws = (char*)workspace;
  StackDims dims{};
  dims.B = d->B; dims.H = d->H; dims.Hp = (d->H + 15) / 16 * 16; dims.Hkv = d->Hkv; dims.Lk = d->Lk; dims.Lp = gw.Lp; dims.r = d->r; dims.F = d->F;
  dims.n_chunk = gw.n_chunk;
  dims.s = (float*)(ws + gw.s);
  dims.part_o = (float*)(ws + gw.part_o);
  dims.part_ml = (float*)(ws + gw.part_ml);
  dims.w = (unsigned short*)(ws + gw.w);
  dims.w_elems = gw.w_elems;
  auto dense = [&](int width) {
    KeyStrides s;
    s.t = 1; s.j = width; s.h = (long long)d->Lmax * width; s.b = s.h * d->Hkv;
    return s;
  };
  KeyStrides klr = dense(d->r);
  if (d->kcache_dim_major) klr.j = 1, klr.t = d->Lmax;
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
    sa.kstd = pa.vs = dense(d->d_k);
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
      sa.std_blocks = d->B * d->Hkv * gw.n_chunk;
      sa.delta_blocks = d->B * ((d->Hkv + 3) / 4) * ((d->Lk + kpw - 1) / kpw);
      sa.w_blocks = (gw.w_elems / 8 + 255) / 256;
      const unsigned grid = sa.n_std * sa.std_blocks + sa.n_lisa * (sa.delta_blocks + sa.w_blocks);
      StageScope prof("k_stack_scores", st);
      if (d->d_k == 128) k_stack_scores<128><<<grid, 256, 0, st>>>(sa);
      else k_stack_scores<64><<<grid, 256, 0, st>>>(sa);
      if ((rc = check_launch())) return rc;
    }
    if (n_chain && (rc = launch_chain(ca, d->act, st))) return rc;
    if ((rc = d->d_k == 128 ? launch_pv<128>(pa, n1 - n0, st) : launch_pv<64>(pa, n1 - n0, st))) return rc;
    if (gw.n_chunk > 1) {
      dim3 grid(d->H, d->B, n1 - n0);
      StageScope prof("k_stack_combine", st);
      if (d->d_k == 128) {
        if (d->out_f32) k_stack_combine<float, 128><<<grid, 256, 0, st>>>(ma);
        else k_stack_combine<bf16_t, 128><<<grid, 256, 0, st>>>(ma);
      } else {
        if (d->out_f32) k_stack_combine<float, 64><<<grid, 256, 0, st>>>(ma);
        else k_stack_combine<bf16_t, 64><<<grid, 256, 0, st>>>(ma);
      }
      if ((rc = check_launch())) return rc;
    }
    if (carry_out) carried = carry_out;
    // (a group of direct-sharing layers alone passes on what it was given)
  }
  return LISA_OK;
}

}  // namespace lisa
