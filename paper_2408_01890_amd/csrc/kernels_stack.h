// One decode step through a stack of layers (Sec. 5.1 table of layer patterns) in four launches per
// group of layers instead of one or two per layer.
//
// What a layer of the stack waits for is narrow: A_n at a key position is made of A_{n-1} at the same
// position, this layer's q and K_LR at it and the FFN.  No position waits for another one, and nothing
// waits for the softmax or P V of the layer before.  So the stack is cut by data flow, not by layer:
//   k_stack_scores   everything that depends on no other layer, all layers at once: a = q K^T of the
//                    standard layers (Eq. 2) and a_delta = q_lr K_LR^T of the LiSA layers (Eq. 3) as
//                    float32 rows in the workspace, and the FFN weights in MFMA operand order;
//   k_stack_chain    A_n = FFN(A_{n-1}) + a_delta along the layers, a wave per 16 key positions and
//                    run of layers, A_{n-1} carried in registers from layer to layer;
//   k_stack_pv       softmax and P V of all layers at once, split over the keys: the V stream, which is
//                    most of the bytes;
//   k_stack_combine  merges the splits of all layers.
// A layer by itself fills the chip only with hundreds of (sequence, 128 keys) units (k_decode_part); a
// stack has that many times the number of layers.
#pragma once
#include <type_traits>

#include "kernels_decode.h"

namespace lisa {

constexpr int STK_MAXL = 48;       // layers of a group (bounded by the size of the kernel arguments)
constexpr int STK_CK = 128;        // keys per unit of the score and P V kernels
constexpr int STK_PB = 16;         // key positions per wave of the chain
// (per-layer numbers in the kernel arguments are ints: a byte has no scalar load, and a vector load in a
// layer loop is waited for together with everything else in flight)

// Workspace of a group: slot s (a layer) holds float32 scores [B][Hp][Lp], the partial results of its
// splits and (LiSA layers) the FFN weights in operand order.
struct StackDims {
  int B, H, Hp, Hkv, Lk, Lp, r, F, n_chunk;   // Hp, Lp: H, Lk rounded up to 16; n_chunk: splits of STK_CK keys
  float* s;              // [slot][B][Hp][Lp]
  float* part_o;         // [slot][B][n_chunk][H][DK]
  float* part_ml;        // [slot][B][n_chunk][H][2]
  unsigned short* w;     // [slot][w_elems]
  int w_elems;
  __host__ __device__ size_t s_at(int slot, int b, int h) const { return (((size_t)slot * B + b) * Hp + h) * Lp; }
};

struct StackScoresArgs {
  StackDims d;
  KeyStrides kstd, klr;
  float std_scale, delta_scale;
  int n_std, n_lisa;
  int std_blocks, delta_blocks, w_blocks;     // workgroups of one layer in each part
  int slot[STK_MAXL];               // standard layers first, then the LiSA layers
  const bf16_t* q[STK_MAXL];
  const bf16_t* k[STK_MAXL];
  const bf16_t* w1[STK_MAXL];
  const bf16_t* w2[STK_MAXL];
};

// FFN weights of one layer in the operand order of k_stack_chain: operands W1 (fb, ks), then W2 (hb, s),
// 64 lanes x 8 halves each.  Both contractions are numbered by what the product before leaves in the
// lanes (mfma_ffn.h): slot (k-step, g, e) is index 16 (2 kstep + e / 4) + 4 g + e % 4, of the heads
// for W1 as well as of the hidden units for W2, so that the chain never moves data between lanes.
__device__ __forceinline__ int stack_slot_index(int kstep, int g, int e) { return 16 * (2 * kstep + (e >> 2)) + 4 * g + (e & 3); }

template <int HB, int FS>
struct StackFfn {
  static constexpr int KS = (HB + 1) / 2, FB = 2 * FS;
  static constexpr int N1 = FB * KS, N2 = HB * FS, NOP = N1 + N2;
};

// grid n_std std_blocks + n_lisa (delta_blocks + w_blocks), block 256
//   std part    workgroup = 128 keys of one key/value head of one sequence: on the matrix cores with the
//               keys as rows and the query heads of the group as columns (no cross-lane sums); bound
//               by the K stream.
//   delta part  dimension-major K_LR with 16-byte aligned rows: a lane per 8 keys, a wave per key/value
//               head; otherwise a lane per key.
//   weight part 256 operand pieces per workgroup.
template <int DK>
__global__ __launch_bounds__(256) void k_stack_scores(StackScoresArgs a) {
  const StackDims& d = a.d;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = d.H / d.Hkv;
  int blk = blockIdx.x;
  if (blk < a.n_std * a.std_blocks) {
    const int l = blk / a.std_blocks;
    blk -= l * a.std_blocks;
    const int chunk = blk % d.n_chunk, kv = blk / d.n_chunk % d.Hkv, b = blk / (d.n_chunk * d.Hkv);
    constexpr int KS = DK / 32;
    const int c = lane & 15, g = lane >> 4;
    const int j0 = chunk * STK_CK + wv * 32;                 // this wave's 32 keys
    if (j0 >= d.Lk) return;
    const bf16_t* kb = a.k[l] + b * a.kstd.b + kv * a.kstd.h + 8 * g;
    u32x4 kreg[2][KS];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        kreg[u][ks] = ld_stream(kb + (size_t)min(j0 + 16 * u + c, d.Lk - 1) * a.kstd.j + 32 * ks);
    const int slot = a.slot[l];
    for (int hb = 0; hb < group; hb += 16) {                 // columns: the query heads of this kv head
      const int h = kv * group + min(hb + c, group - 1);
      const bf16_t* qp = a.q[l] + ((size_t)b * d.H + h) * DK + 8 * g;
      f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 qo = *(const bf16x8*)(qp + 32 * ks);
#pragma unroll
        for (int u = 0; u < 2; ++u)
          acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kreg[u][ks]), qo, acc[u], 0, 0, 0);
      }
      if (hb + c < group) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int j = j0 + 16 * u + 4 * g;                 // keys j .. j + 3 of head h
          if (j >= d.Lk) continue;
          *(f32x4*)(d.s + d.s_at(slot, b, h) + j) = acc[u] * a.std_scale;   // (Lp is a multiple of 16)
        }
      }
    }
    return;
  }
  blk -= a.n_std * a.std_blocks;
  if (blk < a.n_lisa * a.delta_blocks) {
    __shared__ float q_s[64 * 64];                           // [query heads of the workgroup][r]
    const int li = blk / a.delta_blocks, l = a.n_std + li;
    blk -= li * a.delta_blocks;
    const bool vec = a.klr.j == 1 && (a.klr.t & 7) == 0 && (a.klr.h & 7) == 0 && (a.klr.b & 7) == 0;
    const int kpl = vec ? 8 : 1;                             // keys per lane
    const int nx = (d.Lk + 64 * kpl - 1) / (64 * kpl), ny = (d.Hkv + 3) / 4;
    const int x = blk % nx, y = blk / nx % ny, b = blk / (nx * ny);
    const int h0 = 4 * y * group, nh = min(4 * group, d.H - h0);
    for (int e = tid; e < nh * d.r; e += 256)
      q_s[e] = elem<bf16_t>::load(a.q[l] + ((size_t)b * d.H + h0) * d.r + e);
    __syncthreads();
    const int kv = 4 * y + wv;
    const int j = (x * 64 + lane) * kpl;
    if (kv >= d.Hkv || j >= d.Lk) return;
    const bf16_t* kp = a.k[l] + b * a.klr.b + kv * a.klr.h + (size_t)j * a.klr.j;
    float* sp = d.s + d.s_at(a.slot[l], b, kv * group) + j;
    const float* qw = q_s + wv * group * d.r;
    if (vec) {
      constexpr int GC = 4;                                  // query heads per pass over the K_LR rows
      for (int g0 = 0; g0 < group; g0 += GC) {
        float acc[GC][8] = {};
        auto rows = [&](auto n, int t0) __attribute__((always_inline)) {                    // rows t0 .. t0 + n - 1 of the rank axis
          constexpr int N = decltype(n)::value;
          u32x4 kvv[N];
#pragma unroll
          for (int u = 0; u < N; ++u) kvv[u] = ld_stream(kp + (size_t)(t0 + u) * a.klr.t);
#pragma unroll
          for (int u = 0; u < N; ++u) {
            float kf[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              kf[2 * e] = bf16_bits_to_f32(kvv[u][e] & 0xffffu);
              kf[2 * e + 1] = __uint_as_float(kvv[u][e] & 0xffff0000u);
            }
#pragma unroll
            for (int q = 0; q < GC; ++q) {
              if (g0 + q >= group) break;
              const float qt = qw[(g0 + q) * d.r + t0 + u];
#pragma unroll
              for (int e = 0; e < 8; ++e) acc[q][e] += qt * kf[e];
            }
          }
        };
        int t0 = 0;
        for (; t0 + 8 <= d.r; t0 += 8) rows(std::integral_constant<int, 8>{}, t0);
        if (d.r & 4) rows(std::integral_constant<int, 4>{}, t0), t0 += 4;
        if (d.r & 2) rows(std::integral_constant<int, 2>{}, t0), t0 += 2;
        if (d.r & 1) rows(std::integral_constant<int, 1>{}, t0);
#pragma unroll
        for (int q = 0; q < GC; ++q) {
          if (g0 + q >= group) break;
          float4* dst = (float4*)(sp + (size_t)(g0 + q) * d.Lp);
          dst[0] = make_float4(acc[q][0] * a.delta_scale, acc[q][1] * a.delta_scale, acc[q][2] * a.delta_scale, acc[q][3] * a.delta_scale);
          dst[1] = make_float4(acc[q][4] * a.delta_scale, acc[q][5] * a.delta_scale, acc[q][6] * a.delta_scale, acc[q][7] * a.delta_scale);
        }
      }
    } else {
      for (int q = 0; q < group; ++q) {
        float acc = 0.f;
        for (int t = 0; t < d.r; ++t) acc += qw[q * d.r + t] * elem<bf16_t>::load(kp + (size_t)t * a.klr.t);
        sp[(size_t)q * d.Lp] = acc * a.delta_scale;
      }
    }
    return;
  }
  blk -= a.n_lisa * a.delta_blocks;
  {
    const int li = blk / a.w_blocks, l = a.n_std + li;
    blk -= li * a.w_blocks;
    const int HB = (d.H + 15) / 16, KS = (HB + 1) / 2, FS = (d.F + 31) / 32, N1 = 2 * FS * KS;
    const int idx = blk * 256 + tid, o = idx >> 6;
    if (idx * 8 >= d.w_elems) return;
    const int c = lane & 15, g = lane >> 4;
    const bf16_t *w1 = a.w1[l], *w2 = a.w2[l];
    u16x8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float w = 0.f;
      if (o < N1) {
        const int f = 16 * (o / KS) + c, h = stack_slot_index(o % KS, g, e);
        if (f < d.F && h < d.H) w = elem<bf16_t>::load(w1 + (size_t)h * d.F + f);
      } else {
        const int h = 16 * ((o - N1) / FS) + c, f = stack_slot_index((o - N1) % FS, g, e);
        if (f < d.F && h < d.H) w = elem<bf16_t>::load(w2 + (size_t)f * d.H + h);
      }
      out[e] = half_bits(w);
    }
    *(u16x8*)(d.w + (size_t)a.slot[l] * d.w_elems + (size_t)idx * 8) = out;
  }
}

struct StackChainArgs {
  StackDims d;
  int n_seg;
  int first[STK_MAXL], count[STK_MAXL];   // segment: its LiSA layers (entries of slot)
  int from[STK_MAXL];                       // slot of the layer whose scores it starts from; -1: from_row
  int slot[STK_MAXL];
  const half_t* from_row;                           // A of the layer in front of the group
};

// grid (ceil(Lk / 16), B, n_seg), block 64: one wave = 16 key positions, all heads, a run of LiSA layers.
// Bound: the chain of a layer (two dependent products, the activation, two roundings), a few hundred
// cycles, if the operands are there: those of the next NSET - 1 layers are in flight.
template <int HB, int FS, int ACT>
__global__ __launch_bounds__(64) void k_stack_chain(StackChainArgs a) {
  typedef StackFfn<HB, FS> G;
  constexpr int KS = G::KS;
  constexpr int NSET = G::NOP <= 8 ? 3 : G::NOP <= 24 ? 2 : 1;
  const StackDims& d = a.d;
  const int lane = threadIdx.x, c = lane & 15, g = lane >> 4;
  const int b = blockIdx.y, seg = blockIdx.z;
  const int j = blockIdx.x * STK_PB + c;                     // < Lp
  const int first = a.first[seg], count = a.count[seg];
  // lane (c, g) holds heads 16 hb + 4 g + v of position c
  auto head = [&](int hb, int v) { return min(16 * hb + 4 * g + v, d.H - 1); };
  struct Set {
    f16x8 w[G::NOP];
    f32x4 ad[HB];
  };
  auto load_w = [&](int i, Set& t) __attribute__((always_inline)) {
    const unsigned short* wp = d.w + (size_t)a.slot[first + i] * d.w_elems + lane * 8;
#pragma unroll
    for (int o = 0; o < G::NOP; ++o) t.w[o] = *(const f16x8*)(wp + o * 512);
  };
  auto load_ad = [&](int i, Set& t) __attribute__((always_inline)) {
    const float* sp = d.s + d.s_at(a.slot[first + i], b, 0) + j;
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int v = 0; v < 4; ++v) t.ad[hb][v] = sp[(size_t)head(hb, v) * d.Lp];
  };
  f16x8 x[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) x[ks][e] = (_Float16)0.f;
  if (a.from[seg] >= 0) {
    const float* sp = d.s + d.s_at(a.from[seg], b, 0) + j;
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int v = 0; v < 4; ++v) x[hb >> 1][4 * (hb & 1) + v] = f32_to_half_sat(sp[(size_t)head(hb, v) * d.Lp]);
  } else {
    const half_t* sp = a.from_row + (size_t)b * d.H * d.Lk + min(j, d.Lk - 1);
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int v = 0; v < 4; ++v) x[hb >> 1][4 * (hb & 1) + v] = sp[(size_t)head(hb, v) * d.Lk];
  }
  auto layer = [&](int i, const Set& t) __attribute__((always_inline)) {
    f16x8 hid[FS];
#pragma unroll
    for (int fb = 0; fb < G::FB; ++fb) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(t.w[fb * KS + ks], x[ks], acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) hid[fb >> 1][4 * (fb & 1) + v] = MfmaFfn<HB, FS, HB, ACT>::activate(acc[v]);
    }
    float* sp = d.s + d.s_at(a.slot[first + i], b, 0) + j;
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < FS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(t.w[G::N1 + hb * FS + s], hid[s], acc, 0, 0, 0);
      acc += t.ad[hb];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        x[hb >> 1][4 * (hb & 1) + v] = f32_to_half_sat(acc[v]);
        sp[(size_t)(16 * hb + 4 * g + v) * d.Lp] = acc[v];   // (no branch: the loads in flight stay counted)
      }
    }
  };
  // NSET layers in flight (the weights and a_delta of a layer come from the last-level cache, a
  // microsecond away)
  Set set[NSET];
#pragma unroll
  for (int p = 0; p < NSET; ++p) {
    load_w(min(p, count - 1), set[p]);
    load_ad(min(p, count - 1), set[p]);
  }
  int i0 = 0;
  for (; i0 + NSET <= count; i0 += NSET) {                   // (whole rounds, no way out between: the compiler counts
#pragma unroll                                               //  the loads in flight exactly)
    for (int p = 0; p < NSET; ++p) {
      layer(i0 + p, set[p]);
      load_w(min(i0 + p + NSET, count - 1), set[p]);
      load_ad(min(i0 + p + NSET, count - 1), set[p]);
    }
  }
#pragma unroll
  for (int p = 0; p < NSET - 1; ++p) {
    if (i0 + p >= count) break;
    layer(i0 + p, set[p]);
  }
}

struct StackPvArgs {
  StackDims d;
  KeyStrides vs;
  int blocks;                        // workgroups of one layer
  int out_f32;
  int src[STK_MAXL];         // slot of the scores; -1: from_row
  int slot[STK_MAXL];      // slot of the partial results
  int share[STK_MAXL];     // direct sharing: the scores as the half row would hold them
  const bf16_t* v[STK_MAXL];
  half_t* row[STK_MAXL];             // A_n as half [B][H][Lk], or null
  void* out[STK_MAXL];
  const half_t* from_row;
};

// grid n_layers * blocks, blocks = ceil(B Hkv (group / GQ) n_chunk / 4), block 256: the waves that are in
// flight together read neighbouring pieces of V.
// A wave = 128 keys of one key/value head for GQ of its query heads (one pass over V serves them).  The
// first half of the V loads is in flight while the softmax statistics are made.  Bound: the V stream.
// With one split the wave writes the layer's output itself.
template <int DK, int GQ>
__global__ __launch_bounds__(256, GQ == 1 ? 4 : 3) void k_stack_pv(StackPvArgs a) {
  constexpr int LPK = DK / 8, KPW = 64 / LPK, UN = 8, NB = STK_CK / KPW / UN;   // batches of UN loads
  static_assert(NB % 2 == 0, "batches are taken in pairs");
  constexpr int NIT = STK_CK / KPW;                          // loads of a lane
  __shared__ __align__(16) float p_s[4][GQ][STK_CK];         // [key % KPW][key / KPW]: a lane's keys are consecutive
  const StackDims& d = a.d;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = d.H / d.Hkv, subs = group / GQ;
  const int l = blockIdx.x / a.blocks;
  const int unit = (blockIdx.x - l * a.blocks) * 4 + wv;     // (chunk, sub, key/value head, sequence), chunk fastest
  const int chunk = unit % d.n_chunk, hu = unit / d.n_chunk;
  const int sub = hu % subs, kv = hu / subs % d.Hkv, b = hu / (subs * d.Hkv);
  if (b >= d.B) return;                                      // (no barriers below)
  const int h0 = kv * group + sub * GQ;
  const int j0 = chunk * STK_CK, n_here = min(STK_CK, d.Lk - j0);
  const int js = lane / LPK, dc = lane % LPK;
  const char* vb = (const char*)(a.v[l] + b * a.vs.b + kv * a.vs.h + (size_t)j0 * DK);   // wave-uniform
  const unsigned last = (n_here - 1) * (DK * 2u) + dc * 16u;   // this lane's features of the last key
  auto issue = [&](int bt, u32x4 (&vv)[UN]) __attribute__((always_inline)) {   // (keys past the end repeat the last one, with p = 0)
#pragma unroll
    for (int u = 0; u < UN; ++u)
      vv[u] = ld_stream((const bf16_t*)(vb + min(lane * 16u + (bt * UN + u) * 1024u, last)));
  };
  // the scores first: loads complete in order, and the statistics wait for these alone
  float s0[GQ], s1[GQ];
  if (a.src[l] >= 0) {
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
      const float* sp = d.s + d.s_at(a.src[l], b, h0 + q) + j0;
      s0[q] = sp[min(lane, n_here - 1)];
      s1[q] = sp[min(lane + 64, n_here - 1)];
    }
  } else {
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
      const half_t* sp = a.from_row + ((size_t)b * d.H + h0 + q) * d.Lk + j0;
      s0[q] = (float)sp[min(lane, n_here - 1)];
      s1[q] = (float)sp[min(lane + 64, n_here - 1)];
    }
  }
  u32x4 va[UN], vb2[UN];
  issue(0, va);
  issue(1, vb2);
  const bool in0 = lane < n_here, in1 = lane + 64 < n_here;
  float m[GQ], sum[GQ];
#pragma unroll
  for (int q = 0; q < GQ; ++q) {
    const half_t r0 = f32_to_half_sat(s0[q]), r1 = f32_to_half_sat(s1[q]);
    if (a.share[l]) s0[q] = (float)r0, s1[q] = (float)r1;
    if (a.row[l]) {
      half_t* rp = a.row[l] + ((size_t)b * d.H + h0 + q) * d.Lk + j0;
      if (in0) rp[lane] = r0;
      if (in1) rp[lane + 64] = r1;
    }
    if (!in0) s0[q] = -INFINITY;
    if (!in1) s1[q] = -INFINITY;
    m[q] = wave_max(fmaxf(s0[q], s1[q]));
    const float p0 = __expf(s0[q] - m[q]), p1 = __expf(s1[q] - m[q]);
    sum[q] = wave_sum(p0 + p1);
    p_s[wv][q][lane % KPW * NIT + lane / KPW] = p0;
    p_s[wv][q][lane % KPW * NIT + lane / KPW + 64 / KPW] = p1;
  }
  float acc[GQ][8] = {};
  auto consume = [&](int bt, const u32x4 (&vv)[UN]) __attribute__((always_inline)) {
    float p[GQ][UN];
#pragma unroll
    for (int q = 0; q < GQ; ++q)
#pragma unroll
      for (int u = 0; u < UN; u += 4) {
        const float4 x = *(const float4*)&p_s[wv][q][js * NIT + bt * UN + u];
        p[q][u] = x.x, p[q][u + 1] = x.y, p[q][u + 2] = x.z, p[q][u + 3] = x.w;
      }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      u32x4 x = vv[u];
      asm volatile("" : "+v"(x));                            // (unpacked here, not when it arrives: registers)
      float vf[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        vf[2 * e] = bf16_bits_to_f32(x[e] & 0xffffu);
        vf[2 * e + 1] = __uint_as_float(x[e] & 0xffff0000u);
      }
#pragma unroll
      for (int q = 0; q < GQ; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[q][e] += p[q][u] * vf[e];
    }
    // (summed here: the sums of all but the first head are used behind a branch, and the compiler would
    // move their products there, with everything they are made of kept until then)
#pragma unroll
    for (int q = 0; q < GQ; ++q)
      asm volatile("" : "+v"(acc[q][0]), "+v"(acc[q][1]), "+v"(acc[q][2]), "+v"(acc[q][3]), "+v"(acc[q][4]),
                        "+v"(acc[q][5]), "+v"(acc[q][6]), "+v"(acc[q][7]));
  };
  // (no batch is issued twice: the loads are non-temporal, a repeated one goes to memory again; the fences
  // keep the compiler from issuing the next batch before this one is consumed, into registers that it
  // does not have)
#pragma unroll
  for (int bt = 0; bt < NB; bt += 2) {
    __builtin_amdgcn_sched_barrier(0);
    consume(bt, va);
    __builtin_amdgcn_sched_barrier(0);
    if (bt + 2 < NB) issue(bt + 2, va);
    __builtin_amdgcn_sched_barrier(0);
    consume(bt + 1, vb2);
    __builtin_amdgcn_sched_barrier(0);
    if (bt + 3 < NB) issue(bt + 3, vb2);
  }
#pragma unroll
  for (int q = 0; q < GQ; ++q) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int o = LPK; o < 64; o <<= 1) acc[q][e] += __shfl_xor(acc[q][e], o, 64);
    const int h = h0 + q;
    if (d.n_chunk == 1) {
      const float inv = 1.f / sum[q];
      if (js == 0) {
        const size_t at = ((size_t)b * d.H + h) * DK + dc * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (a.out_f32) ((float*)a.out[l])[at + e] = acc[q][e] * inv;
          else elem<bf16_t>::store((bf16_t*)a.out[l] + at + e, acc[q][e] * inv);
        }
      }
    } else {
      const size_t at = (((size_t)a.slot[l] * d.B + b) * d.n_chunk + chunk) * d.H + h;
      if (js == 0) {
        float* po = d.part_o + at * DK + dc * 8;
        *(float4*)po = make_float4(acc[q][0], acc[q][1], acc[q][2], acc[q][3]);
        *(float4*)(po + 4) = make_float4(acc[q][4], acc[q][5], acc[q][6], acc[q][7]);
      }
      if (lane == 0) {
        d.part_ml[at * 2] = m[q];
        d.part_ml[at * 2 + 1] = sum[q];
      }
    }
  }
}

struct StackCombineArgs {
  StackDims d;
  int slot[STK_MAXL];
  void* out[STK_MAXL];
};
// grid (H, B, n_layers), block 256
template <typename O, int DK>
__global__ __launch_bounds__(256) void k_stack_combine(StackCombineArgs a) {
  __shared__ __align__(16) float s_lds[256 * 4 + 64];
  const StackDims& d = a.d;
  const size_t base = (size_t)a.slot[blockIdx.z] * d.B * d.n_chunk * d.H;
  decode_combine_unit<O, DK>(d.part_o + base * DK, d.part_ml + base * 2, (O*)a.out[blockIdx.z], d.H, d.n_chunk,
                             blockIdx.x, blockIdx.y, s_lds);
}

}  // namespace lisa
