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
//                    most of the bytes.  The last of the workgroups that share an output merges them, or
//                    (long streams) k_stack_combine.
// A layer by itself fills the chip only with hundreds of (sequence, 128 keys) units (k_decode_part); a
// stack has that many times the number of layers.  Single layers with fewer units than that run on the
// same kernels, the chain's place taken by k_decode_scores.
#pragma once
#include <cfloat>
#include <type_traits>

#include "kernels_decode.h"
#include "kernels_prefill.h"   // rows_sum

namespace lisa {

constexpr int STK_MAXL = 48;       // layers of a group (bounded by the size of the kernel arguments)
constexpr int STK_CK = 128;        // keys per workgroup of the score kernel's standard part
constexpr int STK_PB = 16;         // key positions per wave of the chain
// (per-layer numbers in the kernel arguments are ints: a byte has no scalar load, and a vector load in a
// layer loop is waited for together with everything else in flight)

// Workspace of a group: slot s (a layer) holds float32 scores [B][Hp][Lp], the partial results of its
// splits and (LiSA layers) the FFN weights in operand order.
struct StackDims {
  int B, H, Hp, Hkv, Lk, Lp, r, F, n_span;    // Hp, Lp: H, Lk rounded up to 16; n_span: splits of the keys in P V
  float* s;              // [slot][B][Hp][Lp]
  float* part_o;         // [slot][B][n_span][H][DK]
  float* part_ml;        // [slot][B][n_span][H][2]
  unsigned* done;        // [slot][B][H]: splits of an output that have left their part (null: k_stack_combine merges)
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
  int n_done;                                 // counters to clear for k_stack_pv
  int slot[STK_MAXL];               // standard layers first, then the LiSA layers
  const bf16_t* q[STK_MAXL];
  const bf16_t* k[STK_MAXL];
  const bf16_t* w1[STK_MAXL];
  const bf16_t* w2[STK_MAXL];
};

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
  for (int e = blk * 256 + tid; e < a.n_done; e += (int)gridDim.x * 256) d.done[e] = 0u;
  if (blk < a.n_std * a.std_blocks) {
    const int l = blk / a.std_blocks;
    blk -= l * a.std_blocks;
    const int nc = (d.Lk + STK_CK - 1) / STK_CK;
    const int chunk = blk % nc, kv = blk / nc % d.Hkv, b = blk / (nc * d.Hkv);
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
    FfnOperands w;
    w.w1 = a.w1[l];
    w.w2 = a.w2[l];
    w.out = d.w + (size_t)a.slot[l] * d.w_elems;
    w.Din = w.HO = d.H;
    w.F = d.F;
    w.HBO = (d.H + 15) / 16;
    w.KS = (w.HBO + 1) / 2;
    w.FS = (d.F + 31) / 32;
    ffn_operand_piece<true>(w, blk * 256 + tid);
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

// ---- one LiSA layer: a_delta and FFN of 64 key positions, all heads ---------------------------------
struct DecodeScoresArgs {
  StackDims d;
  KeyStrides ks;          // K_LR cache
  const bf16_t* q;        // q_lr [B,H,r]
  const bf16_t* k;
  const half_t* prev;     // A_{n-1} [B,H,Lk]
  const unsigned short* w;   // FFN weights in operand order (ffn_operand_piece<false>)
  float scale;
  int n_done;             // counters to clear for k_stack_pv
  int pass_through;       // the module is the identity: mask_to_finite(prev)
};
constexpr int DS_KEYS = 64;
constexpr int DS_ROW = DS_KEYS + 4;                          // floats per head of the a_delta tile
constexpr int decode_scores_lds(int H, int r, int w_bytes) { return (H * DS_ROW + ((H * r + 3) & ~3)) * 4 + w_bytes; }

static __global__ __launch_bounds__(256) void k_ffn_operands(FfnOperands w) {
  ffn_operand_piece<false>(w, blockIdx.x * 256 + threadIdx.x);
}

// grid (ceil(Lk / 64), B), block 256.  ADD: A_n = FFN(A_{n-1}) + a_delta; CONCAT: A_n = FFN([A_{n-1}; a_delta]).
// float32 A_n to d.s for k_stack_pv.  Latency: a_delta and the weights are fetched side by side, then a wave
// takes 16 positions through the FFN.
template <int HBI, int FS, int HBO, int ACT, bool CONCAT>
__global__ __launch_bounds__(256) void k_decode_scores(DecodeScoresArgs a) {
  typedef MfmaFfn<HBI, FS, HBO, ACT> Ffn;
  constexpr int KS = Ffn::KS;
  extern __shared__ __align__(16) float ds_lds[];
  const StackDims& d = a.d;
  const int H = d.H, r = d.r, Din = CONCAT ? 2 * H : H;
  float* a_s = ds_lds;                                       // [H][DS_ROW]
  float* q_s = a_s + H * DS_ROW;                             // [H][r]
  unsigned short* w_s = (unsigned short*)(q_s + ((H * r + 3) & ~3));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y, j0 = blockIdx.x * DS_KEYS;
  const int c = lane & 15, g = lane >> 4;
  const int group = H / d.Hkv;
  for (int e = (b * (int)gridDim.x + blockIdx.x) * 256 + tid; e < a.n_done; e += (int)(gridDim.x * gridDim.y) * 256) d.done[e] = 0u;
  const int pj = 16 * wv + c, j = j0 + pj;                   // this lane's position in the FFN
  f16x8 x[1][KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      x[0][ks][e] = a.prev[((size_t)b * H + min(32 * ks + 8 * g + e, H - 1)) * d.Lk + min(j, d.Lk - 1)];
  for (int e = tid; e < H * r; e += 256) q_s[e] = elem<bf16_t>::load(a.q + (size_t)b * H * r + e);
#pragma unroll
  for (int i = 0; i < (Ffn::kStageBytes + 4095) / 4096; ++i) {
    const int at = (i * 256 + tid) * 16;
    if (Ffn::kStageBytes % 4096 == 0 || at < Ffn::kStageBytes) *(u32x4*)((char*)w_s + at) = *(const u32x4*)((const char*)a.w + at);
  }
  __syncthreads();
  // a_delta of the 64 keys
  if (a.ks.j == 1 && (a.ks.t & 7) == 0 && (a.ks.h & 7) == 0 && (a.ks.b & 7) == 0) {
    // dimension-major cache with 16-byte aligned rows: 8 keys per lane (the cache holds whole octets)
    const int jo = tid & 7, jb = j0 + 8 * jo;
    for (int h = tid >> 3; h < H; h += 32) {
      float acc[8] = {};
      if (jb < d.Lk) {
        const bf16_t* kp = a.k + b * a.ks.b + h / group * a.ks.h + jb;
        const float* qp = q_s + h * r;
        auto rows = [&](auto n, int t0) __attribute__((always_inline)) {
          constexpr int N = decltype(n)::value;
          u32x4 kvv[N];
#pragma unroll
          for (int u = 0; u < N; ++u) kvv[u] = *(const u32x4*)(kp + (size_t)(t0 + u) * a.ks.t);
#pragma unroll
          for (int u = 0; u < N; ++u) {
            const float qt = qp[t0 + u];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              acc[2 * e] += qt * bf16_bits_to_f32(kvv[u][e] & 0xffffu);
              acc[2 * e + 1] += qt * __uint_as_float(kvv[u][e] & 0xffff0000u);
            }
          }
        };
        int t0 = 0;
        for (; t0 + 8 <= r; t0 += 8) rows(std::integral_constant<int, 8>{}, t0);
        if (r & 4) rows(std::integral_constant<int, 4>{}, t0), t0 += 4;
        if (r & 2) rows(std::integral_constant<int, 2>{}, t0), t0 += 2;
        if (r & 1) rows(std::integral_constant<int, 1>{}, t0);
      }
      float4* dst = (float4*)(a_s + h * DS_ROW + 8 * jo);
      dst[0] = make_float4(acc[0] * a.scale, acc[1] * a.scale, acc[2] * a.scale, acc[3] * a.scale);
      dst[1] = make_float4(acc[4] * a.scale, acc[5] * a.scale, acc[6] * a.scale, acc[7] * a.scale);
    }
  } else {
    for (int h = wv; h < H; h += 4) {
      const bf16_t* kp = a.k + b * a.ks.b + h / group * a.ks.h + (size_t)min(j0 + lane, d.Lk - 1) * a.ks.j;
      float acc = 0.f;
      for (int t = 0; t < r; ++t) acc += q_s[h * r + t] * elem<bf16_t>::load(kp + (size_t)t * a.ks.t);
      a_s[h * DS_ROW + lane] = acc * a.scale;
    }
  }
  __syncthreads();
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int ch = 32 * ks + 8 * g + e;
      if (CONCAT && ch >= H) x[0][ks][e] = ch < Din ? f32_to_half_sat(a_s[(ch - H) * DS_ROW + pj]) : (_Float16)0.f;
      else if (ch >= Din) x[0][ks][e] = (_Float16)0.f;
    }
  if (!CONCAT && a.pass_through)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x[0][ks] = mask_to_finite(x[0][ks]);
  f32x4 y[1][HBO];
  if (CONCAT) Ffn::template apply_lds_lean<1>(w_s, x, y);
  else Ffn::template apply_lds<1>(w_s, x, y);
  if (j >= d.Lk) return;
  float* sp = d.s + d.s_at(0, b, 0) + j;
#pragma unroll
  for (int hb = 0; hb < HBO; ++hb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int h = 16 * hb + 4 * g + v;
      if (h < H) sp[(size_t)h * d.Lp] = y[0][hb][v] + (CONCAT ? 0.f : a_s[h * DS_ROW + pj]);
    }
}

struct StackPvArgs {
  StackDims d;
  KeyStrides vs;
  int out_f32;
  int src[STK_MAXL];         // slot of the scores; -1: from_row
  int slot[STK_MAXL];      // slot of the partial results
  int share[STK_MAXL];     // direct sharing: the scores as the half row would hold them
  const bf16_t* v[STK_MAXL];
  half_t* row[STK_MAXL];             // A_n as half [B][H][Lk], or null
  void* out[STK_MAXL];
  const half_t* from_row;
};

// What one workgroup leaves for another one of the same launch: stores and loads at agent scope go past
// the L2 of the XCD, which the other XCDs do not see.
__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store((unsigned*)p, __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
  return __uint_as_float(__hip_atomic_load((const unsigned*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// Sum over the lane groups js of a wave that hold the same features (LPK lanes per key).
template <int LPK>
__device__ __forceinline__ float key_groups_sum(float v) {
  if (LPK == 8) v += dpp_move<0x128>(v);                     // row_ror:8
  return rows_sum(v);
}

// Keys per workgroup of k_stack_pv: 512 at d_k = 128, 1024 at 64 (32 KB ... of V per four waves either way).
constexpr int stack_pv_keys(int dk) { return 65536 / dk; }

// grid (n_span group / GQ, Hkv B, n_layers), block 64 NW.  A workgroup = one key/value head, GQ
// of its query heads (one pass over V serves them) and NW consecutive pieces of the keys, one per wave (NB
// batches of eight 1 KB loads each); n_span of them make up an output.  NB = 4, NW = 4: the long stream.
// NB = 1, NW = 16: all of it in flight at once, where there are few workgroups.  The first batches of V are in
// flight while the softmax statistics are made.  The waves' results are merged through the LDS, the
// spans' by the workgroup that finishes last (in the order of the keys, whoever it is).
// Bound: the V stream.  16 users at 4096 tokens, 32 layers: 17.5 GB fetched in 2.65 ms, 6.6 TB/s; one user at 1023
// tokens: 273 MB in 41 - 44 us.
template <int DK, int GQ, int NB>
__global__ __launch_bounds__(1024 / NB, NB == 1 ? 4 : GQ == 1 ? 4 : 3) void k_stack_pv(StackPvArgs a) {
  constexpr int NW = 16 / NB, THREADS = 64 * NW;
  constexpr int LPK = DK / 8, KPW = 64 / LPK, UN = 8, NIT = NB * UN, CK = NIT * KPW;
  static_assert(LPK == 8 || LPK == 16, "d_k 64 or 128");
  static_assert(NW * CK == stack_pv_keys(DK), "keys per workgroup");
  constexpr int PER = (CK + 63) / 64;                        // scores per lane
  __shared__ __align__(16) float p_s[NW][GQ][CK];             // [key % KPW][key / KPW]: a lane's keys are consecutive
  __shared__ __align__(16) float o_s[NW][GQ][DK];
  __shared__ float m_s[NW][GQ], l_s[NW][GQ];
  __shared__ int last_s;
  const StackDims& d = a.d;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = d.H / d.Hkv, subs = group / GQ;
  const int l = blockIdx.z;
  const int sub = subs == 1 ? 0 : blockIdx.x / d.n_span, span = blockIdx.x - sub * d.n_span;
  const int b = blockIdx.y / d.Hkv, kv = blockIdx.y - b * d.Hkv;
  const int h0 = kv * group + sub * GQ;
  const int j0 = (span * NW + wv) * CK, n_here = min(CK, d.Lk - j0);
  const int js = lane / LPK, dc = lane % LPK;
  if (n_here > 0) {                                          // wave-uniform
    const char* vb = (const char*)(a.v[l] + b * a.vs.b + kv * a.vs.h + (size_t)j0 * DK);   // wave-uniform
    const unsigned last = (n_here - 1) * (DK * 2u) + dc * 16u;   // this lane's features of the last key
    auto issue = [&](int bt, u32x4 (&vv)[UN]) __attribute__((always_inline)) {   // (keys past the end repeat the last one, with p = 0)
#pragma unroll
      for (int u = 0; u < UN; ++u)
        vv[u] = ld_stream((const bf16_t*)(vb + min(lane * 16u + (bt * UN + u) * 1024u, last)));
    };
    // the scores first: loads complete in order, and the statistics wait for these alone
    float s[GQ][PER];
    if (a.src[l] >= 0) {
#pragma unroll
      for (int q = 0; q < GQ; ++q)
#pragma unroll
        for (int i = 0; i < PER; ++i) s[q][i] = d.s[d.s_at(a.src[l], b, h0 + q) + j0 + min(lane + 64 * i, n_here - 1)];
    } else {
#pragma unroll
      for (int q = 0; q < GQ; ++q)
#pragma unroll
        for (int i = 0; i < PER; ++i)
          s[q][i] = (float)a.from_row[((size_t)b * d.H + h0 + q) * d.Lk + j0 + min(lane + 64 * i, n_here - 1)];
    }
    u32x4 va[UN], vb2[UN];
    issue(0, va);
    if (NB > 1) issue(1, vb2);
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
      half_t* rp = a.row[l] ? a.row[l] + ((size_t)b * d.H + h0 + q) * d.Lk + j0 : nullptr;
      float mx = -FLT_MAX;                                   // (finite: a piece masked with -inf throughout weighs nothing)
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const bool in = lane + 64 * i < n_here;
        const half_t rv = f32_to_half_sat(s[q][i]);
        if (a.share[l]) s[q][i] = (float)rv;
        if (rp && in) rp[lane + 64 * i] = rv;
        if (!in) s[q][i] = -INFINITY;
        mx = fmaxf(mx, s[q][i]);
      }
      mx = wave_max(mx);
      float ps = 0.f;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const float p = __expf(s[q][i] - mx);
        ps += p;
        const int key = lane + 64 * i;
        if (CK >= 64 || key < CK) p_s[wv][q][key % KPW * NIT + key / KPW] = p;
      }
      ps = wave_sum(ps);
      if (lane == 0) m_s[wv][q] = mx, l_s[wv][q] = ps;
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
        asm volatile("" : "+v"(x));                          // (unpacked here, not when it arrives: registers)
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
      // (summed here: left alone, the compiler moves the products of all but the first head behind the
      // branches that follow, and keeps everything they are made of until then)
#pragma unroll
      for (int q = 0; q < GQ; ++q)
        asm volatile("" : "+v"(acc[q][0]), "+v"(acc[q][1]), "+v"(acc[q][2]), "+v"(acc[q][3]), "+v"(acc[q][4]),
                          "+v"(acc[q][5]), "+v"(acc[q][6]), "+v"(acc[q][7]));
    };
    // (no batch is issued twice: the loads are non-temporal, a repeated one goes to memory again; the
    // fences keep the compiler from issuing the next batch before this one is consumed, into registers
    // that it does not have)
#pragma unroll
    for (int bt = 0; bt < NB; bt += 2) {
      __builtin_amdgcn_sched_barrier(0);
      consume(bt, va);
      __builtin_amdgcn_sched_barrier(0);
      if (bt + 2 < NB) issue(bt + 2, va);
      __builtin_amdgcn_sched_barrier(0);
      if (bt + 1 < NB) consume(bt + 1, vb2);
      __builtin_amdgcn_sched_barrier(0);
      if (bt + 3 < NB) issue(bt + 3, vb2);
    }
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[q][e] = key_groups_sum<LPK>(acc[q][e]);
      if (js == 0) {
        float* op = &o_s[wv][q][dc * 8];
        *(float4*)op = make_float4(acc[q][0], acc[q][1], acc[q][2], acc[q][3]);
        *(float4*)(op + 4) = make_float4(acc[q][4], acc[q][5], acc[q][6], acc[q][7]);
      }
    }
  } else {                                                   // a piece without keys weighs nothing
    if (lane < GQ) m_s[wv][lane] = -FLT_MAX, l_s[wv][lane] = 0.f;
    for (int e = lane; e < GQ * DK; e += 64) (&o_s[wv][0][0])[e] = 0.f;
  }
  __syncthreads();
  // ---- the pieces (the first one of a span has keys) ------------------------------------------------
  constexpr int EPT = (GQ * DK + THREADS - 1) / THREADS;                 // output elements per thread
  float num[EPT], den[EPT], M[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int e = threadIdx.x + THREADS * i, q = min(e / DK, GQ - 1), f = e % DK;
    M[i] = m_s[0][q];
#pragma unroll
    for (int w = 1; w < NW; ++w) M[i] = fmaxf(M[i], m_s[w][q]);
    num[i] = den[i] = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float c = __expf(m_s[w][q] - M[i]);
      num[i] += c * o_s[w][q][f];
      den[i] += c * l_s[w][q];
    }
  }
  auto store_out = [&](int i, float v) {
    const int e = threadIdx.x + THREADS * i;
    if (e >= GQ * DK) return;
    const size_t at = ((size_t)b * d.H + h0 + e / DK) * DK + e % DK;
    if (a.out_f32) ((float*)a.out[l])[at] = v;
    else elem<bf16_t>::store((bf16_t*)a.out[l] + at, v);
  };
  if (d.n_span == 1) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) store_out(i, num[i] / den[i]);
    return;
  }
  const size_t row0 = ((size_t)a.slot[l] * d.B + b) * d.n_span * d.H + h0;   // span s, head q: row0 + s H + q
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int e = threadIdx.x + THREADS * i, q = e / DK, f = e % DK;
    if (e >= GQ * DK) break;
    const size_t at = row0 + (size_t)span * d.H + q;
    st_agent(d.part_o + at * DK + f, num[i]);
    if (f == 0) {
      st_agent(d.part_ml + at * 2, M[i]);
      st_agent(d.part_ml + at * 2 + 1, den[i]);
    }
  }
  if (!d.done) return;
  // The parts have arrived where every XCD reads them before the count does.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    last_s = (int)__hip_atomic_fetch_add(d.done + ((size_t)a.slot[l] * d.B + b) * d.H + h0, 1u, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) == d.n_span - 1;
  __syncthreads();
  if (!last_s) return;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int e = min((int)threadIdx.x + THREADS * i, GQ * DK - 1), q = e / DK, f = e % DK;
    float Mx = -FLT_MAX, nm = 0.f, dn = 0.f;
    // eight spans at a time: their loads are in flight together
    for (int s0 = 0; s0 < d.n_span; s0 += 8) {
      float po[8], pm[8], pl[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const size_t at = row0 + (size_t)min(s0 + u, d.n_span - 1) * d.H + q;
        po[u] = ld_agent(d.part_o + at * DK + f);
        pm[u] = ld_agent(d.part_ml + at * 2);
        pl[u] = ld_agent(d.part_ml + at * 2 + 1);
      }
      float m8 = Mx;
#pragma unroll
      for (int u = 0; u < 8; ++u) m8 = fmaxf(m8, pm[u]);
      const float c0 = __expf(Mx - m8);
      nm *= c0;
      dn *= c0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float c = s0 + u < d.n_span ? __expf(pm[u] - m8) : 0.f;
        nm += c * po[u];
        dn += c * pl[u];
      }
      Mx = m8;
    }
    store_out(i, nm / dn);
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
  const size_t base = (size_t)a.slot[blockIdx.z] * d.B * d.n_span * d.H;
  decode_combine_unit<O, DK>(d.part_o + base * DK, d.part_ml + base * 2, (O*)a.out[blockIdx.z], d.H, d.n_span,
                             blockIdx.x, blockIdx.y, s_lds);
}

}  // namespace lisa
