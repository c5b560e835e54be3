// Prefill layers (Lq > 1) in float32 arithmetic on the matrix cores: attention, and the scores of a LiSA layer.
// Same arithmetic as the generic kernels (float32 products and sums); they cover any other shape.
// T is the type of the operands (float, or bf16, whose values and products float32 holds exactly), S the
// score type.  bf16 layers come here, from score rows that are no multiple of 8 scores, with the shapes that the
// kernels of kernels_split.h do not take or are slower at (f32_attn_takes(), f32_scores_win()).
#pragma once
#include <type_traits>
#include "kernels_prefill.h"

namespace lisa {

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned f32_u32x2 __attribute__((ext_vector_type(2)));
typedef f16x4 f16x4_a2 __attribute__((aligned(2)));

// Four consecutive elements as they are loaded (8 or 16 bytes, aligned), and as numbers.
template <typename T> struct Quad;
template <> struct Quad<float> {
  f32x4 raw;
  static __device__ __forceinline__ Quad load(const float* p) { return {*(const f32x4*)p}; }
  __device__ __forceinline__ float operator[](int e) const { return raw[e]; }
};
template <> struct Quad<bf16_t> {
  f32_u32x2 raw;
  static __device__ __forceinline__ Quad load(const bf16_t* p) { return {*(const f32_u32x2*)p}; }
  __device__ __forceinline__ float operator[](int e) const {
    return __uint_as_float(e & 1 ? raw[e >> 1] & 0xffff0000u : raw[e >> 1] << 16);
  }
};
// Two bf16 elements, neighbours at an even offset or from anywhere.
struct Pair {
  unsigned raw;
  static __device__ __forceinline__ Pair load(const bf16_t* p) { return {*(const unsigned*)p}; }
  static __device__ __forceinline__ Pair load2(const bf16_t* p, const bf16_t* q) { return {p->bits | (unsigned)q->bits << 16}; }
  __device__ __forceinline__ float operator[](int e) const { return __uint_as_float(e ? raw & 0xffff0000u : raw << 16); }
};
// Four consecutive scores of a row, which starts at any element.
__device__ __forceinline__ void store_scores4(float* p, f32x4 s) { *(f32x4_a4*)p = s; }
__device__ __forceinline__ void store_scores4(half_t* p, f32x4 s) {
  *(f16x4_a2*)p = f16x4{f32_to_half_sat(s[0]), f32_to_half_sat(s[1]), f32_to_half_sat(s[2]), f32_to_half_sat(s[3])};
}

template <typename T, typename S>
struct F32AttnArgs {
  const T* q;             // [B,H,Lq,DK]
  const T* k;             // [B,Hkv,Lk,DK]
  const T* v;             // [B,Hkv,Lk,DK] or null (scores only)
  const float* given;     // GIVEN: scores [B,H,n_rows,Lk] to take instead of Q K^T (then q, k unused)
  S* scores;              // [B,H,Lq,Lk] or null
  void* out;              // [B,Lq,H,DK] (float where out_f32, else T) or null
  int B, H, Hkv, Lq, Lk, causal, out_f32;
  int order, blocks;      // of the workgroups, see f32_attn_order(); parts * row blocks
  int row0, n_rows;       // query rows of this launch (row0 a multiple of 16)
  int parts;              // workgroups that the tiles of a row block are dealt to (1 unless scores only)
  float scale;
};

// grid (parts ceil(n_rows / 16), H, B), (H, B, parts ceil(n_rows / 16)) or all of it in x (order 0, 1, 2), block 64 NW: 16 query rows of one head, the 16-key tiles dealt to the NW
// waves (scores only: of `parts` workgroups), their softmax states merged through the LDS at the end.  16x16x4 float32 MFMAs with the
// query row on lane % 16 for both products, so that a lane's four scores are its B operands of the
// second one.  Short sequences are a matter of latency: a wave holds the operands of its next tile while
// it works on this one, and nothing passes through the LDS before the end.
// Order 2 has them by length over all heads, long ones first, every other 256 of them backwards: a compute unit has numbers i, i + 256,
// .. where all run at once, and with the row blocks as the fastest index these are equally long (two sequences of 504 tokens,
// 8 heads: 18.4 -> 14.7 us, three of 504 25 -> 19).
// The contraction over the features is numbered so that a lane's operands are pieces of four: step s of
// piece i takes feature 16 i + 4 g + s.  For P V the 16 rows of output block i are the features 4 m + i.
template <typename T, typename S, int NDK, bool GIVEN, int NW>
__global__ __launch_bounds__(64 * NW) void k_f32_attn(F32AttnArgs<T, S> a) {
  constexpr int DK = 64 * NDK, NP = DK / 16;                 // pieces of four of a row per lane group
  __shared__ float o_s[NW][16][DK + 4];
  __shared__ float m_s[NW][16], l_s[NW][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const bool z = a.order != 0;                               // (nothing of the grid is read: one load of the arguments less to wait for)
  int h = z ? blockIdx.x : blockIdx.y, b = z ? blockIdx.y : blockIdx.z, xr = a.blocks - 1 - (z ? blockIdx.z : blockIdx.x);   // long row blocks first
  if (a.order == 2) {
    const int heads = a.H * a.B, chunk = blockIdx.x & ~255u;
    const int pos = chunk & 256 ? chunk + min(a.blocks * heads, chunk + 256) - 1 - (int)blockIdx.x : blockIdx.x;
    xr = a.blocks - 1 - pos / heads, h = pos % heads % a.H, b = pos % heads / a.H;
  }
  int rb = xr, t_first = wv, t_step = NW;
  if (a.parts > 1) {
    rb = xr / a.parts;
    t_first += NW * (xr - rb * a.parts);
    t_step = NW * a.parts;
  }
  const int Lq = a.Lq, Lk = a.Lk, i0 = a.row0 + rb * 16;
  const int kv = h / (a.H / a.Hkv);
  const int i_last = min(i0 + 15, Lq - 1), row = min(i0 + c, Lq - 1);
  const int n_keys = n_visible(i_last, Lq, Lk, a.causal), n_tiles = (n_keys + 15) / 16;
  const int vis = i0 + c < Lq ? n_visible(row, Lq, Lk, a.causal) : 0;
  const float LOG2E = 1.4426950408889634f;
  const bool with_v = a.out != nullptr;
  Quad<T> qr[NP];
  if (!GIVEN) {
    const T* qp = a.q + (((size_t)b * a.H + h) * Lq + row) * DK + 4 * g;
#pragma unroll
    for (int i = 0; i < NP; ++i) qr[i] = Quad<T>::load(qp + 16 * i);
  }
  const T* kb = GIVEN ? nullptr : a.k + ((size_t)b * a.Hkv + kv) * Lk * DK + 4 * g;
  const T* vb = a.v + ((size_t)b * a.Hkv + kv) * Lk * DK + 4 * c;
  const size_t srow = (((size_t)b * a.H + h) * Lq + row) * Lk;
  const size_t grow = (((size_t)b * a.H + h) * a.n_rows + row - a.row0) * Lk;
  Quad<T> kr[NP], vr[4][NDK];
  f32x4 sr;
  auto load_k = [&](int tile) {
    if (GIVEN) {
      const int j = tile * 16 + 4 * g;
      if (tile * 16 + 16 <= Lk) {
        sr = *(const f32x4_a4*)(a.given + grow + j);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) sr[v] = a.given[grow + min(j + v, Lk - 1)];
      }
    } else {
      const T* kp = kb + (size_t)min(tile * 16 + c, Lk - 1) * DK;
#pragma unroll
      for (int i = 0; i < NP; ++i) kr[i] = Quad<T>::load(kp + 16 * i);
    }
  };
  auto load_v = [&](int tile) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int n = 0; n < NDK; ++n) vr[v][n] = Quad<T>::load(vb + (size_t)min(tile * 16 + 4 * g + v, Lk - 1) * DK + 64 * n);
  };
  f32x4 o[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  if (t_first < n_tiles) {
    load_k(t_first);
    if (with_v) load_v(t_first);
  }
  for (int tile = t_first; tile < n_tiles; tile += t_step) {
    const int tile_n = min(tile + t_step, n_tiles - 1);
    const int j = tile * 16 + 4 * g;                         // this lane's keys j .. j + 3 of row c
    f32x4 s;
    if (GIVEN) {
      s = sr;
    } else {
      f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[i][e], qr[i][e], acc[i & 1], 0, 0, 0);
      s = (acc[0] + acc[1]) * a.scale;
    }
    load_k(tile_n);
    if (!GIVEN && a.scores) {
      if (j + 4 <= vis) {
        store_scores4(a.scores + srow + j, s);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (j + v < vis) elem<S>::store(a.scores + srow + j + v, s[v]);
      }
    }
    if (with_v) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (j + v >= vis) s[v] = -INFINITY;
      const float m_new = rows_max(max2_raw(max2_raw(s[0], s[1]), max2_raw(s[2], s[3])), m_run);
      // (the maximum is subtracted before the change of base: m log2(e) on its own is rounded to the ulp of
      // the maximum, differently in each wave, and at scores around 200 that is 3e-5 of the result)
      const float m0 = m_new == -INFINITY ? 0.f : m_new;     // (no key seen yet: every p is 0)
      const float alpha = fast_exp2((m_run - m0) * LOG2E);
      m_run = m_new;
      f32x4 p;
#pragma unroll
      for (int v = 0; v < 4; ++v) p[v] = fast_exp2((s[v] - m0) * LOG2E);
      l_run = l_run * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
      for (int i = 0; i < NP; ++i) o[i] *= alpha;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int n = 0; n < NDK; ++n)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[4 * n + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[v][n][e], p[v], o[4 * n + e], 0, 0, 0);
      load_v(tile_n);
    }
  }
  if (!with_v) return;
  const float l = rows_sum(l_run);
  if (g == 0) {
    m_s[wv][c] = m_run;
    l_s[wv][c] = l;
  }
  // o[4 n + e][v]: row c, feature 64 n + 4 (4 g + v) + e
#pragma unroll
  for (int n = 0; n < NDK; ++n)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      *(float4*)&o_s[wv][c][64 * n + 16 * g + 4 * v] = make_float4(o[4 * n][v], o[4 * n + 1][v], o[4 * n + 2][v], o[4 * n + 3][v]);
  __syncthreads();
  for (int e = tid; e < 16 * DK; e += 64 * NW) {
    const int r = e / DK, d = e % DK;
    if (i0 + r >= Lq) break;
    float M = m_s[0][r];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, m_s[w][r]);
    if (M == -INFINITY) M = 0.f;                             // (every score of the row -inf: num = den = 0)
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = fast_exp2((m_s[w][r] - M) * LOG2E);    // (a wave without tiles: 0)
      num += f * o_s[w][r][d];
      den += f * l_s[w][r];
    }
    // (a row that sees nothing gives zeros, as the generic kernel has it; NaN stays NaN)
    const size_t at = (((size_t)b * Lq + i0 + r) * a.H + h) * DK + d;
    const float x = den > 0.f ? num / den : num * 0.f;
    if (a.out_f32) ((float*)a.out)[at] = x;
    else elem<T>::store((T*)a.out + at, x);
  }
}

template <typename T, typename S>
struct F32ScoresArgs {
  const T* q_lr;          // [B,H,Lq,r]
  const T* k_lr;          // [B,Hkv,Lk,r]
  const S* prev;          // [B,H,Lq,Lk]
  const T* w1;            // [Din,F]
  const T* w2;            // [F,H]
  S* scores;              // [B,H,Lq,Lk] or null
  float* exact;           // [B,H,n_rows,Lk] or null: the unrounded copy
  int H, Hkv, Lq, Lk, r, F, causal;
  int row0, n_rows;       // query rows of this launch (row0 a multiple of 16)
  int tiles;              // key tiles per workgroup
  float dscale;
};
constexpr int F32_DROW = 20;                                 // floats per row of the A_delta tile (16 keys, padded)
// LDS bytes for HT padded heads: A_delta tile, then the weights in operand order.
constexpr int f32_scores_lds(int HT, int F, bool concat) {
  return (HT * 16 * F32_DROW + (F + 15) / 16 * ((concat ? 2 : 1) * HT / 4 + (HT + 15) / 16 * 4) * 64) * (int)sizeof(float);
}

// A_n = FFN(A_{n-1}) + A_delta, or FFN([A_{n-1}; A_delta]) (CONCAT).  grid (ceil(key tiles / tiles), ceil(n_rows / 16), B),
// block 256.  A tile = 16 query rows x 16 keys, all heads: the waves make A_delta by heads (16x16x4 float32
// MFMA, keys x rows) and leave it in the LDS, then take the tile's rows, four each: FFN with the 16 keys of
// a row as the columns (mfma_ffn.h's scheme in float32: a lane's hidden units are its operands of the second
// product).
// Bound: at most a third of the time is the float32 MFMAs, the rest loads and stores of 32- and 64-byte pieces in
// H pages per tensor.  32 heads, 2 x 509 rows behind 1022 keys, bf16: 316 us (589 with a wait per load of A_delta and the tests
// of the stores inside their loops), where k_split_scores takes 130 now; few or short rows stay here (f32_scores_win()).
// (One position per lane with the weights through the scalar cache took 17 us where this takes 4, 8 heads, 128 tokens: one
// wave per SIMD waits for every weight.)
// HT: H rounded up to 8, 16, 32 or 40.
template <typename T, typename S, int HT, int ACT, bool CONCAT>
__global__ __launch_bounds__(256) void k_f32_lisa_scores(F32ScoresArgs<T, S> a) {
  constexpr int KH = HT / 4, KS = CONCAT ? 2 * KH : KH;      // k-steps of the heads, of the inputs
  constexpr int HB = (HT + 15) / 16, NB = 4;                 // output blocks, rows per wave
  // bf16: the products of 16 hidden units are summed from zero and added in one step, A_delta last (each step of a sum is
  // rounded at the size of what it has reached): error of O 4.9e-7 -> 1.3e-7 (16 heads, 255 tokens, F = 256), 2.0e-7 ->
  // 1.2e-7 (8 heads, 201 tokens, F = 32); the kernel of three-part products has 1.4e-7 and 1.0e-7.  float32 layers keep one
  // chain: A_delta last alone cost 21.8 -> 23.1 us for a pair of layers of 128 tokens.
  constexpr bool BLOCKS = sizeof(T) == 2;
  extern __shared__ __align__(16) float f32_lds[];
  float* d_s = f32_lds;                                      // [HT][16 rows][F32_DROW]
  const int FB = (a.F + 15) / 16;
  float* w1_s = d_s + HT * 16 * F32_DROW;                    // [FB][KS][64]
  float* w2_s = w1_s + FB * KS * 64;                         // [FB][4][HB][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int H = a.H, Lq = a.Lq, Lk = a.Lk, r = a.r, group = H / a.Hkv;
  const int rb = gridDim.y - 1 - blockIdx.y, b = blockIdx.z, i0 = a.row0 + rb * 16;
  const int n_tiles = (n_visible(min(i0 + 15, Lq - 1), Lq, Lk, a.causal) + 15) / 16;
  const int t0 = blockIdx.x * a.tiles, t1 = min(n_tiles, t0 + a.tiles);
  if (t0 >= t1) return;                                      // (workgroup-uniform)
  for (int e = tid; e < FB * KS * 64; e += 256) {
    const int o = e >> 6, f = 16 * (o / KS) + (e & 15), s = o % KS, h = 4 * (s % KH) + ((e >> 4) & 3);
    w1_s[e] = f < a.F && h < H ? elem<T>::load(a.w1 + (size_t)(s < KH ? h : H + h) * a.F + f) : 0.f;
  }
  for (int e = tid; e < FB * 4 * HB * 64; e += 256) {
    const int o = e >> 6, h = 16 * (o % HB) + (e & 15), f = 16 * (o / (4 * HB)) + 4 * ((e >> 4) & 3) + o / HB % 4;
    w2_s[e] = f < a.F && h < H ? elem<T>::load(a.w2 + (size_t)f * H + h) : 0.f;
  }
  const size_t hs = (size_t)Lq * Lk;                         // from a head's scores to the next head's
  for (int tile = t0; tile < t1; ++tile) {
    const int j = tile * 16 + c, jc = min(j, Lk - 1);
    // this wave's rows of A_{n-1}
    float x[NB][KS];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const S* xp = a.prev + ((size_t)b * H * Lq + min(i0 + wv * NB + n, Lq - 1)) * Lk + jc;
#pragma unroll
      for (int s = 0; s < KH; ++s) {
        const float xs = elem<S>::load(xp + min(4 * s + g, H - 1) * hs);
        x[n][s] = 4 * s + g < H ? xs : 0.f;
      }
    }
    if (tile > t0) __syncthreads();                          // d_s of the tile before has been read
    // A_delta.  bf16: NH heads and 32 ranks at a time with all their loads in flight together; a load per step of the
    // product, each waited for, made this the longest part of the kernel.  The ranks are numbered so that a lane's
    // two steps 2 u, 2 u + 1 take neighbours, one load where the rows (r elements) keep them aligned.
    // float32 operands take twice the registers for it, and what it does for ranks and heads that fill no batch
    // costs the small layers more than the waits: a head and a step at a time there (4 heads, 1024 rows, 44 us
    // against 96 in batches; 32 heads 267 against 328).
    if constexpr (sizeof(T) == 4) {
      for (int h = wv; h < H; h += 4) {
        const T* kp = a.k_lr + (((size_t)b * a.Hkv + h / group) * Lk + jc) * r;
        const T* qp = a.q_lr + (((size_t)b * H + h) * Lq + min(i0 + c, Lq - 1)) * r;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < (r + 3) / 4; ++s) {
          const int t = 4 * s + g;
          const float kx = t < r ? kp[t] : 0.f, qx = t < r ? qp[t] : 0.f;
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(kx, qx, acc, 0, 0, 0);
        }
        *(f32x4*)(d_s + (h * 16 + c) * F32_DROW + 4 * g) = acc * a.dscale;   // row c, keys 4 g ..
      }
    } else {
      constexpr int NH = HT >= 16 ? 4 : 2;
      const bool pairs = (r & 1) == 0;
      for (int h0 = wv; h0 < H; h0 += 4 * NH) {
        f32x4 acc[NH];
  #pragma unroll
        for (int m = 0; m < NH; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int r0 = 0; r0 < r; r0 += 32) {
          Pair kx[NH][4], qx[NH][4];
  #pragma unroll
          for (int m = 0; m < NH; ++m) {
            const int h = min(h0 + 4 * m, H - 1);
            const T* kp = a.k_lr + (((size_t)b * a.Hkv + h / group) * Lk + jc) * r;
            const T* qp = a.q_lr + (((size_t)b * H + h) * Lq + min(i0 + c, Lq - 1)) * r;
  #pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int t = r0 + 8 * u + 2 * g;
              kx[m][u] = pairs ? Pair::load(kp + min(t, r - 2)) : Pair::load2(kp + min(t, r - 1), kp + min(t + 1, r - 1));
              qx[m][u] = pairs ? Pair::load(qp + min(t, r - 2)) : Pair::load2(qp + min(t, r - 1), qp + min(t + 1, r - 1));
            }
          }
  #pragma unroll
          for (int u = 0; u < 4; ++u)
  #pragma unroll
            for (int e = 0; e < 2; ++e) {
              const bool in = r0 + 8 * u + 2 * g + e < r;
  #pragma unroll
              for (int m = 0; m < NH; ++m)
                acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? kx[m][u][e] : 0.f, in ? qx[m][u][e] : 0.f, acc[m], 0, 0, 0);
            }
        }
  #pragma unroll
        for (int m = 0; m < NH; ++m) {
          const int h = h0 + 4 * m;
          if (h < H) *(f32x4*)(d_s + (h * 16 + c) * F32_DROW + 4 * g) = acc[m] * a.dscale;   // row c, keys 4 g ..
        }
      }
    }
    __syncthreads();                                         // (also publishes the weights)
    f32x4 y[NB][HB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      if constexpr (CONCAT) {
#pragma unroll
        for (int s = 0; s < KH; ++s) {
          const int h = 4 * s + g;
          x[n][KH + s] = h < H ? d_s[(h * 16 + wv * NB + n) * F32_DROW + c] : 0.f;
        }
      }
#pragma unroll
      for (int hb = 0; hb < HB; ++hb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int h = min(16 * hb + 4 * g + v, H - 1);
          y[n][hb][v] = CONCAT || BLOCKS ? 0.f : d_s[(h * 16 + wv * NB + n) * F32_DROW + c];
        }
    }
    for (int fb = 0; fb < FB; ++fb) {
      f32x4 u[NB];
#pragma unroll
      for (int n = 0; n < NB; ++n) u[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const float w = w1_s[(fb * KS + s) * 64 + lane];
#pragma unroll
        for (int n = 0; n < NB; ++n) u[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, x[n][s], u[n], 0, 0, 0);
      }
      f32x4 block[NB][HB];
      f32x4 (&sum)[NB][HB] = BLOCKS ? block : y;
      if (BLOCKS)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) block[n][hb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int n = 0; n < NB; ++n) u[n][v] = ACT == 0 ? fmaxf(u[n][v], 0.f) : u[n][v] / (1.f + expf(-u[n][v]));
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
          const float w = w2_s[((fb * 4 + v) * HB + hb) * 64 + lane];
#pragma unroll
          for (int n = 0; n < NB; ++n) sum[n][hb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, u[n][v], sum[n][hb], 0, 0, 0);
        }
      }
      if (BLOCKS)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) y[n][hb] += block[n][hb];
    }
    if constexpr (BLOCKS && !CONCAT) {
#pragma unroll
      for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
#pragma unroll
          for (int v = 0; v < 4; ++v) y[n][hb][v] += d_s[(min(16 * hb + 4 * g + v, H - 1) * 16 + wv * NB + n) * F32_DROW + c];
    }
    // (one test of the tensor and of the heads around each run of stores, not one per element)
    auto store = [&](auto* dst, size_t head_stride, int rows, int row0) {
      typedef std::remove_pointer_t<decltype(dst)> D;
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int i = i0 + wv * NB + n;
        if (i >= Lq || j >= n_visible(i, Lq, Lk, a.causal)) continue;
        D* p = dst + ((size_t)b * H * rows + i - row0) * Lk + j + 4 * g * head_stride;
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
          if (16 * hb + 16 <= H) {
#pragma unroll
            for (int v = 0; v < 4; ++v) elem<D>::store(p + (16 * hb + v) * head_stride, y[n][hb][v]);
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * hb + 4 * g + v < H) elem<D>::store(p + (16 * hb + v) * head_stride, y[n][hb][v]);
          }
        }
      }
    };
    if constexpr (sizeof(T) == 4) {                          // (scores and their copy are the same type and rows: one of them)
      store(a.scores ? a.scores : a.exact, hs, Lq, 0);
    } else {
      if (a.scores) store(a.scores, hs, Lq, 0);
      if (a.exact) store(a.exact, (size_t)a.n_rows * Lk, a.n_rows, a.row0);
    }
  }
}

}  // namespace lisa
