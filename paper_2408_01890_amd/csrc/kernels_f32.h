// float32 prefill layers (Lq > 1): attention on the float32 matrix instructions, and the scores of an
// ADD-form LiSA layer.  Same arithmetic as the generic kernels (float32
// products and sums); they cover any other shape.
#pragma once
#include "kernels_prefill.h"

namespace lisa {

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

struct F32AttnArgs {
  const float* q;         // [B,H,Lq,DK]
  const float* k;         // [B,Hkv,Lk,DK]
  const float* v;         // [B,Hkv,Lk,DK] or null (scores only)
  const float* given;     // GIVEN: scores [B,H,Lq,Lk] to take instead of Q K^T (then q, k unused)
  float* scores;          // [B,H,Lq,Lk] or null
  float* out;             // [B,Lq,H,DK] or null
  int H, Hkv, Lq, Lk, causal;
  float scale;
};

// grid (ceil(Lq / 16), H, B), block 256: 16 query rows of one head, the 16-key tiles dealt to the four
// waves, their softmax states merged through the LDS at the end.  16x16x4 float32 MFMAs with the
// query row on lane % 16 for both products, so that a lane's four scores are its B operands of the
// second one.  Short sequences are a matter of latency: a wave holds the operands of its next tile while
// it works on this one, and nothing passes through the LDS before the end.
// The contraction over the features is numbered so that a lane's operands are 16-byte pieces: step s of
// piece i takes feature 16 i + 4 g + s.  For P V the 16 rows of output block i are the features 4 m + i.
template <int NDK, bool GIVEN>
__global__ __launch_bounds__(256) void k_f32_attn(F32AttnArgs a) {
  constexpr int DK = 64 * NDK, NP = DK / 16;                 // 16-byte pieces of a row per lane group
  __shared__ float o_s[4][16][DK + 4];
  __shared__ float m_s[4][16], l_s[4][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int rb = gridDim.x - 1 - blockIdx.x;                 // long row blocks first
  const int h = blockIdx.y, b = blockIdx.z;
  const int Lq = a.Lq, Lk = a.Lk, i0 = rb * 16;
  const int kv = h / (a.H / a.Hkv);
  const int i_last = min(i0 + 15, Lq - 1), row = min(i0 + c, Lq - 1);
  const int n_keys = n_visible(i_last, Lq, Lk, a.causal), n_tiles = (n_keys + 15) / 16;
  const int vis = i0 + c < Lq ? n_visible(row, Lq, Lk, a.causal) : 0;
  const float LOG2E = 1.4426950408889634f;
  const bool with_v = a.out != nullptr;
  f32x4 qr[NP];
  if (!GIVEN) {
    const float* qp = a.q + (((size_t)b * a.H + h) * Lq + row) * DK + 4 * g;
#pragma unroll
    for (int i = 0; i < NP; ++i) qr[i] = *(const f32x4*)(qp + 16 * i);
  }
  const float* kb = GIVEN ? nullptr : a.k + ((size_t)b * a.Hkv + kv) * Lk * DK + 4 * g;
  const float* vb = a.v + ((size_t)b * a.Hkv + kv) * Lk * DK + 4 * c;
  const size_t srow = (((size_t)b * a.H + h) * Lq + row) * Lk;
  f32x4 kr[NP], sr, vr[4][NDK];
  auto load_k = [&](int tile) {
    if (GIVEN) {
      const int j = tile * 16 + 4 * g;
      if (tile * 16 + 16 <= Lk) {
        sr = *(const f32x4_a4*)(a.given + srow + j);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) sr[v] = a.given[srow + min(j + v, Lk - 1)];
      }
    } else {
      const float* kp = kb + (size_t)min(tile * 16 + c, Lk - 1) * DK;
#pragma unroll
      for (int i = 0; i < NP; ++i) kr[i] = *(const f32x4*)(kp + 16 * i);
    }
  };
  auto load_v = [&](int tile) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int n = 0; n < NDK; ++n) vr[v][n] = *(const f32x4*)(vb + (size_t)min(tile * 16 + 4 * g + v, Lk - 1) * DK + 64 * n);
  };
  f32x4 o[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  if (wv < n_tiles) {
    load_k(wv);
    if (with_v) load_v(wv);
  }
  for (int tile = wv; tile < n_tiles; tile += 4) {
    const int tile_n = min(tile + 4, n_tiles - 1);
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
        *(f32x4_a4*)(a.scores + srow + j) = s;
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (j + v < vis) a.scores[srow + j + v] = s[v];
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
  for (int e = tid; e < 16 * DK; e += 256) {
    const int r = e / DK, d = e % DK;
    if (i0 + r >= Lq) break;
    float M = m_s[0][r];
#pragma unroll
    for (int w = 1; w < 4; ++w) M = fmaxf(M, m_s[w][r]);
    if (M == -INFINITY) M = 0.f;                             // (every score of the row -inf: num = den = 0)
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = fast_exp2((m_s[w][r] - M) * LOG2E);    // (a wave without tiles: 0)
      num += f * o_s[w][r][d];
      den += f * l_s[w][r];
    }
    // (a row that sees nothing gives zeros, as the generic kernel has it; NaN stays NaN)
    a.out[(((size_t)b * Lq + i0 + r) * a.H + h) * DK + d] = den > 0.f ? num / den : num * 0.f;
  }
}

struct F32ScoresArgs {
  const float* q_lr;      // [B,H,Lq,r]
  const float* k_lr;      // [B,Hkv,Lk,r]
  const float* prev;      // [B,H,Lq,Lk]
  const float* w1;        // [H,F]
  const float* w2;        // [F,H]
  float* scores;          // [B,H,Lq,Lk]
  int H, Hkv, Lq, Lk, r, F, causal;
  int tiles;              // key tiles per workgroup
  float dscale;
};
constexpr int F32_DROW = 20;                                 // floats per row of the A_delta tile (16 keys, padded)
// LDS bytes for HT padded heads: A_delta tile, then the weights in operand order.
constexpr int f32_scores_lds(int HT, int F) {
  return (HT * 16 * F32_DROW + (F + 15) / 16 * (HT / 4 + (HT + 15) / 16 * 4) * 64) * (int)sizeof(float);
}

// A_n = FFN(A_{n-1}) + A_delta.  grid (ceil(key tiles / tiles), ceil(Lq / 16), B), block 256.  A tile = 16 query
// rows x 16 keys, all heads: the waves make A_delta by heads (16x16x4 float32 MFMA, keys x rows) and
// leave it in the LDS, then take the tile's rows, four each: FFN with the 16 keys of a row as the columns
// (mfma_ffn.h's scheme in float32: a lane's hidden units are its operands of the second product).
// Bound: the float32 MFMAs of the FFN.  (One position per lane with the weights through the scalar
// cache took 17 us where this takes 4, 8 heads, 128 tokens: one wave per SIMD waits for every weight.)
// HT: H rounded up to 8, 16 or 32.
template <int HT, int ACT>
__global__ __launch_bounds__(256) void k_f32_lisa_scores(F32ScoresArgs a) {
  constexpr int KS = HT / 4, HB = (HT + 15) / 16, NB = 4;    // k-steps of the heads, output blocks, rows per wave
  extern __shared__ __align__(16) float f32_lds[];
  float* d_s = f32_lds;                                      // [HT][16 rows][F32_DROW]
  const int FB = (a.F + 15) / 16;
  float* w1_s = d_s + HT * 16 * F32_DROW;                    // [FB][KS][64]
  float* w2_s = w1_s + FB * KS * 64;                         // [FB][4][HB][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int H = a.H, Lq = a.Lq, Lk = a.Lk, r = a.r, group = H / a.Hkv;
  const int rb = gridDim.y - 1 - blockIdx.y, b = blockIdx.z, i0 = rb * 16;
  const int n_tiles = (n_visible(min(i0 + 15, Lq - 1), Lq, Lk, a.causal) + 15) / 16;
  const int t0 = blockIdx.x * a.tiles, t1 = min(n_tiles, t0 + a.tiles);
  if (t0 >= t1) return;                                      // (workgroup-uniform)
  for (int e = tid; e < FB * KS * 64; e += 256) {
    const int o = e >> 6, f = 16 * (o / KS) + (e & 15), h = 4 * (o % KS) + ((e >> 4) & 3);
    w1_s[e] = f < a.F && h < H ? a.w1[(size_t)h * a.F + f] : 0.f;
  }
  for (int e = tid; e < FB * 4 * HB * 64; e += 256) {
    const int o = e >> 6, h = 16 * (o % HB) + (e & 15), f = 16 * (o / (4 * HB)) + 4 * ((e >> 4) & 3) + o / HB % 4;
    w2_s[e] = f < a.F && h < H ? a.w2[(size_t)f * H + h] : 0.f;
  }
  const size_t hs = (size_t)Lq * Lk;                         // from a head's scores to the next head's
  for (int tile = t0; tile < t1; ++tile) {
    const int j = tile * 16 + c, jc = min(j, Lk - 1);
    // this wave's rows of A_{n-1}
    float x[NB][KS];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const float* xp = a.prev + ((size_t)b * H * Lq + min(i0 + wv * NB + n, Lq - 1)) * Lk + jc;
#pragma unroll
      for (int s = 0; s < KS; ++s) x[n][s] = 4 * s + g < H ? xp[(4 * s + g) * hs] : 0.f;
    }
    if (tile > t0) __syncthreads();                          // d_s of the tile before has been read
    for (int h = wv; h < H; h += 4) {
      const float* kp = a.k_lr + (((size_t)b * a.Hkv + h / group) * Lk + jc) * r;
      const float* qp = a.q_lr + (((size_t)b * H + h) * Lq + min(i0 + c, Lq - 1)) * r;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < (r + 3) / 4; ++s) {
        const int t = 4 * s + g;
        const float kx = t < r ? kp[t] : 0.f, qx = t < r ? qp[t] : 0.f;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(kx, qx, acc, 0, 0, 0);
      }
      *(f32x4*)(d_s + (h * 16 + c) * F32_DROW + 4 * g) = acc * a.dscale;   // row c, keys 4 g ..
    }
    __syncthreads();                                         // (also publishes the weights)
    f32x4 y[NB][HB];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int hb = 0; hb < HB; ++hb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int h = min(16 * hb + 4 * g + v, H - 1);
          y[n][hb][v] = d_s[(h * 16 + wv * NB + n) * F32_DROW + c];
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
#pragma unroll
      for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int n = 0; n < NB; ++n) u[n][v] = ACT == 0 ? fmaxf(u[n][v], 0.f) : u[n][v] / (1.f + expf(-u[n][v]));
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
          const float w = w2_s[((fb * 4 + v) * HB + hb) * 64 + lane];
#pragma unroll
          for (int n = 0; n < NB; ++n) y[n][hb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, u[n][v], y[n][hb], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int i = i0 + wv * NB + n;
      if (i >= Lq || j >= n_visible(i, Lq, Lk, a.causal)) continue;
      float* sp = a.scores + ((size_t)b * H * Lq + i) * Lk + j;
#pragma unroll
      for (int hb = 0; hb < HB; ++hb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int h = 16 * hb + 4 * g + v;
          if (h < H) sp[h * hs] = y[n][hb][v];
        }
    }
  }
}

}  // namespace lisa
