// Prefill layers of bf16 operands in float32 arithmetic on the bf16 matrix instructions: scores of a LiSA layer, and
// attention.  They serve row-major score rows of any length (rows start at any 2-byte boundary), whose layers
// keep probabilities, hidden units, A_delta and A_n in float32.
//
// A product of two bf16 numbers is exact in float32, and a float32 number is the sum of three bf16 numbers without
// remainder: 24 significant bits are the first 8, the next 8 and the last 8.  A product with one bf16 operand (V, W1,
// W2) is therefore three bf16 MFMAs with the other operand cut into its three parts, exact products summed in float32
// like those of the float32 MFMA, at 3/16 of its time (16x16x32 bf16: 16 cycles, 16x16x4 float32: 32, per 32 and 4
// terms).  Half operands (A_{n-1}) are two parts, bf16 ones (Q K^T, Q_LR K_LR^T) one.
#pragma once
#include <type_traits>
#include "kernels_prefill.h"
#include "kernels_scores_mfma.h"
#include "kernels_std_prefill.h"

namespace lisa {

// Accesses of 16 bytes at any element (the hardware takes any alignment; the type keeps the compiler from assuming one).
typedef pf_u32x4 pf_u32x4_a2 __attribute__((aligned(2)));
typedef float f32x4_a4b __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned long long u64_a2 __attribute__((aligned(2)));
typedef unsigned u32_a2 __attribute__((aligned(2)));

// store_row_part() at any 2-byte boundary.
__device__ __forceinline__ void store_row_part_any(half_t* p, pf_u32x4 v, int n) {
  if (n & 4) *(u64_a2*)p = v[0] | (unsigned long long)v[1] << 32;
  if (n & 2) *(u32_a2*)((char*)p + 2 * (n & 4)) = n & 4 ? v[2] : v[0];
  if (n & 1) {
    const unsigned w = n & 4 ? (n & 2 ? v[3] : v[2]) : (n & 2 ? v[1] : v[0]);
    *(unsigned short*)((char*)p + 2 * (n & 6)) = (unsigned short)w;
  }
}

// The upper 16 bits of two floats: a float cut (not rounded) to bf16, which leaves a remainder of its own sign.
__device__ __forceinline__ unsigned cut_pair(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302);
}
__device__ __forceinline__ float cut_rest(float a) { return a - __uint_as_float(__float_as_uint(a) & 0xffff0000u); }

// (Not of what a MFMA has just written.  With the builtin in its place the scores kernel waits for its LDS reads at other
// points, 95.5 -> 97.1 us for a layer of 777 tokens, 32 heads.)
__device__ __forceinline__ float clamp_raw(float a, float top) {
  float r;
  asm("v_med3_f32 %0, %1, -%2, %2" : "=v"(r) : "v"(a), "s"(top));
  return r;
}

// Eight floats as bf16 operands whose sum they are: PARTS = 3 for any float, 2 for the value of a half.
// INF: which infinities may occur.  What is left of one (inf - inf) must not become a number of the other sign, which, times
// the weights and summed, could pass the float32 range and make NaN of the sum: it is taken to be that of the largest
// number of its sign, or 0 where there are no negative numbers (then no rest is, and one maximum does it).
enum { NO_INF, ANY_INF, POSITIVE_INF };
template <int PARTS, int INF>
__device__ __forceinline__ void split_parts(const float (&x)[8], bf16x8 (&p)[PARTS]) {
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = x[e];
#pragma unroll
  for (int k = 0; k < PARTS; ++k) {
    pf_u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = cut_pair(r[2 * e], r[2 * e + 1]);
    p[k] = __builtin_bit_cast(bf16x8, w);
    if (k + 1 < PARTS)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        constexpr float TOP = PARTS == 2 ? 65504.f : 3.40282347e38f;
        r[e] = cut_rest(INF == ANY_INF && k == 0 ? clamp_raw(r[e], TOP) : r[e]);
        if (INF == POSITIVE_INF && k == 0) r[e] = max2_raw(r[e], 0.f);   // (NaN: the other operand)
      }
  }
}

// Where a float32 tile of 16 rows x 32 keys has key 8 g + 4 q .. + 3 of row c: in the order of the lanes that hold it, so
// that a store of a wave is one KB on end.
__host__ __device__ constexpr int split_tile_at(int c, int g, int q) { return q * 256 + (g * 16 + c) * 4; }

// ---- attention ---------------------------------------------------------------------------------
struct SplitAttnArgs {
  const bf16_t* q;        // [B,H,Lq,128]
  const bf16_t* k;        // [B,Hkv,Lk,128]
  const bf16_t* v;        // [B,Hkv,Lk,128] or null (scores only)
  const float* given;     // GIVEN: float32 scores of the rows of this launch to take instead of Q K^T (then q, k unused)
  half_t* scores;         // [B,H,Lq,Lk] or null
  void* out;              // [B,Lq,H,128] float32 or bf16
  int H, Hkv, Lq, Lk, causal, out_f32;
  int row0, n_rows;       // query rows of this launch (row0 a multiple of 16)
  int given_tiled;        // given is [B,ceil(n_rows/16),ceil(Lk/32),H] tiles (split_tile_at), else [B,H,n_rows,Lk] with 32 floats behind it
  int parts;              // scores only: workgroups that the key tiles of a row group are dealt to (1 with V, or not KEYS)
  int by_length;          // row groups of all sequences by length, else sequence by sequence
  float scale;
};

constexpr int SA_OROW = 128 + 4;             // floats per row of a wave's partial result
// LDS of four waves: a K tile, over which the emitted scores are staged, and a V tile each; at the end the partial results.
constexpr int SA_PROW = SP_TK + 1;           // floats per row of a wave's probabilities
constexpr int split_attn_wave_lds(bool with_v, bool given) { return (given ? 0 : SP_KTILE) + (with_v ? SP_VTILE : 0); }
constexpr int split_attn_lds(bool with_v, bool given) {
  const int tiles = 4 * split_attn_wave_lds(with_v, given), merge = with_v ? 4 * (SP_ROWS * SA_OROW + 2 * SP_ROWS) * 4 : 0;
  return tiles > merge ? tiles : merge;
}

// grid (H, B, parts * row groups of 32), or the last two swapped, block 256: 32 query rows of one head, the tiles of 32 keys dealt to the four
// waves, each with LDS of its own (no barrier in the loop); their softmax states are merged at the end.  The scheme of
// k_std_prefill (see there for the operand layouts) with float32 probabilities in three parts, V staged as it is (the
// transposing LDS read hands out its columns), and scores at any 2-byte boundary.  GIVEN: the scores come from memory.
// What bounds it is the chain of a step (1.7 us with one wave per SIMD: scores, softmax, three products one behind the
// other), so the keys are split inside the workgroup: 17 rows of 1501 keys, 32 heads, standard layer 28.7 us (84 with
// the keys in one wave and the tiles shared by the rows of four; 53 in float32 MFMAs); at two 509-row chunks behind 1022
// keys, where V is read from the L2 once per 32 rows instead of 128, still 7 % ahead.
template <bool WITH_V, bool GIVEN>
__global__ __launch_bounds__(256, 2) void k_split_attn(SplitAttnArgs a) {
  constexpr int DK = 128, CH = 8;                              // 16-byte chunks of a tile per lane
  __shared__ __align__(16) unsigned char lds[split_attn_lds(WITH_V, GIVEN)];
  __shared__ int again;                                        // NaN has come out: see `whole`
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char* ks_ = lds + wv * split_attn_wave_lds(WITH_V, GIVEN);   // K tile; the score staging lies over it
  unsigned char* vs_ = ks_ + (GIVEN ? 0 : SP_KTILE);
  // probabilities of a second pass: over the K tile (which has been read), GIVEN behind the V tiles
  float* ps_ = (float*)(GIVEN ? lds + 4 * SP_VTILE + wv * (SP_ROWS * SA_PROW * 4) : ks_);
  static_assert(SP_ROWS * SA_PROW * 4 <= SP_KTILE && (!GIVEN || 4 * (SP_VTILE + SP_ROWS * SA_PROW * 4) <= split_attn_lds(WITH_V, GIVEN)), "");
  const int r = lane & 31, half = lane >> 5;
  const int b = a.by_length ? blockIdx.y : blockIdx.z, h = blockIdx.x;
  const int Lq = a.Lq, Lk = a.Lk, H = a.H, shift = Lk - Lq;
  const int kv = h / (H / a.Hkv);
  const float LOG2E = 1.4426950408889634f;
  const int xr = a.by_length ? gridDim.z - 1 - blockIdx.z : gridDim.y - 1 - blockIdx.y;   // long row groups first
  const int grp = xr / a.parts, part = xr - grp * a.parts;
  const int row_end = a.row0 + a.n_rows;
  const int i0 = a.row0 + grp * SP_ROWS;
  const int my_row = min(i0 + r, row_end - 1);
  const int vis_row = a.causal ? min(Lk, my_row + 1 + shift) : Lk;
  auto tiles_to = [&](int row) { return ((a.causal ? min(Lk, row + 1 + shift) : Lk) + SP_TK - 1) / SP_TK; };
  const int n_tiles = tiles_to(min(i0 + SP_ROWS, row_end) - 1);
  const int t_begin = 4 * part + wv, t_step = 4 * a.parts;
  const int n_full = i0 + SP_ROWS <= row_end ? (a.causal ? min(Lk, i0 + 1 + shift) : Lk) / SP_TK : 0;
  const int key_of_r = 16 * (r >> 4) + 8 * ((r >> 2) & 1) + 4 * ((r >> 3) & 1) + (r & 3);
  const bf16_t* kbase = GIVEN ? nullptr : a.k + ((size_t)b * a.Hkv + kv) * Lk * DK;
  const bf16_t* vbase = WITH_V ? a.v + ((size_t)b * a.Hkv + kv) * Lk * DK : nullptr;
  const int ck_key = lane >> 4, ck_c = lane & 15;              // chunk u: key ck_key + 4 u
  const int k_rd = key_of_r * SP_KROW + half * 16;
  // transposing read: lane s of a 16-lane group passes the address of key s / 4, features 4 (s % 4) .. and receives
  // feature s of keys 0 .. 3; lanes 16 .. 31 of a half take the next 16 features
  const int v_rd = (8 * half + ((lane & 15) >> 2)) * SP_VROW + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;

  bf16x8 qop[GIVEN ? 1 : DK / 16];
  if (!GIVEN) {
    const bf16_t* qp = a.q + (((size_t)b * H + h) * Lq + my_row) * DK + 8 * half;
#pragma unroll
    for (int ks = 0; ks < DK / 16; ++ks) qop[ks] = *(const bf16x8*)(qp + 16 * ks);
  }
  half_t* sbase = a.scores ? a.scores + ((size_t)b * H + h) * Lq * Lk : nullptr;

  // Tiles travel through registers and are written to the LDS where they are used.  V is loaded at the start of its step (it
  // arrives behind the scores and the softmax), K behind the softmax of the step before (behind P V): only one of the
  // two is in flight, which is what the register file has room for.
  auto tile_key = [&](int tile, int u) { return min(tile * SP_TK + ck_key + 4 * u, Lk - 1); };
  pf_u32x4 kr[CH], vr[CH];
  auto load_kt = [&](int tile) {
    if (!GIVEN)
#pragma unroll
      for (int u = 0; u < CH; ++u) kr[u] = *(const pf_u32x4*)(kbase + (size_t)tile_key(tile, u) * DK + 8 * ck_c);
  };
  auto load_vt = [&](int tile) {
    if (WITH_V)
#pragma unroll
      for (int u = 0; u < CH; ++u) vr[u] = *(const pf_u32x4*)(vbase + (size_t)tile_key(tile, u) * DK + 8 * ck_c);
  };
  auto store_kt = [&]() {
    if (!GIVEN)
#pragma unroll
      for (int u = 0; u < CH; ++u) *(pf_u32x4*)(ks_ + (ck_key + 4 * u) * SP_KROW + ck_c * 16) = kr[u];
  };
  auto store_vt = [&]() {
    if (WITH_V)
#pragma unroll
      for (int u = 0; u < CH; ++u) *(pf_u32x4*)(vs_ + (ck_key + 4 * u) * SP_VROW + ck_c * 16) = vr[u];
  };
  // given scores: row my_row, keys 32 tile + 16 u + 8 half .. + 7, loaded a step ahead
  const int n_kt = (Lk + SP_TK - 1) / SP_TK, crow = my_row - a.row0;
  const size_t g_step = a.given_tiled ? (size_t)H * (16 * SP_TK) : SP_TK;
  const int g_u = a.given_tiled ? split_tile_at(0, 2, 0) : 16, g_q = a.given_tiled ? split_tile_at(0, 0, 1) : 4;
  const float* grow =
      !GIVEN          ? nullptr
      : a.given_tiled ? a.given + (((size_t)b * ((a.n_rows + 15) / 16) + (crow >> 4)) * n_kt * H + h) * (16 * SP_TK) + split_tile_at(crow & 15, half, 0)
                      : a.given + (((size_t)b * H + h) * a.n_rows + crow) * Lk + 8 * half;
  f32x4 gq[4];
  auto load_scores = [&](int tile) {
    const float* gp = grow + tile * g_step;
    if (GIVEN)
#pragma unroll
      for (int u = 0; u < 4; ++u) gq[u] = *(const f32x4_a4b*)(gp + g_u * (u >> 1) + g_q * (u & 1));
  };
  auto clamp_tile = [&](int t) { return min(t, n_tiles - 1); };
  f32x16 o[DK / 32];
  float m_run, l_run;
  // A part of a probability may be 0 (1.0 has one part only), and 0 times an infinite element of V is NaN where the probability
  // itself gives infinity.  Where NaN comes out the workgroup goes over its tiles again with `whole` probabilities: one float32
  // product for each visible key.  (A pass of its own: as a branch inside the loop it cost 40 spilled registers.)
  auto pass = [&](auto whole) __attribute__((always_inline)) {
    load_kt(clamp_tile(t_begin));
    load_scores(clamp_tile(t_begin));
#pragma unroll
    for (int db = 0; db < DK / 32; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    m_run = -INFINITY, l_run = 0.f;

    // (the scheduling fences keep the order of the accesses to the tiles and the distance of the loads)
    for (int tile = t_begin; tile < n_tiles; tile += t_step) {
      store_kt();
      load_vt(tile);
      __builtin_amdgcn_sched_barrier(0);
      const int j0 = tile * SP_TK;
      float an[16];                                              // an[8 u + e]: key j0 + 16 u + 8 half + e of row r
      if (GIVEN) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) an[4 * u + e] = gq[u][e];
      } else {
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < DK / 16; ++ks)
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(ks_ + k_rd + 32 * ks), qop[ks], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 16; ++v) an[v] = acc[v] * a.scale;
      }
      const bool full = tile < n_full;
      const int jl = j0 + 8 * half;
      if (!GIVEN && a.scores) {
        __builtin_amdgcn_sched_barrier(0);                       // (the staging tile lies over the K tile, which has been read)
        f16x8 hv0, hv1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          hv0[e] = f32_to_half_sat(an[e]);
          hv1[e] = f32_to_half_sat(an[8 + e]);
        }
        unsigned char* sl = ks_ + r * SP_SROW + 16 * half;
        *(f16x8*)sl = hv0;
        *(f16x8*)(sl + 32) = hv1;
        const int jc = j0 + 8 * (lane & 3);                      // lane -> row lane / 4 (+ 16), 8 keys
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int row = 16 * u + (lane >> 2), gi = i0 + row;
          const pf_u32x4 hv = *(const pf_u32x4*)(ks_ + row * SP_SROW + (lane & 3) * 16);
          const int vis = gi < row_end ? (a.causal ? min(Lk, gi + 1 + shift) : Lk) : 0;
          half_t* sp = sbase + (size_t)min(gi, Lq - 1) * Lk + jc;
          if (full || jc + 8 <= vis) {
            *(pf_u32x4_a2*)sp = hv;
          } else if (jc < vis) {
            int rel = vis - jc;                                  // (kept inside this branch: registers)
            asm volatile("" : "+v"(rel));
            store_row_part_any(sp, hv, rel);
          }
        }
      }
      if (WITH_V) {
        if (!full) {
          const int rel = vis_row - jl;
#pragma unroll
          for (int v = 0; v < 16; ++v) an[v] = 16 * (v >> 3) + (v & 7) < rel ? an[v] : -INFINITY;
        }
        float mx = an[0];
#pragma unroll
        for (int v = 1; v < 15; v += 2) mx = max3_raw(mx, an[v], an[v + 1]);
        mx = halves_max(max2_raw(mx, an[15]));
        const float m_new = max2_raw(m_run, mx);
        // (the maximum is subtracted before the change of base, and no key may have been seen yet: see k_f32_attn)
        const float m0 = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = fast_exp2((m_run - m0) * LOG2E);
        m_run = m_new;
        float ps = 0.f;
        bf16x8 pop[2][3];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          float p[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            p[e] = fast_exp2((an[8 * s + e] - m0) * LOG2E);
            ps += p[e];
          }
          split_parts<3, NO_INF>(p, pop[s]);
        }
        load_scores(clamp_tile(tile + t_step));
        store_vt();
        load_kt(clamp_tile(tile + t_step));
        __builtin_amdgcn_sched_barrier(0);
        l_run = l_run * alpha + ps;
        if (__any(alpha != 1.f)) {                               // wave-uniform: the running maximum rarely moves
#pragma unroll
          for (int db = 0; db < DK / 32; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
        }
        if constexpr (decltype(whole)::value) {
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float p = 0.f;
#pragma unroll
            for (int k = 2; k >= 0; --k) p += (float)pop[v >> 3][k][v & 7];
            ps_[r * SA_PROW + 16 * (v >> 3) + 8 * half + (v & 7)] = p;
          }
#pragma unroll 1
          for (int j = 0; j < SP_TK; ++j) {
            const float p = ps_[r * SA_PROW + j];
            const unsigned seen = j0 + j < vis_row ? ~0u : 0u;
#pragma unroll
            for (int db = 0; db < DK / 32; ++db) {
#pragma unroll
              for (int q4 = 0; q4 < 4; ++q4) {
                const uint2 w = *(const uint2*)(vs_ + j * SP_VROW + (32 * db + 8 * q4 + 4 * half) * 2);
                o[db][4 * q4] += p * __uint_as_float((w.x & seen) << 16);
                o[db][4 * q4 + 1] += p * __uint_as_float(w.x & seen & 0xffff0000u);
                o[db][4 * q4 + 2] += p * __uint_as_float((w.y & seen) << 16);
                o[db][4 * q4 + 3] += p * __uint_as_float(w.y & seen & 0xffff0000u);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        } else {
          // The tile's products are summed from zero and added in one step: what a MFMA adds to its accumulator is
          // rounded (at the accumulator's size) six times per tile otherwise, 4.0e-7 of O against 2.2e-7 (301 rows of 1301 keys).
#pragma unroll
          for (int db = 0; db < DK / 32; ++db) {
            bf16x8 vop[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) vop[s] = read_columns(vs_ + v_rd + 16 * s * SP_VROW + 64 * db);
            f32x16 t;
#pragma unroll
            for (int v = 0; v < 16; ++v) t[v] = 0.f;
#pragma unroll
            for (int k = 2; k >= 0; --k)                           // small terms first
#pragma unroll
              for (int s = 0; s < 2; ++s) t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[s], pop[s][k], t, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] += t[v];
          }
        }
      } else {
        load_kt(clamp_tile(tile + t_step));
      }
      __builtin_amdgcn_sched_barrier(0);                         // (the next step's tile goes over this one's)
    }
  };
  pass(std::false_type{});
  if (!WITH_V) return;

  auto store4 = [&](size_t at, const float (&x)[4]) {
    if (a.out_f32) {
      *(float4*)((float*)a.out + at) = make_float4(x[0], x[1], x[2], x[3]);
    } else {
      uint2 pk;
      pk.x = f32_to_bf16_bits(x[0]) | (f32_to_bf16_bits(x[1]) << 16);
      pk.y = f32_to_bf16_bits(x[2]) | (f32_to_bf16_bits(x[3]) << 16);
      *(uint2*)((bf16_t*)a.out + at) = pk;
    }
  };
  // O[row][h][32 db + 8 (v / 4) + 4 half + v % 4] = o[db][v] / l (a row that sees nothing gives zeros, as the generic kernel
  // has it; NaN stays NaN)
  float* o_s = (float*)lds;                                  // [wave][row][SA_OROW]
  float* ml_s = o_s + 4 * SP_ROWS * SA_OROW;                 // [wave][row][m, l]
  auto merge = [&]() __attribute__((always_inline)) {        // true: the thread has stored NaN
    float nan = 0.f;
    const float l = halves_sum(l_run);
    __syncthreads();                                         // every wave is done with its tiles
    if (half == 0) *(float2*)(ml_s + (wv * SP_ROWS + r) * 2) = make_float2(m_run, l);
#pragma unroll
    for (int db = 0; db < DK / 32; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *(float4*)(o_s + (wv * SP_ROWS + r) * SA_OROW + 32 * db + 8 * q4 + 4 * half) =
            make_float4(o[db][4 * q4], o[db][4 * q4 + 1], o[db][4 * q4 + 2], o[db][4 * q4 + 3]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = tid + 256 * u, row = e >> 5, d = 4 * (e & 31);
      if (i0 + row >= row_end) break;
      float M = -INFINITY, den = 0.f, x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < 4; ++w) M = fmaxf(M, ml_s[(w * SP_ROWS + row) * 2]);
      if (M == -INFINITY) M = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float2 ml = *(const float2*)(ml_s + (w * SP_ROWS + row) * 2);
        const float f = fast_exp2((ml.x - M) * LOG2E);       // (a wave without tiles: 0)
        const float4 ow = *(const float4*)(o_s + (w * SP_ROWS + row) * SA_OROW + d);
        den += f * ml.y;
        x[0] += f * ow.x, x[1] += f * ow.y, x[2] += f * ow.z, x[3] += f * ow.w;
      }
      const float inv = den > 0.f ? 1.f / den : 0.f;
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] *= inv;
      nan += (x[0] + x[1]) + (x[2] + x[3]);
      store4((((size_t)b * Lq + i0 + row) * H + h) * DK + d, x);
    }
    return nan != nan;
  };
  if (tid == 0) again = 0;                                   // (written again behind the barriers of the merge)
  if (merge()) again = 1;
  __syncthreads();
  if (again) {
    pass(std::true_type{});
    merge();
  }
}

// ---- scores of a LiSA layer --------------------------------------------------------------------
struct SplitScoresArgs {
  const bf16_t* qp;       // [B,H,Lqp,32]   Q_LR rows zero-padded to 32 elements
  const bf16_t* kp;       // [B,Hkv,Lkp/32] K_LR tiles in operand order (k_prepare_prefill)
  const half_t* prev;     // [B,H,Lq,Lk]
  const unsigned short* w;  // FFN weights as k_prepare_prefill leaves them (FfnImage)
  half_t* scores;         // [B,H,Lq,Lk] or null
  float* exact;           // [B,ceil(n_rows/16),ceil(Lk/32),H] tiles of 512 (split_tile_at) or null: the unrounded copy
  int B, H, Hkv, Lq, Lk, Lqp, Lkp, F, causal;
  int row0, n_rows;       // query rows of this launch (row0 a multiple of 16)
  long long tiles_b;      // tiles of one sequence: sum over the row blocks of split_scores_tiles()
  float dscale;
};

// Key tiles of tk keys that hold visible keys of the 16 rows from i0 on.
__host__ __device__ inline int split_scores_tiles(int i0, int i_end, int Lq, int Lk, int causal, int tk) {
  return (n_visible((i0 + 16 < i_end ? i0 + 16 : i_end) - 1, Lq, Lk, causal) + tk - 1) / tk;
}
// Geometry for HT padded heads and tiles of 16 TKB keys.
template <int HT, bool CONCAT, int TKB>
struct SplitScoresGeo {
  static constexpr int TK = 16 * TKB, KSA = (HT + 31) / 32, KS = CONCAT ? 2 * KSA : KSA, HB = (HT + 15) / 16;
  static constexpr int XROW = TK * 2, XHEAD = 16 * XROW + (TKB == 2 ? 32 : 16);   // A_{n-1} tile, half
  static constexpr int YROW = TK * 4 + 16, YHEAD = 16 * YROW + 16;                // A_delta / y tile, float32
  // HT heads of A_{n-1} and one of zeros, the float32 tile, the weights in operand order
  static constexpr int lds(int F) { return (HT + 1) * XHEAD + HT * YHEAD + (F + 31) / 32 * (2 * KS + HB) * 1024; }
};

// A_n = FFN(A_{n-1}) + A_delta, or FFN([A_{n-1}; A_delta]) (CONCAT).  grid (G), block 512: the tiles of 16 query rows x
// 16 TKB keys, all heads, in (sequence, row block, key tile) order, cut into G equal runs (see k_lisa_scores_mfma).
// Per tile: every wave runs the FFN on 2 TKB blocks of 16 positions (one row, 16 keys) with the operands in parts, y goes
// to the LDS by heads; then a wave takes heads wv, wv + 8, ..: A_delta by one MFMA per 16 keys, added in registers,
// A_n out in pieces of 8 keys.  CONCAT: A_delta goes through the LDS first, as input of the FFN.
// What bounds it is the number of cache lines that a compute unit's loads and stores name (four lanes in a row, 64 bytes, are
// looked up at a time): K_LR in operand order, the float32 tile in the order of the lanes and A_n turned through the
// LDS into rows take 1/4 of what operand rows and pieces per lane did (11600 per tile of 32 heads: 149 -> 130 us at 2 x 509 rows behind 1022 keys, 32 heads).
template <int HT, int ACT, bool CONCAT, int TKB>
__global__ __launch_bounds__(512) void k_split_scores(SplitScoresArgs a) {
  typedef SplitScoresGeo<HT, CONCAT, TKB> Geo;
  constexpr int TK = Geo::TK, KSA = Geo::KSA, KS = Geo::KS, HB = Geo::HB, NW = 8;
  constexpr int XROW = Geo::XROW, XHEAD = Geo::XHEAD, YROW = Geo::YROW, YHEAD = Geo::YHEAD;
  constexpr int HPW = (HT + NW - 1) / NW;                      // heads per wave
  constexpr int NBW = 2 * TKB;                                 // position blocks per wave
  constexpr int NBLK = KS > 1 ? (NBW < 2 ? NBW : 2) : NBW;     // of them at a time (registers)
  constexpr int HPL = 2 / TKB;                                 // heads per 16-byte load of A_{n-1} by a wave
  constexpr int XCH = (HPW + HPL - 1) / HPL;
  extern __shared__ __align__(16) unsigned char split_lds[];
  unsigned char* xs = split_lds;
  unsigned char* ys = xs + (HT + 1) * XHEAD;
  unsigned char* w_s = ys + HT * YHEAD;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int H = a.H, Lq = a.Lq, Lk = a.Lk, group = H / a.Hkv;
  const int FS = (a.F + 31) / 32, row_end = a.row0 + a.n_rows;
  const int n_rg = (a.n_rows + 15) / 16, n_kt = (Lk + PF_TK - 1) / PF_TK;
  const long long total = a.tiles_b * a.B;
  long long pos = total * blockIdx.x / gridDim.x;
  const long long hi = total * (blockIdx.x + 1) / gridDim.x;
  if (pos >= hi) return;
  int b = (int)(pos / a.tiles_b), rg = 0;
  int tile0 = (int)(pos - b * a.tiles_b);
  auto tiles_of = [&](int q) { return split_scores_tiles(a.row0 + 16 * q, row_end, Lq, Lk, a.causal, TK); };
  for (int nt; tile0 >= (nt = tiles_of(rg)); ++rg) tile0 -= nt;

  // weights in operand order: W1 operands [hidden block][k-step], then W2 [hidden k-step][head block]
  const int n_w1 = FS * 2 * KS;
  stage_image(a.w, (n_w1 + FS * HB) * 64, a.w, (n_w1 + FS * HB) * 64, (unsigned short*)w_s, tid, 512);
  for (int i = tid; i < XHEAD / 4; i += 512) ((unsigned*)(xs + HT * XHEAD))[i] = 0;
  const unsigned char* wl = w_s + lane * 16;

  int xrd[KSA][2];                                             // transposing LDS reads (k_lisa_scores_mfma)
#pragma unroll
  for (int ks = 0; ks < KSA; ++ks)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int h = 32 * ks + 8 * g + 4 * q + (c >> 2);
      xrd[ks][q] = (h < H ? h : HT) * XHEAD + 8 * (c & 3);
    }
  // the 8 elements from `off` on, or (past `limit`) the last 8 of the tensor; shifted into place when they are used
  auto load8 = [&](const void* base, int off, int limit) { return *(const pf_u32x4_a2*)((const char*)base + 2u * (unsigned)min(off, limit)); };
  auto shift8 = [&](pf_u32x4 x, int by) {                      // drop the first `by` (0 .. 7) elements
    unsigned long long lo = x[0] | (unsigned long long)x[1] << 32, up = x[2] | (unsigned long long)x[3] << 32;
    if (by & 4) lo = up, up = 0;
    const int s = 16 * (by & 3);
    if (s) lo = lo >> s | up << (64 - s), up >>= s;
    return pf_u32x4{(unsigned)lo, (unsigned)(lo >> 32), (unsigned)up, (unsigned)(up >> 32)};
  };
  auto limit_of = [&](size_t total_elems, size_t base) { return (int)min((long long)(total_elems - 8 - base), 0x7fffffffLL); };
  const size_t hs = (size_t)Lq * Lk, s_elems = (size_t)a.B * H * hs;
  const int xl = lane & (32 * TKB - 1), x_hl = lane / (32 * TKB);   // A_{n-1} chunk: row, 8 keys, head of the load
  const int x_r = xl / (TK / 8), x_k = 8 * (xl % (TK / 8));
  while (pos < hi) {
    // ---- one row block: key tiles [t_first, t_last) -----------------------------------------------
    const int i0 = a.row0 + 16 * rg, t_first = tile0;
    const int t_last = (int)min((long long)tiles_of(rg), tile0 + (hi - pos));
    const bool last_b = b == a.B - 1;
    bf16x8 qop[HPW];
#pragma unroll
    for (int u = 0; u < HPW; ++u)
      qop[u] = *(const bf16x8*)(a.qp + (((size_t)b * H + min(wv + NW * u, H - 1)) * a.Lqp + i0 + c) * 32 + 8 * g);
    pf_u32x4 xr[XCH];
    bf16x8 kop[HPW][TKB];
    auto x_off = [&](int tile) { return min(i0 + x_r, Lq - 1) * Lk + min(tile * TK + x_k, Lk - 1) + (HPL == 2 ? x_hl * (int)hs : 0); };
    auto x_head = [&](int u) { return min((wv + NW * u) * HPL, (H - 1) / HPL * HPL); };
    auto load_x = [&](int tile) {
#pragma unroll
      for (int u = 0; u < XCH; ++u) {
        const size_t base = ((size_t)b * H + x_head(u)) * hs;
        xr[u] = load8(a.prev + base, x_off(tile), limit_of(s_elems, base));
      }
    };
    auto store_x = [&](int tile) {
#pragma unroll
      for (int u = 0; u < XCH; ++u) {
        const int h = (wv + NW * u) * HPL + x_hl;
        pf_u32x4 x = xr[u];
        if (last_b && tile * TK + TK > Lk - 8) {
          const int off = x_off(tile), lim = limit_of(s_elems, ((size_t)b * H + x_head(u)) * hs);
          if (__any(off > lim)) x = shift8(x, min(max(off - lim, 0), 7));
        }
        if (h < H) *(pf_u32x4*)(xs + h * XHEAD + xl * 16) = x;
      }
    };
    // K_LR operand q of the tile: keys 8 (m / 4) + m % 4 + 4 q in MFMA row m, so that a lane ends with 8 consecutive ones
    // (TKB = 1: key m in row m, 4 consecutive ones)
    auto load_k = [&](int tile, int u) {
      const bf16_t* base = a.kp + (((size_t)b * a.Hkv + min(wv + NW * u, H - 1) / group) * a.Lkp + (size_t)(tile * TKB / 2) * PF_TK) * 32;
#pragma unroll
      for (int q = 0; q < TKB; ++q) {
        int at = q * 512 + lane * 8;
        if (TKB == 1) at = ((c >> 2) & 1) * 512 + (16 * g + 8 * (tile & 1) + 4 * (c >> 3) + (c & 3)) * 8;   // key 16 (tile % 2) + c
        kop[u][q] = *(const bf16x8*)(base + at);
      }
    };
    // A_delta of this wave's head u: row c, keys 4 TKB g + 4 q + v in d[q][v]
    auto delta = [&](int u, f32x4 (&d)[TKB]) {
#pragma unroll
      for (int q = 0; q < TKB; ++q) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        d[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[u][q], qop[u], zero, 0, 0, 0) * a.dscale;
      }
    };
    load_x(t_first);
    if (CONCAT)
#pragma unroll
      for (int u = 0; u < HPW; ++u) load_k(t_first, u);
    store_x(t_first);

    for (int tile = t_first; tile < t_last; ++tile) {
      const int tile_n = min(tile + 1, t_last - 1);
      if constexpr (CONCAT) {
        lds_barrier();                                         // the tile before has left ys
#pragma unroll
        for (int u = 0; u < HPW; ++u) {
          const int h = wv + NW * u;
          f32x4 d[TKB];
          delta(u, d);
          if (h < H)
#pragma unroll
            for (int q = 0; q < TKB; ++q) *(f32x4*)(ys + h * YHEAD + c * YROW + (4 * TKB * g + 4 * q) * 4) = d[q];
        }
      }
      lds_barrier();                                           // xs (CONCAT: and A_delta) complete
      // All loads of a tile go out here and are waited for behind the FFN, ahead of the stores: a load behind a store that
      // sits in a branch could only be waited for together with it (13 us per tile, 32 heads, with the K_LR rows loaded
      // head by head between the stores).
      load_x(tile_n);
#pragma unroll
      for (int u = 0; u < HPW; ++u) load_k(CONCAT ? tile_n : tile, u);
      f32x4 y[NBW][HB];
#pragma unroll
      for (int n0 = 0; n0 < NBW; n0 += NBLK) {
        bf16x8 x[NBLK][KSA][2], xd[CONCAT ? NBLK : 1][KSA][3];
#pragma unroll
        for (int n = 0; n < NBLK; ++n) {
          const int nb = wv + (n0 + n) * NW, i = nb / TKB, kh = nb % TKB;   // block = (row, 16 keys)
#pragma unroll
          for (int ks = 0; ks < KSA; ++ks) {
            float xf[8];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              const f16x4 t = __builtin_bit_cast(f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                            (s16x4 __attribute__((address_space(3)))*)(xs + xrd[ks][q] + i * XROW + 32 * kh)));
#pragma unroll
              for (int e = 0; e < 4; ++e) xf[4 * q + e] = (float)t[e];
            }
            split_parts<2, ANY_INF>(xf, x[n][ks]);
            if constexpr (CONCAT) {
              float df[8];
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                const int h = 32 * ks + 8 * g + e;
                const float t = *(const float*)(ys + min(h, H - 1) * YHEAD + i * YROW + (16 * kh + c) * 4);
                df[e] = h < H ? t : 0.f;
              }
              split_parts<3, ANY_INF>(df, xd[n][ks]);
            }
          }
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) y[n0 + n][hb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 1
        for (int s = 0; s < FS; ++s) {
          f32x4 acc[NBLK][2];
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
#pragma unroll
            for (int n = 0; n < NBLK; ++n) acc[n][hf] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KSA; ++ks) {
              const bf16x8 w = *(const bf16x8*)(wl + ((2 * s + hf) * KS + ks) * 1024);
#pragma unroll
              for (int k = 1; k >= 0; --k)                     // small parts first
#pragma unroll
                for (int n = 0; n < NBLK; ++n) acc[n][hf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x[n][ks][k], acc[n][hf], 0, 0, 0);
              if constexpr (CONCAT) {
                const bf16x8 wd = *(const bf16x8*)(wl + ((2 * s + hf) * KS + KSA + ks) * 1024);
#pragma unroll
                for (int k = 2; k >= 0; --k)
#pragma unroll
                  for (int n = 0; n < NBLK; ++n) acc[n][hf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wd, xd[n][ks][k], acc[n][hf], 0, 0, 0);
              }
            }
          }
          bf16x8 w2[HB];
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) w2[hb] = *(const bf16x8*)(wl + (n_w1 + s * HB + hb) * 1024);
#pragma unroll
          for (int n = 0; n < NBLK; ++n) {
            float u[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float t = acc[n][e >> 2][e & 3];
              // (a median, one instruction; inline assembly may not read what a MFMA has just written.  NaN gives 0.)
              u[e] = ACT == 0 ? __builtin_amdgcn_fmed3f(t, 0.f, INFINITY) : t / (1.f + expf(-t));
            }
            bf16x8 hid[3];
            split_parts<3, ACT == 0 ? POSITIVE_INF : ANY_INF>(u, hid);
#pragma unroll
            for (int k = 2; k >= 0; --k)
#pragma unroll
              for (int hb = 0; hb < HB; ++hb) y[n0 + n][hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2[hb], hid[k], y[n0 + n][hb], 0, 0, 0);
          }
        }
      }
      if constexpr (CONCAT) lds_barrier();                     // every wave has read A_delta
#pragma unroll
      for (int n = 0; n < NBW; ++n) {
        const int nb = wv + n * NW, i = nb / TKB, kh = nb % TKB;
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int h = 16 * hb + 4 * g + v;
            if (HT % 16 == 0 || h < HT) *(float*)(ys + h * YHEAD + i * YROW + (16 * kh + c) * 4) = y[n][hb][v];
          }
      }
      lds_barrier();                                           // ys complete, xs free
      store_x(tile_n);
      f32x4 an[HPW][TKB];
      if constexpr (!CONCAT)
#pragma unroll
        for (int u = 0; u < HPW; ++u) delta(u, an[u]);
      // out as rows: lane -> row lane / (2 TKB), 8 keys
      const int o_r = lane / (2 * TKB), o_k = 8 * (lane % (2 * TKB));
      const int j = tile * TK + o_k, gi = i0 + o_r;
      const int vis = o_r < 16 && gi < row_end ? n_visible(gi, Lq, Lk, a.causal) : 0;
      const bool full = TKB == 2 && i0 + 16 <= row_end && tile * TK + TK <= n_visible(i0, Lq, Lk, a.causal);   // workgroup-uniform
#pragma unroll
      for (int u = 0; u < HPW; ++u) {
        const int h = wv + NW * u;
        if (HT % NW != 0 || HT != H)
          if (h >= H) continue;                                // (wave-uniform)
        f32x4 (&d)[TKB] = an[u];
        unsigned char* yh = ys + h * YHEAD;
#pragma unroll
        for (int q = 0; q < TKB; ++q) {
          const f32x4 yq = *(const f32x4*)(yh + c * YROW + (4 * TKB * g + 4 * q) * 4);
          d[q] = CONCAT ? yq : d[q] + yq;
        }
        if (a.exact) {
          float* ep = a.exact + ((((size_t)b * n_rg + rg) * n_kt + tile * TKB / 2) * H + h) * (16 * PF_TK);
#pragma unroll
          for (int q = 0; q < TKB; ++q)
            *(f32x4*)(ep + (TKB == 2 ? split_tile_at(c, g, q) : split_tile_at(c, 2 * (tile & 1) + (g >> 1), g & 1))) = d[q];
        }
        if (a.scores) {
          // the head's y has been read (by this wave alone): its place takes the half tile, [row][key]
#pragma unroll
          for (int q = 0; q < TKB; ++q)
            *(f16x4*)(yh + c * (2 * TK) + (4 * TKB * g + 4 * q) * 2) =
                f16x4{f32_to_half_sat(d[q][0]), f32_to_half_sat(d[q][1]), f32_to_half_sat(d[q][2]), f32_to_half_sat(d[q][3])};
          const pf_u32x4 w = *(const pf_u32x4*)(yh + (lane % (32 * TKB)) * 16);
          half_t* sp = a.scores + ((size_t)b * H + h) * hs + (unsigned)(min(gi, Lq - 1) * Lk + j);
          if (full || j + 8 <= vis) *(pf_u32x4_a2*)sp = w;
          else if (j < vis) store_row_part_any(sp, w, vis - j);
        }
      }
    }
    pos += t_last - t_first;
    tile0 = 0;
    if (++rg == n_rg) rg = 0, ++b;
  }
}

}  // namespace lisa
